// DyBit matrix product for small outputs: 32 rows by 32 or 64 columns of C per workgroup, K split over its waves.
//
// The tiled kernels put one workgroup on a 64 x 64 or 128 x 128 tile and walk K serially; a product with few
// rows (the classifier of a network, a small batch, a narrow layer) then leaves most compute units idle and takes as
// long as the K loop of one workgroup: 128 x 1000 x 2048 ran on 8 of 256 compute units.  Here a tile is as small as the
// matrix instruction allows and up to 16 waves share its K: wave w takes K steps w, w + S, w + 2 S, ... (64 codes each),
// fetches and decodes the codes of both operands itself, straight into fragments (there is nothing to share between waves
// that work on different k, so no LDS and no barrier inside the loop), and the partial sums are added through LDS in
// log2 S rounds at the end.  The price is decoding: every code of A is decoded once per column tile and every code of
// W once per row tile, at 1/32 of the reuse a full tile would have, which is what bounds the kernel once the
// device is full; the dispatcher takes it below that.
//
// Rows of any length (RAGGED) and convolutions with Cin a multiple of 64 as in the other kernels.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dybit_codec.h"
#include "dybit_codec8.h"
#include "gemm_args.h"
#include "ragged.h"
#include "tile_common.h"
#include "tile_epilogue.h"

#ifndef DYBIT_SMALL_W
#error "compile with -DDYBIT_SMALL_W=<weight format id> (0: 4-bit, 2: 8-bit, 4: 6-bit, 6: 2-bit; signed)"
#endif

namespace dybit {
namespace small {

using namespace fast;

enum : int { ROWS_ALIGNED = 0, CONVOLUTION = 1, RAGGED = 3 };   // how the operands' rows are reached
constexpr int kMaxWaves = 16;

// E4M3: both operands 4- or 2-bit (every value exact in e4m3): one matrix instruction per K step and column block
// instead of four, and decoders that emit bytes.  512 x 512 x 4096, 4-bit pair: fp16 form 9.2, this one 8.4 us.
template <int FMT> constexpr bool low_format() { return FMT == F4S || FMT == F4U || FMT == F2S || FMT == F2U; }

// The order of the tiles: l / per is one coordinate, l % per the other.
struct TileOrder {
    uint32_t tiles;
    Divisor per;
    int by_columns, waves;
};

template <int FMT_A, int FMT_W, int MODE, int CB, int OUT, bool E4M3>
__global__ __launch_bounds__(64 * kMaxWaves) void gemm_small_kernel(const GemmArgs g, const TileOrder order)
{
    using CA = Codec<FMT_A>;
    using CW = Codec<FMT_W>;
    constexpr int BA = CA::BITS, BW = CW::BITS;
    constexpr int NA = MODE == RAGGED ? ragged_regs<BA>() : (BA + 3) / 4, NW = MODE == RAGGED ? ragged_regs<BW>() : (BW + 3) / 4;
    extern __shared__ __attribute__((aligned(16))) float red[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // every argument that the first loads need, read at once, and the scales and biases requested before the K loop: the compiler otherwise
    // reads them in steps that wait for each other.  Kernel times 1 to 7 % shorter (64 x 64 x 256, 4-bit pair 3.33 -> 3.10 us, 128 x 1000 x 2048,
    // 8-bit 8.72 -> 8.55), a call that is waited for, with its absmax and encoder, 1 % (23.4 -> 23.2 and 32.7 -> 32.4).  Not in the
    // write-back build, whose epilogue has no scalar registers to spare (196 rows, three layers of a bottleneck block: 31.5 -> 32.6 us)
    constexpr bool EARLY = OUT == OUT_FP32;
    if (EARLY) asm volatile("" ::"s"(g.M), "s"(g.N), "s"(g.K), "s"(g.A), "s"(g.W), "s"(g.a_bytes), "s"(g.w_bytes), "s"(g.a_scale), "s"(g.w_scale), "s"(g.bias));
    if (EARLY && MODE == CONVOLUTION) asm volatile("" ::"s"(g.H), "s"(g.Wd), "s"(g.Cin), "s"(g.Ho), "s"(g.Wo), "s"(g.kw), "s"(g.stride), "s"(g.pad), "s"(g.pix_bytes));
    const int waves = order.waves, kq = lane >> 5;
    // neighbouring tiles, which share an operand strip, go to the same XCD: by columns when W is the larger operand
    const int l = xcd_contiguous_index();
    if ((u32)l >= order.tiles) return;                               // uniform per workgroup
    const int high = (int)quotient((u32)l, order.per), low = l - high * (int)order.per.d;
    const int tile_m = order.by_columns ? low : high, tile_n = order.by_columns ? high : low;
    const int64_t m0 = (int64_t)tile_m * 32, n0 = (int64_t)tile_n * (32 * CB);

    const __amdgpu_buffer_rsrc_t rsrcA = MODE == RAGGED ? word_descriptor(g.A, g.a_bytes) : code_descriptor(g.A, g.a_bytes);
    const __amdgpu_buffer_rsrc_t rsrcW = MODE == RAGGED ? word_descriptor(g.W, g.w_bytes) : code_descriptor(g.W, g.w_bytes);
    const int a_row_bytes = (int)(g.K * BA / 8), w_row_bytes = (int)(g.K * BW / 8), K = (int)g.K;
    const int pix_bytes = MODE == CONVOLUTION ? g.pix_bytes : 0;
    const int64_t m = m0 + (lane & 31);
    const bool okA = m < g.M;
    u32 offA, offW[CB];
    int hi0 = 0, wi0 = 0;
    TapCounter tap;
    if (MODE == CONVOLUTION) {
        const PixelOrigin o = pixel_origin(g, okA ? m : 0);
        hi0 = o.hi0;
        wi0 = o.wi0;
        offA = (u32)(o.first_pixel * pix_bytes + kq * 4 * BA);
        tap.advance(wave * 64, g);
    } else {
        offA = okA ? (u32)(m * a_row_bytes + kq * 4 * BA) : kOob;
    }
#pragma unroll
    for (int j = 0; j < CB; ++j) {
        const int64_t n = n0 + j * 32 + (lane & 31);
        offW[j] = n < g.N ? (u32)(n * w_row_bytes + kq * 4 * BW) : kOob;
    }
    // RAGGED: the last bytes of the operands, in the lanes whose row they end
    u32 last_a = 0, last_w[CB] = {};
    if (MODE == RAGGED && kq == 1) {
        if (m == g.M - 1) last_a = last_bytes(g.A, g.a_bytes);
#pragma unroll
        for (int j = 0; j < CB; ++j)
            if (n0 + j * 32 + (lane & 31) == g.N - 1) last_w[j] = last_bytes(g.W, g.w_bytes);
    }
    const int steps = (K + 63) / 64, head = MODE == RAGGED ? K - (steps - 1) * 64 : 64;   // codes of K step 0
    auto first_code = [&](int t) { return t == 0 ? 0 : head + (t - 1) * 64; };

    auto load = [&](int t, u32x4 (&a)[NA], u32x4 (&w)[CB][NW]) {
        const bool in = t < steps;
        const int k0 = first_code(t);
        u32 oa;
        if (MODE == CONVOLUTION) {
            oa = in && okA && tap.inside(g, hi0, wi0) ? offA + (u32)tap.byte_offset(g, pix_bytes, BA) : kOob;   // padding reads code 0
            tap.advance(64 * waves, g);
        } else {
            oa = in ? offA + (u32)(k0 * BA / 8) : kOob;
        }
        if constexpr (MODE == RAGGED) load_run_ragged<BA>(rsrcA, oa, a);
        else load_run<BA>(rsrcA, oa, a);
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            const u32 ow = in ? offW[j] + (u32)(k0 * BW / 8) : kOob;
            if constexpr (MODE == RAGGED) load_run_ragged<BW>(rsrcW, ow, w[j]);
            else load_run<BW>(rsrcW, ow, w[j]);
        }
    };

    f32x16 acc[CB];
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.0f;

    auto contract = [&](int t, const u32x4 (&a)[NA], const u32x4 (&w)[CB][NW]) {
        u32x4 ta[(BA + 3) / 4], tw[CB][(BW + 3) / 4];
        if constexpr (MODE == RAGGED) {
            align_run<BA>(a, ta, t == steps - 1 ? last_a : 0u);
#pragma unroll
            for (int j = 0; j < CB; ++j) {
                align_run<BW>(w[j], tw[j], t == steps - 1 ? last_w[j] : 0u);
                if (t == 0) keep_codes<BW>(tw[j], head - 32 * kq);   // uniform: the odd part of K
            }
        }
        if constexpr (E4M3) {
            const f8::i32x8 fa = f8::decode_fragment<FMT_A>(MODE == RAGGED ? ta[0] : a[0]);
#pragma unroll
            for (int j = 0; j < CB; ++j)
                acc[j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fa, f8::decode_fragment<FMT_W>(MODE == RAGGED ? tw[j][0] : w[j][0]), acc[j],
                                                                         0, 0, 0, 0, 0, 0);
            return;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u32 d[4];
            decode_eight<FMT_A>(MODE == RAGGED ? ta : a, q, d);
            const f16x8 fa = __builtin_bit_cast(f16x8, u32x4{d[0], d[1], d[2], d[3]});
#pragma unroll
            for (int j = 0; j < CB; ++j) {
                decode_eight<FMT_W>(MODE == RAGGED ? tw[j] : w[j], q, d);
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa, __builtin_bit_cast(f16x8, u32x4{d[0], d[1], d[2], d[3]}), acc[j], 0, 0, 0);
            }
        }
    };

    // the codes of two further steps are in flight while one is decoded
    u32x4 a0[NA], a1[NA], w0[CB][NW], w1[CB][NW];
    load(wave, a0, w0);
    load(wave + waves, a1, w1);
    // the epilogue's scales and biases, requested now for its wave: its own loads then come out of the caches
    u32 ahead[3] = {0, 0, 0};
    if (EARLY && wave == 0) {
        const u32 n = (u32)(n0 + (lane & (32 * CB - 1))), n_in = n < (u32)g.N ? n : 0u;
        ahead[0] = __builtin_amdgcn_raw_buffer_load_b32(code_descriptor(reinterpret_cast<const uint8_t *>(g.a_scale), 4), 0, 0, 0);
        ahead[1] = __builtin_amdgcn_raw_buffer_load_b32(code_descriptor(reinterpret_cast<const uint8_t *>(g.w_scale), g.w_per_channel ? 4 * g.N : 4), g.w_per_channel ? 4u * n_in : 0u, 0, 0);
        if (g.bias) ahead[2] = __builtin_amdgcn_raw_buffer_load_b32(code_descriptor(reinterpret_cast<const uint8_t *>(g.bias), 4 * g.N), 4u * n_in, 0, 0);
    }
    for (int t = wave; t < steps; t += 2 * waves) {
        contract(t, a0, w0);
        load(t + 2 * waves, a0, w0);
        if (t + waves < steps) contract(t + waves, a1, w1);
        load(t + 3 * waves, a1, w1);
    }

    if (EARLY) asm volatile("" ::"v"(ahead[0]), "v"(ahead[1]), "v"(ahead[2]));

    // ---- add the waves' partial sums: in each round the upper half hands its sums to the lower half
    for (int half = waves >> 1; half > 0; half >>= 1) {
        if (wave >= half && wave < 2 * half) {
#pragma unroll
            for (int j = 0; j < CB; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) red[(((wave - half) * CB + j) * 16 + v) * 64 + lane] = acc[j][v];
        }
        __syncthreads();
        if (wave < half) {
#pragma unroll
            for (int j = 0; j < CB; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[j][v] += red[((wave * CB + j) * 16 + v) * 64 + lane];
        }
        __syncthreads();
    }
    if (wave == 0) epilogue_strip<CB, OUT != OUT_FP32, true, CA::ACC_EXP + CW::ACC_EXP>(g, acc, m0, n0);
}

template <int FA, int FW, int MODE, int CB, bool E4M3>
static void launch_one(const GemmArgs &g, hipStream_t st)
{
    const int tiles_m = (int)((g.M + 31) / 32), tiles_n = (int)((g.N + 32 * CB - 1) / (32 * CB));
    const int64_t tiles = (int64_t)tiles_m * tiles_n;
    const int steps = (int)((g.K + 63) / 64);
    // waves per tile: at most 16 per compute unit in all (what fits at once), and at least one K step each
    int waves = 1;
    while (waves < kMaxWaves && waves * 2 <= steps && tiles * waves * 2 <= 4096) waves *= 2;
    const int lds_bytes = waves / 2 * CB * 16 * 64 * 4;
    const TileOrder order{(uint32_t)tiles, divisor((uint32_t)(g.N > g.M ? tiles_m : tiles_n)), g.N > g.M ? 1 : 0, waves};
    auto k = gemm_small_kernel<FA, FW, MODE, CB, kOut, E4M3>;
    note_kernel(E4M3 ? DYBIT_KERNEL_F8_SMALL : DYBIT_KERNEL_F16_SMALL);
    note_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxWaves / 2 * CB * 16 * 64 * 4));
    hipLaunchKernelGGL(k, dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(64 * waves), lds_bytes, st, g, order);
}

template <int FA, int FW, bool E4M3>
static void launch_path(const GemmArgs &g, bool conv, hipStream_t st)
{
    // 64 columns per tile (half the decoding of A) once that still gives every compute unit a workgroup
    const bool two = ((g.M + 31) / 32) * ((g.N + 63) / 64) >= 256;
    if (conv) return two ? launch_one<FA, FW, CONVOLUTION, 2, E4M3>(g, st) : launch_one<FA, FW, CONVOLUTION, 1, E4M3>(g, st);
    if (g.K % 64) return two ? launch_one<FA, FW, RAGGED, 2, E4M3>(g, st) : launch_one<FA, FW, RAGGED, 1, E4M3>(g, st);
    return two ? launch_one<FA, FW, ROWS_ALIGNED, 2, E4M3>(g, st) : launch_one<FA, FW, ROWS_ALIGNED, 1, E4M3>(g, st);
}

template <int FA, int FW>
static void launch(const GemmArgs &g, bool conv, hipStream_t st)
{
    if constexpr (low_format<FA>() && low_format<FW>())
        if (!dispatch_options().mfma_f16) return launch_path<FA, FW, true>(g, conv, st);
    launch_path<FA, FW, false>(g, conv, st);
}

}  // namespace small

#define DYBIT_SMALL_NAME2(w) DYBIT_WB_NAME(launch_gemm_small_w##w)
#define DYBIT_SMALL_NAME(w) DYBIT_SMALL_NAME2(w)
void DYBIT_SMALL_NAME(DYBIT_SMALL_W)(const GemmArgs &g, int a_bits, bool conv, hipStream_t st)
{
    using namespace fast;
    const int fa = (a_bits == 8 ? F8S : a_bits == 6 ? F6S : a_bits == 2 ? F2S : F4S) + (g.a_signed ? 0 : 1);
    switch (fa) {
        case F2S: return small::launch<F2S, DYBIT_SMALL_W>(g, conv, st);
        case F2U: return small::launch<F2U, DYBIT_SMALL_W>(g, conv, st);
        case F4S: return small::launch<F4S, DYBIT_SMALL_W>(g, conv, st);
        case F4U: return small::launch<F4U, DYBIT_SMALL_W>(g, conv, st);
        case F6S: return small::launch<F6S, DYBIT_SMALL_W>(g, conv, st);
        case F6U: return small::launch<F6U, DYBIT_SMALL_W>(g, conv, st);
        case F8S: return small::launch<F8S, DYBIT_SMALL_W>(g, conv, st);
        case F8U: return small::launch<F8U, DYBIT_SMALL_W>(g, conv, st);
    }
}

}  // namespace dybit
