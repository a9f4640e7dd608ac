// Large DyBit matrix products on the 6-bit matrix path.
//
// `v_mfma_f32_32x32x64_f8f6f4` contracts 64 k in 32 cycles when both operands are 6-bit floats: four times the fp16 and twice
// the e4m3 rate.  The 3-bit significand of e3m2 holds every 2- and 4-bit DyBit value exactly, and the sum of two of them, each
// with a power of two of its own (the instruction's block scale), every signed 8-bit and every 6-bit value: hi, the value
// rounded to the e3m2 grid, and lo, the rest.  So an operand becomes one or two planes of 6-bit floats, and a product as many
// matrix instructions as its operands' planes have pairs -- two for 8-bit by 4-bit, half the matrix time of fp16.
//
// Nothing is rounded on the way.  The instruction adds the products of groups of four k before they join the fp32 sum, and keeps of
// each what lies within 2^13 of the leading bit of the largest (measured: 2^8 + 2^-5 comes out whole, 2^8 + 2^-6 does not).
// The products of two planes span 2^12 at most (hi: 16 in steps of 1/16; 4-bit signed weights: 4 in steps of 1/4), except those of 4-bit unsigned
// values with a hi plane (2^14), which gemm_six_bytes declines.  Against 64-bit sums, 1168 products of all
// format pairs, K from 1024 to 131072, codes of one sign and of both: no error where the kernel before has none, and in the mean at most its error
// elsewhere (4096 x 2304 x 32804, 8- by 4-bit, all codes positive: 4.0e-7 of the result against 6.6e-7).
//
// The planes are made by a pass of their own (split_kernel) into a caller's scratch memory, in the order in which the product's
// lanes use them: decoding inside a tile's K loop costs 4.6 vector instructions per code for each of the N / 256 tiles that use
// it, more than the matrix instructions leave room for; here it is done once, and the loop of the product holds nothing but loads
// to LDS, fragment reads and matrix instructions.
//
// What bounds it, 8192^3: 8- by 4-bit (470 to 510 us over cards, 39 of the split before it; fp16 kernel 775 to 840) the device's power: matrix
// cores busy 76 % of the time at 1.59 GHz, 0.82 of the rate of a loop of the same instruction alone on such values, which holds 1.48 GHz; a 4-bit
// pair (267 to 288 us, 25 of the split; e4m3 kernel 400 to 415; busy 66 %, 0.68 of its loop's rate) the loads to LDS, 24 KiB per 64 k of a
// tile.  For 128 x 128 tiles these are twice as many per matrix instruction.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/dybit.h"
#include "dybit_codec.h"
#include "gemm_args.h"
#include "ragged.h"
#include "tile_common.h"

namespace dybit {
namespace six {

using namespace fast;

typedef _Float16 f16x32 __attribute__((ext_vector_type(32)));
typedef u32 u32x6 __attribute__((ext_vector_type(6)));
typedef u32 u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

// Planes of a format and their powers of two.  hi holds the value rounded to 2^HI times the e3m2 grid (up to 28, in steps of 1/16
// below 1/2): HI is the least that reaches the format's largest value.  What remains is at most half a step of that grid and a
// multiple of the format's own step: 2^LO times an integer of at most three significant bits.
template <int FMT> struct Planes {
    static constexpr bool kTwo = FMT == F8S || FMT == F6S || FMT == F6U;
    static constexpr int COUNT = kTwo ? 2 : 1;
    static constexpr int HI = FMT == F8S ? 2 : FMT == F6U ? 1 : 0;
    static constexpr int LO = FMT == F8S ? -2 : FMT == F6U ? -1 : 0;      // steps of 2^LO / 16: 1/64, 1/32, 1/16
};

// A unit: 32 rows x 128 k of a plane, 3 KiB.  Per 64 k it holds the fragment of one matrix instruction: words 0-3 of the 64 lanes' 32 codes
// (16 bytes a lane), then words 4-5 (8 bytes a lane), so that reads from LDS touch consecutive bytes.  Lane (row, kq) holds k = 32 kq
// .. + 31.  Units of a row block follow one another along k; then come the row blocks, then the planes.
constexpr int kUnit = 3072, kFragment = 1536;
constexpr int kPitch = kUnit + 16;                       // in LDS: 8-byte reads of two units do not become one, whose halves would have to be moved apart

struct SplitArgs {
    const uint8_t *codes;
    int64_t rows, K, bytes;
    int fmt, row_blocks, ktiles;                         // units per plane and row block
    uint8_t *out;
};

// Half h (64 k) of unit kt of row block rb.
template <int FMT, bool RAGGED>
__device__ __forceinline__ void split_half(const SplitArgs &s, const int rb, const int kt, const int h)
{
    using CF = Codec<FMT>;
    using P = Planes<FMT>;
    constexpr int BITS = CF::BITS, N = (BITS + 3) / 4, RUN = 4 * BITS;
    const int lane = threadIdx.x & 63, row = lane & 31, kq = lane >> 5, k = kt * 128 + h * 64 + kq * 32;
    const int64_t r = (int64_t)rb * 32 + row, row_bytes = s.K * BITS / 8;
    const u32 off = r < s.rows && k < s.K ? (u32)(r * row_bytes) + (u32)(k / 32 * RUN) : kOob;
    u32x4 raw[N];
    if constexpr (RAGGED) {
        const __amdgpu_buffer_rsrc_t rsrc = word_descriptor(s.codes, s.bytes);
        u32x4 words[ragged_regs<BITS>()];
        const u32 end = (u32)whole_words(s.bytes);
        if (((int64_t)rb * 32 + 32) * row_bytes + RUN + 4 <= end) {      // uniform: no run of these rows reaches past the tensor's whole words
            load_run_ragged<BITS>(rsrc, off, words);
        } else {
            load_run_bounded<BITS>(rsrc, off, end, last_bytes(s.codes, s.bytes), words);
        }
        align_run<BITS>(words, raw);
        const int64_t left = s.K - k;
        keep_codes<BITS>(raw, left < 0 ? 0 : left > 32 ? 32 : (int)left);
    } else {
        load_run<BITS>(code_descriptor(s.codes, s.bytes), off, raw);
    }
    union { u32 w[16]; f16x32 v; } x;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        decode_eight<FMT>(raw, q, x.w + 4 * q);
        if constexpr (CF::ACC_EXP != 0) {
            static_assert(CF::ACC_EXP == 14, "scale of the arithmetic decoders");
            const f16x2 up = {(_Float16)16384.0f, (_Float16)16384.0f};
#pragma unroll
            for (int v = 0; v < 4; ++v) x.w[4 * q + v] = __builtin_bit_cast(u32, __builtin_bit_cast(f16x2, x.w[4 * q + v]) * up);
        }
    }
    uint8_t *out = s.out + ((int64_t)rb * s.ktiles + kt) * kUnit + h * kFragment;
#pragma unroll
    for (int p = 0; p < P::COUNT; ++p) {
        const float scale = __uint_as_float((u32)(127 + (p ? P::LO : P::HI)) << 23);
        const u32x6 f = __builtin_amdgcn_cvt_scalef32_pk32_bf6_f16(x.v, scale);
        *reinterpret_cast<u32x4 *>(out + lane * 16) = u32x4{f[0], f[1], f[2], f[3]};
        *reinterpret_cast<u32x2 *>(out + 1024 + lane * 8) = u32x2{f[4], f[5]};
        if (p + 1 < P::COUNT) x.v -= __builtin_amdgcn_cvt_scalef32_pk32_f16_bf6(f, scale);
        out += (int64_t)s.row_blocks * s.ktiles * kUnit;
    }
}

// Both operands in one launch: a wave per 64 k of a row block (it is a chain of latencies: with 128 k a wave the smaller products of this
// kernel have too few of them), those of A first.
constexpr int kSplitThreads = 256;
template <bool RAGGED>
__global__ __launch_bounds__(kSplitThreads) void split_kernel(const SplitArgs a, const SplitArgs w)
{
    int u = (int)blockIdx.x * (kSplitThreads / 64) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int halves = 2 * a.ktiles;                     // of both operands
    const bool of_a = u < a.row_blocks * halves;         // uniform per wave, as all below
    const SplitArgs s = of_a ? a : w;
    if (!of_a) u -= a.row_blocks * halves;
    if (u >= s.row_blocks * halves) return;
    const int rb = u / halves, kt = u - rb * halves;
    switch (s.fmt) {
        case F2S: split_half<F2S, RAGGED>(s, rb, kt >> 1, kt & 1); break;
        case F2U: split_half<F2U, RAGGED>(s, rb, kt >> 1, kt & 1); break;
        case F4S: split_half<F4S, RAGGED>(s, rb, kt >> 1, kt & 1); break;
        case F4U: split_half<F4U, RAGGED>(s, rb, kt >> 1, kt & 1); break;
        case F6S: split_half<F6S, RAGGED>(s, rb, kt >> 1, kt & 1); break;
        case F6U: split_half<F6U, RAGGED>(s, rb, kt >> 1, kt & 1); break;
        default: split_half<F8S, RAGGED>(s, rb, kt >> 1, kt & 1); break;
    }
}

struct ProductArgs {
    const uint8_t *a, *w;                                // planes
    int a_bytes, w_bytes;
    int a_blocks, w_blocks, ktiles;                      // row blocks of either operand, units along k
    int scale_a[2], scale_w[2];                          // block scales of the planes
    int tiles_m, tiles_n;
};

// Results of 32 rows x 32 CB columns (tile_epilogue.h).  CACHE 2: stores past the caches; 0: through them, so that those of neighbouring
// columns join there where rows do not begin on cache lines (2999 x 1999 x 1532, 8- by 4-bit: 24.4 -> 20.1 us; with rows on
// lines, 2048^3, it is 14.0 -> 16.3).
template <int CB, int CACHE>
__device__ __forceinline__ void store_results(const GemmArgs &g, const f32x16 (&acc)[CB], const int64_t m_strip, const int64_t n0, const float alpha, const float (&bias)[CB])
{
    const int lane = threadIdx.x & 63;
    int col = lane & 31;
    asm volatile("" : "+v"(col));                        // see store_strip
    const int64_t left = g.M - m_strip;
    const int rows = left <= 0 ? 0 : left < 32 ? (int)left : 32;
    const u32 ldc4 = (u32)g.ldc * 4u;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(g.C + (left <= 0 ? 0 : m_strip) * g.ldc, 0, (int)((u32)rows * ldc4), 0x00020000);
#pragma unroll
    for (int j = 0; j < CB; ++j) {
        const int64_t n = n0 + j * 32 + col;
        const bool n_ok = n < g.N;
        u32 off = (n_ok ? (u32)n * 4u : kOob) + (u32)(4 * (lane >> 5)) * ldc4;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            float c = acc[j][v] * alpha + bias[j];
            if (g.relu) c = fmaxf(c, 0.0f);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(c), rsrc, off, 0, CACHE);
            off += (v & 3) == 3 ? 5u * ldc4 : ldc4;
        }
    }
}

// PA, PW: planes.  WM x WN waves, each with RBW x CBW blocks of 32 x 32.  BUFFERS stages of 128 k in LDS.
template <int PA, int PW, int WM, int WN, int RBW, int CBW, int BUFFERS>
__global__ __launch_bounds__(64 * WM * WN, 2) void product_kernel(const GemmArgs g, const ProductArgs p)
{
    constexpr int WAVES = WM * WN, STAGE = WAVES * (PA + PW) * kPitch, LOADS = 3 * (PA + PW);
    static_assert(WM * RBW == WAVES && WN * CBW == WAVES, "a wave loads one row block of either operand");
    extern __shared__ __attribute__((aligned(16))) char lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    int tile_m, tile_n;
    if (!panel_order_tile(xcd_contiguous_index(), p.tiles_m, p.tiles_n, tile_m, tile_n)) return;   // uniform per workgroup

    // ---- factors and biases, which the epilogue would wait for
    const int64_t m0 = ((int64_t)tile_m * WAVES + wm * RBW) * 32, n0 = ((int64_t)tile_n * WAVES + wn * CBW) * 32;
    const float alpha = (*g.a_scale) * (*g.w_scale);
    float bias[CBW];
#pragma unroll
    for (int c = 0; c < CBW; ++c) {
        const int64_t n = n0 + c * 32 + (lane & 31);
        bias[c] = g.bias ? g.bias[n < g.N ? n : 0] : 0.0f;
    }

    // ---- loads to LDS: this wave's row block of A and of W, every plane, three times 1 KiB each
    const u32 lds_base = (u32)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    auto descriptor = [](const uint8_t *at, int bytes) { return u32x4{(u32)(uintptr_t)at, (u32)((uintptr_t)at >> 32), (u32)bytes, 0x00020000u}; };
    const int rb = min(tile_m * WAVES + wave, p.a_blocks - 1), cb = min(tile_n * WAVES + wave, p.w_blocks - 1);   // past the end: any rows, not stored
    const u32 voff = (u32)lane * 16;
    // Load j of a stage.  Past the last stage (whose units are then named) the descriptors are empty: nothing is read, and no branch
    // splits the loop (the compiler moves the matrix instructions before one behind it).
    auto load = [&](int j, int kt, u32 buffer) {
        const int q = j / 3, plane = q < PA ? q : q - PA;
        const bool w = q >= PA, some = kt < p.ktiles;
        const int at = some ? kt : p.ktiles - 1;
        const u32x4 rsrc = descriptor(w ? p.w : p.a, some ? (w ? p.w_bytes : p.a_bytes) : 0);
        const u32 from = (u32)(((w ? plane * p.w_blocks + cb : plane * p.a_blocks + rb) * p.ktiles + at) * kUnit + j % 3 * 1024);
        const u32 to = lds_base + buffer + (w ? WAVES * PA + wave * PW + plane : wave * PA + plane) * kPitch + j % 3 * 1024;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(to), "v"(voff), "s"(rsrc), "s"(from) : "memory");
    };
    // A fragment: this lane's 16 and its 8 bytes.
    typedef __attribute__((address_space(3))) u32x4 LdsFour;
    typedef __attribute__((address_space(3))) u32x2 LdsTwo;
    struct At { u32 four, two; };
    auto at_units = [&](u32 first) { return At{first + lane * 16, first + 1024 + lane * 8}; };
    auto read = [&](const At &a, int unit, int half) -> i32x8 {
        const u32x4 lo = *(const LdsFour *)(uintptr_t)(a.four + unit * kPitch + half * kFragment);
        const u32x2 hi = *(const LdsTwo *)(uintptr_t)(a.two + unit * kPitch + half * kFragment);
        i32x8 f;                                         // six of its words are used
        f[0] = (int)lo.x; f[1] = (int)lo.y; f[2] = (int)lo.z; f[3] = (int)lo.w; f[4] = (int)hi.x; f[5] = (int)hi.y;
        return f;
    };
    const At ownA = at_units(lds_base + wm * (RBW * PA * kPitch)), ownW = at_units(lds_base + (WAVES * PA + wn * (CBW * PW)) * kPitch);
    auto plus = [](const At &a, u32 o) { return At{a.four + o, a.two + o}; };

    f32x16 acc[RBW][CBW];
#pragma unroll
    for (int r = 0; r < RBW; ++r)
#pragma unroll
        for (int c = 0; c < CBW; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[r][c][v] = 0.0f;

    constexpr int NA = RBW * PA, NW = CBW * PW;          // fragments of a wave per 64 k
    static_assert((NA == 2 || NA == 4) && NW % 2 == 0, "the ring holds four fragments of A");
    i32x8 fa[4], fw[2][NW];
    // A stage: twice (64 k each) NA phases, in each a fragment of A times every fragment of W.  The fragments of A are read two phases
    // ahead, those of W 64 k ahead.  Once a wave has read its last fragment of this buffer (before phase NA - 2 of the second
    // half) it waits for the others and for the next stage, reads on in the next buffer and has this one filled with a
    // new stage, load by load behind the matrix instructions that follow, the last ones of them in the next stage: issued in a row they
    // fill the address unit's queue, and the waves wait before their matrix instructions (8192^3, 8- by 4-bit, all codes zero: 449 -> 414 us).
    constexpr int TOTAL = 2 * NA * NW, FIRST = 2 * NW;   // matrix instructions of a stage, and of its last two phases
    constexpr int SPAN = BUFFERS == 2 ? TOTAL * 5 / 8 : TOTAL;   // those that loads stand behind; two buffers: the last load needs time to arrive
    auto loads_at = [](int n) { int j = 0; while (j < LOADS && j * SPAN / LOADS < n) ++j; return j; };   // loads before the n-th one
    constexpr int HERE = (FIRST * LOADS + SPAN - 1) / SPAN;   // loads_at(FIRST)
    static_assert(HERE <= LOADS, "");
    u32 buffer = 0, before = (BUFFERS - 1) * STAGE;
    auto stage = [&](int kt, f32x16 (&acc)[RBW][CBW]) {
        const u32 next = buffer == (BUFFERS - 1) * STAGE ? 0 : buffer + STAGE;
        const At a = plus(ownA, buffer), w = plus(ownW, buffer), a_next = plus(ownA, next), w_next = plus(ownW, next);
#pragma unroll
        for (int hi = 0; hi < 2 * NA; ++hi) {
            const int h = hi / NA, i = hi % NA;
            const bool ahead = i >= NA - 2, late = h == 1 && ahead;   // reads of the next 64 k; of the next stage
            if (late && i == NA - 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((BUFFERS - 2) * LOADS) : "memory");
#pragma unroll
            for (int c = 0; c < NW; ++c) {
                // the fragment of A, then half of the next 64 k's of W, one before each instruction; past the last stage: not used
                if (c == 0) fa[(hi + 2) & 3] = late ? read(a_next, i + 2 - NA, 0) : ahead ? read(a, i + 2 - NA, 1) : read(a, i + 2, h);
                else if (ahead && c <= NW / 2) {
                    const int n = (i - (NA - 2)) * (NW / 2) + c - 1;
                    fw[h ^ 1][n] = late ? read(w_next, n, 0) : read(w, n, 1);
                }
                acc[i / PA][c / PW] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fa[hi & 3], fw[h][c], acc[i / PA][c / PW], 3, 3, 0, p.scale_a[i % PA], 0, p.scale_w[c % PW]);
                const int n = late ? (i - (NA - 2)) * NW + c : FIRST + hi * NW + c;   // which one since the last wait
                if (loads_at(n) != loads_at(n + 1)) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = loads_at(n); j < loads_at(n + 1); ++j) {
                        if (late) load(j, kt + BUFFERS, buffer);
                        else load(j, kt - 1 + BUFFERS, before);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        before = buffer;
        buffer = next;
    };

#pragma unroll
    for (int b = 0; b < BUFFERS; ++b)
#pragma unroll
        for (int j = 0; j < (b < BUFFERS - 1 ? LOADS : HERE); ++j) load(j, b, b * STAGE);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((BUFFERS - 2) * LOADS + HERE) : "memory");
#pragma unroll
    for (int c = 0; c < NW; ++c) fw[0][c] = read(ownW, c, 0);
    fa[0] = read(ownA, 0, 0);
    fa[1] = read(ownA, 1, 0);
    // Tiles of 128: two sums, of every other stage.  The fp16 kernels that such products ran on add two k-groups where tiles are few,
    // and one sum of everything rounds where two do not (1300 x 1300 x 32772, 8- by 4-bit, all codes positive: 2.3e-6 of the result against 3.8e-8).
    // 0.98 times the time besides (39 products in place of fp16 ones).
    constexpr bool TWO_SUMS = RBW * CBW <= 4;            // tiles of 256 have no registers for it, and replace kernels with one sum
    int kt = 0;
    if constexpr (TWO_SUMS) {
        f32x16 odd[RBW][CBW];
#pragma unroll
        for (int r = 0; r < RBW; ++r)
#pragma unroll
            for (int c = 0; c < CBW; ++c) odd[r][c] = acc[r][c];
#pragma unroll 1
        for (; kt + 1 < p.ktiles; kt += 2) {
            stage(kt, acc);
            stage(kt + 1, odd);
        }
        if (kt < p.ktiles) stage(kt, acc);
#pragma unroll
        for (int r = 0; r < RBW; ++r)
#pragma unroll
            for (int c = 0; c < CBW; ++c) acc[r][c] += odd[r][c];
    } else {
#pragma unroll 1
        for (; kt < p.ktiles; ++kt) stage(kt, acc);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // no load to LDS outlives the workgroup
    if (g.ldc % 32) {                                    // uniform
#pragma unroll
        for (int r = 0; r < RBW; ++r) store_results<CBW, 0>(g, acc[r], m0 + r * 32, n0, alpha, bias);
    } else {
#pragma unroll
        for (int r = 0; r < RBW; ++r) store_results<CBW, 2>(g, acc[r], m0 + r * 32, n0, alpha, bias);
    }
}

template <int PA, int PW, int WM, int WN, int RBW, int CBW, int BUFFERS>
static void launch(const GemmArgs &g, const ProductArgs &p, hipStream_t st)
{
    constexpr int LDS = BUFFERS * WM * WN * (PA + PW) * kPitch;
    auto k = product_kernel<PA, PW, WM, WN, RBW, CBW, BUFFERS>;
    note_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS));
    hipLaunchKernelGGL(k, dim3((unsigned)((p.tiles_m * p.tiles_n + 7) / 8 * 8)), dim3(64 * WM * WN), LDS, st, g, p);
}

// Planes of a format; 0: none (8-bit unsigned values would need three, more matrix time than the e4m3 and fp16 kernels save by).
struct Format {
    int planes, id, hi, lo;
};
static Format format(int bits, int is_signed)
{
    if (bits == 2) return is_signed ? Format{1, F2S, 0, 0} : Format{1, F2U, 0, 0};
    if (bits == 4) return is_signed ? Format{1, F4S, 0, 0} : Format{1, F4U, 0, 0};
    if (bits == 6) return is_signed ? Format{2, F6S, Planes<F6S>::HI, Planes<F6S>::LO} : Format{2, F6U, Planes<F6U>::HI, Planes<F6U>::LO};
    return is_signed ? Format{2, F8S, Planes<F8S>::HI, Planes<F8S>::LO} : Format{};
}
static int64_t plane_bytes(int64_t rows, int64_t K) { return (rows + 31) / 32 * ((K + 127) / 128) * kUnit; }

}  // namespace six

int64_t gemm_six_bytes(int64_t M, int64_t N, int64_t K, int a_bits, int a_signed, int w_bits, int w_signed)
{
    const six::Format a = six::format(a_bits, a_signed), w = six::format(w_bits, w_signed);
    if (!a.planes || !w.planes || !w_signed || a.planes * w.planes > 2 || (a.id == fast::F4U && w.planes == 2) || M < 1 || N < 1 || K < 1) return 0;
    if (M > 1 << 24 || N > 1 << 24 || K > 1 << 24 || M * (K * a_bits / 8) >= 0x7fffffff || N * (K * w_bits / 8) >= 0x7fffffff) return 0;
    const int64_t ba = a.planes * six::plane_bytes(M, K), bw = w.planes * six::plane_bytes(N, K);
    return ba >= 0x7fffffff || bw >= 0x7fffffff ? 0 : ba + bw;
}

void launch_gemm_six(const GemmArgs &g, int a_bits, int w_bits, int tile, uint8_t *scratch, hipStream_t st)
{
    using namespace six;
    const Format a = format(a_bits, g.a_signed), w = format(w_bits, g.w_signed);
    const int kt = (int)((g.K + 127) / 128), a_blocks = (int)((g.M + 31) / 32), w_blocks = (int)((g.N + 31) / 32);
    const int64_t ba = a.planes * plane_bytes(g.M, g.K), bw = w.planes * plane_bytes(g.N, g.K);
    uint8_t *const planes = scratch;
    const SplitArgs sa{g.A, g.M, g.K, g.a_bytes, a.id, a_blocks, kt, planes}, sw{g.W, g.N, g.K, g.w_bytes, w.id, w_blocks, kt, planes + ba};
    const dim3 grid((unsigned)((((int64_t)a_blocks + w_blocks) * 2 * kt + kSplitThreads / 64 - 1) / (kSplitThreads / 64)));
    if (g.K % 64) hipLaunchKernelGGL(split_kernel<true>, grid, dim3(kSplitThreads), 0, st, sa, sw);
    else hipLaunchKernelGGL(split_kernel<false>, grid, dim3(kSplitThreads), 0, st, sa, sw);

    auto block_scale = [](int e) { return 127 + e; };
    const bool wide = tile == 256;
    const ProductArgs p{planes, planes + ba, (int)ba, (int)bw, a_blocks, w_blocks, kt, {block_scale(a.hi), block_scale(a.lo)}, {block_scale(w.hi), block_scale(w.lo)},
                        (int)((g.M + tile - 1) / tile), (int)((g.N + tile - 1) / tile)};
    note_kernel(wide ? DYBIT_KERNEL_F6_256 : DYBIT_KERNEL_F6_128);
    if (wide) {
        if (a.planes == 2) launch<2, 1, 4, 2, 2, 4, 2>(g, p, st);
        else if (w.planes == 2) launch<1, 2, 2, 4, 4, 2, 2>(g, p, st);
        else launch<1, 1, 4, 2, 2, 4, 3>(g, p, st);
    } else {
        if (a.planes == 2) launch<2, 1, 2, 2, 2, 2, 2>(g, p, st);
        else if (w.planes == 2) launch<1, 2, 2, 2, 2, 2, 2>(g, p, st);
        else launch<1, 1, 2, 2, 2, 2, 3>(g, p, st);
    }
}

}  // namespace dybit
