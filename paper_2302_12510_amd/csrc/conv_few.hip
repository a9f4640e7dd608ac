// Convolution of an image with few channels (the first layer of an image network) with its input decoded once.
//
// An implicit-GEMM kernel decodes an input code again for every filter tap it meets -- 16 times for 7 x 7 at stride 2 with its
// rows padded to 8 taps -- and gathers it word by word: 802816 x 64 x 256 at 8 bits spent two thirds of its vector
// instructions there.  Here a workgroup owns R whole output rows of an image: it decodes the input rows they need (with
// padding, as fp16) into LDS once, then its waves take strips of 32 consecutive output pixels and read the fragments of A
// from there: the eight codes of a lane are 8 / Cin neighbouring pixels of one filter row, 16 consecutive bytes.  The weights
// of up to 64 output channels stay in LDS for all units a workgroup of the persistent grid walks over.  A filter row is 32
// codes of K (kw Cin, filled up with zero weights), so the filter needs no padding in memory.
//
// What bounds it then: LDS reads (1.5 KiB per matrix instruction, 64 KiB per strip with the epilogue's factors) and the
// epilogue's vector instructions, which the barriers around a unit keep from overlapping fully.  64 x 112 x 112 x 64 from
// 224 x 224, 8-bit operands: codes out 74.4 -> 50.6 us (46.9 with a kernel per width of the codes), fp32 out 79.3 -> 65.6 us (weight-stationary kernel -> this one).
//
// Decoding is cheap only in whole runs: a thread takes 32 codes of an image row (a group of eight per thread spent 150
// instructions on where it lies, and the kernel was no faster than decoding every tap), written at the padded column with
// the codes in their natural order, so that runs can start at the image's edge and fragments at the padding's.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "codes_epilogue.h"
#include "dybit_codec.h"
#include "gemm_args.h"
#include "ragged.h"
#include "tile_common.h"
#include "tile_epilogue.h"

#ifndef DYBIT_FEW_W
#error "compile with -DDYBIT_FEW_W=<weight format id> (0: 4-bit, 2: 8-bit, 4: 6-bit, 6: 2-bit; signed)"
#endif

namespace dybit {
namespace few {

using namespace fast;

constexpr int CB = 2;                                    // column blocks of 32: output channels of a workgroup
constexpr int kMaxThreads = 512;

struct FewArgs {
    int rows, units_per_image, units;                    // output rows of a unit; units of an image, of the call
    int in_cols, in_rows, pitch;                         // input patch: columns (pixels), rows, bytes per row in LDS
    int row_bytes, parts;                                // LDS bytes of a weight row; groups of 64 output channels
};

// decode_eight() with the codes in their natural order.
template <int FMT>
__device__ __forceinline__ u32x4 decode_eight_in_order(const u32x4 *raw, int q)
{
    u32 d[4];
    decode_eight<FMT>(raw, q, d);                        // (k0,k2), (k1,k3), (k4,k6), (k5,k7)
    return u32x4{__builtin_amdgcn_perm(d[1], d[0], 0x05040100u), __builtin_amdgcn_perm(d[1], d[0], 0x07060302u),
                 __builtin_amdgcn_perm(d[3], d[2], 0x05040100u), __builtin_amdgcn_perm(d[3], d[2], 0x07060302u)};
}

template <int FMT_A, int FMT_W, int OUT, int Q, int R>
__global__ __launch_bounds__(kMaxThreads, 4) void conv_few_kernel(const GemmArgs g, const FewArgs f)
{
    using CA = Codec<FMT_A>;
    using CW = Codec<FMT_W>;
    constexpr int BA = CA::BITS, BW = CW::BITS, ACC = CA::ACC_EXP + CW::ACC_EXP;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char *const patch = lds + CB * 32 * f.row_bytes;
    float *const cols = reinterpret_cast<float *>(patch + f.in_rows * f.pitch);

    const int tid = threadIdx.x, threads = (int)blockDim.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), kq = lane >> 5;
    const int part = (int)blockIdx.x % f.parts, walker = (int)blockIdx.x / f.parts, walkers = (int)gridDim.x / f.parts;
    const int n0 = part * (32 * CB), row_codes = g.kw * g.Cin, K = g.kh * row_codes;

    // ---- weights: filter row by filter row, 32 codes each with zeros behind the row's own
    {
        const __amdgpu_buffer_rsrc_t rsrcW = word_descriptor(g.W, g.w_bytes);
        const u32 w_end = (u32)whole_words(g.w_bytes), w_last = last_bytes(g.W, g.w_bytes);
        for (int r = tid; r < CB * 32 * g.kh; r += threads) {
            const int n = r / g.kh, fr = r - n * g.kh;
            const u32 off = n0 + n < g.N ? (u32)(((int64_t)(n0 + n) * K + fr * row_codes) * BW / 8) : kOob;
            u32x4 raw[ragged_regs<BW>()], t[(BW + 3) / 4];
            load_run_bounded<BW>(rsrcW, off, w_end, w_last, raw);
            align_run<BW>(raw, t);
            keep_codes<BW>(t, row_codes);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<u32x4 *>(lds + n * f.row_bytes + fr * 64 + q * 16) = decode_eight_in_order<FMT_W>(t, q);
        }
    }
    bool big = false;
    OutScale os{};
    if constexpr (OUT == OUT_CODES) {
        big = stage_columns<CB, ACC>(g, n0, cols);
        os = out_scale(g);
    }

    // padding left and right of the image, and everything else no run ever writes
    for (int i = tid; i < f.in_rows * f.pitch / 16; i += threads) *reinterpret_cast<u32x4 *>(patch + i * 16) = u32x4{0u, 0u, 0u, 0u};

    // ---- the runs of a unit: 32 codes each, image row by image row
    const __amdgpu_buffer_rsrc_t rsrcA = word_descriptor(g.A, g.a_bytes);
    const int row_runs = (g.Wd * g.Cin + 31) / 32, last_codes = g.Wd * g.Cin - (row_runs - 1) * 32;
    const u32 rdW = (u32)(lane & 31) * (u32)f.row_bytes + (u32)kq * 16;
    struct Unit {
        int b, ho0, rows, hi_first, runs;
    };
    auto unit_of = [&](int unit) {
        Unit u;
        u.b = unit / f.units_per_image;
        u.ho0 = (unit - u.b * f.units_per_image) * f.rows;
        u.rows = min(f.rows, g.Ho - u.ho0);
        u.hi_first = u.ho0 * g.stride - g.pad;
        u.runs = unit < f.units ? ((u.rows - 1) * g.stride + g.kh) * row_runs : 0;
        return u;
    };
    auto run_offset = [&](const Unit &u, int it) {
        const int iy = (int)((u32)it / (u32)row_runs), run = it - iy * row_runs, hi = u.hi_first + iy;
        const bool in = it < u.runs && (unsigned)hi < (unsigned)g.H;   // a row above or below the image: zeros
        return in ? (u32)((u.b * g.H + hi) * g.Wd * g.pix_bytes + run * 4 * BA) : kOob;
    };
    auto fetch = [&](const Unit &u, int it, u32x4 (&raw)[ragged_regs<BA>()]) { load_run_ragged<BA>(rsrcA, run_offset(u, it), raw); };
    auto decode = [&](const Unit &u, int it, u32x4 (&raw)[ragged_regs<BA>()]) {
        const int iy = (int)((u32)it / (u32)row_runs), run = it - iy * row_runs;
        if (g.a_bytes & 3) {                                           // the tensor ends inside a word: the lanes whose runs hold its last bytes
            const u32 off = run_offset(u, it), end = (u32)whole_words(g.a_bytes);
            if (end - (off & ~3u) <= 4u * BA) join_last_bytes<BA>(off, end, last_bytes(g.A, g.a_bytes), raw);
        }
        u32x4 t[(BA + 3) / 4];
        align_run<BA>(raw, t);
        if (last_codes != 32 && run == row_runs - 1) keep_codes<BA>(t, last_codes);   // behind the image: the next row
        char *o = patch + iy * f.pitch + (g.pad * g.Cin + run * 32) * 2;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const u32x4 d = decode_eight_in_order<FMT_A>(t, q);
            *reinterpret_cast<uint2 *>(o + q * 16) = make_uint2(d.x, d.y);            // pad Cin is a multiple of four: 8-byte aligned
            *reinterpret_cast<uint2 *>(o + q * 16 + 8) = make_uint2(d.z, d.w);
        }
    };

    float run_max = 0.0f;
    u32x4 ahead[ragged_regs<BA>()];                                    // the thread's run of the next unit, fetched while this one's strips are computed
    fetch(unit_of(walker), tid, ahead);
    for (int unit = walker; unit < f.units; unit += walkers) {
        const Unit u = unit_of(unit);
        const int b = u.b, ho0 = u.ho0, rows = u.rows;
        // ---- the unit's input rows, decoded
        __syncthreads();                                               // the previous unit's fragments have been read (first: weights and zeros are written)
        if (tid < u.runs) decode(u, tid, ahead);
        for (int it = tid + threads; it < u.runs; it += threads) {
            u32x4 raw[ragged_regs<BA>()];
            fetch(u, it, raw);
            decode(u, it, raw);
        }
        fetch(unit_of(unit + walkers), tid, ahead);
        __syncthreads();

        // ---- strips of 32 output pixels, consecutive in the output
        const int outputs = rows * g.Wo;
        const int64_t m_unit = ((int64_t)b * g.Ho + ho0) * g.Wo;
        for (int s = wave * 32; s < outputs; s += (threads >> 6) * 32) {
            const int i = min(s + (lane & 31), outputs - 1);           // past the unit: repeats its last pixel, not stored
            const int y = (int)((u32)i / (u32)g.Wo), x = i - y * g.Wo;
            const char *a = patch + y * g.stride * f.pitch + x * g.stride * g.Cin * 2 + kq * 16;
            const char *w = lds + rdW;
            f32x16 acc[CB];
            auto filter_row = [&](auto first) {                        // the first adds to a constant zero
#pragma unroll
                for (int h = 0; h < 2; ++h) {                          // 16 codes of the filter row
                    const f16x8 fa = *reinterpret_cast<const f16x8 *>(a + h * 32);
#pragma unroll
                    for (int j = 0; j < CB; ++j) {
                        const f16x8 fw = *reinterpret_cast<const f16x8 *>(w + h * 32 + j * 32 * f.row_bytes);
                        const f32x16 c = decltype(first)::value && h == 0 ? f32x16{} : acc[j];
                        acc[j] = OUT == OUT_CODES ? __builtin_amdgcn_mfma_f32_32x32x16_f16(fw, fa, c, 0, 0, 0)
                                                  : __builtin_amdgcn_mfma_f32_32x32x16_f16(fa, fw, c, 0, 0, 0);
                    }
                }
                a += f.pitch;
                w += 64;
            };
            int fr = 0;
            if constexpr (OUT == OUT_CODES) {
                filter_row(std::true_type{});
                fr = 1;
            } else {                                                   // a second copy of the loop's body costs this epilogue up to 1.39 times the time
#pragma unroll
                for (int j = 0; j < CB; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[j][v] = 0.0f;
            }
            for (; fr < g.kh; ++fr) filter_row(std::false_type{});
            GemmArgs ge = OUT == OUT_CODES && R != 0 ? reload_args() : g;   // kept over the loop, a shortcut's fill the scalar registers
            ge.M = m_unit + outputs;                                   // the epilogue stores no row past the unit
            if constexpr (OUT == OUT_CODES) run_max = fmaxf(run_max, epilogue_strip_codes<CB, ACC, Q, R>(ge, acc, m_unit + s, n0, cols, big, os));
            else run_max = fmaxf(run_max, epilogue_strip<CB, false, false, ACC>(ge, acc, m_unit + s, n0));
        }
    }

    if (g.absmax_bits) {                                               // one merge per workgroup (see gemm_ws.hip)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) run_max = fmaxf(run_max, __shfl_xor(run_max, off, 64));
        __syncthreads();
        float *red = reinterpret_cast<float *>(lds);
        if (lane == 0) red[wave] = run_max;
        __syncthreads();
        if (tid == 0) {
            float mx = red[0];
            for (int w = 1; w < threads >> 6; ++w) mx = fmaxf(mx, red[w]);
            const uint32_t bits = __float_as_uint(mx);
            if (bits > __hip_atomic_load(g.absmax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(g.absmax_bits, bits);
        }
    }
}

// Unit size: output rows and waves for which the modelled time is least.  A compute unit spends about 500 vector
// instructions on a strip (with the codes-only epilogue) and 130 on 64 runs of 32 codes, issued at full rate by 16 waves (128
// registers) and in proportion by fewer; each round of units the device holds at once (as many workgroups per compute unit as
// their LDS allows) waits for its loads, barriers and last strips for about as long as 6000 of them take.
static bool plan(const GemmArgs &g, FewArgs &f, int &waves, int &lds_bytes, int &resident)
{
    f.parts = (int)((g.N + 32 * CB - 1) / (32 * CB));
    f.row_bytes = g.kh * 64 + 16;
    const int taps = 32 / g.Cin;
    int64_t in_cols = (int64_t)(g.Wo - 1) * g.stride + taps;
    const int64_t written = g.pad + ((int64_t)g.Wd * g.Cin + 31) / 32 * 32 / g.Cin;   // the last run of a row may reach past the image
    if (in_cols < written) in_cols = written;
    if (in_cols * g.Cin * 2 > kLdsLimit) return false;               // no row fits the LDS (padding and stride reach 2^31)
    f.in_cols = (int)in_cols;
    f.pitch = (f.in_cols * g.Cin * 2 + 15) / 16 * 16;
    const int64_t fixed = (int64_t)CB * 32 * f.row_bytes + (kOut == OUT_CODES ? column_bytes<CB>() : 0);
    double best = 0;
    for (int r = 1; r <= 16 && r <= g.Ho; ++r) {
        const int64_t in_rows = (int64_t)(r - 1) * g.stride + g.kh, bytes = fixed + in_rows * f.pitch;
        if (bytes > kLdsLimit) break;
        for (int wv = 4; wv <= 8; ++wv) {
            const int by_lds = (int)(160 * 1024 / (bytes + 160 * 1024 - kLdsLimit)), per_cu = by_lds < 16 / wv ? by_lds : 16 / wv;
            const int rounds = ((r * g.Wo + 31) / 32 + wv - 1) / wv;
            const int64_t units = g.M / ((int64_t)g.Ho * g.Wo) * ((g.Ho + r - 1) / r) * f.parts;
            const double work = rounds * wv * 500.0 + (double)in_rows * f.in_cols * g.Cin / 32 * 130 / 64;
            const double t = (double)((units + 256 * per_cu - 1) / (256 * per_cu)) * (work * 16 / wv + 6000);
            if (best == 0 || t < best) {
                best = t;
                f.rows = r;
                f.in_rows = (int)in_rows;
                waves = wv;
                lds_bytes = (int)bytes;
                resident = 256 * per_cu;
            }
        }
    }
    if (best == 0) return false;
    f.units_per_image = (g.Ho + f.rows - 1) / f.rows;
    const int64_t units = g.M / ((int64_t)g.Ho * g.Wo) * f.units_per_image;
    if (units > 0x3fffffff) return false;
    f.units = (int)units;
    return true;
}

template <int FA, int FW>
static bool launch(const GemmArgs &g, hipStream_t st)
{
    FewArgs f{};
    int waves = 0, lds_bytes = 0, resident = 0;
    if (!plan(g, f, waves, lds_bytes, resident)) return false;
    int walkers = resident / f.parts;
    if (walkers < 1) walkers = 1;
    if (walkers > f.units) walkers = f.units;
    // codes: a kernel per form of them.  One with all forms computes the uniform values of each of them
    // and keeps them in vector registers: 64 x 224 x 224 at 8 bits to 4-bit codes 31.1 -> 27.4 us; with a shortcut, 77 calls, 0.94 times the time
    // (and 0.96 of that with the arguments read again for each strip: 25088 outputs, 4 x 4 taps of 4 to 128, 19.0 -> 15.8)
    auto k = [&] {
        if constexpr (kOut == OUT_CODES) return kernel_for_codes(g, [](auto q, auto r) { return conv_few_kernel<FA, FW, kOut, q(), r()>; });
        else return conv_few_kernel<FA, FW, kOut, 0, 0>;
    }();
    note_kernel(DYBIT_KERNEL_F16_FEW);
    note_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit));
    hipLaunchKernelGGL(k, dim3((unsigned)(walkers * f.parts)), dim3(64 * waves), lds_bytes, st, g, f);
    return true;
}

}  // namespace few

#define DYBIT_FEW_NAME2(w) DYBIT_WB_NAME(launch_conv_few_w##w)
#define DYBIT_FEW_NAME(w) DYBIT_FEW_NAME2(w)
bool DYBIT_FEW_NAME(DYBIT_FEW_W)(const GemmArgs &g, int a_bits, hipStream_t st)
{
    using namespace fast;
    const int fa = (a_bits == 8 ? F8S : a_bits == 6 ? F6S : F4S) + (g.a_signed ? 0 : 1);
    switch (fa) {
        case F4S: return few::launch<F4S, DYBIT_FEW_W>(g, st);
        case F4U: return few::launch<F4U, DYBIT_FEW_W>(g, st);
        case F6S: return few::launch<F6S, DYBIT_FEW_W>(g, st);
        case F6U: return few::launch<F6U, DYBIT_FEW_W>(g, st);
        case F8S: return few::launch<F8S, DYBIT_FEW_W>(g, st);
        case F8U: return few::launch<F8U, DYBIT_FEW_W>(g, st);
        default: return false;
    }
}

}  // namespace dybit
