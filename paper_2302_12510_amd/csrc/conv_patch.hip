// Convolution of 64 and more channels with its input decoded once: the 3 x 3 layers of a residual network.
//
// An implicit-GEMM kernel decodes an input code again for every filter tap (nine times for 3 x 3) and every column tile, and
// stages decoded weights through LDS behind a barrier per K step.  Here the operands change places.  The pixels that a
// workgroup's outputs look at are one range of the image, pixel after pixel (for every stride, as long as no output reaches
// past the image with its first taps, which the dispatcher checks); they are decoded into LDS once, all channels, as e4m3
// bytes (pairs of 4- and 2-bit formats) or as halves, and every tap reads its fragments of A from there, a tap outside the
// image from one pixel of zeros.  The weights never touch LDS: wave (rw, g, cw) owns 128 outputs x 32 channels, and a lane
// decodes the codes of its own channel, two K steps ahead, for the four matrix instructions that use each fragment.  The K loop
// has no barrier.  Two k-groups (kg = 2) halve a serial loop where there are few tiles: each wave gives half of its four
// accumulators to its partner through LDS and stores the other half.
//
// Per matrix instruction: one fragment read from LDS (128 B per clock and compute unit at the full matrix rate, half of what
// the LDS delivers) and, for 4-bit weights, 10 (e4m3) or 4 (fp16) vector instructions against 33 in gemm_f8.hip.  What bounds it:
// of the 30000 cycles of 64 x 14 x 14 x 256 -> 256 with a 4-bit pair 15000 are the K loop (9200 matrix cycles per SIMD), the rest is
// waiting for the first loads, decoding the patch, joining and storing; at N = 64 the encoder of the epilogue.  Loads of all
// constants and the set-up of the lanes' outputs lie between the patch's loads and their use (18.2 -> 15.7 us), and nothing before those loads
// waits twice for arguments, or for other loads (15.7 -> 15.2).
// The kernels it replaces -> this one (us; fp32 or codes out): 64 x 14 x 14 x 256, 4-bit pair 22.8 -> 15.5, 8-bit 25.4 -> 21.4;
// 64 x 7 x 7 x 512 25.8 -> 15.6 and 41.3 -> 25.4; 64 x 28 x 28 x 128 19.8 -> 16.4 and 25.0 -> 22.0; 64 x 56 x 56 x 64 25.7 -> 22.9.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "codes_epilogue.h"
#include "dybit_codec.h"
#include "dybit_codec8.h"
#include "gemm_args.h"
#include "tile_common.h"
#include "tile_epilogue.h"

#ifndef DYBIT_PATCH_W
#error "compile with -DDYBIT_PATCH_W=<weight format id> (0: 4-bit, 2: 8-bit, 4: 6-bit, 6: 2-bit; signed)"
#endif

namespace dybit {
namespace patch {

using namespace fast;
using f8::i32x8;

constexpr int RB = 4;                                    // row blocks of 32 per wave
constexpr int kMaxCols = 256;                            // columns of a workgroup, at most
constexpr int kExchange = 2 * 16 * 64 * 4;               // LDS bytes a wave hands to its partner (two accumulators)

struct PatchArgs {
    int rw, cw_log, kg_log;                              // waves of a workgroup: strips of 128 rows; of 32 columns and k-groups, as powers of two
    int tiles;
    int pitch, zero_at, cols_at;                         // LDS: bytes per pixel, the pixel of zeros, the columns' factors (and a word for the maximum)
    int a_fmt, threads;
    uint32_t run_bytes;                                  // of 32 codes of A
    uint32_t runs_magic;                                 // ceil(2^32 / runs of 32 codes per pixel)
    uint32_t row_bits;                                   // the first tap of every filter row
    Divisor wo, ho, tiles_n;
    int second_step, second_tap, second_block, second_fr, second_fs;   // where the second k-group begins
};
constexpr int kColumnBytes = 2 * kMaxCols * 4;
constexpr int kLds = 160 * 1024 - 256;                   // what a launch may ask for: the codes-only kernels hold 256 bytes themselves (__syncthreads_or)

// First tap of output pixel m (M and the image's pixels are below 2^31).
struct Origin {
    int hi0, wi0, pixel;
};
__device__ __forceinline__ Origin origin(const GemmArgs &g, const PatchArgs &p, u32 m)
{
    const u32 row = quotient(m, p.wo), b = quotient(row, p.ho);
    Origin o;
    o.hi0 = (int)(row - b * (u32)g.Ho) * g.stride - g.pad;
    o.wi0 = (int)(m - row * (u32)g.Wo) * g.stride - g.pad;
    o.pixel = ((int)b * g.H + o.hi0) * g.Wd + o.wi0;
    return o;
}

// Bits [lo, up) of a word, 0 <= lo, up <= 31 (none for up <= lo).
__device__ __forceinline__ u32 bit_range(int lo, int up) { return up > lo ? (1u << up) - (1u << lo) : 0u; }

// The runs of 32 codes of pixels first .. first + pixels - 1 (those before the tensor or behind it read as zeros), which the
// workgroup's threads take in turn, kBatch at a time.
constexpr int kBatch = 4;
struct Runs {
    int first, count, per_pixel, threads;
    u32 magic, pix_bytes, bytes;                         // bytes: of a run
};
// One sequence of instructions for all formats, without branches around the loads: 16 bytes each, and the next 16 where the
// format has them (what a 2- or 6-bit run reads too much stays unused, or is zero behind the tensor).  A variant per format
// made the compiler wait for the weights' loads before the first of these (registers of the variant not taken).
template <int N>
__device__ __forceinline__ void load_batch(const __amdgpu_buffer_rsrc_t rsrcA, const Runs &q, const int r0, u32x4 (&raw)[kBatch][N])
{
    u32 off[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
        const int r = r0 + i * q.threads, px = (int)__umulhi((u32)r, q.magic), at = q.first + px;
        off[i] = ((u32)at * q.pix_bytes + (u32)(r - px * q.per_pixel) * q.bytes) | (r < q.count && at >= 0 ? 0u : kOob);
        raw[i][0] = __builtin_amdgcn_raw_buffer_load_b128(rsrcA, off[i], 0, 0);
    }
    if (N == 2 && q.bytes > 16) {                        // uniform
#pragma unroll
        for (int i = 0; i < kBatch; ++i) raw[i][N - 1] = __builtin_amdgcn_raw_buffer_load_b128(rsrcA, off[i] + 16, 0, 0);
    }
}
// Decodes them into LDS; raw holds the thread's first batch.  fp16: values as they are, not on the 2^-14 scale of the arithmetic
// decoders (a power of two: exact), so that the factor left to the epilogue is that of the weights alone.
template <int FMT, bool F8, int N>
__device__ __forceinline__ void fill(const __amdgpu_buffer_rsrc_t rsrcA, const Runs &q, const int pitch, char *lds, u32x4 (&raw)[kBatch][N])
{
    const int threads = q.threads;
    for (int r0 = threadIdx.x; r0 < q.count; r0 += kBatch * threads) {
        u32x4 ahead[kBatch][N];
        const bool more = r0 - (int)threadIdx.x + kBatch * threads < q.count;   // uniform
        if (more) load_batch(rsrcA, q, r0 + kBatch * threads, ahead);
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int r = r0 + i * threads, px = (int)__umulhi((u32)r, q.magic);
            if (r >= q.count) break;
            char *o = lds + px * pitch + (r - px * q.per_pixel) * (F8 ? 32 : 64);
            if constexpr (F8) {
                const i32x8 f = f8::decode_fragment<FMT, true>(raw[i][0]);
                *reinterpret_cast<u32x4 *>(o) = u32x4{(u32)f[0], (u32)f[1], (u32)f[2], (u32)f[3]};
                *reinterpret_cast<u32x4 *>(o + 16) = u32x4{(u32)f[4], (u32)f[5], (u32)f[6], (u32)f[7]};
            } else {
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    u32 d[4];
                    decode_eight<FMT>(raw[i], h, d);
                    if constexpr (Codec<FMT>::ACC_EXP != 0) {
                        static_assert(Codec<FMT>::ACC_EXP == 14, "scale of the arithmetic decoders");
                        const f16x2 up = {(_Float16)16384.0f, (_Float16)16384.0f};
#pragma unroll
                        for (int v = 0; v < 4; ++v) d[v] = __builtin_bit_cast(u32, __builtin_bit_cast(f16x2, d[v]) * up);
                    }
                    *reinterpret_cast<u32x4 *>(o + h * 16) = u32x4{d[0], d[1], d[2], d[3]};
                }
            }
        }
        if (!more) break;
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
#pragma unroll
            for (int n = 0; n < N; ++n) raw[i][n] = ahead[i][n];
    }
}

// Maximum over the lanes of a wave (non-negative floats order like their bits).
template <int CTRL>
__device__ __forceinline__ u32 max_dpp(u32 v) { return max(v, (u32)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true)); }
__device__ __forceinline__ u32 wave_max(float f)
{
    u32 v = __float_as_uint(f);
    v = max_dpp<0xb1>(v);                                // lanes 1, 0, 3, 2 of each four
    v = max_dpp<0x4e>(v);                                // 2, 3, 0, 1
    v = max_dpp<0x141>(v);                               // mirrored within eight
    v = max_dpp<0x140>(v);                               // mirrored within sixteen
    const u32 a = max((u32)__builtin_amdgcn_readlane((int)v, 0), (u32)__builtin_amdgcn_readlane((int)v, 16));
    const u32 b = max((u32)__builtin_amdgcn_readlane((int)v, 32), (u32)__builtin_amdgcn_readlane((int)v, 48));
    return max(a, b);
}

// fp32 results of 32 `blocks` rows x 32 columns.  The shortcut of the first two blocks has been requested before the k-groups
// were joined; that of block b + 2 is requested once block b is computed, before it is stored (see store_strip).  Rows past M
// fall outside the descriptors.
struct Rows {
    __amdgpu_buffer_rsrc_t c, res;
    u32 off, ldc4;
    int rows;
    bool n_ok;
};
__device__ __forceinline__ Rows rows_of(const GemmArgs &g, const int blocks, const int64_t m_first, const int64_t n0)
{
    Rows o;
    const int lane = threadIdx.x & 63;
    const int64_t left = g.M - m_first, n = n0 + (lane & 31);
    o.rows = left <= 0 ? 0 : left < 32 * blocks ? (int)left : 32 * blocks;
    o.ldc4 = (u32)g.ldc * 4u;
    const int64_t m = left <= 0 ? 0 : m_first;
    o.c = __builtin_amdgcn_make_buffer_rsrc(g.C + m * g.ldc, 0, (int)((u32)o.rows * o.ldc4), 0x00020000);
    o.res = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(g.residual ? g.residual + m * g.ldc : g.C), 0, g.residual ? (int)((u32)o.rows * o.ldc4) : 0, 0x00020000);
    o.n_ok = n < g.N;
    o.off = (o.n_ok ? (u32)n * 4u : kOob) + (u32)(4 * (lane >> 5)) * o.ldc4;
    return o;
}
__device__ __forceinline__ void request_rows(const Rows &o, const int b, float (&res)[16])
{
    u32 off = o.off + (u32)(32 * b) * o.ldc4;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        res[v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(o.res, off, 0, 0));
        off += (v & 3) == 3 ? 5u * o.ldc4 : o.ldc4;
    }
}
template <int ACC, bool HAS_RES>
__device__ __forceinline__ float store_rows(const Rows &o, const f32x16 (&acc)[RB], const int blocks, const float alpha, const float bias,
                                            const bool relu, const bool track, float (&res)[2][16])
{
    const int kq = (threadIdx.x & 63) >> 5;
    float mx = 0.0f;
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        if (b >= blocks) break;                          // uniform
        u32 off = o.off + (u32)(32 * b) * o.ldc4;
        float c[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            c[v] = acc_value<ACC>(acc[b][v]) * alpha + bias;
            if (HAS_RES) c[v] += res[b & 1][v];
            if (relu) c[v] = fmaxf(c[v], 0.0f);
            if (track) mx = fmaxf(mx, (o.n_ok && 32 * b + 8 * (v >> 2) + 4 * kq + (v & 3) < o.rows) ? fabsf(c[v]) : 0.0f);
        }
        if (HAS_RES && b + 2 < RB) request_rows(o, b + 2, res[b & 1]);   // past the strip: the descriptor's end
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(c[v]), o.c, off, 0, 2);
            off += (v & 3) == 3 ? 5u * o.ldc4 : o.ldc4;
        }
    }
    return mx;
}

// Codes of 64 rows x 32 columns (two blocks, one above the other).
template <int ACC, int Q, int R>
__device__ __forceinline__ float codes_of_pair(const GemmArgs &g, f32x16 (&acc)[2], const int64_t m_first, const int64_t n0,
                                               const float *cols, const bool big, const OutScale os)
{
    const int64_t left = g.M - m_first;
    const int rows = left <= 0 ? 0 : left < 64 ? (int)left : 64;
    if (ACC != 0 && big) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][v] = acc_value<ACC>(acc[j][v]);
    }
    return strip_codes<2, true, Q, R>(g, acc, m_first, n0, rows, cols, os, kMaxCols);
}

template <int FMT_W, bool F8, int OUT, int Q, int R>
__global__ __launch_bounds__(512, 3) void conv_patch_kernel(const GemmArgs g, const PatchArgs p)
{
    constexpr int PB = F8 ? 1 : 2;                       // LDS bytes per code
    constexpr int BW = Codec<FMT_W>::BITS, NW = (BW + 3) / 4, RUN_W = 4 * BW, ACC = F8 ? 0 : Codec<FMT_W>::ACC_EXP;
    using Frag = typename std::conditional<F8, i32x8, f16x8>::type;
    extern __shared__ __attribute__((aligned(16))) char lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), kq = lane >> 5;
    // every argument that is needed before the first loads, read at once: the compiler otherwise reads them in five steps that wait for each other
    asm volatile("" ::"s"(g.M), "s"(g.N), "s"(g.K), "s"(g.A), "s"(g.W), "s"(g.a_bytes), "s"(g.w_bytes), "s"(g.a_scale), "s"(g.w_scale), "s"(g.bias));
    asm volatile("" ::"s"(g.H), "s"(g.Wd), "s"(g.Cin), "s"(g.Ho), "s"(g.Wo), "s"(g.kh), "s"(g.kw), "s"(g.stride), "s"(g.pad), "s"(g.pix_bytes), "s"(g.w_per_channel));
    asm volatile("" ::"s"(p.threads), "s"(p.run_bytes), "s"(p.runs_magic), "s"(p.pitch), "s"(p.tiles), "s"(p.rw), "s"(p.cw_log), "s"(p.kg_log), "s"(p.second_step));
    const int cw = 1 << p.cw_log, kg = 1 << p.kg_log;
    const int cwi = wave & (cw - 1), kgp = (wave >> p.cw_log) & (kg - 1), rwi = wave >> (p.cw_log + p.kg_log);
    const int tile = xcd_contiguous_index();             // all column tiles of a strip of rows together
    if (tile >= p.tiles) return;                         // uniform per workgroup
    const int tile_m = (int)quotient((u32)tile, p.tiles_n), tile_n = tile - tile_m * (int)p.tiles_n.d;
    const int64_t m0 = (int64_t)tile_m * (32 * RB * p.rw), m_wave = m0 + rwi * (32 * RB);
    const int64_t n_tile = (int64_t)tile_n * (32 * cw), n0 = n_tile + cwi * 32;

    // ---- weights: this k-group's K steps of 64 codes, the first ones requested before anything else
    const int s0 = kgp ? p.second_step : 0, s1 = kgp || kg == 1 ? (int)(g.K / 64) : p.second_step;
    const __amdgpu_buffer_rsrc_t rsrcW = code_descriptor(g.W, g.w_bytes);
    const int64_t n_lane = n0 + (lane & 31);
    u32 offW = n_lane < g.N ? (u32)((u32)n_lane * (u32)(g.K * BW / 8) + (u32)(s0 * 2 * RUN_W + kq * RUN_W)) : kOob;
    auto load_W = [&](u32x4 (&raw)[NW]) {                // past the last step: read and not used
        load_run<BW>(rsrcW, offW, raw);
        offW += 2 * RUN_W;
    };
    constexpr int AHEAD = F8 ? 4 : 2;                    // K steps whose codes are in registers or on their way
    u32x4 rawW[AHEAD][NW];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) load_W(rawW[i]);

    // ---- the image's pixels that the tile looks at: first codes requested
    const int64_t m_end = m0 + 32 * RB * p.rw < g.M ? m0 + 32 * RB * p.rw : g.M;
    const int first = origin(g, p, (u32)m0).pixel, pixels = origin(g, p, (u32)(m_end - 1)).pixel - first + (g.kh - 1) * g.Wd + g.kw;
    const Runs runs{first, pixels * (g.Cin / 32), g.Cin / 32, p.threads, p.runs_magic, (u32)g.pix_bytes, p.run_bytes};
    const __amdgpu_buffer_rsrc_t rsrcA = code_descriptor(g.A, g.a_bytes);
    u32x4 raw[kBatch][F8 ? 1 : 2];
    load_batch(rsrcA, runs, tid, raw);

    // ---- factors and biases: of the lane's column, or (codes only) of the tile's columns, a thread each
    const int64_t n_own = OUT == OUT_CODES ? n_tile + tid : n_lane;
    const bool n_ok = n_own < g.N;
    const float a_scale = scalar_scale(g.a_scale), w_scale = g.w_scale[g.w_per_channel && n_ok ? n_own : 0];   // no branch, used behind the set-up
    const float bias_read = g.bias ? g.bias[n_ok ? n_own : 0] : 0.0f;

    // ---- the lane's outputs: where their first taps lie in LDS, and which taps lie inside the image
    const u32 lds_base = (u32)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    u32 base[RB], inside[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        const int64_t m = m_wave + 32 * r + (lane & 31);
        const bool ok = m < g.M;
        const Origin o = origin(g, p, ok ? (u32)m : (u32)m0);
        const u32 columns = bit_range(max(0, -o.wi0), min(g.kw, g.Wd - o.wi0));
        const u32 rows = bit_range(max(0, -o.hi0) * g.kw, min(g.kh, g.H - o.hi0) * g.kw) & p.row_bits;
        base[r] = lds_base + (u32)((o.pixel - first) * p.pitch + kq * (32 * PB));
        inside[r] = ok ? columns * rows : 0u;            // the columns' bits, once per row
    }
    const int blocks_of_tap = g.Cin / 64;
    int tap = kgp ? p.second_tap : 0, block = kgp ? p.second_block : 0, fr = kgp ? p.second_fr : 0, fs = kgp ? p.second_fs : 0;   // the step whose A is read next
    const int steps = (n0 < g.N && m_wave < g.M) ? s1 - s0 : 0;

    __builtin_amdgcn_sched_barrier(0);
    const float factor = n_ok ? a_scale * w_scale : 0.0f, bias = n_ok ? bias_read : 0.0f;

    // ---- the pixels, decoded
    float *const cols = reinterpret_cast<float *>(lds + p.cols_at);
    u32 *const top = reinterpret_cast<u32 *>(lds + p.cols_at + (OUT == OUT_CODES ? kColumnBytes : 0));
    if (tid == 0) *top = 0;
    for (int i = tid * 16; i < p.pitch; i += p.threads * 16) *reinterpret_cast<u32x4 *>(lds + p.zero_at + i) = u32x4{0u, 0u, 0u, 0u};
    switch (p.a_fmt) {                                   // uniform
        case F4S: fill<F4S, F8>(rsrcA, runs, p.pitch, lds, raw); break;
        case F4U: fill<F4U, F8>(rsrcA, runs, p.pitch, lds, raw); break;
        case F2S: fill<F2S, F8>(rsrcA, runs, p.pitch, lds, raw); break;
        case F2U: fill<F2U, F8>(rsrcA, runs, p.pitch, lds, raw); break;
        default:
            if constexpr (!F8) {
                if (p.a_fmt == F8S) fill<F8S, F8>(rsrcA, runs, p.pitch, lds, raw);
                else if (p.a_fmt == F8U) fill<F8U, F8>(rsrcA, runs, p.pitch, lds, raw);
                else if (p.a_fmt == F6S) fill<F6S, F8>(rsrcA, runs, p.pitch, lds, raw);
                else fill<F6U, F8>(rsrcA, runs, p.pitch, lds, raw);
            }
    }
    bool big = false;                                    // see stage_columns
    if constexpr (OUT == OUT_CODES) {
        const float up = __uint_as_float((uint32_t)(127 + ACC) << 23);
        big = fabsf(factor) < __builtin_inff() && !(fabsf(factor * up) < __builtin_inff());
        if (tid < 32 * cw) {
            cols[tid] = factor * up;
            cols[kMaxCols + tid] = bias;
        }
    }

    u32 at[RB];
    auto locate = [&](u32 (&a)[RB]) {                    // of the first 64 channels of a tap
        const u32 off = (u32)((fr * g.Wd + fs) * p.pitch), bit = 1u << tap, zero = lds_base + (u32)(p.zero_at + kq * (32 * PB));
#pragma unroll
        for (int r = 0; r < RB; ++r) a[r] = (inside[r] & bit) ? base[r] + off : zero;
    };
    auto advance = [&](const u32 (&a)[RB], u32 (&b)[RB]) {   // the next 64 channels, or the next tap
        if (++block < blocks_of_tap) {                   // uniform
#pragma unroll
            for (int r = 0; r < RB; ++r) b[r] = a[r] + 64 * PB;
            return;
        }
        block = 0;
        ++tap;
        const bool next_row = fs + 1 == g.kw;
        fs = next_row ? 0 : fs + 1;
        fr += next_row ? 1 : 0;
        locate(b);
    };
    auto decode_W = [&](const u32x4 (&raw)[NW], int kk) -> Frag {
        if constexpr (F8) {
            return f8::decode_fragment<FMT_W>(raw[0]);
        } else {
            u32 d[4];
            decode_eight<FMT_W>(raw, kk, d);
            return __builtin_bit_cast(f16x8, u32x4{d[0], d[1], d[2], d[3]});
        }
    };
    auto decode_part = [&](const u32x4 &raw, int r, Frag &f) {   // a quarter of decode_W's fragment (e4m3)
        if constexpr (F8) {
            u32 d[4];
            if constexpr (BW == 2) {
                if (r & 1) return;                       // two words of 16 codes: in every second slot
                f8::Codec8<FMT_W>::word16(r ? raw.y : raw.x, d);
#pragma unroll
                for (int v = 0; v < 4; ++v) f[2 * r + v] = (int)d[v];
            } else {
                f8::Codec8<FMT_W>::word(r == 0 ? raw.x : r == 1 ? raw.y : r == 2 ? raw.z : raw.w, d);
                f[2 * r] = (int)d[0];
                f[2 * r + 1] = (int)d[1];
            }
        }
    };
    typedef __attribute__((address_space(3))) u32x4 LdsWords;
    auto read_A = [&](u32 a, int kk) -> Frag {
        if constexpr (F8) {
            const u32x4 lo = *(const LdsWords *)(uintptr_t)a, hi = *(const LdsWords *)(uintptr_t)(a + 16);
            return i32x8{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
        } else {
            return __builtin_bit_cast(f16x8, *(const LdsWords *)(uintptr_t)(a + kk * 16));
        }
    };
    auto mfma = [&](const Frag &a, const Frag &w, const f32x16 &c) -> f32x16 {
        if constexpr (F8) return OUT == OUT_CODES ? __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(w, a, c, 0, 0, 0, 0, 0, 0)
                                                  : __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, w, c, 0, 0, 0, 0, 0, 0);
        else return OUT == OUT_CODES ? __builtin_amdgcn_mfma_f32_32x32x16_f16(w, a, c, 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_f16(a, w, c, 0, 0, 0);
    };

    f32x16 acc[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[r][v] = 0.0f;
    // Slot r of a weight fragment (its matrix instruction with row block r): the fragment of A two slots on is requested first.
    // The ring of four A fragments is indexed by row block; everything it holds is read by the slot that needs it.
    u32 next[RB];
    locate(at);
#pragma unroll
    for (int r = 0; r < RB; ++r) at[r] += (u32)block * (64 * PB);
    Frag fw = decode_W(rawW[0], 0), fa[RB];
    if constexpr (OUT == OUT_CODES) {
        big = __syncthreads_or(big);                     // the patch is whole
        if (big) {                                       // uniform
            if (tid < 32 * cw) cols[tid] = factor;
            __syncthreads();
        }
    } else {
        __syncthreads();
    }
    fa[0] = read_A(at[0], 0);
    fa[1] = read_A(at[1], 0);
    auto step8 = [&](auto slot_tag) {                    // e4m3: one fragment per K step, a word of the next one decoded per slot
        constexpr int slot = decltype(slot_tag)::value;
        const u32x4 raw = rawW[(slot + 1) % AHEAD][0];
        const Frag w = fw;
        advance(at, next);
        load_W(rawW[slot]);                              // decoded during the step before
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            fa[(r + 2) % RB] = r < 2 ? read_A(at[r + 2], 0) : read_A(next[r - 2], 0);
            acc[r] = mfma(fa[r], w, acc[r]);
            decode_part(raw, r, fw);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) at[r] = next[r];
    };
    auto step16 = [&](auto slot_tag) {                   // fp16: four fragments per K step
        constexpr int slot = decltype(slot_tag)::value;
        advance(at, next);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const Frag w = fw;
            fw = kk < 3 ? decode_W(rawW[slot], kk + 1) : decode_W(rawW[slot ^ 1], 0);
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                fa[(r + 2) % RB] = r < 2 ? read_A(at[r + 2], kk) : kk < 3 ? read_A(at[r - 2], kk + 1) : read_A(next[r - 2], 0);
                acc[r] = mfma(fa[r], w, acc[r]);
            }
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                // DS read
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                // MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, BW == 6 ? 12 : 8, 0); // VALU
            }
            if (kk == 3) load_W(rawW[slot]);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) at[r] = next[r];
    };
    for (int s = 0; s < steps; s += AHEAD) {
        if constexpr (F8) {
            step8(std::integral_constant<int, 0>{});
            if (s + 1 < steps) step8(std::integral_constant<int, 1>{});
            if (s + 2 < steps) step8(std::integral_constant<int, 2>{});
            if (s + 3 < steps) step8(std::integral_constant<int, 3>{});
        } else {
            step16(std::integral_constant<int, 0>{});
            if (s + 1 < steps) step16(std::integral_constant<int, 1>{});
        }
    }

    // ---- what the epilogue waits for: the shortcut, and the maximum so far (an old value costs an atomic, never a wrong result)
    const int blocks = kg == 2 ? RB / 2 : RB;
    const int64_t m_first = m_wave + (kg == 2 && kgp ? 64 : 0);
    Rows out{};
    float res[2][16];
    if constexpr (OUT == OUT_FP32) {
        out = rows_of(g, blocks, m_first, n0);
        if (g.residual) {
            request_rows(out, 0, res[0]);
            request_rows(out, 1, res[1]);
        }
    }
    u32 seen = 0;
    if (g.absmax_bits && tid == 0) seen = __hip_atomic_load(g.absmax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // ---- two k-groups: the wave of group 0 keeps the upper 64 rows, that of group 1 the lower ones
    if (kg == 2) {
        __syncthreads();                                 // every fragment has been read
        float *mine = reinterpret_cast<float *>(lds + wave * kExchange) + lane;
        const float *theirs = reinterpret_cast<const float *>(lds + (kgp ? wave - cw : wave + cw) * kExchange) + lane;
        if (kgp) {                                       // uniform
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) mine[(j * 16 + v) * 64] = acc[j][v];
            acc[0] = acc[2];
            acc[1] = acc[3];
        } else {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) mine[(j * 16 + v) * 64] = acc[j + 2][v];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][v] += theirs[(j * 16 + v) * 64];
    }

    // ---- epilogue
    float mx = 0.0f;
    if (n0 < g.N && m_first < g.M) {
        if constexpr (OUT == OUT_CODES) {
            const OutScale os = out_scale(g);
            f32x16 pair[2] = {acc[0], acc[1]};
#pragma unroll 1
            for (int b = 0; b < blocks; b += 2) {
                mx = fmaxf(mx, codes_of_pair<ACC, Q, R>(g, pair, m_first + 32 * b, n0, cols + cwi * 32, big, os));
                pair[0] = acc[2];
                pair[1] = acc[3];
            }
        } else if constexpr (OUT == OUT_WRITE_BACK) {    // fp32 and codes: a block after the other
            f32x16 one[1] = {acc[0]};
#pragma unroll 1
            for (int b = 0; b < blocks; ++b) {
                mx = fmaxf(mx, epilogue_strip<1, true, false, ACC>(g, one, m_first + 32 * b, n0));
                one[0] = b == 0 ? acc[1] : b == 1 ? acc[2] : acc[3];
            }
        } else {
            const bool relu = g.relu, track = g.absmax_bits != nullptr;
            mx = g.residual ? store_rows<ACC, true>(out, acc, blocks, factor, bias, relu, track, res)
                            : store_rows<ACC, false>(out, acc, blocks, factor, bias, relu, track, res);
        }
    }
    if (g.absmax_bits) {                                 // one merge per workgroup
        const u32 bits = wave_max(mx);
        if (lane == 0) atomicMax(top, bits);
        __syncthreads();
        if (tid == 0 && *top > seen) atomicMax(g.absmax_bits, *top);
    }
}

// The split of a workgroup for which the modelled time (cycles) is least.  A compute unit holds twelve waves (168 registers) and
// the patches that fit its LDS; each round of workgroups it holds at once costs about 9000 cycles of launch, waiting for loads and
// storing, the decoding of the patch, the K loop and the epilogue.  Sharing its SIMD a wave comes to 0.87 of the matrix rate (or
// of the vector rate, where decoding the weights takes longer), alone to 0.56.  Fitted to 56 x 56 x 64 to 7 x 7 x 512 channels.
struct Split {
    int rw, cw, kg, lds_bytes;
    int64_t pixels;
    double cycles;
};
template <int FMT_W, bool F8>
static bool plan(const GemmArgs &g, int pitch, Split &best)
{
    constexpr int kDecode = F8 ? 33 : Codec<FMT_W>::BITS == 6 ? 138 : Codec<FMT_W>::BITS == 8 ? 68 : 48;   // instructions per step
    const double step = F8 ? 256 : 4 * (kDecode + 20) > 512 ? 4 * (kDecode + 20) : 512, steps = (double)g.K / 64;
    best.cycles = 0;
    for (int rw = 1; rw <= 2; ++rw) {
        const int64_t rows = 32 * RB * rw, pixels = strip_pixels(g, rows < g.M ? rows : g.M);
        if ((pixels + 1) * pitch > kLds) break;
        for (int cw = 1; cw <= 8; cw *= 2)
            for (int kg = 1; kg <= 2; ++kg) {
                const int waves = rw * cw * kg;
                if (waves < 4 || waves > 8 || (cw > 1 && g.N <= 16 * cw)) continue;
                const int patch = (int)((pixels + 1) * pitch), exchange = kg == 2 ? waves * kExchange : 0;
                const int lds = (patch > exchange ? patch : exchange) + (kOut == OUT_CODES ? kColumnBytes : 0) + 16;
                if (lds > kLds) continue;
                const int by_lds = 160 * 1024 / (lds + 256), resident = by_lds < 12 / waves ? by_lds : 12 / waves;
                const int64_t tiles = (g.M + rows - 1) / rows * ((g.N + 32 * cw - 1) / (32 * cw)), per_cu = (tiles + 255) / 256;
                auto round = [&](double workgroups) {
                    const double s = workgroups * waves / 4;
                    const double shared = s * steps / kg * step * 1.15, alone = steps / kg * step * 1.8;
                    return 9000.0 + (kg == 2 ? 2500.0 : 0.0) + (double)((pixels * (g.Cin / 32) + 64 * waves - 1) / (64 * waves)) * (F8 ? 320 : 560) * s +
                           (shared > alone ? shared : alone) + 64.0 / kg * 48 * s;
                };
                const double t = (double)(per_cu / resident) * round(resident) + (per_cu % resident ? round((double)(per_cu % resident)) : 0.0);
                if (best.cycles == 0 || t < best.cycles) best = Split{rw, cw, kg, lds, pixels, t};
            }
    }
    return best.cycles != 0;
}

template <int FMT_W, bool F8>
static bool launch(const GemmArgs &g, int a_fmt, hipStream_t st)
{
    PatchArgs p{};
    Split sp;
    p.pitch = g.Cin * (F8 ? 1 : 2) + 16;
    if (!plan<FMT_W, F8>(g, p.pitch, sp)) return false;
    const int cw = sp.cw, kg = sp.kg, waves = sp.rw * cw * kg;
    const int64_t rows = 32 * RB * sp.rw;
    p.rw = sp.rw;
    p.cw_log = cw == 8 ? 3 : cw == 4 ? 2 : cw == 2 ? 1 : 0;
    p.kg_log = kg - 1;
    p.a_fmt = a_fmt;
    p.threads = 64 * waves;
    p.run_bytes = a_fmt >= F2S ? 8 : a_fmt >= F6S ? 24 : a_fmt >= F8S ? 32 : 16;
    p.runs_magic = (uint32_t)((1ull << 32) / (unsigned)(g.Cin / 32) + 1);
    p.wo = divisor((uint32_t)g.Wo);
    p.ho = divisor((uint32_t)g.Ho);
    p.zero_at = (int)(sp.pixels * p.pitch);
    p.cols_at = p.zero_at + p.pitch;
    if (kg == 2 && p.cols_at < waves * kExchange) p.cols_at = waves * kExchange;
    const int64_t tiles_n = (g.N + 32 * cw - 1) / (32 * cw), tiles = (g.M + rows - 1) / rows * tiles_n;
    if (tiles > 0x3fffffff) return false;
    p.tiles = (int)tiles;
    p.tiles_n = divisor((uint32_t)tiles_n);
    for (int f = 0; f < g.kh; ++f) p.row_bits |= 1u << (f * g.kw);
    const int per_tap = g.Cin / 64;
    p.second_step = kg == 2 ? (int)(g.K / 128) : 0;
    p.second_tap = p.second_step / per_tap;
    p.second_block = p.second_step % per_tap;
    p.second_fr = p.second_tap / g.kw;
    p.second_fs = p.second_tap % g.kw;
    auto k = [&] {
        if constexpr (kOut == OUT_CODES) return kernel_for_codes(g, [](auto q, auto r) { return conv_patch_kernel<FMT_W, F8, kOut, q(), r()>; });
        else return conv_patch_kernel<FMT_W, F8, kOut, 0, 0>;
    }();
    note_kernel(F8 ? DYBIT_KERNEL_F8_PATCH : DYBIT_KERNEL_F16_PATCH);
    note_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kLds));
    hipLaunchKernelGGL(k, dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(64 * waves), sp.lds_bytes, st, g, p);
    return true;
}

}  // namespace patch

// One translation unit per weight format; the activation format is an argument of the kernel.
#define DYBIT_PATCH_NAME2(w) DYBIT_WB_NAME(launch_conv_patch_w##w)
#define DYBIT_PATCH_NAME(w) DYBIT_PATCH_NAME2(w)
bool DYBIT_PATCH_NAME(DYBIT_PATCH_W)(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st)
{
    using namespace fast;
    const int fa = (a_bits == 8 ? F8S : a_bits == 6 ? F6S : a_bits == 2 ? F2S : F4S) + (g.a_signed ? 0 : 1);
#if DYBIT_PATCH_W == 0 || DYBIT_PATCH_W == 6
    if (low_pair) return patch::launch<DYBIT_PATCH_W, true>(g, fa, st);
#endif
    return patch::launch<DYBIT_PATCH_W, false>(g, fa, st);
}

}  // namespace dybit
