// Depthwise convolution on DyBit codes for gfx950 (the layer type of the depthwise-separable
// network of Sec. IV): Y[b,ho,wo,c] = sA sW sum_{r,s} x[b,hi,wi,c] w[r,s,c] (+ bias[c]) (ReLU).
//
// Nine multiply-adds per output and no contraction over channels: this is not matrix-core work.  With fp32 results the bound is
// their 4 bytes each, as long as the vector instructions per output stay few.
//
// 3 x 3 filters at stride 1 and 2 (dw3_kernel): no LDS and no barrier.  A thread owns four neighbouring channels of a strip of
// output rows, four columns wide (two at stride 2).  It reads the codes of its input rows itself -- a quad of codes is
// one load, neighbouring threads share the lines -- decodes two quads at a time in registers (dybit_codec.h) and keeps a window
// of three input rows and the taps as fp16; the multiply-adds read the halves directly (v_fma_mix_f32: the product of
// two halves is exact, so the sums are those of fp32 operands).  The next row's codes load while a row is
// computed.  A staged patch (codes -> table of values in LDS -> fp32 window) took 36 lane-instructions per output and two
// barriers per 128 pixels; this takes 18.  64 x 56 x 56 x 144, 4-bit, fp32 results: 41.0 -> 28.5 us (115 MB written); 8-bit
// 52.0 -> 28.9; codes alone 49.2 -> 31.4; stride 2 28.1 -> 12.1; one image of 7 x 7 x 960 4.6 -> 4.2.
// Every other geometry (dwconv_kernel): a workgroup decodes a patch for 8 x 8 output pixels of 32 channels through a table of the
// format's values into LDS as fp32 and walks over it with run-time bounds.  Image, filter and output are channel-innermost,
// so global loads and stores (float4) are contiguous per pixel.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "dybit_codec.h"
#include "dybit_device.h"
#include "dybit_host.h"
#include "gemm_args.h"
#include "requant.h"

namespace dybit {
namespace {

constexpr int kThreads = 256;
constexpr int TH = 8, TW = 8, CG = 32;             // dwconv_kernel: output patch and channel group of a workgroup
constexpr int kMaxLdsBytes = 64 * 1024;
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct DwArgs {
    const uint32_t *X, *Wt;                        // packed codes, read as whole words
    const float *x_scale, *w_scale, *bias;
    float *Y;                                      // may be NULL when q_out is given
    uint32_t *absmax_bits;
    int w_per_channel;                             // w_scale holds one value per channel
    uint8_t *q_out;                                // optional write-back as DyBit codes, packed along C like the image
    const float *q_scale;
    int q_bits, q_signed;
    int *async_error;
    int B, H, W, C, Ho, Wo, kh, kw, stride, pad, relu;
    int a_bits, a_signed, w_bits, w_signed;
    int tiles_h, tiles_w, groups;
    int images, rows;                              // dw3_kernel: images of a grid row, output rows of a thread (tiles_h = strips, tiles_w = column groups)
    int pad_top;                                   // dw3_kernel: padding above the image (pad, but for the later bands of a large image)
};

// Scale, bias, ReLU, maximum and the stores of four neighbouring channels; elem is the index of the first.
// The four codes of a write-back are 16 bits (4-bit formats) or one word (8-bit formats) of the packed pixel.
__device__ __forceinline__ void finish_quad(const DwArgs &a, const Requant &rq, const f32x4 acc, const f32x4 alpha, const f32x4 bv,
                                            float &mx, int64_t elem)
{
    f32x4 y;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        y[u] = acc[u] * alpha[u] + bv[u];
        if (a.relu) y[u] = fmaxf(y[u], 0.0f);
        mx = fmaxf(mx, fabsf(y[u]));
    }
    if (a.Y) __builtin_nontemporal_store(y, reinterpret_cast<f32x4 *>(a.Y + elem));
    if (a.q_out && rq.ok) {
        uint32_t zb[4], code[4], key = ~0u;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            zb[u] = requant_rounded(y[u], rq);
            key = min(key, requant_settle_key(zb[u]));
            code[u] = requant_magnitude(zb[u], rq);
        }
        if (__builtin_amdgcn_ballot_w64(key == 0u)) {             // some value of the wave on a decision point: rare
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (requant_needs_settling(zb[u])) code[u] = requant_settle(y[u], code[u], rq);
        }
        if (rq.is_signed) {
#pragma unroll
            for (int u = 0; u < 4; ++u) code[u] = requant_with_sign(code[u], y[u], rq);
        }
        const uint32_t w = ((code[3] << a.q_bits | code[2]) << a.q_bits | code[1]) << a.q_bits | code[0];
        if (a.q_bits == 8) *reinterpret_cast<uint32_t *>(a.q_out + elem) = w;
        else *reinterpret_cast<uint16_t *>(a.q_out + (elem >> 1)) = (uint16_t)w;
    }
}

// ---- 3 x 3 filters at stride 1 and 2 -------------------------------------------------------------
constexpr int cols_of(int stride) { return stride == 1 ? 4 : 2; }    // output columns of a thread (four at stride 2 do not fit 128 registers)
constexpr uint32_t kRowOob = 0x40000000u;          // row and column offsets past the end: their sums stay past it and below 2^32
using fast::u32;

template <int FMT>
__device__ __forceinline__ u32 load_quad(const __amdgpu_buffer_rsrc_t rsrc, u32 off)        // four codes in the low bits
{
    if constexpr (fast::Codec<FMT>::BITS == 8) return __builtin_amdgcn_raw_buffer_load_b32(rsrc, off, 0, 0);
    else if constexpr (fast::Codec<FMT>::BITS == 4) return __builtin_amdgcn_raw_buffer_load_b16(rsrc, off, 0, 0);
    else return __builtin_amdgcn_raw_buffer_load_b8(rsrc, off, 0, 0);
}

// The quads of two pixels -> fp16: d[0], d[1] = channels (0,2), (1,3) of the first, d[2], d[3] of the second.
template <int FMT>
__device__ __forceinline__ void decode_quads(u32 q0, u32 q1, u32 *d)
{
    if constexpr (fast::Codec<FMT>::BITS == 8) fast::Codec<FMT>::two_words(q0, q1, d);
    else if constexpr (fast::Codec<FMT>::BITS == 4) fast::Codec<FMT>::word(q0 | (q1 << 16), d);
    else fast::Codec<FMT>::half_word(q0 | (q1 << 8), d);
}

// acc + x[X] * w[X] with the halves X of two registers, converted inside the multiply-add (the compiler keeps converted copies
// of every value instead, 108 registers).  FIRST: acc is 0.
template <int X, bool FIRST>
__device__ __forceinline__ float fma_half(u32 x, u32 w, float acc)
{
    if constexpr (FIRST) {
        if constexpr (X) asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,1,0] op_sel_hi:[1,1,0]" : "=v"(acc) : "v"(x), "v"(w));
        else asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[1,1,0]" : "=v"(acc) : "v"(x), "v"(w));
    } else {
        if constexpr (X) asm("v_fma_mix_f32 %0, %1, %2, %0 op_sel:[1,1,0] op_sel_hi:[1,1,0]" : "+v"(acc) : "v"(x), "v"(w));
        else asm("v_fma_mix_f32 %0, %1, %2, %0 op_sel_hi:[1,1,0]" : "+v"(acc) : "v"(x), "v"(w));
    }
    return acc;
}

// Wait states between the decoders' packed instructions and asm that reads their results (which the compiler does not see into).
__device__ __forceinline__ void settle(u32 (*px)[2], int n)
{
    for (int p = 0; p < n; ++p) asm volatile("" : "+v"(px[p][0]), "+v"(px[p][1]));
    asm volatile("s_nop 1" ::: "memory");
    for (int p = 0; p < n; ++p) asm volatile("" : "+v"(px[p][0]), "+v"(px[p][1]));
}

template <int FA, int FW, int S>
__global__ __launch_bounds__(kThreads, 4) void dw3_kernel(const DwArgs a)
{
    constexpr int BA = fast::Codec<FA>::BITS, BW = fast::Codec<FW>::BITS;
    constexpr int DW = cols_of(S), NP = (DW - 1) * S + 3;                          // input columns of a thread
    constexpr float kExp = (float)(1u << fast::Codec<FA>::ACC_EXP) * (float)(1u << fast::Codec<FW>::ACC_EXP);
    const int b_first = blockIdx.y * a.images;                    // first image of this grid row, images in it
    const int images = min(a.images, a.B - b_first);
    const int quads = a.C / 4;
    int id = blockIdx.x * kThreads + threadIdx.x;
    const int quad = id % quads; id /= quads;
    const int colg = id % a.tiles_w; id /= a.tiles_w;
    const int strip = id % a.tiles_h;
    const int b = id / a.tiles_h;
    const bool live = b < images;
    const int c = quad * 4, wo = colg * DW, ho = strip * a.rows;
    const u32 pix_bytes = a.C * BA / 8, row_bytes = a.W * pix_bytes, image_bytes = a.H * row_bytes;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(reinterpret_cast<const uint8_t *>(a.X)) + (int64_t)b_first * image_bytes, 0, images * image_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.Wt), 0, 9u * a.C * BW / 8, 0x00020000);

    u32 col_off[NP];                                              // a column outside the image reads zeros: code 0 is 0.0
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int wi = wo * S - a.pad + p;
        col_off[p] = (live && (unsigned)wi < (unsigned)a.W) ? wi * pix_bytes + c * BA / 8 : fast::kOob;
    }
    int hi = ho * S - a.pad_top;                                  // next input row to read
    auto load_row = [&](u32 *raw) {
        const u32 row = (unsigned)hi < (unsigned)a.H ? b * image_bytes + hi * row_bytes : kRowOob;
#pragma unroll
        for (int p = 0; p < NP; ++p) raw[p] = load_quad<FA>(rx, row + col_off[p]);
        ++hi;
    };
    auto decode_row = [&](const u32 *raw, u32 (*px)[2]) {
#pragma unroll
        for (int p = 0; p < NP; p += 2) {
            u32 d[4];
            decode_quads<FA>(raw[p], p + 1 < NP ? raw[p + 1] : 0u, d);
            px[p][0] = d[0]; px[p][1] = d[1];
            if (p + 1 < NP) { px[p + 1][0] = d[2]; px[p + 1][1] = d[3]; }
        }
        settle(px, NP);
    };
    u32 win[3][NP][2], raw[3][NP];
#pragma unroll
    for (int r = 0; r < 3; ++r) load_row(raw[r]);
    u32 taps[10][2];
    {
        u32 wr[10];
#pragma unroll
        for (int t = 0; t < 9; ++t) wr[t] = load_quad<FW>(rw, live ? (t * a.C + c) * BW / 8 : fast::kOob);
        wr[9] = 0;
#pragma unroll
        for (int t = 0; t < 10; t += 2) {
            u32 d[4];
            decode_quads<FW>(wr[t], wr[t + 1], d);
            taps[t][0] = d[0]; taps[t][1] = d[1]; taps[t + 1][0] = d[2]; taps[t + 1][1] = d[3];
        }
        settle(taps, 9);
    }
    f32x4 alpha, bv = {0.f, 0.f, 0.f, 0.f};
    {
        const float sx = *a.x_scale;
#pragma unroll
        for (int u = 0; u < 4; ++u) alpha[u] = sx * (a.w_per_channel ? a.w_scale[c + u] : a.w_scale[0]);
        if (a.bias) bv = *reinterpret_cast<const f32x4 *>(a.bias + c);
    }
    Requant rq{};
    const bool wb = a.q_out != nullptr;
    if (wb) {
        rq = make_requant(a.q_scale, a.q_bits, a.q_signed);
        if (!rq.ok && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *a.async_error = DYBIT_ERR_BAD_SCALE;
    }
    float mx = 0.0f;
    int64_t elem = (((int64_t)(b_first + b) * a.Ho + ho) * a.Wo + wo) * a.C + c;
#pragma unroll
    for (int r = 0; r < 3 - S; ++r) decode_row(raw[r], win[r]);
#pragma unroll 1
    for (int i = 0; i < a.rows; ++i) {
#pragma unroll
        for (int r = 3 - S; r < 3; ++r) decode_row(raw[r], win[r]);
        if (i + 1 < a.rows) {                                     // the next row's codes are on their way while this one is computed
#pragma unroll
            for (int r = 3 - S; r < 3; ++r) load_row(raw[r]);
        }
        const bool row_ok = live && ho + i < a.Ho;
#pragma unroll
        for (int j = 0; j < DW; ++j) {
            f32x4 y;
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const u32 *x = win[r][j * S + q], *w = taps[r * 3 + q];
                    if (r + q == 0) y = f32x4{fma_half<0, true>(x[0], w[0], 0.f), fma_half<0, true>(x[1], w[1], 0.f),
                                              fma_half<1, true>(x[0], w[0], 0.f), fma_half<1, true>(x[1], w[1], 0.f)};
                    else y = f32x4{fma_half<0, false>(x[0], w[0], y[0]), fma_half<0, false>(x[1], w[1], y[1]),
                                   fma_half<1, false>(x[0], w[0], y[2]), fma_half<1, false>(x[1], w[1], y[3])};
                }
            if (kExp != 1.0f) y *= kExp;                          // the decoders' power of two: exact
            if (row_ok && wo + j < a.Wo) finish_quad(a, rq, y, alpha, bv, mx, elem + j * a.C);
        }
        elem += (int64_t)a.Wo * a.C;
#pragma unroll
        for (int r = 0; r < 3 - S; ++r)
#pragma unroll
            for (int p = 0; p < NP; ++p) { win[r][p][0] = win[r + S][p][0]; win[r][p][1] = win[r + S][p][1]; }
    }
    if (a.absmax_bits) fold_absmax(a.absmax_bits, mx);            // every lane of every wave arrives here
}

// ---- any other geometry -----------------------------------------------------------------------------
// BA, BW: code widths of image and filter (2, 4 or 8).
template <int BA, int BW>
__global__ __launch_bounds__(kThreads) void dwconv_kernel(const DwArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int kh = a.kh, kw = a.kw, stride = a.stride;
    const int in_h = (TH - 1) * stride + kh, in_w = (TW - 1) * stride + kw;
    float *tile = lds;                                           // [in_h * in_w][CG]
    float *taps = tile + (size_t)in_h * in_w * CG;               // [kh * kw][CG]
    float *lut_a = taps + (size_t)kh * kw * CG;                  // value of every code of the two formats
    float *lut_w = lut_a + (1 << BA);
    const int tid = threadIdx.x;
    int id = blockIdx.x;
    const int cg = id % a.groups; id /= a.groups;
    const int tw = id % a.tiles_w; id /= a.tiles_w;
    const int th = id % a.tiles_h;
    const int b = id / a.tiles_h;
    const int ho0 = th * TH, wo0 = tw * TW, c_first = cg * CG;

    if (tid < (1 << BA)) lut_a[tid] = code_value(tid, BA, a.a_signed);
    if (tid < (1 << BW)) lut_w[tid] = code_value(tid, BW, a.w_signed);
    __syncthreads();

    // Writes the values of the CPW codes of one word to consecutive floats, four at a time.
    auto expand = [&](uint32_t word, const float *lut, auto bits_tag, float *dst) {
        constexpr int BITS = decltype(bits_tag)::value, CPW = 32 / BITS;
#pragma unroll
        for (int j = 0; j < CPW; j += 4) {
            f32x4 v;
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = lut[(word >> ((j + u) * BITS)) & ((1u << BITS) - 1u)];
            *reinterpret_cast<f32x4 *>(dst + j) = v;
        }
    };
    // ---- stage the input patch: one item = one word of codes of one pixel (offsets inside one image fit 32 bits)
    {
        constexpr int WPP = CG * BA / 32, CPW = 32 / BA;                  // words per pixel and group, codes per word
        const int row_words = a.C * BA / 32;                              // words per pixel in the image
        const uint32_t *image = a.X + (int64_t)b * a.H * a.W * row_words + c_first * BA / 32;
        const int items = in_h * in_w * WPP;
        const int hi0 = ho0 * stride - a.pad, wi0 = wo0 * stride - a.pad;
        for (int it = tid; it < items; it += kThreads) {
            const int pix = it / WPP, wd = it % WPP;
            const int iy = pix / in_w, ix = pix - iy * in_w;
            const int hi = hi0 + iy, wi = wi0 + ix;
            const bool in = (unsigned)hi < (unsigned)a.H && (unsigned)wi < (unsigned)a.W && c_first + wd * CPW < a.C;
            const uint32_t word = in ? image[(hi * a.W + wi) * row_words + wd] : 0u;
            expand(word, lut_a, std::integral_constant<int, BA>{}, tile + pix * CG + wd * CPW);   // code 0 is 0.0: padding, channels past C
        }
    }
    // ---- stage the filter taps of the group's channels
    {
        constexpr int WPP = CG * BW / 32, CPW = 32 / BW;
        const int row_words = a.C * BW / 32;
        const int items = kh * kw * WPP;
        for (int it = tid; it < items; it += kThreads) {
            const int tap = it / WPP, wd = it % WPP;
            const bool in = c_first + wd * CPW < a.C;
            const uint32_t word = in ? a.Wt[tap * row_words + c_first * BW / 32 + wd] : 0u;
            expand(word, lut_w, std::integral_constant<int, BW>{}, taps + tap * CG + wd * CPW);
        }
    }
    __syncthreads();

    // ---- accumulate.  A thread's four channels are the same for all its outputs: their scales are read once.
    const int c_thread = c_first + (tid & (CG / 4 - 1)) * 4;
    f32x4 alpha;
    {
        const float sx = *a.x_scale;
        const bool pc = a.w_per_channel && c_thread < a.C;
#pragma unroll
        for (int u = 0; u < 4; ++u) alpha[u] = sx * (pc ? a.w_scale[c_thread + u] : a.w_scale[0]);
    }
    Requant rq{};
    const bool wb = a.q_out != nullptr;
    if (wb) {
        rq = make_requant(a.q_scale, a.q_bits, a.q_signed);
        if (!rq.ok && blockIdx.x == 0 && tid == 0) *a.async_error = DYBIT_ERR_BAD_SCALE;   // no codes, flag the call
    }
    float mx = 0.0f;
    {
        // one item = four neighbouring channels of one output pixel
        const int quad = tid & (CG / 4 - 1);
        for (int it = tid; it < TH * TW * (CG / 4); it += kThreads) {
            const int pix = it / (CG / 4);
            const int py = pix / TW, px = pix % TW;
            const int ho = ho0 + py, wo = wo0 + px, c = c_first + quad * 4;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            const float *origin = tile + ((py * stride) * in_w + px * stride) * CG + quad * 4;
            for (int r = 0; r < kh; ++r)
                for (int q = 0; q < kw; ++q) {
                    const f32x4 x = *reinterpret_cast<const f32x4 *>(origin + (r * in_w + q) * CG);
                    const f32x4 w = *reinterpret_cast<const f32x4 *>(taps + (r * kw + q) * CG + quad * 4);
#pragma unroll
                    for (int u = 0; u < 4; ++u) acc[u] = fmaf(x[u], w[u], acc[u]);
                }
            if (ho < a.Ho && wo < a.Wo && c < a.C) {
                f32x4 bv = {0.f, 0.f, 0.f, 0.f};
                if (a.bias) bv = *reinterpret_cast<const f32x4 *>(a.bias + c);
                finish_quad(a, rq, acc, alpha, bv, mx, (((int64_t)b * a.Ho + ho) * a.Wo + wo) * a.C + c);
            }
        }
    }
    if (a.absmax_bits) fold_absmax(a.absmax_bits, mx);           // every lane of every wave arrives here
}

template <int BA, int BW>
void launch_dw(const DwArgs &a, size_t lds_bytes, hipStream_t st, unsigned blocks)
{
    note_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(dwconv_kernel<BA, BW>), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes));
    hipLaunchKernelGGL((dwconv_kernel<BA, BW>), dim3(blocks), dim3(kThreads), lds_bytes, st, a);
}

template <int FA, int FW>
void launch_dw3(const DwArgs &a, hipStream_t st, dim3 grid)
{
    if (a.stride == 1) hipLaunchKernelGGL((dw3_kernel<FA, FW, 1>), grid, dim3(kThreads), 0, st, a);
    else hipLaunchKernelGGL((dw3_kernel<FA, FW, 2>), grid, dim3(kThreads), 0, st, a);
}

// Plans dw3_kernel: the rows of a thread and the images of a grid row.  False: the call is outside its range (an image of 2^30
// bytes or more, see launch_bands: byte offsets with room for the out-of-range ones are 32-bit), or not a 3 x 3 filter at stride 1 or 2.
bool plan_dw3(DwArgs &a, dim3 &grid)
{
    if (a.kh != 3 || a.kw != 3 || a.stride > 2 || a.C > (1 << 20)) return false;
    const int64_t image_bytes = (int64_t)a.H * a.W * a.C * a.a_bits / 8;
    if (image_bytes >= kRowOob) return false;
    const int64_t quads = a.C / 4, colg = (a.Wo + cols_of(a.stride) - 1) / cols_of(a.stride);
    // Rows: what a thread does once (two rows more to decode, taps, scales, addresses) is worth about 1.2 rows, so long strips do
    // less work, short ones fill the chip.  The longest of 1 .. 16 rows with the least (waves per SIMD, 4 at least) x (rows + 1.2)
    // is taken: 7 rows for 64 x 56 x 56 x 144 (3.9 waves per SIMD).  With 0.6 in place of 1.2, 64 x 14 x 14 x 384 ran one row
    // per thread in 9.2 us instead of two in 7.8.
    int64_t best = INT64_MAX;
    for (int rows = 1; rows <= 16 && rows <= a.Ho; ++rows) {
        const int64_t threads = (int64_t)a.B * ((a.Ho + rows - 1) / rows) * colg * quads;
        int64_t waves = (threads + 64 * 1024 - 1) / (64 * 1024);
        if (waves < 4) waves = 4;
        const int64_t cost = waves * (10 * rows + 12);
        if (cost <= best) { best = cost; a.rows = rows; }
    }
    a.tiles_h = (a.Ho + a.rows - 1) / a.rows;
    a.tiles_w = (int)colg;
    const int64_t image_threads = a.tiles_h * colg * quads;
    int64_t images = image_bytes ? (kRowOob - 1) / image_bytes : 1;
    if (images > a.B) images = a.B;
    if (images * image_threads > 0x7fffff00) images = 0x7fffff00 / image_threads;
    if (images < 1 || (a.B + images - 1) / images > 65535) return false;
    a.images = (int)images;
    grid = dim3((unsigned)((images * image_threads + kThreads - 1) / kThreads), (unsigned)((a.B + images - 1) / images));
    return true;
}

// launch(arguments, grid) for a 3 x 3 filter: once, or for images of 2^30 bytes and more once per image and band of output rows that
// reads less than that.  False, with nothing launched: another kernel has to take the call (a last such case: three rows of the
// image hold 2^30 bytes).  One image of 8192 x 8192 x 16, 8-bit, fp32 results: run-time-geometry kernel 3446 us at stride 1, 2258 at
// stride 2; in bands 1529 and 510.
template <class F>
bool launch_bands(DwArgs a, F launch)
{
    a.pad_top = a.pad;
    dim3 grid;
    if (plan_dw3(a, grid)) {
        launch(a, grid);
        return true;
    }
    if (a.kh != 3 || a.kw != 3 || a.stride > 2) return false;
    const int64_t row_bytes = (int64_t)a.W * a.C * a.a_bits / 8, in_rows = (kRowOob - 1) / row_bytes;
    if (a.H * row_bytes < kRowOob || in_rows < 3) return false;
    const int64_t band = (in_rows - 3) / a.stride + 1;
    for (int pass = 0; pass < 2; ++pass)                          // every band is planned before the first is launched
        for (int64_t b = 0; b < a.B; ++b)
            for (int64_t ho = 0; ho < a.Ho; ho += band) {
                DwArgs s = a;
                s.B = 1;
                s.Ho = (int)(a.Ho - ho < band ? a.Ho - ho : band);
                const int64_t top = ho * a.stride - a.pad, first = top > 0 ? top : 0, end = top + (s.Ho - 1) * (int64_t)a.stride + 3;
                s.H = (int)((end < a.H ? end : a.H) - first);
                if (s.H < 0) s.H = 0;                             // padding only
                else s.X += (b * a.H + first) * row_bytes / 4;
                s.pad_top = (int)(first - top);
                const int64_t elem = (b * a.Ho + ho) * a.Wo * a.C;
                if (s.Y) s.Y += elem;
                if (s.q_out) s.q_out += elem * a.q_bits / 8;
                if (!plan_dw3(s, grid)) return false;
                if (pass) launch(s, grid);
            }
    return true;
}

}  // namespace
}  // namespace dybit

using namespace dybit;

static dybit_status dwconv_impl(int64_t B, int64_t H, int64_t W, int64_t C,
                                int32_t kh, int32_t kw, int32_t stride, int32_t pad,
                                const uint8_t *X_codes, dybit_fmt x_fmt, const float *x_scale,
                                const uint8_t *Wt_codes, dybit_fmt w_fmt, const float *w_scale, int32_t w_per_channel,
                                const float *bias, int32_t relu, float *Y, float *y_absmax,
                                dybit_fmt y_fmt, const float *y_scale, uint8_t *Y_codes, dybit_stream stream)
{
    dybit_status st = check_fmt(x_fmt);
    if (st == DYBIT_OK) st = check_fmt(w_fmt);
    if (st != DYBIT_OK) return st;
    if (x_fmt.bits == 6 || w_fmt.bits == 6) return DYBIT_ERR_UNSUPPORTED_BITS;      // whole codes per 32-bit word only
    if (B < 0 || H < 1 || W < 1 || C < 0 || kh < 1 || kw < 1 || stride < 1 || pad < 0 || (relu != 0 && relu != 1) ||
        H > (1 << 24) || W > (1 << 24) || C > (1 << 24) || kh > 64 || kw > 64 || stride > 64)
        return DYBIT_ERR_INVALID_ARG;
    if (H + 2 * (int64_t)pad < kh || W + 2 * (int64_t)pad < kw) return DYBIT_ERR_INVALID_ARG;
    if ((C * x_fmt.bits) % 32 || (C * w_fmt.bits) % 32) return DYBIT_ERR_ALIGNMENT;   // a pixel's codes are whole words
    if (w_per_channel != 0 && w_per_channel != 1) return DYBIT_ERR_INVALID_ARG;
    if (Y_codes) {
        if ((st = check_fmt(y_fmt)) != DYBIT_OK) return st;
        if (y_fmt.bits != 4 && y_fmt.bits != 8) return DYBIT_ERR_UNSUPPORTED_BITS;     // four codes of a thread are 16 or 32 bits
        if ((C * y_fmt.bits) % 32) return DYBIT_ERR_ALIGNMENT;
        if (!y_scale) return DYBIT_ERR_NULL;
        if (reinterpret_cast<uintptr_t>(Y_codes) & 3u) return DYBIT_ERR_ALIGNMENT;
    }
    const int64_t Ho = (H + 2 * pad - kh) / stride + 1, Wo = (W + 2 * pad - kw) / stride + 1;
    const int in_h = (TH - 1) * stride + kh, in_w = (TW - 1) * stride + kw;
    const int64_t lds_bytes = ((int64_t)in_h * in_w + (int64_t)kh * kw) * CG * 4 + 4 * ((1 << x_fmt.bits) + (1 << w_fmt.bits));
    if (lds_bytes > kMaxLdsBytes) return DYBIT_ERR_INVALID_ARG;                    // filter / stride too large for one patch
    if (H * W * (C * x_fmt.bits / 32) > 0x7fffffff || (int64_t)kh * kw * (C * w_fmt.bits / 32) > 0x7fffffff)
        return DYBIT_ERR_INVALID_ARG;                                              // offsets inside one image are 32-bit
    if (B == 0 || C == 0) return DYBIT_OK;
    if (!x_scale || !w_scale || !X_codes || !Wt_codes || (!Y && !Y_codes)) return DYBIT_ERR_NULL;
    if (!aligned16(X_codes) || !aligned16(Wt_codes) || !aligned16(Y) || (bias && !aligned16(bias))) return DYBIT_ERR_ALIGNMENT;
    clear_call_record();
    DwArgs a{};
    a.X = reinterpret_cast<const uint32_t *>(X_codes); a.Wt = reinterpret_cast<const uint32_t *>(Wt_codes);
    a.x_scale = x_scale; a.w_scale = w_scale; a.bias = bias; a.Y = Y;
    a.absmax_bits = reinterpret_cast<uint32_t *>(y_absmax);
    a.w_per_channel = w_per_channel;
    if (Y_codes) {
        a.q_out = Y_codes; a.q_scale = y_scale; a.q_bits = y_fmt.bits; a.q_signed = y_fmt.is_signed;
        a.async_error = async_error_word();
        if (!a.async_error) return DYBIT_ERR_HIP;
    }
    a.B = (int)B; a.H = (int)H; a.W = (int)W; a.C = (int)C; a.Ho = (int)Ho; a.Wo = (int)Wo;
    a.kh = kh; a.kw = kw; a.stride = stride; a.pad = pad; a.relu = relu;
    a.a_bits = x_fmt.bits; a.a_signed = x_fmt.is_signed; a.w_bits = w_fmt.bits; a.w_signed = w_fmt.is_signed;
    a.tiles_h = (int)((Ho + TH - 1) / TH); a.tiles_w = (int)((Wo + TW - 1) / TW); a.groups = (int)((C + CG - 1) / CG);
    const int64_t blocks = B * a.tiles_h * a.tiles_w * a.groups;
    if (blocks > 0x7fffffff || B > 0x7fffffff) return DYBIT_ERR_INVALID_ARG;
    hipStream_t hs = (hipStream_t)stream;
    // the plan fills in its own tiles in a copy; the general kernel keeps those of a
    const bool done = launch_bands(a, [&](const DwArgs &a3, dim3 grid) {
        using namespace fast;
        auto with_image = [&](auto fa) {
            constexpr int FA = decltype(fa)::value;
            switch (w_fmt.bits * 2 + w_fmt.is_signed) {
                case 4: launch_dw3<FA, F2U>(a3, hs, grid); break;   case 5: launch_dw3<FA, F2S>(a3, hs, grid); break;
                case 8: launch_dw3<FA, F4U>(a3, hs, grid); break;   case 9: launch_dw3<FA, F4S>(a3, hs, grid); break;
                case 16: launch_dw3<FA, F8U>(a3, hs, grid); break;  case 17: launch_dw3<FA, F8S>(a3, hs, grid); break;
            }
        };
        switch (x_fmt.bits * 2 + x_fmt.is_signed) {
            case 4: with_image(std::integral_constant<int, F2U>{}); break;   case 5: with_image(std::integral_constant<int, F2S>{}); break;
            case 8: with_image(std::integral_constant<int, F4U>{}); break;   case 9: with_image(std::integral_constant<int, F4S>{}); break;
            case 16: with_image(std::integral_constant<int, F8U>{}); break;  case 17: with_image(std::integral_constant<int, F8S>{}); break;
        }
    });
    if (done) return launch_status();
#define DYBIT_DW(BA, BW) launch_dw<BA, BW>(a, (size_t)lds_bytes, hs, (unsigned)blocks)
    switch (x_fmt.bits * 16 + w_fmt.bits) {
        case 0x22: DYBIT_DW(2, 2); break;  case 0x24: DYBIT_DW(2, 4); break;  case 0x28: DYBIT_DW(2, 8); break;
        case 0x42: DYBIT_DW(4, 2); break;  case 0x44: DYBIT_DW(4, 4); break;  case 0x48: DYBIT_DW(4, 8); break;
        case 0x82: DYBIT_DW(8, 2); break;  case 0x84: DYBIT_DW(8, 4); break;  case 0x88: DYBIT_DW(8, 8); break;
    }
#undef DYBIT_DW
    return launch_status();
}

extern "C" dybit_status dybit_dwconv2d(int64_t B, int64_t H, int64_t W, int64_t C,
                                       int32_t kh, int32_t kw, int32_t stride, int32_t pad,
                                       const uint8_t *X_codes, dybit_fmt x_fmt, const float *x_scale,
                                       const uint8_t *Wt_codes, dybit_fmt w_fmt, const float *w_scale,
                                       const float *bias, int32_t relu, float *Y, float *y_absmax, dybit_stream stream)
{
    if (!Y && B && C) return DYBIT_ERR_NULL;
    return dwconv_impl(B, H, W, C, kh, kw, stride, pad, X_codes, x_fmt, x_scale, Wt_codes, w_fmt, w_scale, 0, bias, relu,
                       Y, y_absmax, dybit_fmt{0, 0}, nullptr, nullptr, stream);
}

extern "C" dybit_status dybit_dwconv2d_wb(int64_t B, int64_t H, int64_t W, int64_t C,
                                          int32_t kh, int32_t kw, int32_t stride, int32_t pad,
                                          const uint8_t *X_codes, dybit_fmt x_fmt, const float *x_scale,
                                          const uint8_t *Wt_codes, dybit_fmt w_fmt, const float *w_scale, int32_t w_per_channel,
                                          const float *bias, int32_t relu, float *Y, float *y_absmax,
                                          dybit_fmt y_fmt, const float *y_scale, uint8_t *Y_codes, dybit_stream stream)
{
    return dwconv_impl(B, H, W, C, kh, kw, stride, pad, X_codes, x_fmt, x_scale, Wt_codes, w_fmt, w_scale, w_per_channel, bias, relu,
                       Y, y_absmax, y_fmt, y_scale, Y_codes, stream);
}
