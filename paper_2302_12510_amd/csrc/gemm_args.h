// Argument block shared by the DyBit matrix-product kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#ifndef DYBIT_WB
#define DYBIT_WB 0
#endif
#if DYBIT_WB == 2
#define DYBIT_WB_NAME(name) name##_co
#elif DYBIT_WB
#define DYBIT_WB_NAME(name) name##_wb
#else
#define DYBIT_WB_NAME(name) name
#endif

namespace dybit {

// The builds of a kernel source, by what its epilogue writes: fp32 results; fp32 results and / or their DyBit codes;
// codes only (codes_epilogue.h).  Which source has which: at the launch functions below.
enum : int { OUT_FP32 = 0, OUT_WRITE_BACK = 1, OUT_CODES = 2 };
constexpr int kOut = DYBIT_WB;
constexpr bool kWriteBack = DYBIT_WB != 0;

// The dynamic LDS that a launch may ask for: all of a compute unit's, less the 256 bytes that the codes-only kernels hold themselves
// (__syncthreads_or).  Kernels of varying sizes set it as their limit with every launch: the limit is one per kernel and process, and with
// the size of the call two threads could set it against each other.
constexpr int kLdsLimit = 160 * 1024 - (kOut == OUT_CODES ? 256 : 0);

struct GemmArgs {
    int64_t M, N, K;                 // conv: M = B*Ho*Wo, N = Cout, K = kh*kw*Cin
    const uint8_t *A, *W;            // packed codes, K-contiguous rows (conv: NHWC image / [Cout][kh][kw][Cin])
    int a_signed, w_signed;
    const float *a_scale, *w_scale, *bias;
    int w_per_channel;               // 0: *w_scale is the scale of the whole tensor; 1: w_scale[n] per output column n
    const float *residual;           // optional: fp32 tensor laid out like C (same ldc), added before the ReLU
    // the shortcut as DyBit codes instead (write-back build only; at most one of the two forms): M rows of
    // res_row_bytes bytes holding N codes of res_bits bits (4, 6 or 8), value = *res_scale * value(code)
    const uint8_t *res_codes;
    const float *res_scale;
    int res_bits, res_signed;
    int64_t res_row_bytes;
    int relu;
    uint32_t *absmax_bits;           // optional: running max |C| of the written values, as float bits (atomic max)
    float *C;                        // may be NULL when q_out is given
    int64_t ldc;
    // optional write-back of the result as DyBit codes: M rows of q_row_bytes bytes (N codes, whole 32-bit words)
    uint8_t *q_out;
    const float *q_scale;
    int q_bits, q_signed;
    int64_t q_row_bytes;
    int *async_error;                // device word that receives DYBIT_ERR_BAD_SCALE when *q_scale is unusable
    // convolution geometry (conv only)
    int H, Wd, Cin, Ho, Wo, kh, kw, stride, pad;
    int pix_bytes;                   // bytes from a pixel to the next one in the image: Cin * bits / 8, or more when A
                                     // points at one channel group of a wider image (grouped convolution)
    int64_t a_bytes, w_bytes;        // sizes of the two code buffers
};

// Whether a write-back call can take the codes-only build (codes_epilogue.h): no fp32 output or shortcut; results that
// an unsigned format can hold (that epilogue encodes magnitudes); a shortcut given as codes in whole, aligned words
// per row (rows of codes out are whole words by the entry points' checks).
inline bool codes_only(const GemmArgs &g)
{
    return g.q_out && !g.C && !g.residual && (g.relu || g.q_signed) &&
           (!g.res_codes || (g.res_row_bytes % 4 == 0 && (reinterpret_cast<uintptr_t>(g.res_codes) & 3u) == 0));
}

// Overrides of the automatic kernel choice (0 = automatic everywhere).  They start from the
// environment, read once when the library is first used (DYBIT_GEMM_KERNEL, DYBIT_GEMM_MFMA,
// DYBIT_MID_TILE, DYBIT_MID_KGROUPS, DYBIT_GEMM_WS), and change only through dybit_set_option.
struct DispatchOptions {
    int kernel;        // 0 automatic, else DYBIT_FORCE_*
    int mfma_f16;      // 1: pairs of 4- and 2-bit operands stay on the fp16 kernels
    int mid_tile;      // 0 automatic, 64 or 128: tile of the fp8-path kernel when it is not the 256 x 256 one
    int mid_kgroups;   // 0 automatic, 1 or 2: k-groups of the 128 x 128 kernels
    int ws_off;        // 1: the weight-stationary kernel is left out of the automatic choice
};
enum { DYBIT_FORCE_GENERAL = 1, DYBIT_FORCE_MID = 2, DYBIT_FORCE_LARGE = 3, DYBIT_FORCE_WS = 4, DYBIT_FORCE_SMALL = 5, DYBIT_FORCE_FEW = 6, DYBIT_FORCE_PATCH = 7, DYBIT_FORCE_SIX = 8 };
DispatchOptions dispatch_options();
// Record of the kernel a launch function started, per host thread (dybit_last_gemm_kernel reads it),
// and of a HIP error met on the way (hipFuncSetAttribute, ...), which the entry point then reports.
void note_kernel(int id);
void note_hip(hipError_t e);
void clear_call_record();          // an entry point calls this first
hipError_t take_hip_error();       // ... and this last: the first error noted since, or hipSuccess

// Tiled MFMA kernels for 4- and 8-bit operands with signed weights: the large-tile kernel
// (gemm_fast.hip, 256 x 256) and the mid-size-tile kernel (gemm_mid.hip, 128 x 128), one
// translation unit per weight format.  a_bits is 4 or 8; signedness comes from g.
// Builds: plain; with DYBIT_WB=1 (_wb) the write-back build whose epilogue also encodes the results (g.q_out must then be
// set); with DYBIT_WB=2 (_co) the build for calls that want codes only (codes_only() above).  The general, 256 x 256 and
// small-output kernels have the first two, the weight-stationary, 128 x 128 and e4m3 kernels and the many-channel convolution all three, the
// few-channel convolution plain and _co, the grouped convolution the plain one.
bool launch_gemm_fast_w0(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);   // W 4-bit signed
bool launch_gemm_fast_w2(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);   // W 8-bit signed
bool launch_gemm_fast_w4(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);   // W 6-bit signed
bool launch_gemm_fast_w6(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);   // W 2-bit signed; a_bits 2, 4, 6 or 8 for all four; false:
                                                                                      // K (Cin) is not a multiple of 128 while an operand is 2- or 6-bit
bool launch_gemm_mid_w0(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_mid_w2(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_mid_w4(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);    // W 6-bit signed
bool launch_gemm_mid_w6(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);    // W 2-bit signed; a_bits 2, 4, 6 or 8 for all four
bool launch_gemm_fast_w0_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_fast_w2_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_fast_w4_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_fast_w6_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_mid_w0_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_mid_w2_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_mid_w4_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_mid_w6_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_mid_w0_co(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_mid_w2_co(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_mid_w4_co(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_mid_w6_co(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);

// Weight-stationary kernel (gemm_ws.hip) for layers whose decoded weight matrix fits the LDS of a
// compute unit (N <= 128, N rounded up to 64 or 128 rows of 2 K + 16 bytes within 160 KiB); one
// translation unit per weight format as above.  Returns false when the weights do not fit.
bool launch_gemm_ws_w0(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_ws_w2(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_ws_w4(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_ws_w6(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_ws_w0_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_ws_w2_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_ws_w4_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_ws_w6_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_ws_w0_co(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_ws_w2_co(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_ws_w4_co(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
bool launch_gemm_ws_w6_co(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);

// Small-output kernel (gemm_small.hip): 32-row tiles, K split over the waves of a workgroup; also K not a multiple of 64.
void launch_gemm_small_w0(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
void launch_gemm_small_w2(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
void launch_gemm_small_w4(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
void launch_gemm_small_w6(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
void launch_gemm_small_w0_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
void launch_gemm_small_w2_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
void launch_gemm_small_w4_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);
void launch_gemm_small_w6_wb(const GemmArgs &g, int a_bits, bool conv, hipStream_t st);

// Few-channel convolution with its input decoded once (conv_few.hip); plain and codes-only builds.  false: no unit of output
// rows fits the LDS.
bool launch_conv_few_w0(const GemmArgs &g, int a_bits, hipStream_t st);
bool launch_conv_few_w2(const GemmArgs &g, int a_bits, hipStream_t st);
bool launch_conv_few_w4(const GemmArgs &g, int a_bits, hipStream_t st);
bool launch_conv_few_w6(const GemmArgs &g, int a_bits, hipStream_t st);
bool launch_conv_few_w0_co(const GemmArgs &g, int a_bits, hipStream_t st);
bool launch_conv_few_w2_co(const GemmArgs &g, int a_bits, hipStream_t st);
bool launch_conv_few_w4_co(const GemmArgs &g, int a_bits, hipStream_t st);
bool launch_conv_few_w6_co(const GemmArgs &g, int a_bits, hipStream_t st);

// Pixels from the first tap of a strip's first output to the last tap of its last one, at most: `rows` outputs advance rows - 1
// times, by a pixel step each or, at an image row's or an image's end, by more (row_ends may count one too many, which must not
// shorten the strip).  No output's first tap may reach past the image, which bounds every step by the image's pixels: with one
// row of outputs every row's end is an image's, and with one column no step is a pixel step, whatever the stride.
inline int64_t strip_pixels(const GemmArgs &g, int64_t rows)
{
    const int64_t steps = rows - 1, row_ends = (steps + g.Wo - 1) / g.Wo, image_ends = (steps + (int64_t)g.Ho * g.Wo - 1) / ((int64_t)g.Ho * g.Wo);
    const int64_t back = (int64_t)(g.Wo - 1) * g.stride, image_step = (g.H - (int64_t)(g.Ho - 1) * g.stride) * g.Wd - back;
    const int64_t row_step = g.Ho > 1 ? (int64_t)g.stride * g.Wd - back : g.Wo > 1 && g.stride > image_step ? g.stride : image_step;
    const int64_t further = row_step > image_step ? row_step : image_step;
    const int64_t inner = steps > row_ends ? steps - row_ends : 0;
    return (g.Wo > 1 ? inner * g.stride : 0) + row_ends * row_step + image_ends * (further - row_step) + (int64_t)(g.kh - 1) * g.Wd + g.kw;
}

// Convolution of 64 and more channels with its input decoded once (conv_patch.hip), all three builds.  false: the pixels of 128 outputs
// (up to 32 columns: of 256, which their four waves take together) do not fit the LDS.
bool launch_conv_patch_w0(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);
bool launch_conv_patch_w2(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);
bool launch_conv_patch_w4(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);
bool launch_conv_patch_w6(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);
bool launch_conv_patch_w0_wb(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);
bool launch_conv_patch_w2_wb(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);
bool launch_conv_patch_w4_wb(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);
bool launch_conv_patch_w6_wb(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);
bool launch_conv_patch_w0_co(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);
bool launch_conv_patch_w2_co(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);
bool launch_conv_patch_w4_co(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);
bool launch_conv_patch_w6_co(const GemmArgs &g, int a_bits, bool low_pair, hipStream_t st);

// Grouped convolution in one launch (gemm_group.hip): g describes the whole layer (N of all groups, Cin and K of one).  false:
// a group's channels are not whole words, or its weights do not fit the LDS of a compute unit.
bool launch_group_conv_w0(const GemmArgs &g, int a_bits, int groups, hipStream_t st);
bool launch_group_conv_w2(const GemmArgs &g, int a_bits, int groups, hipStream_t st);
bool launch_group_conv_w4(const GemmArgs &g, int a_bits, int groups, hipStream_t st);
bool launch_group_conv_w6(const GemmArgs &g, int a_bits, int groups, hipStream_t st);
bool launch_group_conv(const GemmArgs &g, int a_bits, int w_bits, int groups, hipStream_t st);   // gemm_dispatch.cpp

// fp8 matrix path for pairs of 4-bit formats with signed weights (gemm_f8.hip): the 256 x 256 tile
// when `large`, else the 128 x 128 tile.
bool launch_gemm_f8_w0(const GemmArgs &g, int a_bits, bool conv, bool large, hipStream_t st);      // W 4-bit signed
bool launch_gemm_f8_w6(const GemmArgs &g, int a_bits, bool conv, bool large, hipStream_t st);      // W 2-bit signed
bool launch_gemm_f8_w0_wb(const GemmArgs &g, int a_bits, bool conv, bool large, hipStream_t st);
bool launch_gemm_f8_w6_wb(const GemmArgs &g, int a_bits, bool conv, bool large, hipStream_t st);
bool launch_gemm_f8_w0_co(const GemmArgs &g, int a_bits, bool conv, bool large, hipStream_t st);
bool launch_gemm_f8_w6_co(const GemmArgs &g, int a_bits, bool conv, bool large, hipStream_t st);

// Large products on split operands (gemm_six.hip).  Bytes of scratch (0: the kernel does not take the product), the tile it is faster
// with than the other kernels (0: none; gemm_dispatch.cpp), and the launch (`scratch` holds so many bytes).
int64_t gemm_six_bytes(int64_t M, int64_t N, int64_t K, int a_bits, int a_signed, int w_bits, int w_signed);
int gemm_six_tile(int64_t M, int64_t N, int64_t K, int a_bits, int w_bits);
void launch_gemm_six(const GemmArgs &g, int a_bits, int w_bits, int tile, uint8_t *scratch, hipStream_t st);

// General kernel (gemm.hip): any format pair and shape.  mode: 0 operands fetched code by code;
// 1 operands are 16-byte aligned and K (convolution: Cin) is a multiple of 16; 2 (convolution
// only) aligned operands, Cin divides 16 and kw * Cin is a multiple of 16, tensor below 2 GiB.
void launch_gemm_general(const GemmArgs &g, int a_bits, int w_bits, bool conv, int mode, hipStream_t st);
void launch_gemm_general_wb(const GemmArgs &g, int a_bits, int w_bits, bool conv, int mode, hipStream_t st);
// the write-back build's kernels, one translation unit per activation width (gemm_dispatch.cpp joins them)
void launch_gemm_general_a2_wb(const GemmArgs &g, int w_bits, bool conv, int mode, hipStream_t st);
void launch_gemm_general_a4_wb(const GemmArgs &g, int w_bits, bool conv, int mode, hipStream_t st);
void launch_gemm_general_a6_wb(const GemmArgs &g, int w_bits, bool conv, int mode, hipStream_t st);
void launch_gemm_general_a8_wb(const GemmArgs &g, int w_bits, bool conv, int mode, hipStream_t st);

// Picks a tiled kernel for the problem (gemm_dispatch.cpp).  Returns false when the problem does
// not meet their preconditions; the caller then uses the general kernel.
bool launch_gemm_tiled(const GemmArgs &g, int a_bits, int w_bits, bool conv, hipStream_t st);

// Folds a lane's maximum of |c| into the running maximum: wave reduction, then at most one atomic
// per wave.  Non-negative floats order like their bit patterns; fmaxf has already dropped NaNs.
// Atomics on one address serialise (about 10 ns each), and a large layer has tens of thousands of
// waves, so a wave first reads the word (at device scope, from L2) and only competes when it would
// raise it: the running maximum of a sequence is raised only about log(count) times.  A stale read
// can only cause a needless atomic, never a wrong result.
#ifdef __HIPCC__
__device__ __forceinline__ void fold_absmax(uint32_t *absmax_bits, float mx)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    if ((threadIdx.x & 63) == 0) {
        const uint32_t bits = __float_as_uint(mx);
        if (bits > __hip_atomic_load(absmax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(absmax_bits, bits);
    }
}
#endif

}  // namespace dybit
