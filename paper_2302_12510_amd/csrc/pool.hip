// Max pooling on packed DyBit codes (Sec. III-B: between layers the activations exist as codes only).
// The encoder is monotone -- a larger value never gets a code of smaller value -- so the code of the
// maximum of a window equals the maximum, by value, of the window's codes: pooling the codes gives bit for
// bit what quantizing the pooled fp32 tensor under the same scale would give, at 1/8 .. 1/4 of the bytes.
//
// Layout: NHWC, a pixel is C codes packed along C (C * bits a multiple of 32).  A thread owns one 32-bit word of a
// pixel (32 / bits channels).  Fields are compared as the halves of a register, two channels per packed 16-bit maximum.
// Unsigned codes order like their values.  Sign-magnitude codes are first mapped to
// offset keys (non-negative: code + 2^(bits-1); negative: 2^(bits-1) - 1 - magnitude), which order like the
// values, and mapped back at the end; value zero is always written as the all-zero code.
//
// 3 x 3 windows at stride 2 (maxpool3s2_kernel, the pooling of the ResNets): a thread walks down kRows output rows of one column;
// all its loads are in flight at once and the row that two windows share is reduced once.  A field is shifted to the top of its
// half and what lies below it is left there: the maximum by the top bits is all that is read back.  Taps outside the image
// are moved to the nearest pixel inside, which the window holds too.  64 x 112 x 112 x 64, 4-bit: 22.1 -> 8.6 us (32 MB;
// the word-per-thread form spends its time on 64-bit divisions and on loads one after the other); 8-bit 30.3 -> 12.0; one image 4.5 -> 3.6.
// Every other window (maxpool_codes_kernel): one output word per thread, its k x k window walked tap by tap, taps outside the
// image skipped (a window always has one inside: 2 pad <= k).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/dybit.h"
#include "dybit_host.h"

namespace dybit {
namespace {

constexpr int kThreads = 256;

struct PoolArgs {
    const uint32_t *x;
    uint32_t *y;
    int H, W, Ho, Wo, k, stride, pad;
    int words;                    // 32-bit words per pixel
    int strips;                   // maxpool3s2_kernel: strips of kRows output rows
    int64_t total;                // output words (maxpool3s2_kernel: threads)
    int is_signed;
};

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

template <int BITS>
__global__ __launch_bounds__(kThreads) void maxpool_codes_kernel(const PoolArgs a)
{
    constexpr int PLANES = 16 / BITS;                               // fields per 16-bit half
    constexpr uint32_t kField = (1u << BITS) - 1u;
    constexpr uint32_t kPlane = kField | (kField << 16);            // field 0 of both halves
    constexpr uint32_t kSign = (1u << (BITS - 1)) * 0x00010001u, kMag = ((1u << (BITS - 1)) - 1u) * 0x00010001u;
    const bool is_signed = a.is_signed != 0;                        // uniform
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < a.total; i += (int64_t)gridDim.x * kThreads) {
        const int64_t pix = i / a.words;
        const int word = (int)(i - pix * a.words);
        const int wo = (int)(pix % a.Wo);
        const int64_t t = pix / a.Wo;
        const int ho = (int)(t % a.Ho);
        const int64_t b = t / a.Ho;
        const int h_lo = ho * a.stride - a.pad, w_lo = wo * a.stride - a.pad;
        uint32_t best[PLANES];
#pragma unroll
        for (int p = 0; p < PLANES; ++p) best[p] = 0u;              // the smallest key
        for (int r = max(h_lo, 0); r < min(h_lo + a.k, a.H); ++r) {
            const uint32_t *row = a.x + ((b * a.H + r) * a.W) * a.words + word;
            for (int s = max(w_lo, 0); s < min(w_lo + a.k, a.W); ++s) {
                const uint32_t w = row[(int64_t)s * a.words];
#pragma unroll
                for (int p = 0; p < PLANES; ++p) {
                    uint32_t c = (w >> (p * BITS)) & kPlane;
                    if (is_signed) {
                        const uint32_t sg = c & kSign;               // key = c ^ sign bit, magnitude inverted where the sign is set
                        c ^= kSign ^ (sg - (sg >> (BITS - 1)));
                    }
                    const u16x2 m = __builtin_elementwise_max(__builtin_bit_cast(u16x2, best[p]), __builtin_bit_cast(u16x2, c));
                    best[p] = __builtin_bit_cast(uint32_t, m);
                }
            }
        }
        uint32_t out = 0;
#pragma unroll
        for (int p = 0; p < PLANES; ++p) {
            uint32_t c = best[p];
            if (is_signed) {
                // keys >= 2^(bits-1) are the non-negative codes; below: negative, magnitude 2^(bits-1) - 1 - key,
                // and magnitude 0 (the negative zero) becomes the all-zero code
                const uint32_t pos = c & kSign;                      // set: non-negative
                const uint32_t neg = (pos ^ kSign) - ((pos ^ kSign) >> (BITS - 1));   // kMag where negative
                const uint32_t mag = (c ^ neg) & kMag;
                const uint32_t nz = (mag | (mag >> 1) | (mag >> 2) | (mag >> 3) | (mag >> 4) | (mag >> 5) | (mag >> 6)) & 0x00010001u;
                c = mag | ((pos ^ kSign) & (nz << (BITS - 1)));      // sign only with a non-zero magnitude
            }
            out |= c << (p * BITS);
        }
        a.y[i] = out;
    }
}

constexpr int kRows = 4;                          // output rows of a thread of maxpool3s2_kernel: 27 loads

template <int BITS>
__device__ __forceinline__ uint32_t to_keys(uint32_t w)             // sign-magnitude fields -> keys that order like the values
{
    constexpr uint32_t kOnes = 0xffffffffu / ((1u << BITS) - 1u), kSigns = kOnes << (BITS - 1);
    const uint32_t sg = w & kSigns;
    return w ^ kSigns ^ (sg - (sg >> (BITS - 1)));
}

template <int BITS>
__device__ __forceinline__ uint32_t from_keys(uint32_t key)
{
    constexpr uint32_t kOnes = 0xffffffffu / ((1u << BITS) - 1u), kSigns = kOnes << (BITS - 1);
    const uint32_t minus = ~key & kSigns;                            // set: negative
    const uint32_t mag = (key ^ (minus - (minus >> (BITS - 1)))) & ~kSigns;
    uint32_t nz = mag;
#pragma unroll
    for (int j = 1; j < BITS - 1; ++j) nz |= mag >> j;
    return mag | (minus & ((nz & kOnes) << (BITS - 1)));             // sign only with a non-zero magnitude
}

template <int BITS, bool SIGNED>
__global__ __launch_bounds__(kThreads) void maxpool3s2_kernel(const PoolArgs a)
{
    constexpr int PLANES = 16 / BITS;
    constexpr uint32_t kPlane = ((1u << BITS) - 1u) * 0x00010001u;
    const uint32_t id = blockIdx.x * kThreads + threadIdx.x;
    if (id >= (uint32_t)a.total) return;
    const uint32_t word = id % a.words, t0 = id / a.words;
    const uint32_t wo = t0 % a.Wo, t1 = t0 / a.Wo;
    const uint32_t strip = t1 % a.strips, b = t1 / a.strips;
    const int ho = strip * kRows, hi = ho * 2 - a.pad, wi = wo * 2 - a.pad;
    const uint32_t *image = a.x + (int64_t)b * a.H * a.W * a.words + word;
    uint32_t col[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) col[s] = min(max(wi + s, 0), a.W - 1) * a.words;
    uint32_t raw[2 * kRows + 1][3];
#pragma unroll
    for (int r = 0; r < 2 * kRows + 1; ++r) {
        const uint32_t row = (uint32_t)min(max(hi + r, 0), a.H - 1) * a.W * a.words;
#pragma unroll
        for (int s = 0; s < 3; ++s) raw[r][s] = image[row + col[s]];
    }
    auto fold = [](uint32_t m, uint32_t c) {
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, m), __builtin_bit_cast(u16x2, c)));
    };
    uint32_t best[PLANES], next[PLANES];
    auto row_max = [&](const uint32_t *w, uint32_t *m, bool first) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const uint32_t k = SIGNED ? to_keys<BITS>(w[s]) : w[s];
#pragma unroll
            for (int p = 0; p < PLANES; ++p) {
                const uint32_t c = k << (16 - BITS - p * BITS);
                m[p] = first && s == 0 ? c : fold(m[p], c);
            }
        }
    };
    row_max(raw[0], next, true);
    uint32_t *out = a.y + (((int64_t)b * a.Ho + ho) * a.Wo + wo) * a.words + word;
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
#pragma unroll
        for (int p = 0; p < PLANES; ++p) best[p] = next[p];
        row_max(raw[2 * i + 1], best, false);
        row_max(raw[2 * i + 2], next, true);
        uint32_t key = 0;
#pragma unroll
        for (int p = 0; p < PLANES; ++p) key |= ((fold(best[p], next[p]) >> (16 - BITS)) & kPlane) << (p * BITS);
        if (ho + i < a.Ho) out[(int64_t)i * a.Wo * a.words] = SIGNED ? from_keys<BITS>(key) : key;
    }
}

template <int BITS>
void launch_pool(PoolArgs a, int64_t B, hipStream_t st)
{
    a.strips = (a.Ho + kRows - 1) / kRows;
    const int64_t strips = B * a.strips * a.Wo * a.words;
    // 32-bit thread numbers and word offsets inside an image
    if (a.k == 3 && a.stride == 2 && strips <= 0x7fffffff - kThreads && (int64_t)a.H * a.W * a.words <= 0x7fffffff) {
        a.total = strips;
        const dim3 grid((unsigned)((strips + kThreads - 1) / kThreads)), block(kThreads);
        if (a.is_signed) hipLaunchKernelGGL((maxpool3s2_kernel<BITS, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((maxpool3s2_kernel<BITS, false>), grid, block, 0, st, a);
        return;
    }
    const int64_t blocks = (a.total + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(maxpool_codes_kernel<BITS>, dim3((unsigned)(blocks < 256 * 32 ? blocks : 256 * 32)), dim3(kThreads), 0, st, a);
}

}  // namespace
}  // namespace dybit

using namespace dybit;

extern "C" dybit_status dybit_maxpool2d_codes(int64_t B, int64_t H, int64_t W, int64_t C,
                                              int32_t k, int32_t stride, int32_t pad,
                                              const uint8_t *X_codes, dybit_fmt fmt, uint8_t *Y_codes, dybit_stream stream)
{
    if (fmt.bits != 2 && fmt.bits != 4 && fmt.bits != 8) return DYBIT_ERR_UNSUPPORTED_BITS;
    if (fmt.is_signed != 0 && fmt.is_signed != 1) return DYBIT_ERR_INVALID_ARG;
    if (B < 0 || H < 1 || W < 1 || C < 1 || k < 1 || stride < 1 || pad < 0 || 2 * pad > k) return DYBIT_ERR_INVALID_ARG;
    if (H > (1 << 24) || W > (1 << 24) || H + 2 * (int64_t)pad < k || W + 2 * (int64_t)pad < k) return DYBIT_ERR_INVALID_ARG;
    if ((C * fmt.bits) % 32) return DYBIT_ERR_ALIGNMENT;
    if (B == 0) return DYBIT_OK;
    if (!X_codes || !Y_codes) return DYBIT_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(X_codes) | reinterpret_cast<uintptr_t>(Y_codes)) & 3u) return DYBIT_ERR_ALIGNMENT;
    PoolArgs a{};
    a.x = reinterpret_cast<const uint32_t *>(X_codes);
    a.y = reinterpret_cast<uint32_t *>(Y_codes);
    a.H = (int)H; a.W = (int)W; a.k = k; a.stride = stride; a.pad = pad;
    a.Ho = (int)((H + 2 * pad - k) / stride + 1);
    a.Wo = (int)((W + 2 * pad - k) / stride + 1);
    a.words = (int)(C * fmt.bits / 32);
    a.total = B * a.Ho * a.Wo * a.words;
    a.is_signed = fmt.is_signed;
    hipStream_t st = (hipStream_t)stream;
    switch (fmt.bits) {
        case 2: launch_pool<2>(a, B, st); break;
        case 4: launch_pool<4>(a, B, st); break;
        default: launch_pool<8>(a, B, st); break;
    }
    return launch_status();
}
