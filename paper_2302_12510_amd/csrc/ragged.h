// Rows of packed codes that start at any byte: matrix products whose K is not a multiple of 64, so that neither the
// rows nor the last K step fall on word boundaries.
//
// A run of 32 codes is fetched as the aligned words that hold it (one more than the run has) and shifted into place
// when it is decoded.  The odd part of K comes first: K step 0 covers the first `head` = K mod TK codes (TK when that is
// 0) with a full-width run whose codes past `head` are cleared in W, and every later step is whole and starts at
// head + (t - 1) TK.  So every run lies inside its row (K >= TK), the main loop has no tail, and masking one operand once
// is enough: every code decodes to a finite value, and finite times zero is zero.
// Loads are whole words: the last word of a tensor may hold up to three bytes past its end, inside the same aligned
// word and hence the same page; their codes are shifted out or multiplied by zero.
#ifndef DYBIT_RAGGED_H
#define DYBIT_RAGGED_H

#include "dybit_codec.h"
#include "gemm_args.h"
#include "tile_common.h"

namespace dybit {
namespace fast {

// Registers (of four words) that hold a run's words, one extra word and, in the last word, the byte shift.
template <int BITS> constexpr int ragged_regs() { return (BITS + 2 + 3) / 4; }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t word_descriptor(const uint8_t *p, int64_t bytes)
{
    return code_descriptor(p, (bytes + 3) & ~(int64_t)3);
}

// off: byte offset of the run's first code (any byte), or at least kOob.
template <int BITS>
__device__ __forceinline__ void load_run_ragged(const __amdgpu_buffer_rsrc_t rsrc, u32 off, u32x4 (&raw)[ragged_regs<BITS>()])
{
    constexpr int N = ragged_regs<BITS>();
    const u32 base = off & ~3u;
    u32 w[4 * N];
#pragma unroll
    for (int i = 0; i < 4 * N; ++i) w[i] = 0;
    if constexpr (BITS == 2) {
        const auto a = __builtin_amdgcn_raw_buffer_load_b64(rsrc, base, 0, 0);
        w[0] = a[0]; w[1] = a[1];
    } else {
#pragma unroll
        for (int i = 0; i + 4 <= BITS; i += 4) {
            const auto a = __builtin_amdgcn_raw_buffer_load_b128(rsrc, base + 4 * i, 0, 0);
            w[i] = a[0]; w[i + 1] = a[1]; w[i + 2] = a[2]; w[i + 3] = a[3];
        }
        if constexpr (BITS == 6) {
            const auto a = __builtin_amdgcn_raw_buffer_load_b64(rsrc, base + 16, 0, 0);
            w[4] = a[0]; w[5] = a[1];
        }
    }
    w[BITS] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, base + 4 * BITS, 0, 0);
    w[4 * N - 1] = off & 3u;
#pragma unroll
    for (int p = 0; p < N; ++p) raw[p] = u32x4{w[4 * p], w[4 * p + 1], w[4 * p + 2], w[4 * p + 3]};
}

// The run's words in place, as load_run() would have fetched them from an aligned address.
template <int BITS>
__device__ __forceinline__ void align_run(const u32x4 *raw, u32x4 (&t)[(BITS + 3) / 4])
{
    const u32 shift = raw[ragged_regs<BITS>() - 1].w;
#pragma unroll
    for (int p = 0; p < (BITS + 3) / 4; ++p) t[p] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < BITS; ++i)
        t[i >> 2][i & 3] = __builtin_amdgcn_alignbyte(raw[(i + 1) >> 2][(i + 1) & 3], raw[i >> 2][i & 3], shift);
}

// Clears the codes from number `keep` on (0 .. 32) of an aligned run.
template <int BITS>
__device__ __forceinline__ void keep_codes(u32x4 (&t)[(BITS + 3) / 4], int keep)
{
#pragma unroll
    for (int i = 0; i < BITS; ++i) {
        const int bits = min(max(keep * BITS - 32 * i, 0), 32);
        t[i >> 2][i & 3] &= bits >= 32 ? ~0u : (1u << bits) - 1u;
    }
}

}  // namespace fast
}  // namespace dybit
#endif
