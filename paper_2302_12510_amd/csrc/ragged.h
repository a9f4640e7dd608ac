// Rows of packed codes that start at any byte: matrix products whose K is not a multiple of 64, so that neither the
// rows nor the last K step fall on word boundaries.
//
// A run of 32 codes is fetched as the aligned words that hold it (one more than the run has) and shifted into place
// when it is decoded.  The odd part of K comes first: K step 0 covers the first `head` = K mod TK codes (TK when that is
// 0) with a full-width run whose codes past `head` are cleared in W, and every later step is whole and starts at
// head + (t - 1) TK.  So every run lies inside its row (K >= TK), the main loop has no tail, and masking one operand once
// is enough: every code decodes to a finite value, and finite times zero is zero.
//
// Nothing past a tensor is read.  Loads are whole words, the descriptor ends with the last whole word of the tensor, and the one to
// three bytes that may follow are read byte by byte, once (last_bytes), and joined to the run they belong to: a word past the
// descriptor reads 0.  In a matrix product that is the extra word of the last run of the last row, so its lane alone
// holds them and joins them in the last K step (align_run); a run that may end behind its row looks for them (join_last_bytes).
#ifndef DYBIT_RAGGED_H
#define DYBIT_RAGGED_H

#include "dybit_codec.h"
#include "gemm_args.h"
#include "tile_common.h"

namespace dybit {
namespace fast {

// Registers (of four words) that hold a run's words, one extra word and, in the last word, the byte shift.
template <int BITS> constexpr int ragged_regs() { return (BITS + 2 + 3) / 4; }

constexpr __host__ __device__ int64_t whole_words(int64_t bytes) { return bytes & ~(int64_t)3; }
static_assert(whole_words(4) == 4 && whole_words(7) == 4 && whole_words(0x7ffffffe) == 0x7ffffffc, "ends inside the tensor");

__device__ __forceinline__ __amdgpu_buffer_rsrc_t word_descriptor(const uint8_t *p, int64_t bytes)
{
    return code_descriptor(p, whole_words(bytes));
}

// The tensor's bytes behind its last whole word, from the lowest byte on; 0 where there are none.
__device__ __forceinline__ u32 last_bytes(const uint8_t *p, int64_t bytes)
{
    u32 w = 0;
    for (int i = 0; i < (int)(bytes & 3); ++i) w |= (u32)p[whole_words(bytes) + i] << (8 * i);
    return w;
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

// Joins the tensor's last bytes to a run at byte offset `off` that may reach past the tensor; end: whole_words of the tensor.
template <int BITS>
__device__ __forceinline__ void join_last_bytes(u32 off, u32 end, u32 last, u32x4 (&raw)[ragged_regs<BITS>()])
{
#pragma unroll
    for (int i = 0; i <= BITS; ++i) raw[i >> 2][i & 3] |= (off & ~3u) + 4 * i == end ? last : 0u;
}

// load_run_ragged() for a run that may reach past the tensor, word by word (each with its own bound), with the tensor's last bytes.
template <int BITS>
__device__ __forceinline__ void load_run_bounded(const __amdgpu_buffer_rsrc_t rsrc, u32 off, u32 end, u32 last, u32x4 (&raw)[ragged_regs<BITS>()])
{
    constexpr int N = ragged_regs<BITS>();
    u32 w[4 * N];
#pragma unroll
    for (int i = 0; i < 4 * N; ++i) w[i] = i <= BITS ? __builtin_amdgcn_raw_buffer_load_b32(rsrc, (off & ~3u) + 4 * i, 0, 0) : 0u;
    w[4 * N - 1] = off & 3u;
#pragma unroll
    for (int p = 0; p < N; ++p) raw[p] = u32x4{w[4 * p], w[4 * p + 1], w[4 * p + 2], w[4 * p + 3]};
    if (end - (off & ~3u) <= 4u * BITS) join_last_bytes<BITS>(off, end, last, raw);   // hardly any run: skipped by whole waves
}

// The run's words in place, as load_run() would have fetched them from an aligned address.  last: bytes to join to the extra word.
template <int BITS>
__device__ __forceinline__ void align_run(const u32x4 *raw, u32x4 (&t)[(BITS + 3) / 4], u32 last = 0)
{
    const u32 shift = raw[ragged_regs<BITS>() - 1].w;
#pragma unroll
    for (int p = 0; p < (BITS + 3) / 4; ++p) t[p] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < BITS; ++i)
        t[i >> 2][i & 3] = __builtin_amdgcn_alignbyte(raw[(i + 1) >> 2][(i + 1) & 3] | (i + 1 == BITS ? last : 0u), raw[i >> 2][i & 3], shift);
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
