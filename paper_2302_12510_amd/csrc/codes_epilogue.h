// Write-back epilogue for calls that want the results as DyBit codes only (no fp32 output): the codes-only
// chain of Sec. III-B, where activations exist in memory as codes.
//
// The kernels that use it pass W as the first operand of the matrix instruction and A as the second, so that
// a lane holds one output row and, per 32 x 32 block, four runs of four neighbouring columns: accumulator v
// of a lane is column 8 (v / 4) + 4 (lane / 32) + v % 4 and row lane % 32 of its block.  Against the layout of
// store_strip_wb (a lane holds one column) this removes what that epilogue spends most on, next to the encoder
// itself, whose arithmetic is the same: codes are packed inside the lane, without cross-lane permutes; one
// exchange between the half-waves (v_permlane32_swap) per two blocks gives every lane the 32 neighbouring
// columns of one block, so that a row's codes leave as 128-bit words (4-bit codes: one store instruction per
// 2048 results, against 32 byte stores) and a shortcut given as codes arrives the same way; and a row past M
// is a lane that stores nothing, so the running maximum needs no selection per value.
// Per result: 9 vector-ALU instructions for 4- and 6-bit codes, 11 for 8-bit ones (20 there), and 1/32 of a store (2 there); a
// shortcut adds 6.  Maximum without a branch, shortcut product as one mixed-precision instruction, and three halves a minimum: 3 fewer per
// result with a shortcut than before (last layer below 24.9 -> 23.6 with its K loop, 84.4 -> 83.0 us; block 169.9 -> 168.7).
// What bounds the layers that use it is still vector-ALU issue: decode of A plus these.  The two instructions of difference are
// the shift that tests a value for a decision point and the extraction of its code: with 16 fraction bits the first is a
// minimum of half-words, the second is done by the byte permutes that pack (first layer below 57.0 -> 54.1 us with its encoder,
// block 182.6 -> 177.6).  A variant per sign of the format would save one more; it doubled the variants, and what the compiler
// keeps for all of them spilled 11 to 51 registers (first layer 60.4).  Measured, batch 64 to 128, store_strip_wb -> here: first layer of a
// residual network (802816 x 64 x 256, 8-bit, 4-bit codes out) with its input encoding 104.5 -> 82.8 us; a bottleneck block
// on 56 x 56 (401408 rows, 256 -> 64 -> 64 -> 256 channels, mixed widths, 6-bit codes out, 8-bit shortcut) 273 -> 186 us.
//
// It does not pay for fp32 results: 32 rows times 16 bytes per store instruction are partial cache lines.
#ifndef DYBIT_CODES_EPILOGUE_H
#define DYBIT_CODES_EPILOGUE_H

#include <type_traits>

#include "../../include/dybit.h"
#include "dybit_codec.h"
#include "gemm_args.h"
#include "requant.h"
#include "tile_epilogue.h"

namespace dybit {

// Per-column factors in LDS, staged once per workgroup: [columns] result factors (scales times the
// accumulators' power of two), then [columns] biases.
template <int CB> constexpr int column_bytes() { return CB * 32 * 8; }

// Fills them for columns n0 .. n0 + 32 CB - 1 (zeros past N, so that nothing from there reaches the maximum).
// Returns whether some factor leaves the float range when the power of two joins it (scales beyond 2^100):
// the factors are then stored without it.  Contains barriers: every thread of the workgroup calls it.
template <int CB, int ACC_EXP>
__device__ __forceinline__ bool stage_columns(const GemmArgs &g, const int64_t n0, float *cols)
{
    const float p = __uint_as_float((uint32_t)(127 + ACC_EXP) << 23);
    bool big = false;
    for (int c = threadIdx.x; c < CB * 32; c += blockDim.x) {
        const int64_t n = n0 + c;
        const float al = n < g.N ? (*g.a_scale) * g.w_scale[g.w_per_channel ? n : 0] : 0.0f;
        big |= fabsf(al) < __builtin_inff() && !(fabsf(al * p) < __builtin_inff());
        cols[c] = al * p;
        cols[CB * 32 + c] = (g.bias && n < g.N) ? g.bias[n] : 0.0f;
    }
    const bool any = __syncthreads_or(big);
    if (any) {
        for (int c = threadIdx.x; c < CB * 32; c += blockDim.x) {
            const int64_t n = n0 + c;
            cols[c] = n < g.N ? (*g.a_scale) * g.w_scale[g.w_per_channel ? n : 0] : 0.0f;
        }
        __syncthreads();
    }
    return any;
}

// The kernel's arguments, read again from the kernel-argument segment by each call: a persistent loop's uniform values are otherwise
// computed once, before the loop, and where they exceed the scalar registers (the few-channel kernel with a shortcut: 73 to 84
// spilled, each a v_readlane per strip) the scalar loads are cheaper.
__device__ __forceinline__ GemmArgs reload_args()
{
    struct Words { uint64_t w[sizeof(GemmArgs) / 8]; } words;
    static_assert(sizeof(Words) == sizeof(GemmArgs), "whole 64-bit words");
    uint64_t at = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();     // GemmArgs is the kernels' first argument
    asm volatile("" : "+s"(at));
    const auto *p = (const __attribute__((address_space(4))) uint64_t *)at;
#pragma unroll
    for (unsigned i = 0; i < sizeof(GemmArgs) / 8; ++i) words.w[i] = p[i];
    const GemmArgs a = __builtin_bit_cast(GemmArgs, words);
    return a;
}

// A scale, read with a scalar load (no kernel changes a scale that it reads).
__device__ __forceinline__ float scalar_scale(const float *p)
{
    return *(const __attribute__((address_space(4))) float *)(uint64_t)p;
}

// The output scale and its reciprocal, in scalar registers: once per workgroup, not once per strip.
struct OutScale {
    float s, rinv;
};
__device__ __forceinline__ OutScale out_scale(const GemmArgs &g)
{
    OutScale o;
    o.s = scalar_scale(g.q_scale);
    o.rinv = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(1.0f / o.s)));
    return o;
}

// Exchange between the half-waves: afterwards `a` holds, in both halves, what the lower half had in a (lower)
// and b (upper half's lanes), and `b` what the upper half had in a and b.
__device__ __forceinline__ void swap_halves(uint32_t &a, uint32_t &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

// 32 codes of a row (BITS words of 32 bits) <-> eight groups of four codes.
template <int BITS>
__device__ __forceinline__ void words_to_quads(const uint32_t (&w)[BITS], uint32_t (&t)[8])
{
    if constexpr (BITS == 8) {
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = w[i];
    } else if constexpr (BITS == 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { t[2 * i] = w[i] & 0xffffu; t[2 * i + 1] = w[i] >> 16; }
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {                                   // bits above 24 are ignored by the decoder
            t[4 * i] = w[3 * i];
            t[4 * i + 1] = __builtin_amdgcn_alignbit(w[3 * i + 1], w[3 * i], 24);
            t[4 * i + 2] = __builtin_amdgcn_alignbit(w[3 * i + 2], w[3 * i + 1], 16);
            t[4 * i + 3] = w[3 * i + 2] >> 8;
        }
    }
}
template <int BITS>
__device__ __forceinline__ void quads_to_words(const uint32_t (&t)[8], uint32_t (&w)[BITS])
{
    if constexpr (BITS == 8) {
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = t[i];
    } else {
        static_assert(BITS == 6, "4-bit codes are packed by permutes");
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            w[3 * i] = t[4 * i] | (t[4 * i + 1] << 24);
            w[3 * i + 1] = (t[4 * i + 1] >> 8) | (t[4 * i + 2] << 16);
            w[3 * i + 2] = (t[4 * i + 2] >> 16) | (t[4 * i + 3] << 8);
        }
    }
}

// 32 consecutive codes of the lane's row, BITS words at byte offset `off` (a multiple of 4): whole words, each
// with its own bound when the block reaches past the row (`left` bytes of the row remain).
template <int BITS>
__device__ __forceinline__ void store_words(const __amdgpu_buffer_rsrc_t rsrc, uint32_t off, const uint32_t (&w)[BITS], bool whole, int left)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    if (whole) {
#pragma unroll
        for (int i = 0; i + 4 <= BITS; i += 4)
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{w[i], w[i + 1], w[i + 2], w[i + 3]}, rsrc, off + 4 * i, 0, 0);
        if constexpr (BITS == 6) __builtin_amdgcn_raw_buffer_store_b64(u32x2{w[4], w[5]}, rsrc, off + 16, 0, 0);
    } else {
#pragma unroll
        for (int i = 0; i < BITS; ++i)
            __builtin_amdgcn_raw_buffer_store_b32(w[i], rsrc, 4 * i < left ? off + 4 * i : fast::kOob, 0, 0);
    }
}
template <int BITS>
__device__ __forceinline__ void load_words(const __amdgpu_buffer_rsrc_t rsrc, uint32_t off, uint32_t (&w)[BITS], bool whole, int left)
{
    if (whole) {
#pragma unroll
        for (int i = 0; i + 4 <= BITS; i += 4) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + 4 * i, 0, 0);
            w[i] = v[0]; w[i + 1] = v[1]; w[i + 2] = v[2]; w[i + 3] = v[3];
        }
        if constexpr (BITS == 6) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, off + 16, 0, 0);
            w[4] = v[0]; w[5] = v[1];
        }
    } else {
#pragma unroll
        for (int i = 0; i < BITS; ++i) w[i] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, 4 * i < left ? off + 4 * i : fast::kOob, 0, 0);
    }
}

// Four shortcut codes of RB bits in the low bits of t -> fl(s value), the numbers dybit_dequantize writes: the
// arithmetic decoder of dybit_codec.h with the format's constants in (uniform) registers, brought from its
// 2^-14 scale to the value by one packed multiplication (a power of two: exact) before the one that rounds.
struct ShortcutFormat {
    uint32_t mag_mask, k2, sign_mask, sign_shift;   // magnitude bits in every byte; constant of the subtraction; 0x80008000 or 0; 16 - bits
    _Float16 base;
    float s;
};
__device__ __forceinline__ ShortcutFormat shortcut_format(const GemmArgs &g)
{
    const int m = g.res_signed ? g.res_bits - 1 : g.res_bits;
    ShortcutFormat f;
    f.mag_mask = ((1u << m) - 1u) * 0x01010101u;
    f.k2 = ((uint32_t)(15 + m) << 10) * 0x00010001u;
    f.sign_mask = g.res_signed ? 0x80008000u : 0u;
    f.sign_shift = 16u - (uint32_t)g.res_bits;
    f.base = (_Float16)(float)(1024 + (1 << m));
    f.s = scalar_scale(g.res_scale);
    return f;
}
// One instruction (v_fma_mix_f32 takes the half as it is); adding zero rounds nothing, and only a product of -0 comes out as +0,
// which neither a code nor the maximum shows.
__device__ __forceinline__ float shortcut_product(_Float16 v, float s)
{
    return __builtin_fmaf((float)v, s, 0.0f);        // rounded here, before it is added
}
template <int RB>
__device__ __forceinline__ void shortcut_values(uint32_t t, const ShortcutFormat &f, float (&r)[4])
{
    using fast::f16x2;
    if constexpr (RB == 6) t = fast::unpack_six(t);
    else if constexpr (RB == 4) t = (t & 0xfu) | ((t << 4) & 0xf00u) | ((t << 8) & 0xf0000u) | ((t << 12) & 0xf000000u);
    const uint32_t c = t & f.mag_mask;
    const uint32_t h0 = __builtin_amdgcn_perm(0x64646464u, c, 0x04020400u), h1 = __builtin_amdgcn_perm(0x64646464u, c, 0x04030401u);
    const uint32_t d0 = fast::recip_decode_pair(h0, f.base, f.k2) | ((t << f.sign_shift) & f.sign_mask);
    const uint32_t d1 = fast::recip_decode_pair(h1, f.base, f.k2) | ((t << (f.sign_shift - 8u)) & f.sign_mask);
    const f16x2 up = {(_Float16)16384.0f, (_Float16)16384.0f};
    const f16x2 v0 = __builtin_bit_cast(f16x2, d0) * up, v1 = __builtin_bit_cast(f16x2, d1) * up;
    r[0] = shortcut_product(v0[0], f.s);
    r[1] = shortcut_product(v1[0], f.s);
    r[2] = shortcut_product(v0[1], f.s);
    r[3] = shortcut_product(v1[1], f.s);
}

// The least of eight lower halves.
__device__ __forceinline__ uint16_t lower_halves_min(const uint32_t (&z)[8])
{
    uint32_t a, b, c;                                // the compiler's own form pairs them up with permutes: eight instructions
    asm("v_min3_u16 %0, %1, %2, %3" : "=v"(a) : "v"(z[0]), "v"(z[1]), "v"(z[2]));
    asm("v_min3_u16 %0, %1, %2, %3" : "=v"(b) : "v"(z[3]), "v"(z[4]), "v"(z[5]));
    asm("v_min3_u16 %0, %1, %2, %3" : "=v"(c) : "v"(a), "v"(z[6]), "v"(z[7]));
    return min((uint16_t)b, (uint16_t)c);
}

// The strip of 32 rows by 32 CB columns a wave holds or, STACKED, of 32 CB rows by 32 columns (block j is then rows 32 j ..
// + 31).  RB: bits of the shortcut's codes (0: none).  cols: the factors stage_columns has left in LDS, for the strip's first
// column on, the biases `staged` columns behind.  Returns the lane's maximum of |result|.
template <int CB, int RB, int BITS, bool STACKED = false>
__device__ __forceinline__ float store_strip_codes(const GemmArgs &g, const fast::f32x16 (&acc)[CB], const int64_t m_strip,
                                                   const int64_t n0, const int rows, const float *cols, const OutScale os, const int staged = CB * 32)
{
    static_assert(CB % 2 == 0, "column blocks are stored in pairs");
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, kq = lane >> 5;
    int row = lane & 31;
    asm volatile("" : "+v"(row));                                       // see store_strip
    const uint32_t qrow = (uint32_t)g.q_row_bytes, rrow = RB ? (uint32_t)g.res_row_bytes : 0u;
    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(g.q_out + m_strip * g.q_row_bytes, 0,
                                                                        (int)((uint32_t)rows * qrow), 0x00020000);
    const __amdgpu_buffer_rsrc_t rres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(RB ? g.res_codes + m_strip * g.res_row_bytes : reinterpret_cast<const uint8_t *>(g.a_scale)), 0,
        RB ? (int)((uint32_t)rows * rrow) : 0, 0x00020000);
    const Requant rqp = make_requant(os.s, os.rinv, BITS, g.q_signed);
    if (!rqp.ok && m_strip == 0 && n0 == 0 && lane == 0) *g.async_error = DYBIT_ERR_BAD_SCALE;   // no codes, flag the call
    ShortcutFormat sf{};
    if (RB) sf = shortcut_format(g);
    uint32_t floor_bits = (uint32_t)__builtin_amdgcn_readfirstlane(g.relu ? 0 : 0x7fc00000);
    asm volatile("" : "+s"(floor_bits));                                // see store_strip_wb
    const float relu_floor = __uint_as_float(floor_bits);
    constexpr int GB = requant_fraction<BITS>();
    constexpr uint32_t kOnes = BITS == 8 ? 0x01010101u : BITS == 6 ? 0x00041041u : 0x11111111u;   // a word's fields: four codes, 4-bit: eight
    constexpr uint32_t kSign = kOnes << (BITS - 1), kMag = kSign - kOnes;
    const uint32_t mag_fields = kOnes * ((1u << rqp.m) - 1u);
    float mx = 0.0f;

    // the lane's own 32 shortcut codes of each block pair (lower half-wave: first block, upper: second)
    uint32_t rw[RB ? RB : 1];
    auto block_base = [&](int jp) { return (uint32_t)(STACKED ? n0 : n0 + 64 * jp + 32 * kq); };
    auto whole_pair = [&](int jp) { return (STACKED ? n0 + 32 : n0 + 64 * (jp + 1)) <= g.N; };   // uniform
    auto lane_row = [&](int jp) { return (uint32_t)(STACKED ? 64 * jp + 32 * kq + row : row); };
    auto request_shortcut = [&](int jp) {
        if constexpr (RB != 0) {
            const uint32_t at = block_base(jp) * RB / 8;
            load_words<RB>(rres, at < rrow ? lane_row(jp) * rrow + at : fast::kOob, rw, whole_pair(jp), (int)rrow - (int)at);
        }
    };
    request_shortcut(0);
#pragma unroll
    for (int jp = 0; jp < CB / 2; ++jp) {
        uint32_t rt[2][4];                                              // shortcut codes of the lane's quads, per block of the pair
        if constexpr (RB != 0) {
            uint32_t t[8];
            words_to_quads<RB>(rw, t);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                rt[0][q] = t[2 * q]; rt[1][q] = t[2 * q + 1];
                swap_halves(rt[0][q], rt[1][q]);
            }
            if (jp + 1 < CB / 2) request_shortcut(jp + 1);
        }
        uint32_t out[2][BITS == 4 ? 2 : 4];                             // packed quads of the two blocks
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            const int j = 2 * jp + jb;
            float block_max = 0.0f;
#pragma unroll
            for (int h = 0; h < 2; ++h) {                               // two quads at a time: fewer live registers
                float c[8];
                uint32_t zb[8];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int q = 2 * h + i;
                    const f32x4 al = *reinterpret_cast<const f32x4 *>(cols + (STACKED ? 0 : 32 * j) + 8 * q + 4 * kq);
                    const f32x4 bv = *reinterpret_cast<const f32x4 *>(cols + staged + (STACKED ? 0 : 32 * j) + 8 * q + 4 * kq);
                    float r[4];
                    if constexpr (RB != 0) shortcut_values<RB>(rt[jb][q], sf, r);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        float v = fmaf(acc[j][4 * q + u], al[u], bv[u]);
                        if constexpr (RB != 0) v += r[u];
                        c[4 * i + u] = fmaxf(v, relu_floor);
                    }
                }
                float &top = STACKED ? block_max : mx;                  // kept whether asked for or not: behind a branch the magnitudes
#pragma unroll                                                          // would be computed by themselves, two instructions against one
                for (int u = 0; u < 8; u += 2) top = fmaxf(fmaxf(top, fabsf(c[u])), fabsf(c[u + 1]));
#pragma unroll
                for (int u = 0; u < 8; ++u) zb[u] = requant_lower<BITS>(c[u], rqp);
                bool settle;                                            // whether some fraction reads zero
                if constexpr (GB == 16) {
                    settle = lower_halves_min(zb) == 0;
                } else {
                    uint32_t key = 0xffffffffu;
#pragma unroll
                    for (int u = 0; u < 8; ++u) key = min(key, zb[u] << (32 - GB));
                    settle = key == 0;
                }
                if (__builtin_amdgcn_ballot_w64(settle)) {              // some value on a decision point: the exact decision,
                    uint32_t open = 0;                                  // a lane's values one after the other
#pragma unroll
                    for (int u = 0; u < 8; ++u) open |= (zb[u] << (32 - GB)) == 0u ? 1u << u : 0u;
                    while (__builtin_amdgcn_ballot_w64(open != 0u)) {
                        const uint32_t first = open & (0u - open);
                        float x = 0.0f;
                        uint32_t k = 0;
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            if (first & (1u << u)) { x = c[u]; k = requant_complement<BITS>(zb[u], rqp); }
                        const uint32_t top = (1u << rqp.m) - 1u, fixed = (top - requant_settle(x, top + 1u - k, rqp)) << GB;
#pragma unroll
                        for (int u = 0; u < 8; ++u) zb[u] = (first & (1u << u)) ? fixed : zb[u];
                        open &= open - 1u;
                    }
                }
                // the complements of the magnitude codes, packed: bytes 2 of the words, 8-bit codes by extraction
                constexpr int PER = BITS == 4 ? 8 : 4, WORDS = 8 / PER;
                uint32_t w[WORDS];
                if constexpr (BITS == 4) {
                    const uint32_t even = __builtin_amdgcn_perm(zb[2], zb[0], 0x0c0c0602u), even_up = __builtin_amdgcn_perm(zb[6], zb[4], 0x06020c0cu);
                    const uint32_t odd = __builtin_amdgcn_perm(zb[3], zb[1], 0x0c0c0602u) | __builtin_amdgcn_perm(zb[7], zb[5], 0x06020c0cu);
                    w[0] = (odd << 4 | even) | even_up;
                } else if constexpr (BITS == 6) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const uint32_t even = __builtin_amdgcn_perm(zb[4 * i + 2], zb[4 * i], 0x0c060c02u), odd = __builtin_amdgcn_perm(zb[4 * i + 3], zb[4 * i + 1], 0x0c060c02u);
                        const uint32_t pairs = odd << 6 | even;          // 12 bits in each half
                        w[i] = (pairs & 0xfffu) | ((pairs >> 4) & ~0xfffu);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        uint32_t k[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) k[u] = requant_complement<BITS>(zb[4 * i + u], rqp);
                        w[i] = (((k[3] << BITS | k[2]) << BITS | k[1]) << BITS) | k[0];
                    }
                }
#pragma unroll
                for (int i = 0; i < WORDS; ++i) {
                    w[i] ^= mag_fields;
                    if (rqp.is_signed) {                                // uniform
#pragma unroll
                        for (int u = 0; u < PER; ++u) w[i] |= ((__float_as_uint(c[PER * i + u]) >> rqp.sign_shift) & rqp.sign_mask) << (u * BITS);
                        // a field whose magnitude is zero loses its sign
                        const uint32_t t = w[i] & kMag;
                        w[i] = t | (w[i] & (t + kMag) & kSign);
                    }
                    out[jb][WORDS * h + i] = w[i];
                }
            }
            if (STACKED) mx = fmaxf(mx, 32 * j + row < rows ? block_max : 0.0f);
        }
        uint32_t words[BITS];
        if constexpr (BITS == 4) {                                      // out: two groups of four codes in a word
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                swap_halves(out[0][h], out[1][h]);                      // lower half: block 0, upper half: block 1
                words[2 * h] = __builtin_amdgcn_perm(out[1][h], out[0][h], 0x05040100u);
                words[2 * h + 1] = __builtin_amdgcn_perm(out[1][h], out[0][h], 0x07060302u);
            }
        } else {
            uint32_t t[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                swap_halves(out[0][q], out[1][q]);
                t[2 * q] = out[0][q];
                t[2 * q + 1] = out[1][q];
            }
            quads_to_words<BITS>(t, words);
        }
        const uint32_t at = block_base(jp) * BITS / 8;
        const uint32_t off = (rqp.ok && at < qrow) ? lane_row(jp) * qrow + at : fast::kOob;
        store_words<BITS>(rq, off, words, whole_pair(jp), (int)qrow - (int)at);
    }
    return STACKED || row < rows ? mx : 0.0f;
}

// Picks the variant for the call's formats.  Q and R: bits of the codes and of the shortcut's codes (0: none) in a kernel that was
// compiled for them; Q = 0: any.
template <int CB, bool STACKED, int Q = 0, int R = 0>
__device__ __forceinline__ float strip_codes(const GemmArgs &g, const fast::f32x16 (&acc)[CB], const int64_t m_strip, const int64_t n0, const int rows,
                                             const float *cols, const OutScale os, const int staged)
{
#define DYBIT_CODES_STRIP(RB_) \
    return g.q_bits == 4 ? store_strip_codes<CB, RB_, 4, STACKED>(g, acc, m_strip, n0, rows, cols, os, staged) \
         : g.q_bits == 8 ? store_strip_codes<CB, RB_, 8, STACKED>(g, acc, m_strip, n0, rows, cols, os, staged) \
                         : store_strip_codes<CB, RB_, 6, STACKED>(g, acc, m_strip, n0, rows, cols, os, staged)
    if constexpr (Q != 0) return store_strip_codes<CB, R, Q, STACKED>(g, acc, m_strip, n0, rows, cols, os, staged);
    if (!g.res_codes) { DYBIT_CODES_STRIP(0); }
    if (g.res_bits == 8) { DYBIT_CODES_STRIP(8); }
    if (g.res_bits == 4) { DYBIT_CODES_STRIP(4); }
    DYBIT_CODES_STRIP(6);
#undef DYBIT_CODES_STRIP
}

// The kernel for a call's formats: what f(Q, R) returns, with strip_codes' Q and R as constants.
template <int V> using Bits = std::integral_constant<int, V>;
template <typename F> inline auto kernel_for_codes(const GemmArgs &g, F f)
{
    auto with_shortcut = [&](auto q) {
        return !g.res_codes ? f(q, Bits<0>{}) : g.res_bits == 8 ? f(q, Bits<8>{}) : g.res_bits == 4 ? f(q, Bits<4>{}) : f(q, Bits<6>{});
    };
    return g.q_bits == 4 ? with_shortcut(Bits<4>{}) : g.q_bits == 8 ? with_shortcut(Bits<8>{}) : with_shortcut(Bits<6>{});
}

// big: what stage_columns returned; acc is brought to scale here then.
template <int CB, int ACC_EXP, int Q = 0, int R = 0>
__device__ __forceinline__ float epilogue_strip_codes(const GemmArgs &g, fast::f32x16 (&acc)[CB], const int64_t m_strip, const int64_t n0,
                                                      const float *cols, const bool big, const OutScale os)
{
    const int64_t rows_left = g.M - m_strip;
    const int rows = rows_left >= 32 ? 32 : rows_left > 0 ? (int)rows_left : 0;
    if (ACC_EXP != 0 && big) {
#pragma unroll
        for (int j = 0; j < CB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][v] = acc_value<ACC_EXP>(acc[j][v]);
    }
    return strip_codes<CB, false, Q, R>(g, acc, m_strip, n0, rows, cols, os, CB * 32);
}

}  // namespace dybit
#endif
