// Grouped convolution on DyBit codes for gfx950 in one launch: every group is a narrow product of its own (Cout / groups
// columns, kh kw Cin / groups codes of K), and a launch per group leaves most of the device idle -- eight groups of 32
// channels on 64 x 14 x 14 took eight launches of 13 us on the general kernel.
//
// Weight-stationary, as gemm_ws.hip: a workgroup decodes the weights of one group (of up to 64 of its columns) into LDS
// once and its eight waves walk over 256-row slabs of output pixels without further barriers; the workgroups of the groups
// walk side by side on one XCD, so that an image line (which holds the channels of several groups) is read from HBM once.
// What is new is how a lane reaches its 32 codes of a K step: a group's channels are few, so the run is made of pieces of
// P = 32, 16 or 8 codes, each inside one filter tap.  Where the pieces lie -- filter row, filter column, byte offset -- is
// the same for every output pixel, so a table of all pieces is built in LDS once and the two half-waves (k quarters) read
// their entries as broadcasts.  K is padded to a multiple of 64 by pieces that read code 0; the weights beside them need no
// clearing (a finite value times zero).
//
// What bounds it: vector-ALU issue (decoding A for 32 or 64 columns of use) and, at the benchmark's size, the fp32 results.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dybit_codec.h"
#include "gemm_args.h"
#include "ragged.h"
#include "tile_common.h"
#include "tile_epilogue.h"

#ifndef DYBIT_GROUP_W
#error "compile with -DDYBIT_GROUP_W=<weight format id> (0: 4-bit, 2: 8-bit, 4: 6-bit, 6: 2-bit; signed)"
#endif

namespace dybit {
namespace group {

using namespace fast;

constexpr int kThreads = 512, kSlab = 256;

struct GroupArgs {
    int groups, Cg, Cog;             // groups of the convolution, input and output channels of each
    int parts;                       // workgroups that share a group's columns (32 CB each)
    int slabs, ktiles, row_bytes;    // row slabs; K steps of 64; LDS bytes of a weight row
};

template <int FMT_A, int FMT_W, int P, int CB>
__global__ __launch_bounds__(kThreads, 4) void group_conv_kernel(const GemmArgs g, const GroupArgs c)
{
    using CA = Codec<FMT_A>;
    using CW = Codec<FMT_W>;
    constexpr int BA = CA::BITS, BW = CW::BITS, PIECES = 32 / P, WORDS = P * BA / 32;   // pieces of a run, words of a piece
    constexpr int NA = (BA + 3) / 4;
    static_assert(P * BA % 32 == 0, "a piece is whole words");
    extern __shared__ __attribute__((aligned(16))) char lds[];
    int2 *const pieces = reinterpret_cast<int2 *>(lds + CB * 32 * c.row_bytes);         // {byte offset, filter row << 16 | column; negative: none}

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), kq = lane >> 5;
    // workgroups of neighbouring groups are neighbours in an XCD's launch order and follow the same slabs
    const int total = c.groups * c.parts, local = (int)blockIdx.x >> 3;
    const int mine = local % total, walker = (local / total) * 8 + ((int)blockIdx.x & 7), walkers = (int)gridDim.x / total;
    const int gi = mine / c.parts, n0 = gi * c.Cog + (mine % c.parts) * (32 * CB), n_end = (gi + 1) * c.Cog;
    const int K = (int)g.K;

    // ---- weights of the group's columns, decoded once; rows are K codes, which may start at any byte: fetched word by word
    {
        const __amdgpu_buffer_rsrc_t rsrcW = word_descriptor(g.W, g.w_bytes);
        const u32 w_end = (u32)whole_words(g.w_bytes), w_last = last_bytes(g.W, g.w_bytes);
        const int runs = c.ktiles * 2;
        for (int r = tid; r < CB * 32 * runs; r += kThreads) {
            const int row = r / runs, run = r - row * runs;
            const u32 first = (u32)(((int64_t)(n0 + row) * K + run * 32) * BW / 8);
            const u32 off = n0 + row < n_end && run * 32 < K ? first : kOob;
            u32x4 raw[ragged_regs<BW>()], t[(BW + 3) / 4];
            load_run_bounded<BW>(rsrcW, off, w_end, w_last, raw);
            align_run<BW>(raw, t);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                u32 d[4];
                decode_eight<FMT_W>(t, q, d);
                *reinterpret_cast<u32x4 *>(lds + row * c.row_bytes + run * 64 + q * 16) = u32x4{d[0], d[1], d[2], d[3]};
            }
        }
    }
    // ---- the pieces of K: P codes of one filter tap; past K: none
    const int n_pieces = c.ktiles * 2 * PIECES;
    for (int i = tid; i < n_pieces; i += kThreads) {
        const int k = i * P, tap = k / c.Cg, ch = k - tap * c.Cg, fr = tap / g.kw, fs = tap - fr * g.kw;
        pieces[i] = k < K ? make_int2((fr * g.Wd + fs) * g.pix_bytes + ch * BA / 8, fr << 16 | fs)   : make_int2(0, -1);
    }
    __syncthreads();

    GemmArgs ge = g;                                                 // what the epilogue sees: columns up to the group's end
    ge.N = n_end;
    const __amdgpu_buffer_rsrc_t rsrcA = code_descriptor(g.A, g.a_bytes);
    const u32 rdW = (u32)(lane & 31) * (u32)c.row_bytes + (u32)kq * 64;   // K step adds 128 B, block kk 16 B, column block j 32 rows
    const u32 plane = (u32)g.Ho * (u32)g.Wo;

    float run_max = 0.0f;
    for (int slab = walker; slab < c.slabs; slab += walkers) {
        const int64_t m_strip = (int64_t)slab * kSlab + wave * 32;
        if (m_strip >= g.M) continue;                                // uniform per wave; no barriers below
        const u32 mm = m_strip + (lane & 31) < g.M ? (u32)m_strip + (lane & 31) : 0u;   // a row past M: pixel 0, not stored
        const u32 b = mm / plane, rem = mm - b * plane, ho = rem / (u32)g.Wo, wo = rem - ho * (u32)g.Wo;
        const int hi0 = (int)ho * g.stride - g.pad, wi0 = (int)wo * g.stride - g.pad;
        const int offA = (((int)b * g.H + hi0) * g.Wd + wi0) * g.pix_bytes + gi * (c.Cg * BA / 8);   // the image is under 2 GiB; a group is whole words

        auto load_A = [&](int kt, u32x4 (&raw)[NA]) {
            u32 w[4 * NA];
#pragma unroll
            for (int i = 0; i < 4 * NA; ++i) w[i] = 0;
#pragma unroll
            for (int p = 0; p < PIECES; ++p) {
                const int2 at = kt < c.ktiles ? pieces[(kt * 2 + kq) * PIECES + p] : make_int2(0, -1);
                const bool in = at.y >= 0 && (unsigned)(hi0 + (at.y >> 16)) < (unsigned)g.H && (unsigned)(wi0 + (at.y & 0xffff)) < (unsigned)g.Wd;
                const u32 off = in ? (u32)(offA + at.x) : kOob;      // padding reads code 0
                u32 *o = w + p * WORDS;
                int i = 0;
#pragma unroll
                for (; i + 4 <= WORDS; i += 4) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rsrcA, off + 4 * i, 0, 0);
                    o[i] = v[0]; o[i + 1] = v[1]; o[i + 2] = v[2]; o[i + 3] = v[3];
                }
                if constexpr (WORDS % 4 >= 2) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b64(rsrcA, off + 4 * (WORDS & ~3), 0, 0);
                    o[WORDS & ~3] = v[0]; o[(WORDS & ~3) + 1] = v[1];
                }
                if constexpr (WORDS % 2 == 1) o[WORDS - 1] = __builtin_amdgcn_raw_buffer_load_b32(rsrcA, off + 4 * (WORDS - 1), 0, 0);
            }
#pragma unroll
            for (int p = 0; p < NA; ++p) raw[p] = u32x4{w[4 * p], w[4 * p + 1], w[4 * p + 2], w[4 * p + 3]};
        };

        f32x16 acc[CB];
#pragma unroll
        for (int j = 0; j < CB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][v] = 0.0f;
        auto contract = [&](int kt, const u32x4 (&raw)[NA]) {
            const char *wk = lds + rdW + kt * 128;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                u32 d[4];
                decode_eight<FMT_A>(raw, q, d);
                const f16x8 fa = __builtin_bit_cast(f16x8, u32x4{d[0], d[1], d[2], d[3]});
#pragma unroll
                for (int j = 0; j < CB; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa, *reinterpret_cast<const f16x8 *>(wk + q * 16 + j * 32 * c.row_bytes), acc[j], 0, 0, 0);
            }
        };
        // the codes of the next two K steps are in flight while one is decoded
        u32x4 raw0[NA], raw1[NA];
        load_A(0, raw0);
        load_A(1, raw1);
        for (int kt = 0; kt < c.ktiles; kt += 2) {
            contract(kt, raw0);
            load_A(kt + 2, raw0);
            if (kt + 1 < c.ktiles) contract(kt + 1, raw1);
            load_A(kt + 3, raw1);
        }
        run_max = fmaxf(run_max, epilogue_strip<CB, false, false, CA::ACC_EXP + CW::ACC_EXP>(ge, acc, m_strip, n0));
    }

    // ---- running maximum: one merge per workgroup (see gemm_ws.hip)
    if (g.absmax_bits) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) run_max = fmaxf(run_max, __shfl_xor(run_max, off, 64));
        __syncthreads();                                             // every wave is done with the weight tile
        float *red = reinterpret_cast<float *>(lds);
        if (lane == 0) red[wave] = run_max;
        __syncthreads();
        if (tid == 0) {
            float mx = red[0];
#pragma unroll
            for (int w = 1; w < kThreads / 64; ++w) mx = fmaxf(mx, red[w]);
            const uint32_t bits = __float_as_uint(mx);
            if (bits > __hip_atomic_load(g.absmax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(g.absmax_bits, bits);
        }
    }
}

// The sizes behind the LDS request and the grid are computed in 64 bits: K goes up to 2^31, groups x columns to as many.
template <int FA, int FW, int P, int CB>
static bool launch_p(const GemmArgs &g, GroupArgs c, hipStream_t st)
{
    if constexpr (P * Codec<FA>::BITS % 32 != 0) {
        return false;
    } else {
        const int64_t ktiles = (g.K + 63) / 64, row_bytes = ktiles * 128 + 16;
        const int64_t lds_bytes = CB * 32 * row_bytes + ktiles * 2 * (32 / P) * 8;
        if (lds_bytes > kLdsLimit) return false;
        c.ktiles = (int)ktiles;
        c.row_bytes = (int)row_bytes;
        c.parts = (c.Cog + 32 * CB - 1) / (32 * CB);
        c.slabs = (int)((g.M + kSlab - 1) / kSlab);
        // resident: two workgroups per compute unit (512 threads at 128 registers) where their weights fit
        const int64_t columns = (int64_t)c.groups * c.parts, resident = lds_bytes <= 80 * 1024 ? 512 : 256;
        int64_t walkers = resident / (8 * columns) * 8;
        if (walkers < 8) walkers = 8;
        if (walkers > (c.slabs + 7) / 8 * 8) walkers = (c.slabs + 7) / 8 * 8;
        const int64_t grid = walkers * columns;
        if (grid * kThreads > 0xffffffff) return false;               // a launch is less than 2^32 threads
        auto k = group_conv_kernel<FA, FW, P, CB>;
        note_kernel(DYBIT_KERNEL_F16_GROUP);
        note_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit));
        hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(kThreads), (int)lds_bytes, st, g, c);
        return true;
    }
}

template <int FA, int FW>
static bool launch(const GemmArgs &g, int groups, hipStream_t st)
{
    GroupArgs c{};
    c.groups = groups;
    c.Cg = g.Cin;
    c.Cog = (int)(g.N / groups);
    const bool one = c.Cog <= 32;
    if (c.Cg % 32 == 0) return one ? launch_p<FA, FW, 32, 1>(g, c, st) : launch_p<FA, FW, 32, 2>(g, c, st);
    if (c.Cg % 16 == 0) return one ? launch_p<FA, FW, 16, 1>(g, c, st) : launch_p<FA, FW, 16, 2>(g, c, st);
    return one ? launch_p<FA, FW, 8, 1>(g, c, st) : launch_p<FA, FW, 8, 2>(g, c, st);
}

}  // namespace group

#define DYBIT_GROUP_NAME2(w) launch_group_conv_w##w
#define DYBIT_GROUP_NAME(w) DYBIT_GROUP_NAME2(w)
bool DYBIT_GROUP_NAME(DYBIT_GROUP_W)(const GemmArgs &g, int a_bits, int groups, hipStream_t st)
{
    using namespace fast;
    const int fa = (a_bits == 8 ? F8S : a_bits == 6 ? F6S : a_bits == 2 ? F2S : F4S) + (g.a_signed ? 0 : 1);
    switch (fa) {
        case F2S: return group::launch<F2S, DYBIT_GROUP_W>(g, groups, st);
        case F2U: return group::launch<F2U, DYBIT_GROUP_W>(g, groups, st);
        case F4S: return group::launch<F4S, DYBIT_GROUP_W>(g, groups, st);
        case F4U: return group::launch<F4U, DYBIT_GROUP_W>(g, groups, st);
        case F6S: return group::launch<F6S, DYBIT_GROUP_W>(g, groups, st);
        case F6U: return group::launch<F6U, DYBIT_GROUP_W>(g, groups, st);
        case F8S: return group::launch<F8S, DYBIT_GROUP_W>(g, groups, st);
        case F8U: return group::launch<F8U, DYBIT_GROUP_W>(g, groups, st);
        default: return false;
    }
}

}  // namespace dybit
