// Chooses between the tiled MFMA kernels of the DyBit matrix product.
//
// All need signed weights, K (convolution: Cin) a multiple of 64 (2- and 6-bit operands on the 256 x 256 kernel: of 128) so that
// a 64-wide k group is one run of whole 128-bit loads inside one filter tap, 16-byte aligned
// code buffers, and buffers below 2 GiB (32-bit buffer offsets).  A matrix product with any other K from 64 on (rows that
// start at any byte, ragged.h) runs on the small-output and the 128 x 128 fp16 kernel.  The 256 x 256 kernel does the
// least decode work per MFMA and is used when its tiles can fill the 256 compute units, N is
// wide enough for them and K is long enough for the main loop to outweigh the epilogue; the
// 128 x 128 kernel takes the rest.  dybit_set_option (initial values: the environment, read once)
// overrides the choice whenever the named kernel's preconditions hold; every launch records the kernel
// it started, which dybit_last_gemm_kernel reports, so a test can tell which kernel it exercised.
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>

#include "../../include/dybit.h"
#include "gemm_args.h"

namespace dybit {

namespace {

std::atomic<int> opt_kernel{0}, opt_mfma_f16{0}, opt_mid_tile{0}, opt_mid_kgroups{0}, opt_ws_off{0};
// A look of the max-abs kernel's last workgroup takes 0.2 us (100000 of them 23 ms): some 15 s, where a launch ends within milliseconds.
constexpr unsigned kAbsmaxLooks = 1u << 26;
std::atomic<unsigned> opt_absmax_looks{kAbsmaxLooks};
thread_local int last_kernel = DYBIT_KERNEL_NONE;
thread_local hipError_t pending_hip_error = hipSuccess;

// name / value -> option; false for an unknown pair.  "auto" resets an option.
bool apply_option(const char *name, const char *value)
{
    const bool is_auto = !strcmp(value, "auto");
    if (!strcmp(name, "gemm_kernel")) {
        const int v = is_auto ? 0 : !strcmp(value, "general") ? DYBIT_FORCE_GENERAL : !strcmp(value, "mid") ? DYBIT_FORCE_MID
                    : !strcmp(value, "large") ? DYBIT_FORCE_LARGE : !strcmp(value, "ws") ? DYBIT_FORCE_WS
                    : !strcmp(value, "small") ? DYBIT_FORCE_SMALL : !strcmp(value, "few") ? DYBIT_FORCE_FEW
                    : !strcmp(value, "patch") ? DYBIT_FORCE_PATCH : !strcmp(value, "six") ? DYBIT_FORCE_SIX : -1;
        if (v < 0) return false;
        opt_kernel = v;
    } else if (!strcmp(name, "gemm_mfma")) {
        if (!is_auto && strcmp(value, "f16")) return false;
        opt_mfma_f16 = is_auto ? 0 : 1;
    } else if (!strcmp(name, "mid_tile")) {
        const int v = is_auto ? 0 : !strcmp(value, "64") ? 64 : !strcmp(value, "128") ? 128 : -1;
        if (v < 0) return false;
        opt_mid_tile = v;
    } else if (!strcmp(name, "mid_kgroups")) {
        const int v = is_auto ? 0 : !strcmp(value, "1") ? 1 : !strcmp(value, "2") ? 2 : -1;
        if (v < 0) return false;
        opt_mid_kgroups = v;
    } else if (!strcmp(name, "gemm_ws")) {
        if (!is_auto && strcmp(value, "off")) return false;
        opt_ws_off = is_auto ? 0 : 1;
    } else if (!strcmp(name, "absmax_looks")) {
        char *end = nullptr;
        const unsigned long v = is_auto ? kAbsmaxLooks : strtoul(value, &end, 10);
        if (v < 1 || v > kAbsmaxLooks || (end && *end)) return false;
        opt_absmax_looks = (unsigned)v;
    } else {
        return false;
    }
    return true;
}

// The environment gives the initial values, once; values it cannot hold are ignored.
void options_from_environment()
{
    static const bool done = [] {
        static const char *const vars[][2] = {{"DYBIT_GEMM_KERNEL", "gemm_kernel"}, {"DYBIT_GEMM_MFMA", "gemm_mfma"},
                                              {"DYBIT_MID_TILE", "mid_tile"}, {"DYBIT_MID_KGROUPS", "mid_kgroups"}};
        for (const auto &v : vars) {
            const char *e = getenv(v[0]);
            if (e && *e) apply_option(v[1], e);
        }
        const char *ws = getenv("DYBIT_GEMM_WS");
        if (ws && !strcmp(ws, "0")) apply_option("gemm_ws", "off");
        return true;
    }();
    (void)done;
}

}  // namespace

DispatchOptions dispatch_options()
{
    options_from_environment();
    return DispatchOptions{opt_kernel.load(), opt_mfma_f16.load(), opt_mid_tile.load(), opt_mid_kgroups.load(), opt_ws_off.load()};
}

unsigned absmax_looks() { return opt_absmax_looks.load(); }

void note_kernel(int id) { last_kernel = id; }
void note_hip(hipError_t e)
{
    if (e != hipSuccess && pending_hip_error == hipSuccess) pending_hip_error = e;
}
void clear_call_record()
{
    last_kernel = DYBIT_KERNEL_NONE;
    pending_hip_error = hipSuccess;
}
hipError_t take_hip_error()
{
    const hipError_t e = pending_hip_error;
    pending_hip_error = hipSuccess;
    return e;
}

void launch_gemm_general_wb(const GemmArgs &g, int a_bits, int w_bits, bool conv, int mode, hipStream_t st)
{
    switch (a_bits) {
        case 2: launch_gemm_general_a2_wb(g, w_bits, conv, mode, st); break;
        case 4: launch_gemm_general_a4_wb(g, w_bits, conv, mode, st); break;
        case 6: launch_gemm_general_a6_wb(g, w_bits, conv, mode, st); break;
        case 8: launch_gemm_general_a8_wb(g, w_bits, conv, mode, st); break;
    }
}

// Whether the small-output kernel is the faster one: it decodes each code for 32 rows or columns of use where a tile of the
// others decodes it for 64 to 256, so it wins as long as those leave most of the device idle.  The line is drawn in tiles of
// 64 x 64.  Measured over M from 1 to 12544, N from 32 to 4096, K from 256 to 4608 (us, the kernel it replaces -> this one):
// against the 128 x 128 fp16 kernel (8-bit pair) 128 x 1000 x 1024 (32 tiles) 13.4 -> 7.4, 3136 x 256 x 1024 (196) 15.4 -> 13.7,
// 1024 x 1024 x 4096 (256) 35.4 -> 29.1, but 12544 x 128 x 1152 (392) 17.5 -> 20.8; against the 64 x 64 e4m3 kernel (4-bit
// pair) 512 x 512 x 4096 (64) 13.9 -> 8.4, 784 x 512 x 4608 (104) 17.7 -> 13.3, but 128 x 4096 x 1024 (128) 6.7 -> 7.6.  Rows
// that start at any byte, 1200 x 1200 x 1532 (361) against the 128 x 128 fp16 kernel: 8-bit x 4-bit 17.9 -> 20.6, a 4-bit pair
// (which has its e4m3 form only here) 16.9 -> 14.3, but 2999 x 1999 x 1532 (1504) 34.5 -> 39.9.  Long and narrow products stay
// on the weight-stationary kernel.  The line was measured for K up to 2^18 (1024 x 1024, 8-bit pair: 467 -> 393 at K = 2^16, 1866 ->
// 1757 at 2^18), with rows at any byte up to 2^14 (1024 x 1024 x 9220, 8-bit x 4-bit 73.3 -> 59.2, 8-bit pair 78.8 -> 82.0).  A longer
// K outgrows the caches, which this kernel's tiles lean on most, and the line halves: 1024 x 1024 x 2^20, 8-bit x 4-bit 6890 -> 8009,
// 784 x 512 with a 4-bit pair 2558 -> 2715, but 512 x 512 2560 -> 1362; at any byte 1024 x 1024 x 65540, 8-bit pair 477 -> 619, and once
// more from 2^19 on (1024 x 640 x 1048580 10353 -> 12993, 512 x 512 10712 -> 3584).
static bool small_output(const GemmArgs &g, bool ragged, bool low_pair)
{
    if (!ragged && g.M >= 16384) return false;
    int line = !low_pair ? 256 : ragged ? 384 : 104;
    if (ragged && g.K > 1 << 14) line /= 2;
    if (g.K > 1 << 19) line /= 2;
    return ((g.M + 63) / 64) * ((g.N + 63) / 64) <= line;
}

// Whether the few-channel kernel is the faster one (us, the kernel it replaces -> this one; stride 1 or 2, N output channels, M outputs).
// Filters that the weight-stationary and 128 x 128 kernels' row mode takes as well (rows of exactly 32 codes, an even number of them):
//   N <= 128: 8 x 8 taps of 4 channels, 64 out, 8-bit: codes out at M = 50176 11.5 -> 11.6, 100352 16.5 -> 13.7, 802816 74.4 -> 50.6;
//     fp32 out at 200704 24.8 -> 25.5, 401408 41.0 -> 40.0, 802816 79.3 -> 65.6.
//   N > 128: fp32 out only with K >= 256 and M from 393216 on (8 x 8 taps of 4, 256 out: 401408 123.9 -> 104.8, but 192 out at 12544
//     10.2 -> 18.1; 4 x 4 of 8, 256 out: 254016 52.5 -> 68.4); codes out with K >= 128 and 3 * 2^30 multiply-adds (8 x 8 of 4, 160 out:
//     200704 50.6 -> 42.5, but 12544 11.2 -> 12.0, and 2 x 2 of 16, 160 out, 50176: 1.1 to 1.4 times as long).
// Any other filter would run on the general kernel (below 2048 outputs it does).  Codes out take 0.1 to 0.9 of its time everywhere.  fp32
// out, with `units` the outputs times the groups of 128 columns that kernel walks over:
//   where it reads code by code (7 x 7 of 4 at M = 9409 28.8 -> 8.9): with K >= 112 or units from 98304 on (0.2 to 0.95), with K >= 64 but for
//     8-bit images at 16384 to 40960 units (there 1.0 to 1.1, else 0.3 to 1.0), with less K only small calls of narrower codes (0.8 to 0.95;
//     8-bit and more columns 1.0 to 1.5);
//   where it reads 16 codes at a time: with K >= 128 from 98304 units on (0.4 to 1.05); with at most 64 columns in the last 128, K >= 80 and
//     M from 98304 on (0.5 to 1.0) or less K and M from 2^17 on (0.5 to 1.1); below 1.0 to 1.9.
static bool few_channels_pay(const GemmArgs &g, int a_bits, bool codes)
{
    const bool whole_words = g.a_bytes % 4 == 0;
    if (g.kw * g.Cin == 32 && g.kh % 2 == 0 && whole_words) {
        if (g.N <= 128) return g.M >= (codes ? 1 << 16 : 1 << 18);
        return codes ? g.K >= 128 && (double)g.M * (double)(g.N * g.K) >= 3.0 * (1 << 30) : g.K >= 256 && g.M >= 3 << 17;
    }
    if (g.M < 2048) return false;
    if (codes) return true;
    const bool aligned = ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.W)) & 15) == 0;
    const int64_t units = g.M * ((g.N + 127) / 128);
    if (aligned && (g.Cin == 16 || (g.kw * g.Cin % 16 == 0 && whole_words)))
        return g.K >= 128 ? units >= 3 << 15 : (g.N - 1) % 128 < 64 && g.M >= (g.K >= 80 ? 3 << 15 : 1 << 17);
    if (g.K >= 112 || units >= 3 << 15) return true;
    if (g.K >= 64) return a_bits < 8 || units < 1 << 14 || units >= 5 << 13;
    return a_bits < 8 && g.M < 1 << 14 && g.N <= 128;
}

// The few-channel kernel takes a convolution whose filter rows fit 32 codes with at least two taps (with one, no code would be
// decoded twice) and whose fragments start on groups of eight codes.
static bool launch_conv_few(const GemmArgs &g, int a_bits, int w_bits, bool forced, hipStream_t st)
{
    const bool dense = (int64_t)g.pix_bytes * 8 == (int64_t)g.Cin * a_bits, codes = codes_only(g);
    if (!dense || a_bits == 2 || (g.Cin != 4 && g.Cin != 8 && g.Cin != 16) || g.kw < 2 || g.kw * g.Cin > 32 || g.stride * (int64_t)g.Cin % 8) return false;
    if (g.N > 256 || g.M > 0x7fffffff || (g.q_out && !codes) || (!forced && !few_channels_pay(g, a_bits, codes))) return false;
    if (g.a_bytes >= 0x7fffffff || g.w_bytes >= 0x7fffffff || ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.W)) & 3)) return false;
    switch (w_bits) {
        case 4: return (codes ? launch_conv_few_w0_co : launch_conv_few_w0)(g, a_bits, st);
        case 8: return (codes ? launch_conv_few_w2_co : launch_conv_few_w2)(g, a_bits, st);
        case 6: return (codes ? launch_conv_few_w4_co : launch_conv_few_w4)(g, a_bits, st);
        case 2: return (codes ? launch_conv_few_w6_co : launch_conv_few_w6)(g, a_bits, st);
        default: return false;
    }
}

// Whether the many-channel kernel is the faster one.  It decodes an input code once per tile, so it lives on taps that share their
// pixels: `share` of them look at a pixel of a strip of 128 outputs, on average (3 x 3 at stride 1: 8.0 on 7 x 7, 4.8 on 56 x 56, 1.2 on
// 400 columns, where a strip looks at three image rows all along; at stride 2 on 56 x 56 1.8).  Measured over 5300 convolutions of 64 to
// 1024 channels and 2 to 778752 outputs, 1 x 2 to 5 x 5 and 7 x 1 taps, all formats and outputs, and over 24000 calls that it took on images of 4 to
// 160 pixels a side (us, the kernel it replaces -> this one):
//   filters in two dimensions: share from 1.75 on (64 x 64 x 64, 192 to 160 at stride 2, 4-bit pair 44.7 -> 36.1; below, 400 x 400, 64 to 64,
//     8- by 4-bit 22.0 -> 35.0, 4-bit pair 19.7 -> 32.8, and 2 x 2 at stride 2, 63 x 49 x 49, 128 to 256: 14.9 -> 22.6); in one from 3 on
//     (1 x 3 of 384 channels, 69 x 75 x 32, to 128, 8-bit pair: 63.6 -> 81.6);
//   K from 320 on: a shorter loop ends before the strip is decoded (2 taps of 64, 2 x 40 x 40, to 160, 8-bit pair: 5.6 -> 7.4);
//   small-output kernel: not a pair of 4- and 2-bit formats to the line of that kernel (3267 outputs, 256 to 64: 7.9 -> 10.5), others from
//     137 tiles of 64 x 64 on (15 x 23 x 23, 128 to 64, 124 tiles: 9.2 -> 10.8; 36 x 16 x 16, 144 tiles: 13.6 -> 11.9) and K from 512 on
//     (2 x 2 taps of 64, 2 x 40 x 40, to 256: 6.4 -> 7.7); fp32 results with 4- and 2-bit weights, whose decoding that kernel
//     spreads over the most waves, only at stride 1 (16 x 22 x 22, 128 to 512 at stride 2, 6- by 4-bit 11.0 -> 13.2), and with 4-bit weights strips of more
//     than 64 KiB only with a share from 4.5 on (2 x 7 x 129, 192 to 320, 8- by 4-bit 11.0 -> 13.6; 56 x 56, 256 to 256, 4.8, 15.6 -> 14.5);
//   weight-stationary kernel: at stride 1 with 4- and 2-bit weights everywhere (64 x 56 x 56, 64 to 64, 4-bit pair 25.7 -> 22.8, 6- by 4-bit
//     35.8 -> 29.5); wider weights take a lane longer to decode, and at stride 2 a tile looks at four pixels per output, of which fewer fit the
//     LDS: below 40960 outputs (25088: 11.6 -> 10.0 to 28.0 -> 18.0; 50176: 8-bit pair 11.9 -> 11.7, 8- by 6-bit 12.9 -> 14.6, stride 2
//     11.4 -> 11.2 to 14.2 -> 20.3);
//   256 x 256 kernel: not fp16 with 6- and 8-bit weights (64 x 28 x 28 x 256, 8-bit pair: 64.5 -> 69.8), unless that kernel declines and
//     leaves them to the 128 x 128 one (a 6- or 2-bit operand, 64 x 28 x 28, 192 to 192, 6-bit pair: 85.0 -> 51.7);
//   64 x 64 e4m3 kernel: K from 512 on, and 264 tiles, where that one needs a second round (64 x 14 x 14, 256 to 512 at stride 2, 392 tiles,
//     coded shortcut: 20.3 -> 16.1), or a share of 3, codes only 2.5 (16 x 39 x 17, 256 to 160 at stride 2, 135 tiles: 11.9 -> 13.2; 6 x 26 x 72, 320
//     to 40, 3 x 2 taps, 9.9 -> 12.0);
//   128 x 128 kernels: everywhere (64 x 14 x 14 x 256, 4-bit pair 22.8 -> 15.5; 64 x 7 x 7 x 512, 6-bit pair 58.6 -> 31.5);
//   against these and the weight-stationary kernel, which have rounds enough from 513 tiles of 128 x 128 on to hide their fixed times, and a strip of
//     more than 56 KiB, of which a compute unit holds one or two and each waits for its own loads: share from 2.5 on (53 x 90 x 90, 64 to 64, 8- by
//     4-bit, codes 43.1 -> 73.2; 14 x 91 x 91, 128 to 64, 26.3 -> 40.4), with codes beside the fp32 results and more than 64 columns 3.5 (7 x 127 x 127,
//     128 to 160, 2- by 4-bit 58.4 -> 75.6); 4-bit activations of a pair whose bytes decode faster: 2 up to 64 columns (73 x 20 x 128, 192 to 64, codes
//     1.25 times as long), none beyond (64 x 56 x 56, 128 to 256 at stride 2 35.6 -> 31.8), nor for up to 32 columns of any pair (0.84 times).
// Calls that write fp32 results and codes have the long epilogue (20 vector instructions per result, a column per lane), which this kernel
// has fewer waves to hide behind than the ones with small tiles.  They gain as above against tiles of 128 (64 x 7 x 7 x 512, 8-bit pair
// 44.8 -> 28.2), but with K from 512 on; against the small-output kernel with 6-bit weights at stride 1 (40 x 14 x 14, 128 to 96, 6-bit pair
// 16.4 -> 15.2, 8- by 4-bit 12.0 -> 13.2, 29 x 35 x 34, 64 to 64 at stride 2, 8- by 6-bit 12.0 -> 13.8) and with 8-bit ones from K = 1536 on; against the
// 64 x 64 kernel from 264 tiles (64 x 7 x 7 x 512, 4-bit pair 30.2 -> 20.4, but 20 x 16 x 16, 64 to 128, 160 tiles, 2-bit pair 8.9 -> 10.3) or K = 2560
// and a share of 4 on (5 x 5 of 256, 9 x 33 x 33, to 64, 25.9 -> 21.4, but 55 x 17 x 17, 512 to 64, 3 x 2 taps, 15.8 -> 18.6);
// against the weight-stationary kernel with more than 64 columns, for which that one holds twice the weights, or K from 832 on (64 to 64,
// 13 x 56 x 56, 8- by 4-bit 14.2 -> 17.0, 64 x 56 x 56, 2-bit pair 25.4 -> 29.6).
static bool many_channels_pay(const GemmArgs &g, int a_bits, int w_bits, bool f8, bool large)
{
    if (g.K < 320) return false;
    const int64_t strip = g.M < 128 ? g.M : 128;
    const int64_t pixels = strip_pixels(g, strip);
    const double share = (double)(g.kh * (int64_t)g.kw * strip) / (double)pixels;
    if (share < (g.kh > 1 && g.kw > 1 ? 1.75 : 3.0)) return false;
    const int64_t strip_bytes = (pixels + 1) * (g.Cin * (f8 ? 1 : 2) + 16);
    const bool both = g.q_out && !codes_only(g);
    const int64_t tiles64 = ((g.M + 63) / 64) * ((g.N + 63) / 64);
    if (both && g.K < 512) return false;
    if (small_output(g, false, f8)) {
        if (f8 || g.K < 512 || tiles64 <= 136 || (both && (w_bits <= 4 || (w_bits == 8 && g.K < 1536)))) return false;
        if (g.stride > 1 && (g.q_out ? both && w_bits == 6 : w_bits <= 4)) return false;
        if (!g.q_out && w_bits == 4 && strip_bytes > 64 * 1024 && share < 4.5) return false;
    }
    const bool declines = (a_bits == 6 || a_bits == 2 || w_bits == 6) && g.Cin % 128 != 0;   // see gemm_fast.hip
    const bool tiles_of_256 = large && (f8 || !declines);
    if (tiles_of_256 && !f8 && w_bits > 4) return false;
    const int64_t tiles128 = ((g.M + 127) / 128) * ((g.N + 127) / 128);
    if (!tiles_of_256 && tiles128 > 512 && strip_bytes > 56 * 1024 && (!f8 || g.N > 32) &&
        share < (both && g.N > 64 ? 3.5 : !f8 || a_bits == 2 ? 2.5 : g.N > 64 ? 0.0 : 2.0)) return false;
    const int64_t ws_bytes = (g.N <= 64 ? 64 : 128) * (g.K * (f8 ? 1 : 2) + 16);
    if (g.M >= 16384 && g.N <= 128 && ws_bytes <= 160 * 1024) return (g.M < 40960 || (g.stride == 1 && w_bits <= 4)) && (!both || g.N > 64 || g.K >= 832);
    const bool tiles_of_64 = f8 && tiles128 <= 128;   // see gemm_f8.hip
    return !tiles_of_64 || (g.K >= 512 && (tiles64 >= 264 || (both ? g.K >= 2560 && share >= 4.0 : share >= (g.q_out ? 2.5 : 3.0))));
}

// It takes a convolution with 64-code k groups inside one filter tap whose outputs look at consecutive pixels,
// one after the other (no output reaches past the image with its first taps).
static bool launch_conv_patch(const GemmArgs &g, int a_bits, int w_bits, bool low_pair, hipStream_t st)
{
    const bool codes = codes_only(g), wb = g.q_out != nullptr;
    if (g.Cin % 64 || g.kh * (int64_t)g.kw < 2 || g.kh * (int64_t)g.kw > 30 || g.M > 0x7fffffff || g.N > 1 << 16) return false;
    if ((g.Ho - 1) * (int64_t)g.stride >= g.H || (g.Wo - 1) * (int64_t)g.stride >= g.Wd || g.pad >= g.kh || g.pad >= g.kw) return false;
    if (g.ldc > 1 << 20 || (g.q_out && g.q_row_bytes > 1 << 20) || (g.res_codes && g.res_row_bytes > 1 << 20)) return false;
    if (g.M / ((int64_t)g.Ho * g.Wo) * g.H * (int64_t)g.Wd > 0x3fffffff) return false;
    switch (w_bits) {
        case 4: return (codes ? launch_conv_patch_w0_co : wb ? launch_conv_patch_w0_wb : launch_conv_patch_w0)(g, a_bits, low_pair, st);
        case 8: return (codes ? launch_conv_patch_w2_co : wb ? launch_conv_patch_w2_wb : launch_conv_patch_w2)(g, a_bits, low_pair, st);
        case 6: return (codes ? launch_conv_patch_w4_co : wb ? launch_conv_patch_w4_wb : launch_conv_patch_w4)(g, a_bits, low_pair, st);
        case 2: return (codes ? launch_conv_patch_w6_co : wb ? launch_conv_patch_w6_wb : launch_conv_patch_w6)(g, a_bits, low_pair, st);
        default: return false;
    }
}

bool launch_gemm_tiled(const GemmArgs &g, int a_bits, int w_bits, bool conv, hipStream_t st)
{
    if (!g.w_signed) return false;                                  // every width 2, 4, 6, 8 has a decoder; weights are signed
    const DispatchOptions opt = dispatch_options();
    const bool few = opt.kernel == DYBIT_FORCE_FEW;
    if (conv && g.M >= 1 && g.N >= 1 && (few || (!opt.kernel && !opt.mid_tile && !opt.mid_kgroups)) && launch_conv_few(g, a_bits, w_bits, few, st)) return true;
    if (g.M < 1 || g.N < 1 || g.K < 64 || (conv && g.K % 64)) return false;
    const bool ragged = g.K % 64 != 0;                              // a matrix product whose rows start at any byte
    // a convolution needs whole 64-code k groups inside a filter tap, or (few channels) filter rows of
    // exactly 32 codes, which the 128 x 128 kernel fetches row by row
    const bool dense = conv && (int64_t)g.pix_bytes * 8 == (int64_t)g.Cin * a_bits;   // not one channel group of a wider image
    const bool rows = dense && g.Cin < 64 && (int64_t)g.kw * g.Cin == 32 && g.a_bytes % 4 == 0;   // fetched as aligned words: none may reach past the tensor
    if (conv && g.Cin % 64 && !rows) return false;
    if ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.W)) & 15) return false;
    if (g.a_bytes >= 0x7fffffff || g.w_bytes >= 0x7fffffff) return false;

    // which build of a kernel family writes what the call asks for
    const bool wb = g.q_out != nullptr, codes = codes_only(g);
#define DYBIT_BUILD_OF(name) (codes ? name##_co : wb ? name##_wb : name)

    const bool low_pair = (a_bits == 4 || a_bits == 2) && (w_bits == 4 || w_bits == 2);
    const int force = few || opt.kernel == DYBIT_FORCE_PATCH || opt.kernel == DYBIT_FORCE_SIX ? 0 : opt.kernel;
    if (force == DYBIT_FORCE_GENERAL) return false;
    const bool f8 = low_pair && !opt.mfma_f16;

    // Too few 256 x 256 tiles cannot fill 256 compute units, and a narrow N wastes most of a
    // 256-wide tile.  With a short K the epilogue (the stores of C, the loads of the shortcut)
    // dominates, and the 128 x 128 kernel with three workgroups per compute unit keeps more
    // of those memory operations in flight: measured over M x N from 6272 x 2048 to
    // 401408 x 256, it is 1.1 to 1.7 times faster up to K = 512, level at K = 1024 (fp16
    // kernels) or K = 2048 (fp8 kernels), and 10 to 30 % slower beyond.
    const int64_t tiles256 = ((g.M + 255) / 256) * ((g.N + 255) / 256);
    bool large = g.N > 128 && tiles256 >= 128 && g.K >= (low_pair ? 2048 : 1024);

    // Convolution with its input decoded once per tile
    const bool choose = !force && !opt.mid_tile && !opt.mid_kgroups && !opt.ws_off;
    if (conv && (opt.kernel == DYBIT_FORCE_PATCH || (choose && many_channels_pay(g, a_bits, w_bits, f8, large))) &&
        launch_conv_patch(g, a_bits, w_bits, f8, st)) return true;

    // Small outputs: so few 128 x 128 tiles that most compute units would idle through a serial K loop.  That kernel counts the codes
    // of K and the bits of a row in 32 bits (its waves look up to 3072 codes ahead); longer rows go to the others.
    const bool short_rows = g.K < 0x7fff0000 / (a_bits > w_bits ? a_bits : w_bits);
    if (!rows && short_rows && (force == DYBIT_FORCE_SMALL || (!force && !opt.mid_tile && !opt.mid_kgroups && small_output(g, ragged, f8)))) {
        switch (w_bits) {
            case 4: (wb ? launch_gemm_small_w0_wb : launch_gemm_small_w0)(g, a_bits, conv, st); return true;
            case 8: (wb ? launch_gemm_small_w2_wb : launch_gemm_small_w2)(g, a_bits, conv, st); return true;
            case 6: (wb ? launch_gemm_small_w4_wb : launch_gemm_small_w4)(g, a_bits, conv, st); return true;
            default: (wb ? launch_gemm_small_w6_wb : launch_gemm_small_w6)(g, a_bits, conv, st); return true;
        }
    }

    // Weight-stationary kernel: the decoded weights of up to 128 columns (N > 128: of a group of 64) stay in
    // LDS, for many rows against few weights (it declines when the weights do not fit).  Wider than 128 columns
    // it is taken where it was measured faster than the 128 x 128 kernel (M x N x K from 401408 x 256 x 64 to
    // 25088 x 1024 x 256): with the write-back epilogue and a short K, 1.05 to 1.25 times; with fp32 results
    // only its 256-byte row segments lose to the tile's 512-byte ones.
    const bool ws_wide = g.q_out != nullptr && g.K <= 256 && (g.C == nullptr || g.K >= 128);
    if (!ragged && (force == DYBIT_FORCE_WS || (!force && !opt.ws_off && g.M >= 16384 && (g.N <= 128 || ws_wide)))) {
        bool done = false;
        switch (w_bits) {
            case 4: done = DYBIT_BUILD_OF(launch_gemm_ws_w0)(g, a_bits, conv, st); break;
            case 8: done = DYBIT_BUILD_OF(launch_gemm_ws_w2)(g, a_bits, conv, st); break;
            case 6: done = DYBIT_BUILD_OF(launch_gemm_ws_w4)(g, a_bits, conv, st); break;
            case 2: done = DYBIT_BUILD_OF(launch_gemm_ws_w6)(g, a_bits, conv, st); break;
        }
        if (done) return true;
    }
    if (force == DYBIT_FORCE_LARGE) {
        large = true;
    } else if (force == DYBIT_FORCE_MID) {
        large = false;
    }
    // two operands of 4 or 2 bits: every value is exact in e4m3, so the fp8 matrix path (twice the
    // fp16 rate, byte decoders) takes them unless the "gemm_mfma" option asks for the fp16 kernels
    if (f8 && !rows && !ragged) {
        if (w_bits == 4) return DYBIT_BUILD_OF(launch_gemm_f8_w0)(g, a_bits, conv, large, st);
        return DYBIT_BUILD_OF(launch_gemm_f8_w6)(g, a_bits, conv, large, st);
    }
    if (rows || ragged) large = false;
    if (large) {                                                   // declines a 2- or 6-bit operand unless K (Cin) is a multiple of 128
        bool done;
        if (w_bits == 4) done = (wb ? launch_gemm_fast_w0_wb : launch_gemm_fast_w0)(g, a_bits, conv, st);
        else if (w_bits == 6) done = (wb ? launch_gemm_fast_w4_wb : launch_gemm_fast_w4)(g, a_bits, conv, st);
        else if (w_bits == 2) done = (wb ? launch_gemm_fast_w6_wb : launch_gemm_fast_w6)(g, a_bits, conv, st);
        else done = (wb ? launch_gemm_fast_w2_wb : launch_gemm_fast_w2)(g, a_bits, conv, st);
        if (done) return true;
    }
    if (w_bits == 4) return DYBIT_BUILD_OF(launch_gemm_mid_w0)(g, a_bits, conv, st);
    if (w_bits == 6) return DYBIT_BUILD_OF(launch_gemm_mid_w4)(g, a_bits, conv, st);
    if (w_bits == 2) return DYBIT_BUILD_OF(launch_gemm_mid_w6)(g, a_bits, conv, st);
    return DYBIT_BUILD_OF(launch_gemm_mid_w2)(g, a_bits, conv, st);
#undef DYBIT_BUILD_OF
}

// The tile with which the product on split operands (gemm_six.hip) is faster than the kernel that launch_gemm_tiled would take, or 0.
// That kernel's matrix time is half of fp16's (two planes: an operand of 6 or 8 bits) or of e4m3's (one), and rows that start at any byte cost
// it only a slower split; but the operands go through memory once more, and its tiles have the longer fill.  Measured over 9000 products
// (M, N from 96 and K from 200 to 9000, all formats it takes; us, the kernel before -> this one, the split included); of the 2078 taken, 0.63 times
// the time in the geometric mean, 12 more than the same, at most 1.05 times:
//   more than 256 tiles of 128 x 128: two planes with K from 1024 on (8192^3, 8- by 4-bit 775 to 840 -> 470 to 510 over cards; 5203 x 3732 x 1144 68.1 -> 51.5, but
//     5351 x 2368 x 320 20.3 -> 22.3); one plane where the e4m3 kernels have their 256 x 256 tile or K from 3072 on (8192^3, 4-bit
//     pair 400 to 415 -> 267 to 288; 4657 x 4891 x 3968 139 -> 76, but 2196 x 2672 x 960 14.2 -> 16.5); one plane and ragged rows, which have no e4m3 form
//     there, with K from 512 on (2368 x 6144 x 1740, 2-bit pair 70.4 -> 33.7);
//   from there down to the line of the small-output kernel: one plane and ragged rows, K from 1536 on (3281 x 800 x 3004, 4-bit pair 0.5 to 0.9
//     times); two planes, K from 2560 and both sides from 768 on (1874 x 1024 x 8584 75.5 -> 59.2; with one short side the split is most of
//     the work: 7473 x 226 x 8768 68.4 -> 77.7), with a 6-bit operand, whose decoding costs the fp16 kernels most, K from 2048 on or one
//     short side and K from 3072 on (5442 x 193 x 6592 59.9 -> 53.0).
// The 256 x 256 tile where its rounds over the compute units are at most 0.35 times those of 128 x 128: of the faster one of both 1.004 times
// on average, at most 1.26.
int gemm_six_tile(int64_t M, int64_t N, int64_t K, int a_bits, int w_bits)
{
    const DispatchOptions opt = dispatch_options();
    if (opt.kernel == DYBIT_FORCE_SIX) return opt.mid_tile == 128 ? 128 : 256;
    if (opt.kernel || opt.mfma_f16 || opt.mid_tile || opt.mid_kgroups || opt.ws_off) return 0;
    if (M < 1 || N < 1 || K < 512 || M > 1 << 24 || N > 1 << 24 || (M >= 16384 && N <= 128)) return 0;
    GemmArgs g{};
    g.M = M; g.N = N; g.K = K;
    const bool one = a_bits <= 4 && w_bits <= 4, ragged = K % 64 != 0, six = a_bits == 6 || w_bits == 6;
    if (small_output(g, ragged, one)) return 0;
    const int64_t tiles128 = ((M + 127) / 128) * ((N + 127) / 128), tiles256 = ((M + 255) / 256) * ((N + 255) / 256), shorter = M < N ? M : N;
    bool pays;
    if (tiles128 > 256) pays = one ? ragged || K >= 3072 || (K >= 2048 && N > 128 && tiles256 >= 128) : K >= 1024;
    else if (one) pays = ragged && K >= 1536;
    else pays = shorter >= 768 ? K >= (six ? 2048 : 2560) : six && K >= 3072;
    if (!pays) return 0;
    return 20 * ((tiles256 + 255) / 256) <= 7 * ((tiles128 + 255) / 256) ? 256 : 128;
}

// Whether a launch per group beats the one-launch kernel.  For a pair of 4- and 2-bit formats in groups of whole 64-channel k groups
// the other kernels have e4m3 forms, the one-launch kernel is fp16; so with weights of some size (its own advantage on small ones is
// that it fills the device), more columns than its 32-column form takes and enough multiply-adds per group for the number of
// groups, they win.  One launch -> one per group (us on the device, launches back to back), 3 x 3, 4-bit pair: 2 groups of
// 128 -> 128 channels, M = 50176: 52.9 -> 30.1, 4 groups 81.5 -> 55.6; M = 200704, 2 groups 148.8 -> 78.1.  The line was drawn where the 128 x 128
// kernels met the one-launch kernel; with 3 x 3 groups on the many-channel kernel it is on the safe side: of 531 geometries measured (64 to 512
// channels, 1 x 1 to 3 x 3, 2 to 8 groups) two are up to 1.08 times slower than in one launch, and 79 that stay in one launch up to 1.38
// times slower than a launch per group (128 -> 128 channels, 8 groups, M = 50176 152 against 115, 2 groups, M = 12544 19.0 against 16.5).
static bool launch_per_group(const GemmArgs &g, int a_bits, int w_bits, int groups)
{
    if (a_bits > 4 || w_bits > 4 || g.Cin % 64 || dispatch_options().mfma_f16) return false;
    if ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.W)) & 15) return false;
    const int64_t Cog = g.N / groups, columns = (Cog + 63) / 64 * 64, weights = columns * g.K;
    return Cog > 32 && (Cog <= 128 || g.K >= 512) && weights > 64 * 576 && (double)g.M * (double)weights >= 1.25e9 * groups;
}

bool launch_group_conv(const GemmArgs &g, int a_bits, int w_bits, int groups, hipStream_t st)
{
    const int Cg = g.Cin;
    // pieces of 8, 16 or 32 codes, whole words, inside one filter tap; 32-bit buffer offsets; no kernel forced
    if (!g.w_signed || Cg % 8 || (Cg * a_bits) % 32 || g.N / groups > 0x7fffffff || g.M > 0x7fffffff || g.a_bytes >= 0x7fffffff || g.w_bytes >= 0x7fffffff) return false;
    if ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.W)) & 3) return false;
    if (dispatch_options().kernel || launch_per_group(g, a_bits, w_bits, groups)) return false;
    switch (w_bits) {
        case 4: return launch_group_conv_w0(g, a_bits, groups, st);
        case 8: return launch_group_conv_w2(g, a_bits, groups, st);
        case 6: return launch_group_conv_w4(g, a_bits, groups, st);
        case 2: return launch_group_conv_w6(g, a_bits, groups, st);
        default: return false;
    }
}

}  // namespace dybit

extern "C" int32_t dybit_last_gemm_kernel(void) { return dybit::last_kernel; }

extern "C" dybit_status dybit_set_option(const char *name, const char *value)
{
    if (!name || !value) return DYBIT_ERR_NULL;
    dybit::options_from_environment();                              // so that a later first use does not overwrite this
    return dybit::apply_option(name, value) ? DYBIT_OK : DYBIT_ERR_INVALID_ARG;
}
