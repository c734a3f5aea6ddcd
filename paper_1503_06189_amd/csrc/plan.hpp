// plan.hpp -- how one frame is split into workgroups (host and device).
//
// The triangle of 32x32 input-block tiles (I <= J) of each channel is cut
// into "super-blocks" of 8x8 tiles (256 x 256 inputs).  A workgroup of eight
// waves, two per SIMD, takes one tile group:
//   * a diagonal super-block: a triangle of 36 tiles over two 128-input
//     groups of four blocks;
//   * half of an off-diagonal super-block: 4 tile rows (a 128-input group) x
//     8 tile columns (two groups).
// How the waves share a group's tiles is the kernels' matter.  Super-blocks
// at the edge of the triangle are padded: tiles past N are computed but never
// stored, so every wave has a fixed, compile-time tile pattern.  With
// ns = ceil(blocks / 8) super-rows there are ns diagonal groups and
// ns(ns-1)/2 off-diagonal super-blocks of two halves each: ns^2 groups.  Each
// workgroup integrates its tiles over one chunk of the frame's time samples;
// chunk 0 writes the output and a merge kernel adds the other chunks.
//
// Second geometry ("halves", for N <= 128, one 128-input group): the padded
// super-block would compute 36 tiles for the 10 of the group's triangle.
// Instead waves integrate the whole triangle over their own part of the
// samples, and the sums are added at the end.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define XE_HD __host__ __device__
#else
#define XE_HD
#endif

namespace xe {

constexpr int kBlk = 32;          // inputs per tile edge (one 32x32 MFMA)
constexpr int kStep = 32;         // unit of time chunks, in samples
constexpr int kLoop = 64;         // samples per loop step of the kernels
constexpr int kSuper = 8;         // tile blocks per super-block edge
constexpr int kGroupInputs = 128; // inputs of four strided blocks
constexpr int kMaxSlots = 12;     // input blocks staged per workgroup
constexpr int kSuperWaves = 8, kSuperThreads = 64 * kSuperWaves;
constexpr int kSmallWaves = 4, kSmallThreads = 64 * kSmallWaves;   // halves geometry
// Workspace of one tile group and time chunk, in int32 values: at least the
// chunk's copy of the group's share of the output.
constexpr int64_t kGroupPartial = 81920;
// Short time chunks run on the int8 kernel (short_kernels.hpp), longer ones on
// the 6-bit kernels (xcorr_kernels.hpp), which pay more per workgroup and less
// per sample.  Measured, accumulating unchunked frames, int8 | 6-bit, us per
// call:
//   128 inputs, 256 channels:  512 samples 15.9 | 26.1, 1536: 28.2 | 33.7,
//                              2048: 34 | 36, 4096: 66 | 49
//   256 inputs, 256 channels:  512 samples 32.3 | 35.5, 800: 57 | 60,
//                              1024: 60 | 62, 1280: 67 | 66, 2048: 91 | 80
//   512 inputs, 294 channels:  800: 281 | 326, 1024: 312 | 333, 1536: 413 | 383
//   768 inputs, 130 channels:  800: 277 | 291, 1024: 300 | 304, 1280: 345 | 330
//   2048 inputs, 16 channels:  256 samples 86 | 97, 768: 134 | 138,
//                              2048: 283 | 231
//   1024 inputs, 32 channels:  768: 96 | 96, 800: 104 | 100, 1024: 110 | 105
// Padding of the super geometry (inputs past N up to whole super-blocks) costs
// the 6-bit kernel more:
//   132 inputs, 1177 channels: 800: 186 | 233, 1280: 245 | 273, 2048: 360 | 360
//   260 inputs, 294 channels:  800: 185 | 246, 1280: 238 | 282, 2048: 343 | 340
//   516 inputs, 130 channels:  800: 187 | 219, 1280: 242 | 257, 1536: 288 | 283
//   640 inputs, 130 channels:  800: 227 | 253, 1280: 294 | 299, 1536: 335 | 331
// Rows that are not 4-byte aligned cost the int8 kernel more, in its
// off-diagonal groups above all:
//   250 inputs, 1177 channels: 800: 300 | 332, 1024: 325 | 341, 1280: 368 | 365
//   257 inputs, 294 channels:  768: 248 | 244, 800: 274 | 252
//   601 inputs, 130 channels:  768: 272 | 270, 800: 296 | 258
// kShortSteps is also the most validity words that the int8 kernel keeps (one
// per lane).
constexpr int kShortSteps = 64;         // halves geometry
constexpr int kShortSuperSteps = 24;    // super geometry: many inputs, unaligned rows
constexpr int kShortFewSteps = 32;      // up to three super-blocks
constexpr int kShortPaddedSteps = 40;   // of which padding takes a quarter
XE_HD inline int short_steps(int small, int N, int aligned) {
    const int edge = kSuper * kBlk, ns = (N + edge - 1) / edge;
    if (small) return kShortSteps;
    if (ns > 3 || (ns > 1 && !aligned)) return kShortSuperSteps;
    return 4 * N <= 3 * ns * edge ? kShortPaddedSteps : kShortFewSteps;
}
// longest chunk: 2^18 steps (8,388,608 samples)
constexpr int kMaxStepsPerChunk = 1 << 18;
// Chunk lengths are multiples of kDepth steps.  A chunk of n steps is loaded
// n + 3 kDepth steps far at most, lookahead included, and byte offsets within
// that stay below 2^31.
#ifndef XE_DEPTH
#define XE_DEPTH 4
#endif
constexpr int kDepth = XE_DEPTH;

// Longest chunk (in steps) for F channels of N inputs, kDepth steps at least:
// these fit for every F * N that the ABI accepts (asserted with its check).
inline int64_t max_steps_per_chunk(int64_t F, int64_t N) {
    int64_t m = (((int64_t)1 << 31) - 1) / (F * N * kStep) - 4 * kDepth;
    if (m > kMaxStepsPerChunk) m = kMaxStepsPerChunk;
    if (m < kDepth) m = kDepth;
    return m - m % kDepth;
}

// round a chunk length up
inline int round_steps(int sps) { return (sps + kDepth - 1) / kDepth * kDepth; }

// One tile group, in scalars (no arrays: kept in scalar registers on the
// device).  Its 128-input groups are
//   diagonal:      input0, input0 + 128
//   off-diagonal:  input0 (rows), column0 and column0 + 128
struct Group {
    int diag;
    int input0, column0;
};

// the halves geometry applies to frames of at most 4 input blocks
XE_HD inline int use_halves(int halves, int nb) { return halves && nb <= 4 ? 1 : 0; }

XE_HD inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

XE_HD inline int super_rows(int nb) { return ceil_div(nb, kSuper); }

XE_HD inline int groups_per_channel(int nb) {
    int ns = super_rows(nb);
    return ns * ns;
}

// off-diagonal super-block number p (row-major over R < C) -> (R, C)
XE_HD inline void offdiag_pair(int ns, int p, int *R, int *C) {
    int r = 0;
    while (p >= ns - 1 - r) {
        p -= ns - 1 - r;
        ++r;
    }
    *R = r;
    *C = r + 1 + p;
}

XE_HD inline Group make_group(int nb, int gid) {
    Group g;
    int ns = super_rows(nb);
    if (gid < ns) {
        g.diag = 1;
        g.input0 = gid * kSuper * kBlk;
        g.column0 = g.input0 + kGroupInputs;
    } else {
        int q = gid - ns;
        int R, C;
        offdiag_pair(ns, q / 2, &R, &C);
        g.diag = 0;
        g.input0 = R * kSuper * kBlk + (q % 2) * kGroupInputs;  // R is never the last super-row
        g.column0 = C * kSuper * kBlk;
    }
    return g;
}

// first input of 128-input group k of a tile group
XE_HD inline int group_input(const Group &g, int k) {
    return k == 0 ? g.input0 : g.column0 + (k - 1) * kGroupInputs;
}

// 32x32 tiles computed per channel: 36 per diagonal group (8 x 9), 32 per
// off-diagonal half (4 x 8); padded tiles past N included.  The halves
// geometry computes the 10 tiles of the 4-block triangle.
inline int64_t tiles_per_channel(int nb, int halves) {
    if (use_halves(halves, nb)) return 10;
    int64_t ns = super_rows(nb);
    return ns * 36 + ns * (ns - 1) * 32;
}

// Time split: enough workgroups to cover `n_cu` compute units once, but
// at least `min_steps` staged steps per chunk.
inline void choose_split(int64_t units, int steps, int n_cu, int *splits,
                         int *steps_per_split) {
    const int min_steps = 8;
    int64_t want = (n_cu + units - 1) / units;
    int64_t cap = steps / min_steps;
    if (cap < 1) cap = 1;
    int64_t s = want < cap ? want : cap;
    if (s < 1) s = 1;
    int sps = round_steps(ceil_div(steps, (int)s));
    *steps_per_split = sps;
    *splits = ceil_div(steps, sps);
}

// Which kernel counts flags: that of flag_kernels.hpp (in units of 8 or 10 tiles,
// groups^2 per channel) or that of flag_wide_kernels.hpp.  Measured, unit kernel
// | wide kernel, us per call: bursts of 32 over 0.01 - 0.1% of the points, then 1
// - 5% scattered:
//   128 inputs, 128 channels, 16,384 samples:  8.5 - 10.6 |  9 - 13,   25 |   64
//   256 inputs,  64 channels, 16,384 samples:  9.8 - 14.7 |  9 - 13,   41 |  123
//   256 inputs, 128 channels, 16,384 samples:   19 - 27   | 14 - 20,   77 |  191
//   130 inputs, 128 channels, 16,384 samples:   17 - 27   | 13 - 17,   60 |   79
//   256 inputs, 160 channels,  2,048 samples:   11 - 16   |  9 -  9,   37 |   66
//   130 inputs, 400 channels,  2,048 samples:   22 - 32   | 15 - 19,   61 |   60
//   256 inputs, 400 channels,  2,048 samples:   23 - 33   | 11 - 16,   80 |  133
//   512 inputs,  32 channels, 16,384 samples:   24 - 28   | 20 - 36,   80 |  780
//   512 inputs,  64 channels, 16,384 samples:   47 - 53   | 31 - 47,  154 | 1155
//   640 inputs,  25 channels, 16,384 samples, bursts:  42 | 30
//   768 inputs,  21 channels, 16,384 samples:   50 | 26,  122 | 824
//   1024 inputs,  2 channels,  8,192 samples, bursts:  12 | 25
//   1024 inputs,  4 channels, 16,384 samples, bursts:  22 | 19
// How dense the flags are is not known before they are read.  Up to two units
// per compute unit the unit kernel is taken: bursts cost it 10 us more at most,
// and scattered flags mostly between a half and a tenth.  Beyond, bursts, which
// are the method's case, cost it up to twice as much, and decide.  Rows of more
// than 64 bytes reach that point at half a unit per compute unit; a single
// group's units load every word once, and never do.
inline bool use_wide_flags(int64_t F, int groups, int n_cu) {
    const int64_t units = F * groups * groups;
    return groups > 1 && units > (groups <= 4 ? 2 * (int64_t)n_cu : n_cu / 2);
}

}  // namespace xe
