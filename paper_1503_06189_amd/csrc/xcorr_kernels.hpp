// xcorr_kernels.hpp -- gfx950 kernels of the correlator.
//
// Correlation (Sec. II-B: cross-correlate every input pair of a channel and
// add into the previous output), on the 6-bit matrix path.
//
// A sample is x = a + i b, a = A - 8 and b = B - 8 with the packed nibbles
// A, B in 0..15.  The 6-bit format E2M3 is linear below 2: code u means u/8
// for u in 0..15, so a nibble is an operand once its two upper bits are
// cleared, and bit 5 is the sign.  v_mfma_f32_32x32x64_f8f6f4 runs these at
// twice the rate of the int8 instruction (7.1 against 3.6 Pop/s, registers
// only) and takes 6 instead of 8 bits per value from LDS.  Its sums are
// float32, in units of 1/64: exact while |sum| <= 2^24 units, so a workgroup
// turns its sums into int32 at least every kSegSteps loop steps (below).
// With R_ij = sum A_i A_j + B_i B_j and I_ij = sum B_i A_j - A_i B_j over the
// valid samples, n of them (lost samples are staged as A = B = 0),
//   Re V_ij = R_ij - 8 (T_i + T_j) + 128 n      T_i = sum A_i + B_i
//   Im V_ij = I_ij + 8 (D_i - D_j)              D_i = sum A_i - B_i.
// T and D come from the matrix cores too: one 16x16x128 instruction of a 0/1
// pattern against an operand sums it for its 32 inputs.
//
// Blocks of 32 inputs are strided: block c of a 128-input group holds inputs
// 4 q + c, q = 0..31.  A dword of the frame is one sample of inputs
// 4 q .. 4 q + 3, so lane q (and q + 32, for other samples) that loads it
// holds row q of all four blocks: after a 4x4 byte transpose in registers
// the operands are complete, with no exchange between lanes.  The order of
// the samples inside K is arbitrary, but the same for every block.
//
// Packing: per 4 samples, three dwords hold (for 4 inputs, a byte each) the
// bytes of the 24-bit string of four 6-bit codes; a byte transpose of these
// gives each input's string.  16 samples of one component are 3 dwords; an
// operand (32 samples of a lane, 64 of the instruction) is 6.
//
// Geometries (plan.hpp).  Super: a workgroup of eight waves, two per SIMD,
// takes a tile group.  Per loop step of 64 samples the waves pack the group's
// input blocks into LDS, two steps ahead, and run 16 (2 x 2 tiles) or 20 (half
// the triangle of a 128-input group) matrix instructions each on operands read
// from LDS; the packing and the reads are woven between them, and while one
// wave of a SIMD waits the other issues.  Halves (N <= 128): four waves, each
// packs its own 64 samples of the one group and runs the triangle from
// registers, without barriers; the waves' sums are added at the end.
// Short chunks run on another kernel (short_kernels.hpp).
//
// What bounds it: 256 inputs, 64 channels, 16,384 samples (four chunks each)
// take 127 us on average and 118 at best, where the int8 kernel took 163 and
// 149, and the matrix cores are busy 27% of the fastest dispatch.  Packing, LDS
// and matrix work overlap only in part: in copies of the loop with parts left
// out, a step's 2,080 clocks became 1,830 without the hand-over of loaded
// bytes, 1,280 without packing and 1,390 without matrix instructions, which
// alone take 1,150.  Timed over the frame's length (256 channels, one chunk), a
// step takes 1.37 us and a call 37 us besides, of which the launch is about 6.
// 2048 inputs, 16 channels, 8,192 samples take 0.70 ms on quantised noise and
// 0.86 on random bytes (1.01 and 1.16 before).  One wave per SIMD with 2 x 4
// tiles read fewer operands but could not overlap packing with the matrix
// instructions: 122 against 116 us at 256 inputs x 256 channels x 4,096
// samples, 748 against 725 us at 2048 inputs.
//
// Diagonal tiles: block c against itself is Hermitian, so one tile
//   Q = R + I,  R = (Q + Q^T) / 2,  I = (Q - Q^T) / 2  (exact)
// keeps 16 instead of 32 accumulator registers.
//
// Output: chunk 0 of a tile group (or its only chunk) writes its sums with
// plain stores (overwrite) or read-add-write (accumulate).  Chunks 1.. do the
// same in a copy of the output in the workspace, and merge_kernel, launched
// next on the same stream, adds the copies into the output.  Integer sums,
// so the order of chunks does not matter and the result is exact.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "plan.hpp"

namespace xe {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v3i __attribute__((ext_vector_type(3)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v6i __attribute__((ext_vector_type(6)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
// four int32 of the output: vis is only 8-byte aligned
typedef v4i v4i_a8 __attribute__((aligned(8)));

// one component of a block per loop step: 64 lanes x 6 dwords, kept as 64 x
// 16 B (dwords 0..3) and 64 x 8 B (dwords 4, 5)
constexpr int kCompBytes = 64 * 24;
constexpr int kHiOff = 64 * 16;
constexpr int kSlotBytes = 2 * kCompBytes;   // real part, imaginary part
constexpr int kBufBytes = kMaxSlots * kSlotBytes;
constexpr int kBufs = 3;

// Exactness: a tile element grows by at most 2 * 15 * 15 = 450 units of 1/64
// per sample and a Q element by 3 * 15 * 15 = 675, and must stay within
// 2^24: at most 24,855 samples.
constexpr int kSegSteps = 384;               // 24,576 samples
static_assert((int64_t)kSegSteps * kLoop * 675 <= (int64_t)1 << 24, "float32 sums must be exact");

// A triangle's accumulators in LDS: 16 units of 16 registers (Q of block c in
// unit c, R and I of block pair t in units 4 + 2 t and 5 + 2 t).  Element
// (row r, column c) of a unit is word
//   kRowGroup (r / 4) + (r % 4 ^ rotation) + 4 c,
// so a lane stores 4 registers with 16 bytes.  The output reads a row of the
// four units of one block together: their rotations differ, so lanes along c
// meet on no bank, and kRowGroup and kUnit spread lanes along r.
constexpr int kRowGroup = 4 * kBlk + 4;
constexpr int kUnit = 8 * kRowGroup + 16;
constexpr int kDump = 16 * kUnit;

struct CorrArgs {
    const uint8_t *packed;
    const uint8_t *mask;  // may be null
    int32_t *vis;
    int64_t *count;       // null: counted elsewhere
    int32_t *partials;    // [splits - 1][partial_stride] when splits > 1
    int64_t partial_stride;
    int N, F, T, B;
    int nblk_mask;        // ceil(T / B)
    int nb;               // ceil(N / 32)
    int groups;           // groups per channel
    int splits;
    int steps_per_split;  // 32-sample steps
    int overwrite;
};

// ---------------------------------------------------------------------------
// packing
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
    return __builtin_amdgcn_perm(hi, lo, sel);
}

// 4x4 byte transpose: out[c] = bytes c of d[0..3]
__device__ __forceinline__ void transpose4(const uint32_t *d, uint32_t out[4]) {
    uint32_t e0 = perm(d[1], d[0], 0x05010400u);  // d00 d10 d01 d11
    uint32_t e1 = perm(d[1], d[0], 0x07030602u);  // d02 d12 d03 d13
    uint32_t e2 = perm(d[3], d[2], 0x05010400u);  // d20 d30 d21 d31
    uint32_t e3 = perm(d[3], d[2], 0x07030602u);  // d22 d32 d23 d33
    out[0] = perm(e2, e0, 0x05040100u);
    out[1] = perm(e2, e0, 0x07060302u);
    out[2] = perm(e3, e1, 0x05040100u);
    out[3] = perm(e3, e1, 0x07060302u);
}

// One component of 4 samples (d[e] = sample e of 4 inputs, a byte each) as
// the three bytes of four 6-bit codes, per input:
//   byte 0 = n0 | n1 << 6,  byte 1 = n1 >> 2 | n2 << 4,  byte 2 = n3 << 2
template <bool kRe>
__device__ __forceinline__ void pack4(const uint32_t *d, uint32_t *o) {
    if (kRe) {  // high nibbles
        o[0] = ((d[0] >> 4) & 0x0f0f0f0fu) | ((d[1] << 2) & 0xc0c0c0c0u);
        o[1] = ((d[1] >> 6) & 0x03030303u) | (d[2] & 0xf0f0f0f0u);
        o[2] = (d[3] >> 2) & 0x3c3c3c3cu;
    } else {
        o[0] = (d[0] & 0x0f0f0f0fu) | ((d[1] << 6) & 0xc0c0c0c0u);
        o[1] = ((d[1] >> 2) & 0x03030303u) | ((d[2] << 4) & 0xf0f0f0f0u);
        o[2] = (d[3] << 2) & 0x3c3c3c3cu;
    }
}

// A half-unit: 16 samples of 4 inputs per lane (lanes 0..31: samples 0..15 of
// a 32-sample step, lanes 32..63: samples 16..31).  A component is packed in pieces of about 8
// vector instructions, which the loops place between matrix instructions: pack<kRe, g> for each 4 samples,
// then transpose<k>, k = 0..2, after which w[c] are the 3 dwords of input
// c.  (The asm: computed there, and not moved to where the result is used.)
struct Packer {
    uint32_t x[12];
    v3i w[4];
    template <bool kRe, int G>
    __device__ __forceinline__ void pack(const uint32_t (&raw)[16]) {
        uint32_t *o = x + 3 * G;
        pack4<kRe>(raw + 4 * G, o);
        asm volatile("" : "+v"(o[0]), "+v"(o[1]), "+v"(o[2]));
    }
    template <int K>
    __device__ __forceinline__ void transpose() {
        uint32_t t[4];
        transpose4(x + 4 * K, t);
        asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]));
        w[0][K] = (int)t[0];
        w[1][K] = (int)t[1];
        w[2][K] = (int)t[2];
        w[3][K] = (int)t[3];
    }
    // dwords 3 p .. 3 p + 2 of the component in LDS, dst = slot of input 0's
    // block, component and lane 0
    template <int C>
    __device__ __forceinline__ void write_first(uint8_t *d) const {
        if constexpr (C < 4) {
            *(v3i *)(d + C * kSlotBytes) = w[C];
            write_first<C + 1>(d);
        }
    }
    template <int C>
    __device__ __forceinline__ void write_second(uint8_t *d, uint8_t *e) const {
        if constexpr (C < 4) {
            *(int *)(d + C * kSlotBytes) = w[C].x;
            *(v2i *)(e + C * kSlotBytes) = w[C].yz;
            write_second<C + 1>(d, e);
        }
    }
    __device__ __forceinline__ void write(uint8_t *dst, int p, int lane) const {
        if (p == 0)
            write_first<0>(dst + lane * 16);
        else
            write_second<0>(dst + lane * 16 + 12, dst + kHiOff + lane * 8);
    }
    // the same into operands held in registers
    template <int P, int E>
    __device__ __forceinline__ void keep(v6i (&x)[4]) const {
        if constexpr (E < 12) {
            int t = w[E / 3][E % 3];
            asm volatile("" : "+v"(t));   // (else both arrays stay in memory)
            x[E / 3][3 * P + E % 3] = t;
            keep<P, E + 1>(x);
        }
    }
};

// sign flips of 6-bit codes in an operand (bit 5 of every code)
__device__ __forceinline__ v6i negate(v6i x) {
    constexpr int k0 = 0x20820820, k1 = 0x08208208, k2 = (int)0x82082082u;
    return x ^ (v6i){k0, k1, k2, k0, k1, k2};
}

__device__ __forceinline__ v8i wide(v6i x) {
    return __builtin_shufflevector(x, x, 0, 1, 2, 3, 4, 5, -1, -1);
}

__device__ __forceinline__ v16f mfma(v6i a, v6i b, v16f c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wide(a), wide(b), c, 2, 2, 0, 0, 0, 0);
}

// Input sums of an operand: rows of a 0/1 pattern (4-bit codes, 2 = 1.0).  In
// the 16x16x128 instruction lane l of the pattern is row l % 16, and of an
// operand column l % 16, both at K quarter l / 16; the operand's lanes l and
// l + 32 belong to input l % 32, so quarters 0 and 2 are inputs 0..15, 1 and 3
// inputs 16..31.  Pattern of the real part: row 0 = quarters 0, 2 and row 1
// = quarters 1, 3; of the imaginary part: rows 2 and 3.  Lane c < 16 of the
// result then holds (sum A, sum A', sum B, sum B') / 8 of inputs c and
// c + 16.
__device__ __forceinline__ v4i sum_pattern(bool im, int lane) {
    const int row = lane & 15, odd = (lane >> 4) & 1;
    const int x = row == (im ? 2 : 0) + odd ? 0x22222222 : 0;
    return (v4i){x, x, x, x};
}

// Inline asm, because the four accumulators have to live in ordinary
// registers: in the halves geometry the tiles take every AGPR, and the compiler
// gives the builtin's only those, at 8 register moves per instruction (a third
// of a step's issue slots).  The compiler keeps no distances around it:
//   * a register that a vector instruction has just written may be read 2 wait
//     states later at the earliest, as any of the three operands: the s_nop
//     (with it, two of these may also follow each other on one accumulator);
//   * its result must not be touched for 20 wait states: every use below
//     follows it by at least 8 of the 32-cycle tile instructions, or by a
//     barrier.
__device__ __forceinline__ void sum_mfma(v4i pat, v6i b, v4f &c) {
    asm volatile("s_nop 1\n\t"
                 "v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0 cbsz:4 blgp:2"
                 : "+v"(c)
                 : "v"(pat), "v"(b));
}

__device__ __forceinline__ int units(float x) { return (int)(x * 64.0f); }

// ---------------------------------------------------------------------------
// loads
// ---------------------------------------------------------------------------

// The chunk of a workgroup: samples [t_begin, t_end) of channel f.  Loads go
// through a buffer resource whose range ends with the last dword of the
// chunk's last row, so every dword is checked by the hardware and reads 0
// past it.  All members are wave-uniform.
// 16-byte pieces past N are not loaded; inputs past N in the last piece read the
// next channel's bytes or 0, and their products are never stored.  Only the
// frame's end may cut a dword off (N % 4 != 0): see Tail.
struct Chunk {
    uint64_t base;   // address of (t_begin, f, input 0)
    uint32_t row;    // F * N: bytes between consecutive samples
    int extent;      // bytes from base that may be read, < 2^31
    int t_begin, t_end;
};

__device__ __forceinline__ uint32_t uniform(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

__device__ __forceinline__ Chunk make_chunk(const CorrArgs &a, int f, int t_begin, int t_end) {
    Chunk c;
    const uint64_t base =
        (uint64_t)(uintptr_t)(a.packed + ((int64_t)t_begin * a.F + f) * a.N);
    c.base = ((uint64_t)uniform((uint32_t)(base >> 32)) << 32) | uniform((uint32_t)base);
    c.row = uniform((uint32_t)a.F * (uint32_t)a.N);
    const int64_t rows = (int64_t)(t_end - t_begin - 1) * c.row;
    const int64_t left = ((int64_t)(a.T - 1 - t_begin) * a.F + (a.F - 1 - f)) * a.N + a.N;
    const int64_t want = rows + (a.N + 3) / 4 * 4;
    c.extent = (int)uniform((uint32_t)(want < left ? want : left));
    c.t_begin = t_begin;
    c.t_end = t_end;
    return c;
}

// The chunk from `skip` bytes on (whole rows plus a group's first input).  The
// lookahead past a chunk may pass 2^32 where F * N is above 2^20 (halves
// geometry, 20 loop steps): what wraps into the chunk reads bytes of it, which
// the zero validity words of those steps discard.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t chunk_rsrc(const Chunk &ch, uint32_t skip) {
    uint64_t p = ch.base + skip;
    p = ((uint64_t)uniform((uint32_t)(p >> 32)) << 32) | uniform((uint32_t)p);
    const int left = skip < (uint32_t)ch.extent ? (int)((uint32_t)ch.extent - skip) : 0;
    return __builtin_amdgcn_make_buffer_rsrc((void *)(uintptr_t)p, (short)0,
                                             (int)uniform((uint32_t)left), 0x00020000);
}

// A half-unit (32 samples of a 128-input group) is loaded as 4 x 16 bytes per
// lane, piece k = samples 8 k .. 8 k + 7, kept in registers for two loop steps
// and then put into LDS as rows of 128 bytes, from which the lanes read their
// dwords.  Loading the dwords themselves (one sample of 4 inputs per lane)
// costs an address cycle per quad of lanes: 23 bytes per ns and CU against 72
// with 16-byte loads, less than the matrix cores take in.  Rows 16..31 lie
// 128 bytes further, on the other 32 banks.  The loads may have any byte
// alignment.  Pieces of inputs past N, `inputs` from the group's first, have an
// offset out of range: loaded as bytes of the next channels they cost frames of
// 132 to 388 inputs 2% (260 inputs, 300 channels, 1,200 samples: 284 | 277 us).
constexpr uint32_t kNowhere = 0x80000000u;   // an offset out of every range
constexpr int kRawBytes = 32 * kGroupInputs + 128;

__device__ __forceinline__ void raw_offsets(uint32_t (&voff)[4], uint32_t row, int inputs,
                                            int lane) {
    const uint32_t col = 16 * (lane & 7) < inputs ? 16 * (uint32_t)(lane & 7) : kNowhere;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        voff[k] = (uint32_t)(8 * k + (lane >> 3)) * row + col;
}

template <int kFrom, int kTo>
__device__ __forceinline__ void load_raw(__amdgpu_buffer_rsrc_t r, const uint32_t (&voff)[4],
                                         v4i (&d)[kTo - kFrom]) {
#pragma unroll
    for (int k = kFrom; k < kTo; ++k)
        d[k - kFrom] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff[k], 0, 0);
}

// The end of the frame when N % 4 != 0: the dword of inputs that straddles N
// is out of range in the channel's last row where the frame ends within it
// (and in up to two rows more when F * N < 4).  These dwords are assembled
// from bytes once per segment, into LDS, and replace the loaded ones.
constexpr int kMaxCut = 3;
struct Tail {
    int last;   // last sample of the frame, from the segment's first
    int cut;    // rows whose dword is cut off
};

// Threads 0 .. cut - 1 fill tails[k] = the dword of row T - 1 - k.
__device__ __forceinline__ Tail make_tail(const CorrArgs &a, int f, int t_seg, uint32_t *tails) {
    Tail t;
    t.last = a.T - 1 - t_seg;
    t.cut = 0;
    if (a.N % 4 == 0) return t;
    for (int k = 0; k < kMaxCut && k < a.T; ++k)
        t.cut += (int64_t)(k * a.F + a.F - f) * a.N < (a.N + 3) / 4 * 4 ? 1 : 0;
    const int k = threadIdx.x, n0 = a.N / 4 * 4;
    if (k < t.cut) {
        const uint8_t *p = a.packed + ((int64_t)(a.T - 1 - k) * a.F + f) * a.N;
        uint32_t x = 0;
        for (int c = 0; n0 + c < a.N; ++c) x |= (uint32_t)p[n0 + c] << (8 * c);
        tails[k] = x;
    }
    return t;
}

// Pieces kFrom .. kTo - 1 of a half-unit (32-sample step `word` of the segment,
// validity `bits`, first input input0) into LDS: lost samples zeroed, cut
// rows replaced.
template <int kFrom, int kTo>
__device__ __forceinline__ void store_raw(uint8_t *raw, v4i (&d)[kTo - kFrom], uint32_t bits,
                                          int word, const Tail &t, const uint32_t *tails, int N,
                                          int input0, int lane) {
    if (bits != 0xffffffffu) {
        const int mine = (int)(bits >> (lane >> 3));
#pragma unroll
        for (int k = kFrom; k < kTo; ++k) {
            const int m = __builtin_amdgcn_sbfe(mine, 8 * k, 1);
            d[k - kFrom] &= (v4i){m, m, m, m};
        }
    }
#pragma unroll
    for (int k = kFrom; k < kTo; ++k)
        *(v4i *)(raw + 1024 * k + (k >= 2 ? 128 : 0) + 16 * lane) = d[k - kFrom];
    const int n0 = N / 4 * 4 - input0;   // the straddling dword's byte in a row
    if (t.cut > 0 && n0 >= 0 && n0 < kGroupInputs &&
        (word == t.last >> 5 || word == (t.last - t.cut + 1) >> 5)) {
        const int row = t.last - lane - 32 * word;
        if (lane < t.cut && row >= 8 * kFrom && row < 8 * kTo)
            *(uint32_t *)(raw + 128 * row + (row >= 16 ? 128 : 0) + n0) =
                (bits >> row) & 1u ? tails[lane] : 0u;
    }
}

// a lane's 16 rows (16 (lane / 32) .. + 15)
__device__ __forceinline__ void read_raw(const uint8_t *raw, int lane, uint32_t (&r)[16]) {
    const uint8_t *p = raw + (lane >> 5) * (16 * 128 + 128) + 4 * (lane & 31);
#pragma unroll
    for (int e = 0; e < 16; ++e) r[e] = *(const uint32_t *)(p + 128 * e);
}

// Keeps what is computed from x (output addresses) from being moved ahead of
// the main loop, where it would take the loop's registers.
__device__ __forceinline__ int keep_late(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// n validity words of the samples from t0 on: bit k of word w = sample
// t0 + 32 w + k lies before t1 and not in a lost block.  All threads take
// part; returns the valid samples of the words this thread wrote.
template <int kThreads>
__device__ inline int fill_words(const CorrArgs &a, int f, int t0, int t1, int n,
                                 uint32_t *words) {
    const uint8_t *m = a.mask ? a.mask + (int64_t)f * a.nblk_mask : nullptr;
    int valid = 0;
    for (int w = threadIdx.x; w < n; w += kThreads) {
        const int tb = t0 + 32 * w;
        const int left = t1 - tb;
        uint32_t bits = left >= 32 ? 0xffffffffu : left > 0 ? (1u << left) - 1u : 0u;
        if (m && left > 0) {
            int blk = tb / a.B;
            for (int k0 = blk * a.B - tb; k0 < 32 && blk < a.nblk_mask; k0 += a.B, ++blk) {
                if (m[blk]) {
                    int lo = k0 < 0 ? 0 : k0;
                    int hi = k0 + a.B > 32 ? 32 : k0 + a.B;
                    uint32_t range =
                        (hi - lo >= 32) ? 0xffffffffu : (((1u << (hi - lo)) - 1u) << lo);
                    bits &= ~range;
                }
            }
        }
        words[w] = bits;
        valid += __popc(bits);
    }
    return valid;
}

// ---------------------------------------------------------------------------
// output
// ---------------------------------------------------------------------------

// Where a workgroup's sums of one channel go, and how: the output itself
// (chunk 0) or the chunk's copy of it in the workspace.  Accesses go through a
// buffer resource over the channel's sums, and elements that are not to be
// written have an offset out of its range: without branches around them the
// compiler can tell how many accesses are in flight, and loads of old sums
// need not wait for the stores before them.
struct Dest {
    __amdgpu_buffer_rsrc_t rsrc;   // [P][2] of the channel, P * 8 < 2^27 bytes
    bool add;
};

__device__ __forceinline__ Dest make_dest(const CorrArgs &a, int f, int split, bool first_seg) {
    const int64_t P = (int64_t)a.N * (a.N + 1) / 2;
    const int32_t *out =
        (split == 0 ? a.vis : a.partials + (int64_t)(split - 1) * a.partial_stride) +
        (int64_t)f * P * 2;
    const uint64_t p = (uint64_t)(uintptr_t)out;
    Dest d;
    d.rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(uintptr_t)(((uint64_t)uniform((uint32_t)(p >> 32)) << 32) | uniform((uint32_t)p)),
        (short)0, (int)uniform((uint32_t)P * 8), 0x00020000);
    d.add = !first_seg || (split == 0 && !a.overwrite);
    return d;
}

// byte offset of (i, j) in the packed triangle
__device__ __forceinline__ uint32_t tri_bytes(int N, int i, int j) {
    return 4u * (uint32_t)(i * (2 * N - i + 1)) + 8u * (uint32_t)(j - i);
}

// which word of its four a row takes: r % 4 ^ rotation (of a pair, c ^ c')
__device__ constexpr int unit_rotation(int u) {
    constexpr int pair[6] = {1, 2, 3, 3, 2, 1};
    return u < 4 ? 0 : pair[(u - 4) / 2];
}

// registers of unit U into a dump (kAdd: added to it)
template <bool kAdd, int U>
__device__ __forceinline__ void put_unit(float *dump, const v16f &acc, int lane) {
    constexpr int x = unit_rotation(U);
#pragma unroll
    for (int g = 0; g < 4; ++g) {   // rows 8 g + 4 (lane / 32) .. + 3
        v4f *d = (v4f *)(dump + U * kUnit + (2 * g + (lane >> 5)) * kRowGroup + 4 * (lane & 31));
        v4f y = {acc[4 * g + (0 ^ x)], acc[4 * g + (1 ^ x)], acc[4 * g + (2 ^ x)],
                 acc[4 * g + (3 ^ x)]};
        if (kAdd) y += *d;
        *d = y;
    }
}
template <bool kAdd, int U>
__device__ __forceinline__ void put_triangle(float *dump, const v16f (&acc)[16], int lane) {
    if constexpr (U < 16) {
        put_unit<kAdd, U>(dump, acc[U], lane);
        put_triangle<kAdd, U + 1>(dump, acc, lane);
    }
}

// Output rows of the triangle of one 128-input group (first input in0) from
// its dump: rows 4 q + ci for q = q0, q0 + dq, ... < q1 and every ci; lane l
// takes columns l and l + 64.  A lane reads two words x, y per element and
// gets R and I as linear combinations: for ci < cj (cj = l % 4) x, y = R, I of
// the pair's element (q, q'), for ci > cj those of (q', q), conjugated, and on
// a diagonal tile x, y = Q, Q^T.  Where a row's words lie differs between
// lanes only in whether the row steps along r or along c.  Batches of kRows
// rows, with the old sums of the next one (kAdd) requested before this one's
// are stored.
template <bool kAdd, int kRows>
__device__ __forceinline__ void write_triangle_as(const float *dump, const v2i *sums,
                                                  int valid128, int in0, int N,
                                                  __amdgpu_buffer_rsrc_t out, int q0, int q1,
                                                  int dq, int lane) {
    const int rows = N - in0 < kGroupInputs ? N - in0 : kGroupInputs;
    const int cj = lane & 3, qj = lane >> 2;
    v2i sj[2];
    sj[0] = sums[cj * kBlk + qj];
    sj[1] = sums[cj * kBlk + qj + 16];
    sj[0].x = valid128 - sj[0].x;
    sj[1].x = valid128 - sj[1].x;
    const int batches = (q1 - q0 + kRows * dq - 1) / (kRows * dq);
    auto offset = [&](int b, int r, int s) -> uint32_t {
        const int ci = b / batches, q = q0 + (b % batches * kRows + r) * dq;
        const int i = 4 * q + ci, j = 64 * s + lane;
        const uint32_t at = tri_bytes(N, in0 + i, in0 + j);
        return q < q1 && i < rows && j >= i && j < rows ? at : kNowhere;
    };
    v2i old[kRows][2];
    auto load_old = [&](int b) {
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                old[r][s] = __builtin_amdgcn_raw_buffer_load_b64(out, (int)offset(b, r, s), 0, 0);
    };
    if (kAdd) load_old(0);
#pragma clang loop unroll(disable)
    for (int b = 0; b < 4 * batches; ++b) {
        const int ci = b / batches, qb = q0 + b % batches * kRows * dq;
        const bool q = ci == cj, t = ci > cj;   // diagonal tile, transposed pair
        const int lo = t ? cj : ci, hi = t ? ci : cj;
        const int pair = lo == 0 ? hi - 1 : lo + hi;   // 01 02 03 12 13 23
        const int ux = q ? ci : 4 + 2 * pair, uy = q ? ci : 5 + 2 * pair;
        const bool ty = q || t;                         // y is read along c
        const int rot = ci ^ cj, col = 4 * qj;
        const int trans = kRowGroup * (qj >> 2) + ((qj & 3) ^ rot);
        const float *px = dump + ux * kUnit + (t ? trans : col);
        const float *py = dump + uy * kUnit + (ty ? trans : col);
        // 16 columns further: 4 row groups, or 64 words
        const int dx = t ? 4 * kRowGroup : 64, dy = ty ? 4 * kRowGroup : 64;
        const float rx = q ? 32.0f : 64.0f, ry = q ? 32.0f : 0.0f;
        const float ix = q ? 32.0f : 0.0f, iy = q ? -32.0f : t ? -64.0f : 64.0f;
        float u[kRows][2], w[kRows][2];
        v2i si[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int qi = qb + r * dq < kBlk ? qb + r * dq : 0;
            const int along_r = kRowGroup * (qi >> 2) + ((qi & 3) ^ rot), along_c = 4 * qi;
            const float *ax = px + (t ? along_c : along_r), *ay = py + (ty ? along_c : along_r);
            si[r] = sums[ci * kBlk + qi];
            u[r][0] = ax[0];
            u[r][1] = ax[dx];
            w[r][0] = ay[0];
            w[r][1] = ay[dy];
        }
        v2i x[kRows][2];
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                x[r][s].x = (int)__builtin_fmaf(w[r][s], ry, u[r][s] * rx) + sj[s].x - si[r].x;
                x[r][s].y = (int)__builtin_fmaf(w[r][s], iy, u[r][s] * ix) - sj[s].y + si[r].y;
                if (kAdd) x[r][s] += old[r][s];
            }
        if (kAdd && b + 1 < 4 * batches) load_old(b + 1);
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                __builtin_amdgcn_raw_buffer_store_b64(x[r][s], out, (int)offset(b, r, s), 0, 0);
    }
}

template <int kRows>
__device__ __forceinline__ void write_triangle(const float *dump, const v2i *sums, int valid128,
                                               int in0, int N, const Dest &d, int q0, int q1,
                                               int dq, int lane) {
    if (d.add)
        write_triangle_as<true, kRows>(dump, sums, valid128, in0, N, d.rsrc, q0, q1, dq, lane);
    else
        write_triangle_as<false, kRows>(dump, sums, valid128, in0, N, d.rsrc, q0, q1, dq, lane);
}

// ---------------------------------------------------------------------------
// super geometry
// ---------------------------------------------------------------------------

// Roles of the eight waves of a group (waves w and w + 4 share a SIMD).
// Diagonal: waves 0..3 take 2 x 2 tiles of the first 128-input group against
// the second, waves 4, 5 (6, 7) the two halves of the triangle of the first
// (second) group; waves w and w + 4 pack the real and the imaginary part of one
// half-unit.  Off-diagonal half: every wave takes 2 x 2 tiles, rows 2 (w % 2),
// + 1 and columns 2 (w / 2), + 1; waves 0..3 pack a half-unit of the column
// groups each, waves 4..7 a component of one of the row group.
enum Role { kDiagRect = 0, kTriA = 1, kTriB = 2, kOffFull = 3, kOffRe = 4, kOffIm = 5 };

struct SuperLds {
    union {
        struct {
            uint8_t stage[kBufs * kBufBytes];
            // diagonal: [step parity][half-unit]; off-diagonal: 0..3 the next
            // step of waves 0..3, 4 + [step parity][32-sample step] the rows
            uint8_t raw[8][kRawBytes];
        };
        float dump[2][kDump];
    };
    uint32_t words[2 * kSegSteps];
    v2i sums[kMaxSlots * kBlk];   // (8 T, 8 D) of input 4 q + c at [slot][q]
    uint32_t tails[kMaxCut];
    int valid;
};
static_assert(sizeof(SuperLds) <= 160 * 1024, "LDS of a compute unit");

// Matrix instruction M (0..19) of half a triangle's loop step.  Tiles of half
// A: Q0, Q1 and pairs 01 02 03; of half B: Q2, Q3 and 12 13 23, as acc[0, 1]
// and (re, im) in acc[2 ..].  0..4: A against A, 5..9: B rows against A
// columns, 10..14: -A rows against B, 15..19: B against B.  A block of A is
// negated after its last use as a column.
struct TriOp {
    int row, col, acc;
};
template <bool kHalfB>
__device__ constexpr TriOp tri_op(int m) {
    constexpr TriOp a[20] = {{0, 0, 0}, {0, 1, 2}, {1, 1, 1}, {0, 2, 4}, {0, 3, 6},
                             {0, 0, 0}, {0, 1, 3}, {1, 1, 1}, {0, 2, 5}, {0, 3, 7},
                             {0, 0, 0}, {0, 1, 3}, {0, 2, 5}, {0, 3, 7}, {1, 1, 1},
                             {0, 0, 0}, {0, 1, 2}, {0, 2, 4}, {0, 3, 6}, {1, 1, 1}};
    constexpr TriOp b[20] = {{1, 2, 2}, {1, 3, 4}, {2, 2, 0}, {2, 3, 6}, {3, 3, 1},
                             {1, 2, 3}, {2, 2, 0}, {1, 3, 5}, {2, 3, 7}, {3, 3, 1},
                             {1, 2, 3}, {1, 3, 5}, {2, 2, 0}, {2, 3, 7}, {3, 3, 1},
                             {1, 2, 2}, {1, 3, 4}, {2, 2, 0}, {2, 3, 6}, {3, 3, 1}};
    return kHalfB ? b[m] : a[m];
}
// dump unit of acc[k]
template <bool kHalfB>
__device__ constexpr int tri_unit(int k) {
    return kHalfB ? (k < 2 ? 2 + k : 8 + k) : (k < 2 ? k : 2 + k);
}

__device__ __forceinline__ v6i read_op(const uint8_t *comp, int lane) {
    const v4i x = *(const v4i *)(comp + lane * 16);
    const v2i y = *(const v2i *)(comp + kHiOff + lane * 8);
    return (v6i){x.x, x.y, x.z, x.w, y.x, y.y};
}

template <int ROLE>
struct SuperWave {
    static constexpr bool kTri = ROLE == kTriA || ROLE == kTriB, kHalfB = ROLE == kTriB;
    static constexpr bool kOff = ROLE >= kOffFull;
    static constexpr int kOps = kTri ? 20 : 16;
    // pieces of packing per step, 8 per component
    static constexpr int kAll = ROLE == kOffFull ? 16 : 8;
    static constexpr bool kRe = ROLE == kDiagRect || ROLE == kOffRe;   // (of one component)
    // the first piece (its rows are read after matrix instruction 0), and the
    // end, by which the last piece lands before the barrier
    static constexpr int kLead = 2, kSpan = kOps - 1;
    // 16-byte pieces of its half-unit that the wave loads
    static constexpr int kFrom = ROLE == kOffFull || kRe ? 0 : 2;
    static constexpr int kTo = ROLE == kOffFull ? 4 : kFrom + 2;
    static constexpr int kSets = ROLE == kOffFull ? 1 : 2;   // steps in flight

    const Chunk &ch;
    SuperLds &lds;
    const Tail &tail;
    int N, lane;
    int p, grp, in0;     // its half-unit: 32-sample step, group, the group's first input
    int place;           // of the half-unit in lds.raw (even steps)
    // operand slots: rect rows r0, r0 + 1 and columns c0, c0 + 1, triangle
    // c0 .. c0 + 3; a rect's a, b: which of these it sums
    int r0, c0, a, b;
    int n;               // loop steps of the segment
    int cur, nxt, dec;   // LDS buffers of steps s, s + 1, s + 2
    uint32_t skip, step_bytes, cache;
    v4i pat_re, pat_im;
    uint32_t voff[4];
    v4i in[kSets][kTo - kFrom];   // steps in flight
    uint32_t r[16];           // rows being packed
    Packer pk;
    v6i A[4], B[4];           // triangle blocks; rect: rows A[0..1], B[0..1], columns A[2..3]
    v16f acc[8];              // rect: re, im of tile (i, c) at 4 i + 2 c
    v4f sum[2];               // triangle: its two diagonal blocks; rect: column a, row b

    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rows(int j) const {
        return chunk_rsrc(ch, (uint32_t)j * step_bytes + skip);
    }
    // validity of the half-unit's samples in step j (ascending)
    __device__ __forceinline__ uint32_t bits_of(int j) {
        if ((j & 31) == 0 && j < n) cache = lds.words[2 * j + lane];
        return j < n ? (uint32_t)__builtin_amdgcn_readlane((int)cache, 2 * (j & 31) + p) : 0u;
    }
    __device__ __forceinline__ uint8_t *raw(int x) const {
        return lds.raw[place + (ROLE == kOffFull ? 0 : x * (kOff ? 2 : 4))];
    }
    // Step j (parity X) from registers into LDS, and step j + 2 requested.  A
    // wave with a half-unit of its own has read its previous one; the others
    // alternate between two places, with a barrier between writers and readers.
    template <int X>
    __device__ __forceinline__ void hand_over(int j) {
        constexpr int set = X % kSets;
        store_raw<kFrom, kTo>(raw(X), in[set], bits_of(j), 2 * j + p, tail, lds.tails, N, in0,
                              lane);
        load_raw<kFrom, kTo>(rows(j + kSets), voff, in[set]);
    }
    // Piece K of packing a step (parity X) into buffer dst; the step after
    // (j + 1) is handed over in between.
    template <int X, int K>
    __device__ __forceinline__ void piece(int j, uint8_t *dst) {
        constexpr int k = K % 8;
        constexpr bool re = ROLE == kOffFull ? K >= 8 : kRe;
        if constexpr (K == 1) hand_over<1 - X>(j + 1);
        if constexpr (k < 4)
            pk.template pack<re, k>(r);
        else if constexpr (k < 7)
            pk.template transpose<k - 4>();
        else
            pk.write(dst + 4 * grp * kSlotBytes + (re ? 0 : kCompBytes), p, lane);
    }
    // the pieces that follow matrix instruction M (M < 0: all)
    template <int X, int M, int K>
    __device__ __forceinline__ void pieces_at(int j, uint8_t *dst) {
        if constexpr (K < kAll) {
            if constexpr (M < 0 || kLead + K * (kSpan - kLead) / kAll == M) piece<X, K>(j, dst);
            pieces_at<X, M, K + 1>(j, dst);
        }
    }
    __device__ __forceinline__ v6i op_at(int buf, int slot, int comp) const {
        return read_op(lds.stage + buf + slot * kSlotBytes + comp * kCompBytes, lane);
    }
    // Matrix instruction M of the step, and the operand reads and input sums
    // that follow it.  A register set is read again as soon as its last use
    // is issued.
    template <int M>
    __device__ __forceinline__ void op() {
        if constexpr (kTri) {
            constexpr TriOp t = tri_op<kHalfB>(M);
            constexpr bool row_a = M < 5 || (M >= 10 && M < 15);
            acc[t.acc] = mfma(row_a ? A[t.row] : B[t.row], M < 10 ? A[t.col] : B[t.col], acc[t.acc]);
            constexpr int s = kHalfB ? 2 : 0;   // its diagonal blocks: s, s + 1
            if constexpr (M < 2) sum_mfma(pat_re, A[s + M], sum[M]);
            if constexpr (M == 10 || M == 11) sum_mfma(pat_im, B[s + M - 10], sum[M - 10]);
            if constexpr (M < (kHalfB ? 3 : 4)) B[M + (kHalfB ? 1 : 0)] =
                op_at(cur, c0 + M + (kHalfB ? 1 : 0), 1);
            if constexpr (!kHalfB) {
                if constexpr (M == 5) A[0] = negate(A[0]);
                if constexpr (M == 7) A[1] = negate(A[1]);
                if constexpr (M == 10) A[2] = op_at(nxt, c0 + 2, 0);
                if constexpr (M == 11) A[3] = op_at(nxt, c0 + 3, 0);
                if constexpr (M == 14) A[0] = op_at(nxt, c0, 0);
                if constexpr (M == 15) A[1] = op_at(nxt, c0 + 1, 0);
            } else {
                if constexpr (M == 4) A[1] = negate(A[1]);
                if constexpr (M == 6) A[2] = negate(A[2]);
                if constexpr (M == 9) A[3] = negate(A[3]);
                if constexpr (M == 12) A[1] = op_at(nxt, c0 + 1, 0);
                if constexpr (M == 14) A[2] = op_at(nxt, c0 + 2, 0);
                if constexpr (M == 15) A[3] = op_at(nxt, c0 + 3, 0);
            }
        } else {
            // by column: A rows, B rows x A of column 0; B, A rows x A of
            // column 1; then B rows, -A rows x B of column 0; -A, B x B of 1
            constexpr int i = M & 1, ph = M / 2, c = (ph >> 1) & 1;
            constexpr bool row_a = ph == 0 || ph == 3 || ph == 5 || ph == 6;
            constexpr bool im = (ph < 4) != row_a;
            constexpr int y = 4 * i + 2 * c + (im ? 1 : 0);
            acc[y] = mfma(row_a ? A[i] : B[i], A[2 + c], acc[y]);
            if constexpr (kOff) {
                if constexpr (M == 1 || M == 9)
                    if (a == 0) sum_mfma(M == 1 ? pat_re : pat_im, A[2], sum[0]);
                if constexpr (M == 5 || M == 13)
                    if (a == 1) sum_mfma(M == 5 ? pat_re : pat_im, A[3], sum[0]);
                if constexpr (M == 3) {
                    if (b == 0) {
                        sum_mfma(pat_re, A[0], sum[1]);
                        sum_mfma(pat_im, B[0], sum[1]);
                    }
                    if (b == 1) {
                        sum_mfma(pat_re, A[1], sum[1]);
                        sum_mfma(pat_im, B[1], sum[1]);
                    }
                }
            }
            if constexpr (M == 3) A[2] = op_at(cur, c0, 1);
            if constexpr (M == 7) A[3] = op_at(cur, c0 + 1, 1);
            if constexpr (M == 6 || M == 7) A[M - 6] = negate(A[M - 6]);
            if constexpr (M == 11) A[2] = op_at(nxt, c0, 0);
            if constexpr (M == 12 || M == 13) A[M - 12] = op_at(nxt, r0 + M - 12, 0);
            if constexpr (M == 14 || M == 15) B[M - 14] = op_at(nxt, r0 + M - 14, 1);
            if constexpr (M == 15) A[3] = op_at(nxt, c0 + 1, 0);
        }
    }
    template <int X, int M>
    __device__ __forceinline__ void ops(int j, uint8_t *dst) {
        if constexpr (M < kOps) {
            op<M>();
            if constexpr (M == 0) read_raw(raw(X), lane, r);
            pieces_at<X, M, 0>(j, dst);
            __builtin_amdgcn_sched_barrier(0);
            ops<X, M + 1>(j, dst);
        }
    }
    // matrix instructions of step s (parity X), packing of step s + 2
    template <int X>
    __device__ __forceinline__ void step(int s) {
        ops<X, 0>(s + 2, lds.stage + dec);
        __syncthreads();
        const int t = cur;
        cur = nxt;
        nxt = dec;
        dec = t;
    }
    template <int X>
    __device__ __forceinline__ void prologue_step() {
        read_raw(raw(X), lane, r);
        pieces_at<X, -1, 0>(X, lds.stage + X * kBufBytes);
        __syncthreads();
    }
    // the operands that the first step expects
    __device__ __forceinline__ void first_ops() {
        if constexpr (kTri) {
#pragma unroll
            for (int c = kHalfB ? 1 : 0; c < 4; ++c) A[c] = op_at(0, c0 + c, 0);
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                A[i] = op_at(0, r0 + i, 0);
                B[i] = op_at(0, r0 + i, 1);
                A[2 + i] = op_at(0, c0 + i, 0);
            }
        }
    }
    // input sums into LDS, in units of 1/8 of an input's T and D
    __device__ __forceinline__ void put_sum(int slot, const v4f &x) {
        v2i *d = lds.sums + slot * kBlk + lane;
        d[0] = (v2i){units(x.x + x.z), units(x.x - x.z)};
        d[16] = (v2i){units(x.y + x.w), units(x.y - x.w)};
    }
    __device__ __forceinline__ void put_sums() {
        if (lane >= 16) return;
        if constexpr (kTri) {
            put_sum(c0 + (kHalfB ? 2 : 0), sum[0]);
            put_sum(c0 + (kHalfB ? 3 : 1), sum[1]);
        } else if constexpr (kOff) {
            put_sum(c0 + a, sum[0]);
            if (b < 2) put_sum(r0 + b, sum[1]);
        }
    }
    // accumulators of slice S of a rect: rows 8 (S % 4) .. of row block S / 4,
    // t[4 v + 2 c + (0 re, 1 im)]
    template <int S, int E>
    __device__ __forceinline__ void take(float (&t)[16]) const {
        if constexpr (E < 16) {
            t[E] = acc[4 * (S / 4) + E % 4][4 * (S % 4) + E / 4];
            take<S, E + 1>(t);
        }
    }
    // the accumulators into a triangle's dump
    template <int K>
    __device__ __forceinline__ void put_dump(float *dump, int ln) const {
        if constexpr (K < 8) {
            put_unit<false, tri_unit<kHalfB>(K)>(dump, acc[K], ln);
            put_dump<K + 1>(dump, ln);
        }
    }
};

// The tiles of a rect wave: a lane holds 2 consecutive inputs j of a row, 16
// bytes of the output (another wave the next two).  In a loop of 8 slices of 4
// rows (per lane), so that the code stays small: it runs once per workgroup,
// from a cold instruction cache, and unrolled over all accumulators of four
// waves it took 70 us.
template <int ROLE, bool kAdd>
__device__ __forceinline__ void write_rect_as(const SuperWave<ROLE> &w, const v2i *sums,
                                              int valid128, int row_in0, int col_in0, int N,
                                              __amdgpu_buffer_rsrc_t out, int lane) {
    const int jj = lane & 31, j0 = col_in0 + 4 * jj + (w.c0 & 3);
    v2i sj[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        sj[c] = sums[(w.c0 + c) * kBlk + jj];
        sj[c].x = valid128 - sj[c].x;
    }
    // row v of slice s, from element c on
    auto offset = [&](int s, int v, int c) -> uint32_t {
        const int i = row_in0 + 4 * (8 * (s & 3) + 4 * (lane >> 5) + v) + ((w.r0 + (s >> 2)) & 3);
        const uint32_t at = tri_bytes(N, i, j0 + c);
        return i < N && j0 + c < N ? at : kNowhere;
    };
    const bool pairs = N % 2 == 0;   // uniform: whole pairs, else element by element
    v4i old[4];
    auto load_old = [&](int s) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (pairs) {
                old[v] = __builtin_amdgcn_raw_buffer_load_b128(out, (int)offset(s, v, 0), 0, 0);
            } else {
                const v2i y = __builtin_amdgcn_raw_buffer_load_b64(out, (int)offset(s, v, 0), 0, 0);
                const v2i z = __builtin_amdgcn_raw_buffer_load_b64(out, (int)offset(s, v, 1), 0, 0);
                old[v] = (v4i){y.x, y.y, z.x, z.y};
            }
        }
    };
    if (kAdd) load_old(0);
#pragma clang loop unroll(disable)
    for (int s = 0; s < 8; ++s) {
        float t[16];
        switch (s) {
            case 0: w.template take<0, 0>(t); break;
            case 1: w.template take<1, 0>(t); break;
            case 2: w.template take<2, 0>(t); break;
            case 3: w.template take<3, 0>(t); break;
            case 4: w.template take<4, 0>(t); break;
            case 5: w.template take<5, 0>(t); break;
            case 6: w.template take<6, 0>(t); break;
            default: w.template take<7, 0>(t); break;
        }
        v4i x[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const v2i si = sums[(w.r0 + (s >> 2)) * kBlk + 8 * (s & 3) + 4 * (lane >> 5) + v];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                x[v][2 * c] = units(t[4 * v + 2 * c]) + sj[c].x - si.x;
                x[v][2 * c + 1] = units(t[4 * v + 2 * c + 1]) - sj[c].y + si.y;
            }
            if (kAdd) x[v] += old[v];
        }
        if (kAdd && s < 7) load_old(s + 1);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (pairs) {
                __builtin_amdgcn_raw_buffer_store_b128(x[v], out, (int)offset(s, v, 0), 0, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b64(x[v].xy, out, (int)offset(s, v, 0), 0, 0);
                __builtin_amdgcn_raw_buffer_store_b64(x[v].zw, out, (int)offset(s, v, 1), 0, 0);
            }
        }
    }
}

template <int ROLE>
__device__ __forceinline__ void write_rect(const SuperWave<ROLE> &w, const v2i *sums, int valid128,
                                           int row_in0, int col_in0, int N, const Dest &d,
                                           int lane) {
    if (d.add)
        write_rect_as<ROLE, true>(w, sums, valid128, row_in0, col_in0, N, d.rsrc, lane);
    else
        write_rect_as<ROLE, false>(w, sums, valid128, row_in0, col_in0, N, d.rsrc, lane);
}

template <int ROLE>
__device__ __forceinline__ void run_super(const CorrArgs &a, const Group &g, int f, int gid,
                                          int split, int wave, SuperLds &lds) {
    using W = SuperWave<ROLE>;
    const int t_begin = split * a.steps_per_split * kStep;
    int t_end = t_begin + a.steps_per_split * kStep;
    if (t_end > a.T) t_end = a.T;
    const int loops = (t_end - t_begin + kLoop - 1) / kLoop;
    const int segs = (loops + kSegSteps - 1) / kSegSteps;
    const int per = (loops + segs - 1) / segs;
    int counted = 0;

    for (int seg = 0; seg < segs; ++seg) {
        const int t_seg = t_begin + seg * per * kLoop;
        const int t_stop = t_seg + per * kLoop < t_end ? t_seg + per * kLoop : t_end;
        const Chunk ch = make_chunk(a, f, t_seg, t_stop);
        const Tail tail = make_tail(a, f, t_seg, lds.tails);
        W w = {ch, lds, tail};
        w.N = a.N;
        w.lane = threadIdx.x & 63;
        w.p = (wave >> 1) & 1;
        w.grp = !W::kOff ? wave & 1 : ROLE == kOffFull ? 1 + (wave & 1) : 0;
        w.in0 = group_input(g, w.grp);
        w.place = !W::kOff ? wave & 3 : ROLE == kOffFull ? wave : 4 + w.p;
        w.a = wave & 1;
        w.b = wave >> 1;
        w.r0 = 2 * w.a;
        w.c0 = W::kTri ? 4 * (wave >> 1 & 1) : 4 + 2 * w.b;
        w.n = (t_stop - t_seg + kLoop - 1) / kLoop;
        w.step_bytes = kLoop * ch.row;
        w.skip = 32u * (uint32_t)w.p * ch.row + (uint32_t)w.in0;
        w.cache = 0;
        w.pat_re = sum_pattern(false, w.lane);
        w.pat_im = sum_pattern(true, w.lane);
        raw_offsets(w.voff, ch.row, a.N - w.in0, w.lane);
        load_raw<W::kFrom, W::kTo>(w.rows(0), w.voff, w.in[0]);
        if constexpr (W::kSets == 2) load_raw<W::kFrom, W::kTo>(w.rows(1), w.voff, w.in[1]);
        if (threadIdx.x == 0) lds.valid = 0;
        const int my_valid = fill_words<kSuperThreads>(a, f, t_seg, t_stop, 2 * w.n, lds.words);
#pragma unroll
        for (int k = 0; k < 8; ++k) w.acc[k] = (v16f){0};
#pragma unroll
        for (int k = 0; k < 2; ++k) w.sum[k] = (v4f){0};
        __syncthreads();
        w.template hand_over<0>(0);
        __syncthreads();
        w.template prologue_step<0>();
        w.template prologue_step<1>();
        w.cur = 0;
        w.nxt = kBufBytes;
        w.dec = 2 * kBufBytes;
        w.first_ops();
        // pairs of steps (two register sets in flight); a step past the
        // segment's last adds zeros
        for (int s = 0; s < w.n; s += 2) {
            w.template step<0>(s);
            w.template step<1>(s + 1);
        }

        // ---- sums out -----------------------------------------------------
        const int lane = keep_late(threadIdx.x & 63);
        atomicAdd(&lds.valid, my_valid);
        if constexpr (W::kTri) w.template put_dump<0>(lds.dump[w.c0 >> 2], lane);
        w.put_sums();
        __syncthreads();
        const int valid = lds.valid;
        counted += valid;
        const Dest d = make_dest(a, f, split, seg == 0);
        if constexpr (!W::kTri)
            write_rect(w, lds.sums, 128 * valid, group_input(g, 0), group_input(g, w.c0 >> 2), a.N,
                       d, lane);
        // The triangles' 32 row quads each: 6 per triangle wave, 2 (of the
        // short rows) per rect wave, which has its own tiles to write.
        if constexpr (!W::kOff) {
            const int q0 = W::kTri ? wave - 4 : 24 + 2 * wave;
            const int q1 = W::kTri ? 24 : q0 + 2;
#pragma clang loop unroll(disable)
            for (int k = 0; k < 2; ++k)
                write_triangle<W::kTri ? 6 : 2>(lds.dump[k], lds.sums + 4 * k * kBlk, 128 * valid,
                                                group_input(g, k), a.N, d, q0, q1,
                                                W::kTri ? 4 : 1, lane);
        }
        if (seg + 1 < segs) __syncthreads();   // the dump and sums are free
    }
    if (a.count && gid == 0 && threadIdx.x == 0)
        a.count[f] = a.overwrite ? counted : a.count[f] + counted;
}

// ---------------------------------------------------------------------------
// halves geometry
// ---------------------------------------------------------------------------

// A whole triangle: Q[c] = acc[c], pair t (01 02 03 12 13 23) re = acc[4 + 2 t],
// im = the next.
__device__ constexpr int pair_lo(int t) { return t < 3 ? 0 : t < 5 ? 1 : 2; }
__device__ constexpr int pair_hi(int t) { return t < 3 ? t + 1 : t < 5 ? t - 1 : 3; }
constexpr int kTriOps = 40;

// Matrix instruction m of a triangle's loop step on the components A, B of
// its four blocks.  0..9: A against A; 10..19: B rows against A columns,
// column block by column block, so that block c of A may be negated once
// its column is done (m == neg_after(c)); 20..29: -A rows against B; 30..39:
// B against B.
__device__ constexpr int tri_tile(int k) {   // k = 0..9 by column block: Q0 | 01 Q1 | 02 12 Q2 | ...
    return k == 0 ? 0 : k == 1 ? 4 : k == 2 ? 1 : k == 3 ? 5 : k == 4 ? 7 : k == 5 ? 2
         : k == 6 ? 6 : k == 7 ? 8 : k == 8 ? 9 : 3;
}
__device__ constexpr int tri_row_block(int tile) { return tile < 4 ? tile : pair_lo(tile - 4); }
__device__ constexpr int tri_col_block(int tile) { return tile < 4 ? tile : pair_hi(tile - 4); }
// by row block: Q0 01 02 03 | Q1 12 13 | ...
__device__ constexpr int tri_tile_rows(int k) {
    return k == 0 ? 0 : k < 4 ? k + 3 : k == 4 ? 1 : k < 7 ? k + 2 : k == 7 ? 2 : k == 8 ? 9 : 3;
}

template <int M>
__device__ __forceinline__ void tri_mfma(const v6i (&A)[4], const v6i (&B)[4], v16f (&acc)[16]) {
    constexpr int k = M % 10, ph = M / 10;
    constexpr int tile = ph == 2 ? tri_tile_rows(k) : tri_tile(k);
    constexpr int r = tri_row_block(tile), c = tri_col_block(tile);
    constexpr bool im = ph == 1 || ph == 2;
    constexpr int x = tile < 4 ? tile : 4 + 2 * (tile - 4) + (im ? 1 : 0);
    acc[x] = mfma(ph == 0 || ph == 2 ? A[r] : B[r], ph < 2 ? A[c] : B[c], acc[x]);
}
// the matrix instruction after which block c of A is free as a column
template <int M>
__device__ __forceinline__ void tri_negate(v6i (&A)[4]) {
    if constexpr (M == 10) A[0] = negate(A[0]);
    if constexpr (M == 12) A[1] = negate(A[1]);
    if constexpr (M == 15) A[2] = negate(A[2]);
    if constexpr (M == 19) A[3] = negate(A[3]);
}

struct SmallLds {
    union {
        uint8_t raw[kSmallWaves][2][kRawBytes];   // a wave's next loop step
        float dump[2][kDump];
    };
    uint32_t words[2 * kSegSteps];
    int sums[4 * kBlk * 2];
    uint32_t tails[kMaxCut];
    int valid;
};

struct SmallWave {
    static constexpr int kAll = 32;   // pieces of packing per step
    const Chunk &ch;
    SmallLds &lds;
    const Tail &tail;
    int N, lane, in0, n;
    v4i pat_re, pat_im;
    int wave;
    uint32_t voff[4];
    v4i in[2][2][4];      // steps in flight: [set][32-sample step]
    uint32_t r[16];       // rows being packed
    uint32_t cache;
    Packer pk;
    v6i A[2][4], B[2][4];
    v16f acc[16];
    v4f sum[4];

    // 32-sample step P of step j
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rows(int j, int P) const {
        return chunk_rsrc(ch, (uint32_t)(2 * j + P) * 32 * ch.row + (uint32_t)in0);
    }
    // Validity of 32-sample step P of step j = wave + 4 i (ascending): a lane
    // keeps the words of the next 32 steps of the wave.
    template <int P>
    __device__ __forceinline__ uint32_t bits_of(int j) {
        const int i = (j - wave) >> 2;
        if (P == 0 && (i & 31) == 0 && j < n) {
            const int w = 2 * (j + 4 * (lane >> 1)) + (lane & 1);
            cache = lds.words[w < 2 * n ? w : 0];
        }
        return j < n ? (uint32_t)__builtin_amdgcn_readlane((int)cache, 2 * (i & 31) + P) : 0u;
    }
    // 32-sample step P of step j (set X) from registers into LDS, and of step
    // j + 8 requested
    template <int X, int P>
    __device__ __forceinline__ void hand_over(int j) {
        const uint32_t bits = bits_of<P>(j);
        store_raw<0, 4>(lds.raw[wave][P], in[X][P], bits, 2 * j + P, tail, lds.tails, N, in0,
                        lane);
        load_raw<0, 4>(rows(j + 8, P), voff, in[X][P]);
    }
    // Piece K of packing step j (set X) into operands An, Bn, handing over
    // step j + 4
    template <int X, int K>
    __device__ __forceinline__ void piece(int j, v6i (&An)[4], v6i (&Bn)[4]) {
        constexpr int P = K / 16, k = K % 8;
        constexpr bool re = K / 8 % 2 == 1;
        if constexpr (K == 1 || K == 17) hand_over<1 - X, P>(j + 4);
        if constexpr (K == 12) read_raw(lds.raw[wave][1], lane, r);
        if constexpr (k < 4)
            pk.template pack<re, k>(r);
        else if constexpr (k < 7)
            pk.template transpose<k - 4>();
        else
            pk.template keep<P, 0>(re ? An : Bn);
    }
    // the pieces that follow matrix instruction M (M < 0: all)
    template <int X, int M, int K>
    __device__ __forceinline__ void pieces_at(int j, v6i (&An)[4], v6i (&Bn)[4]) {
        if constexpr (K < kAll) {
            if constexpr (M < 0 || 4 + K * (kTriOps - 4) / kAll == M) piece<X, K>(j, An, Bn);
            pieces_at<X, M, K + 1>(j, An, Bn);
        }
    }
    template <int X, int M>
    __device__ __forceinline__ void ops(int j, v6i (&Ac)[4], v6i (&Bc)[4], v6i (&An)[4],
                                        v6i (&Bn)[4]) {
        if constexpr (M < kTriOps) {
            tri_mfma<M>(Ac, Bc, acc);
            if constexpr (M < 4) sum_mfma(pat_re, Ac[M], sum[M]);
            if constexpr (M >= 10 && M < 14) sum_mfma(pat_im, Bc[M - 10], sum[M - 10]);
            tri_negate<M>(Ac);
            if constexpr (M == 0) read_raw(lds.raw[wave][0], lane, r);
            pieces_at<X, M, 0>(j, An, Bn);
            __builtin_amdgcn_sched_barrier(0);
            ops<X, M + 1>(j, Ac, Bc, An, Bn);
        }
    }
    // step j from the operands of set K; the wave's next is packed into the
    // other
    template <int K>
    __device__ __forceinline__ void step(int j) {
        ops<1 - K, 0>(j + 4, A[K], B[K], A[1 - K], B[1 - K]);
    }
};

// Wave w takes loop steps w, w + 4, ... of the chunk.
__device__ __forceinline__ void run_small(const CorrArgs &a, const Group &g, int f, int split,
                                          int wave, SmallLds &lds) {
    const int t_begin = split * a.steps_per_split * kStep;
    int t_end = t_begin + a.steps_per_split * kStep;
    if (t_end > a.T) t_end = a.T;
    const int loops = (t_end - t_begin + kLoop - 1) / kLoop;
    const int segs = (loops + kSegSteps - 1) / kSegSteps;
    const int per = (loops + segs - 1) / segs;
    int counted = 0;

    for (int seg = 0; seg < segs; ++seg) {
        const int t_seg = t_begin + seg * per * kLoop;
        const int t_stop = t_seg + per * kLoop < t_end ? t_seg + per * kLoop : t_end;
        const Chunk ch = make_chunk(a, f, t_seg, t_stop);
        const Tail tail = make_tail(a, f, t_seg, lds.tails);
        SmallWave w = {ch, lds, tail};
        w.N = a.N;
        w.lane = threadIdx.x & 63;
        w.in0 = group_input(g, 0);
        w.n = (t_stop - t_seg + kLoop - 1) / kLoop;
        w.pat_re = sum_pattern(false, w.lane);
        w.pat_im = sum_pattern(true, w.lane);
        w.wave = wave;
        raw_offsets(w.voff, ch.row, a.N - w.in0, w.lane);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int P = 0; P < 2; ++P) load_raw<0, 4>(w.rows(wave + 4 * k, P), w.voff, w.in[k][P]);
        if (threadIdx.x == 0) lds.valid = 0;
        for (int e = threadIdx.x; e < 4 * kBlk * 2; e += kSmallThreads) lds.sums[e] = 0;
        const int my_valid = fill_words<kSmallThreads>(a, f, t_seg, t_stop, 2 * w.n, lds.words);
#pragma unroll
        for (int k = 0; k < 16; ++k) w.acc[k] = (v16f){0};
#pragma unroll
        for (int k = 0; k < 4; ++k) w.sum[k] = (v4f){0};
        __syncthreads();
        w.hand_over<0, 0>(wave);
        w.hand_over<0, 1>(wave);
        read_raw(lds.raw[wave][0], w.lane, w.r);
        w.pieces_at<0, -1, 0>(wave, w.A[0], w.B[0]);
        // pairs of steps; a step past the segment's last adds zeros
        for (int j = wave; j < w.n; j += 8) {
            w.step<0>(j);
            w.step<1>(j + 4);
        }

        // ---- the waves' sums, added in LDS: 0 and 1 store theirs, 2 and 3 add
        // to these, and all add the two (exact: the bound of kSegSteps covers
        // the four of them) ----------------------------------------------------
        const int lane = keep_late(threadIdx.x & 63);
        __syncthreads();
        if (wave < 2) put_triangle<false, 0>(lds.dump[wave], w.acc, lane);
        __syncthreads();
        if (wave >= 2) put_triangle<true, 0>(lds.dump[wave - 2], w.acc, lane);
        atomicAdd(&lds.valid, my_valid);
        if (lane < 16) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                int *s = lds.sums + 2 * (c * kBlk + lane);
                atomicAdd(s, units(w.sum[c].x + w.sum[c].z));
                atomicAdd(s + 1, units(w.sum[c].x - w.sum[c].z));
                atomicAdd(s + 32, units(w.sum[c].y + w.sum[c].w));
                atomicAdd(s + 33, units(w.sum[c].y - w.sum[c].w));
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < kDump / 4; e += kSmallThreads)
            ((v4f *)lds.dump[0])[e] += ((const v4f *)lds.dump[1])[e];
        __syncthreads();
        const int valid = lds.valid;
        counted += valid;
        write_triangle<4>(lds.dump[0], (const v2i *)lds.sums, 128 * valid, w.in0, a.N,
                       make_dest(a, f, split, seg == 0), wave, kBlk, kSmallWaves, lane);
        if (seg + 1 < segs) __syncthreads();
    }
    if (a.count && threadIdx.x == 0)
        a.count[f] = a.overwrite ? counted : a.count[f] + counted;
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------

// Workgroup b runs on XCD b % 8 (round-robin dispatch); number the work so
// that consecutive work items (the time chunks and groups of one channel)
// share an XCD and its L2.
__device__ __forceinline__ int64_t xcd_local_index(int64_t b, int64_t total) {
    const int64_t per = total / 8, rem = total % 8;
    const int64_t x = b % 8, idx = b / 8;
    return x * per + (x < rem ? x : rem) + idx;
}

// the two kernels of one geometry each, so that each is register-allocated
// for its own roles
template <bool kSmall>
using Lds = typename std::conditional<kSmall, SmallLds, SuperLds>::type;

// One work item: tile group gid of channel f over time chunk `split`.
// Every wave of a super group runs the same number of barriers; the tile
// pattern is fixed per group kind.
template <bool kSmall>
__device__ __forceinline__ void run_item(const CorrArgs &a, int f, int gid, int split,
                                         Lds<kSmall> &lds) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Group g = make_group(a.nb, gid);
    if constexpr (kSmall) {
        run_small(a, g, f, split, wave, lds);
    } else if (g.diag) {
        if (wave < 4)
            run_super<kDiagRect>(a, g, f, gid, split, wave, lds);
        else if ((wave & 1) == 0)
            run_super<kTriA>(a, g, f, gid, split, wave, lds);
        else
            run_super<kTriB>(a, g, f, gid, split, wave, lds);
    } else {
        if (wave < 4)
            run_super<kOffFull>(a, g, f, gid, split, wave, lds);
        else if ((wave & 1) == 0)
            run_super<kOffRe>(a, g, f, gid, split, wave, lds);
        else
            run_super<kOffIm>(a, g, f, gid, split, wave, lds);
    }
}

// One frame: workgroup -> (channel, group, chunk), groups of a channel
// and chunks of a (channel, group) numbered next to each other.
template <bool kSmall>
constexpr int kThreadsOf = kSmall ? kSmallThreads : kSuperThreads;

template <bool kSmall>
__global__ __launch_bounds__(kThreadsOf<kSmall>, kSmall ? 1 : 2) void corr_kernel(CorrArgs a) {
    __shared__ __attribute__((aligned(16))) Lds<kSmall> lds;
    const int G = a.groups;
    const int64_t total = (int64_t)a.F * G * a.splits;
    int64_t w = xcd_local_index(blockIdx.x, total);
    const int gid = (int)(w % G);
    w /= G;
    const int split = (int)(w % a.splits);
    const int f = (int)(w / a.splits);
    run_item<kSmall>(a, f, gid, split, lds);
}

// ---------------------------------------------------------------------------
// batched persistent launch
// ---------------------------------------------------------------------------

// One correlator instance of a batch, as the kernel sees it.
struct BatchInstance {
    const uint8_t *packed;
    const uint8_t *mask;
    int32_t *vis;
    int64_t *count;
    int32_t N, F, T, B;
    int32_t nblk_mask, nb, groups, splits;
    int32_t steps_per_split, pad_;
    int64_t partial_base;    // first int32 of its chunk copies
    int64_t partial_stride;  // int32s per chunk copy
};

struct BatchItem {
    int32_t inst, f, gid, split;
};

// A grid of one workgroup per CU pulls work items from a queue until it is
// empty (every workgroup reaches the exit).  The last workgroup to finish
// resets the queue, so the next launch of the same plan starts clean and
// the launch can be replayed from a graph.  Items are accumulated into their
// instances' resident sums.  A batch has one list of items per geometry,
// each drained by its own launch of this kernel.
template <bool kSmall>
__global__ __launch_bounds__(kThreadsOf<kSmall>, kSmall ? 1 : 2) void batch_kernel(
    const BatchInstance *inst, const BatchItem *items, int n_items, int *queue,
    int32_t *partials) {
    __shared__ __attribute__((aligned(16))) Lds<kSmall> lds;
    __shared__ int s_item;
    for (;;) {
        __syncthreads();  // the previous item has released LDS
        if (threadIdx.x == 0) s_item = atomicAdd(&queue[0], 1);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(s_item);  // uniform: scalar loads below
        if (it >= n_items) break;
        // every field is wave-uniform: readfirstlane keeps them in scalar
        // registers (buffer resources and offsets must live there)
        auto u32 = [](int32_t v) { return (int32_t)__builtin_amdgcn_readfirstlane(v); };
        auto u64 = [](int64_t v) {
            uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
            uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
            return (int64_t)(((uint64_t)hi << 32) | lo);
        };
        auto ptr = [&](const void *p) { return (void *)(uintptr_t)u64((int64_t)(uintptr_t)p); };
        const BatchItem w = items[it];
        const int wi = u32(w.inst), wf = u32(w.f), wg = u32(w.gid), ws = u32(w.split);
        const BatchInstance &bi = inst[wi];
        CorrArgs a;
        a.packed = (const uint8_t *)ptr(bi.packed);
        a.mask = (const uint8_t *)ptr(bi.mask);
        a.vis = (int32_t *)ptr(bi.vis);
        a.count = nullptr;   // count_list_kernel
        a.partials = partials + u64(bi.partial_base);
        a.partial_stride = u64(bi.partial_stride);
        a.N = u32(bi.N);
        a.F = u32(bi.F);
        a.T = u32(bi.T);
        a.B = u32(bi.B);
        a.nblk_mask = u32(bi.nblk_mask);
        a.nb = u32(bi.nb);
        a.groups = u32(bi.groups);
        a.splits = u32(bi.splits);
        a.steps_per_split = u32(bi.steps_per_split);
        a.overwrite = 0;
        run_item<kSmall>(a, wf, wg, ws, lds);
    }
    if (threadIdx.x == 0) {
        int done = atomicAdd(&queue[1], 1);
        if (done == (int)gridDim.x - 1) {
            queue[0] = 0;
            queue[1] = 0;
        }
    }
}

// ---------------------------------------------------------------------------
// merge of time chunks, valid-sample counts
// ---------------------------------------------------------------------------

// Valid samples of one channel (mask row m of nblk blocks of B samples, T
// samples), counted by one wave: lane l takes blocks l, l + 64, ..., four
// per pass with every load issued before the first is used (indices clamped
// in range), then the lanes' sums are added; every lane gets the total.
__device__ inline int64_t valid_count(const uint8_t *m, int nblk, int B, int T, int lane) {
    if (m == nullptr) return T;
    const int last = nblk - 1;
    int n = 0;  // <= T < 2^24
    for (int b0 = 0; b0 <= last; b0 += 64 * 4) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = m[min(b0 + 64 * u + lane, last)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = b0 + 64 * u + lane;
            const int64_t lo = (int64_t)b * B;
            const int64_t hi = lo + B < T ? lo + B : T;
            n += (b <= last && v[u] == 0u) ? (int)(hi - lo) : 0;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
    return n;
}

// An instance whose time chunks are merged: chunk 0 has written its sums to
// `vis`, chunks 1 .. splits-1 left theirs in copies of it, `stride` int32s
// apart.
struct MergeInst {
    int32_t *vis;
    const int32_t *partials;
    int64_t ints;         // of one copy
    int64_t stride;
    int splits, pad_;
    int64_t block_begin;  // first merge block of the instance (batch lists)
};

constexpr int kMergeThreads = 256;
constexpr int64_t kMergeInts = kMergeThreads * 4;   // int32s of a merge block

// Block b of an instance adds its 16 bytes per thread of every copy; the
// loads of four copies are in flight together.
__device__ __forceinline__ void merge_block(const MergeInst &m, int64_t b) {
    const int64_t e = (b * kMergeThreads + threadIdx.x) * 4;
    if (e >= m.ints) return;
    const bool whole = e + 4 <= m.ints;   // else 2 are left (ints is even)
    int32_t *o = m.vis + e;
    v4i x;
    if (whole) {
        x = *(const v4i_a8 *)o;
    } else {
        const v2i y = *(const v2i *)o;
        x = (v4i){y.x, y.y, 0, 0};
    }
    for (int s0 = 1; s0 < m.splits; s0 += 4) {
        v4i v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)   // a copy's last 16 bytes lie inside its stride
            v[k] = *(const v4i *)(m.partials +
                                  (int64_t)(s0 + k < m.splits ? s0 + k - 1 : 0) * m.stride + e);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (s0 + k < m.splits) x += v[k];
    }
    if (whole)
        *(v4i_a8 *)o = x;
    else
        *(v2i *)o = (v2i){x.x, x.y};
}

// Valid-sample counts of a frame, taken by extra blocks of its merge launch
// (block first_block + k counts channels 4 k .. 4 k + 3, one per wave), so a
// chunked frame needs no launch of its own for them.
struct CountArgs {
    const uint8_t *mask;
    int64_t *count;
    int nblk, B, T, F, overwrite;
    int64_t first_block;
};

__global__ __launch_bounds__(kMergeThreads) void merge_kernel(MergeInst m, CountArgs c) {
    if ((int64_t)blockIdx.x >= c.first_block) {
        const int f = (int)(blockIdx.x - c.first_block) * (kMergeThreads / 64) +
                      (int)(threadIdx.x >> 6);
        if (f >= c.F) return;
        const int lane = threadIdx.x & 63;
        const int64_t n = valid_count(c.mask ? c.mask + (int64_t)f * c.nblk : nullptr, c.nblk,
                                      c.B, c.T, lane);
        if (lane == 0) c.count[f] = c.overwrite ? n : c.count[f] + n;
        return;
    }
    merge_block(m, blockIdx.x);
}

// a batch's chunked instances, sorted by block_begin; block b belongs to the
// last instance whose first block is <= b
__global__ __launch_bounds__(kMergeThreads) void merge_list_kernel(const MergeInst *list, int n) {
    const int64_t b = blockIdx.x;
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (list[mid].block_begin <= b)
            lo = mid;
        else
            hi = mid - 1;
    }
    const MergeInst m = list[lo];
    merge_block(m, b - m.block_begin);
}

// The counts of every instance of a batch (block (b, y): instance b, whose
// channels the waves of its gridDim.y blocks take in turn); batches
// accumulate.  A channel is a chain of loads and lane exchanges, so channels
// are spread: 8 instances in one block each took 13.5 us, in 16 each
// 4.1.
constexpr int kCountWaves = 4;

__global__ __launch_bounds__(64 * kCountWaves) void count_list_kernel(const BatchInstance *inst) {
    const BatchInstance &x = inst[blockIdx.x];
    const int lane = threadIdx.x & 63;
    for (int f = (int)blockIdx.y * kCountWaves + (int)(threadIdx.x >> 6); f < x.F;
         f += (int)gridDim.y * kCountWaves) {
        const int64_t n = valid_count(x.mask ? x.mask + (int64_t)f * x.nblk_mask : nullptr,
                                      x.nblk_mask, x.B, x.T, lane);
        if (lane == 0) x.count[f] += n;
    }
}

// ---------------------------------------------------------------------------
// normalisation
// ---------------------------------------------------------------------------

// out = (float)((double)v / (double)n), 0 when n == 0; four values per
// thread and iteration (16-byte accesses when kVec: both pointers aligned)
template <bool kVec>
__global__ void normalize_kernel(const int32_t *vis, const int64_t *count, float *out,
                                 int64_t per_channel, int F) {
    const int64_t total = per_channel * F;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x * 4;
    for (int64_t k = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) * 4; k < total;
         k += stride) {
        if (kVec && k + 4 <= total && (k / per_channel) == ((k + 3) / per_channel)) {
            int64_t n = count[k / per_channel];
            v4i v = *(const v4i *)(vis + k);
            double dn = (double)n;
            float4 o;
            o.x = n == 0 ? 0.0f : (float)((double)v.x / dn);
            o.y = n == 0 ? 0.0f : (float)((double)v.y / dn);
            o.z = n == 0 ? 0.0f : (float)((double)v.z / dn);
            o.w = n == 0 ? 0.0f : (float)((double)v.w / dn);
            *(float4 *)(out + k) = o;
        } else {
            for (int64_t e = k; e < k + 4 && e < total; ++e) {
                int64_t n = count[e / per_channel];
                out[e] = n == 0 ? 0.0f : (float)((double)vis[e] / (double)n);
            }
        }
    }
}

}  // namespace xe
