// short_kernels.hpp -- the correlator's kernel for short time chunks (gfx950).
//
// The 6-bit kernels (xcorr_kernels.hpp) run their loop at about twice this
// one's rate but cost more per workgroup: more code to fetch into a cold
// instruction cache, sums in float32 that pass through LDS and are turned
// back, and input sums to be applied.  This one integrates in int8, whose
// sums are the output as they stand.  Where each is faster: see
// short_steps() in plan.hpp.
//
//   x = a + i b.  With the real K-vector of one input laid out as the pairs
//   (a_t, b_t) and the derived vector (b_t, -a_t),
//     Re V_ij = sum_k Xr_i[k] Xr_j[k]      Im V_ij = sum_k Xp_i[k] Xr_j[k]
//   with Xr = (a, b), Xp = (b, -a): two real int8 GEMMs with K = 2T on the
//   matrix cores, exact int32 accumulation.  Only tiles with I <= J run.
//   A diagonal tile (I = J) is Hermitian, so it runs one GEMM:
//     Q = Xs Xr^T with Xs = Xr + Xp = (a + b, b - a)  (fits int8),
//     Re = (Q + Q^T) / 2,  Im = (Q - Q^T) / 2  (exact: Q + Q^T = 2 Re).
//
// A workgroup of eight waves integrates one tile group (plan.hpp) of one
// channel over one chunk of time, in blocks of 32 consecutive inputs.  Per
// staged step of 32 samples it
//   1. loads the packed bytes of its input blocks with dword buffer loads
//      along the input axis (the buffer range ends at the chunk), kDepth
//      steps ahead, into a ring of register sets;
//   2. substitutes 0x88 (= 0) for lost samples, samples past the chunk and
//      inputs past N, transposes 4x4 byte blocks in registers so that each
//      dword holds 4 samples of one input, decodes nibbles to signed int8
//      with carry-free byte arithmetic and writes LDS in the operand layout
//      of v_mfma_i32_32x32x32_i8: per block and 16-sample sub-step, lane l
//      reads 16 bytes = 8 samples of input l % 32.  Both operands use the
//      same K order, so the order of samples inside K does not change the
//      sum;
//   3. runs its tiles: A operand (rows) in Xr, Xp (and Xs) form, B Xr.
// The loop is software-pipelined over three LDS buffers: the decode of step
// s+2 and the operand reads of step s+1 overlap the MFMAs of step s; one
// barrier per step; eight waves, two per SIMD, so that one wave's decode
// and waits overlap the other's MFMAs.
//
// Halves geometry (N <= 128): the 8 staged slots hold blocks 0..3 at two
// consecutive 32-sample steps (slots 4..7 one step later), so a loop step
// covers 64 samples: waves 4 and 5 integrate the triangle over the even
// steps, waves 6 and 7 over the odd ones, and the rectangle waves only
// stage.  At the end waves 6 and 7 hand their sums to 4 and 5 through LDS,
// which write them.
//
// Output: as in xcorr_kernels.hpp, through range-checked accesses with every
// address in 32 bits, so that no branch stands between a tile's loads and
// stores.  With branches around them, a separate launch for the counts and
// unaligned rows loaded byte by byte, 128 inputs x 256 channels x 512 samples
// took 22.3 us and take 15.9, 256 x 256 x 64 23.5 and 20.1, 98 x 256 x 2048 67
// and 35.  Short chunks are bound by the latency of their one pass: loads,
// a few steps, the output read and written.
#pragma once

#include "xcorr_kernels.hpp"

namespace xe {
namespace brief {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kRing = 4;                      // steps of raw bytes in flight
constexpr int kFragBytes = kBlk * kStep * 2;  // one decoded operand of a block per step
// A diagonal group stages Xr and Xs per block (8 slots x 2 operands), an
// off-diagonal half stages Xr only (12 slots)
constexpr int kBufBytes = 16 * kFragBytes;

// Slot s of the staged blocks holds the inputs from slot_input on:
//   diagonal:      block s                          (s < 8)
//   off-diagonal:  row block s for s < 4, column block s - 4 otherwise
//   halves:        block s % 4 (slots 4..7 one step later)
__device__ __forceinline__ int slot_input(const Group &g, bool small, int s) {
    return small                 ? (s & 3) * kBlk
           : (g.diag || s < 4) ? g.input0 + s * kBlk
                                 : g.column0 + (s - 4) * kBlk;
}

// nibble u in 0..15 per byte -> u - 8 as int8: (u + 0x78) ^ 0x80
__device__ __forceinline__ uint32_t nib_to_s8(uint32_t u) {
    return (u + 0x78787878u) ^ 0x80808080u;
}

// -x per byte for x in [-8, 7]: ((x ^ 0x7f) + 1) ^ 0x80, no byte overflows
__device__ __forceinline__ uint32_t neg_s8(uint32_t x) {
    return ((x ^ 0x7f7f7f7fu) + 0x01010101u) ^ 0x80808080u;
}

// 4 validity bits -> 4 byte masks (0xff = valid)
__device__ __forceinline__ uint32_t bits_to_bytes(uint32_t b4) {
    uint32_t m = (b4 * 0x00204081u) & 0x01010101u;  // bit k -> byte k
    return (m << 8) - m;
}

// A 16-byte operand chunk holds, for 8 samples of one input,
// (a0..3 | b0..3 | a4..7 | b4..7).  Xr chunk -> Xp chunk (b | -a).
__device__ __forceinline__ v4i make_xp(v4i x) {
    v4i p;
    p.x = x.y;
    p.y = (int)neg_s8((uint32_t)x.x);
    p.z = x.w;
    p.w = (int)neg_s8((uint32_t)x.z);
    return p;
}

__device__ __forceinline__ v16i mfma(v4i a, v4i b, v16i c) {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}

// LDS position of the 16-byte chunk c (= lane-group g * 32 + row r) of
// (block slot s, operand op, sub-step u).  The 64 chunks of one (s, op, u)
// form 1 KB; lane l of a reading wave takes chunk l, stored at
//   phys(l, s) = l ^ (s & 1) ^ (bit 4 of l) << 1,
// a permutation inside aligned groups of 4 chunks, so a wave's 16-byte
// reads stay conflict-free while the stagers' 8-byte writes (below) hit all
// 64 banks exactly once per half-wave.
__device__ __forceinline__ int phys_chunk(int c, int s) {
    return c ^ (s & 1) ^ (((c >> 4) & 1) << 1);
}
__device__ __forceinline__ int chunk_off(int slot_bytes, int s, int op, int u, int c) {
    return s * slot_bytes + op * kFragBytes + u * 1024 + (phys_chunk(c, s) << 4);
}

// ---------------------------------------------------------------------------
// staging: global packed bytes -> decoded int8 operand layout in LDS
// ---------------------------------------------------------------------------

// One staging unit = 4 inputs (n0..n0+3) x 4 samples (sample quad sq of the
// step) of block slot s.  Units come in rounds of 64 per wave: lane bits
// (q = lane & 7, s_lo = bit 3, h = bit 4, s_hi = bit 5) give input quad q,
// slot 4 sg + s_lo + 2 s_hi and sample quad 2 o + h, with the octet o and
// the slot group sg fixed per wave-round.  Coordinates do not change along
// the time loop.
struct Unit {
    int s, q, sq;
    uint32_t voff;  // byte offset of (sample 4 sq, input n0) within the chunk;
                    // out of range (reads 0) when the inputs lie past N
    bool act;       // inputs lie below N (else staged as 0)
    bool hi;        // halves geometry, slots 4..7: the odd step of the pair
};

template <int UPT>
struct Prefetch {
    uint32_t d[UPT][4];
};

// The chunk of a workgroup: samples [t_begin, t_end) of channel f, read
// through a buffer resource, so that every load is bounds-checked by the
// hardware (a dword past its range reads 0; such samples are replaced below).
// Aligned frames: the range ends with the chunk.  Others: dwords are loaded
// from any byte address, and a row's last dword may hold bytes of the next
// row, of inputs whose products are never stored; the range ends with the
// frame, and a dword that would be cut off there is loaded from the frame's
// last 4 bytes and shifted.  (Its bytes, one by one: 2.5 times the time of a
// 2048-sample frame of 250 inputs.)  It starts up to 3 bytes before the chunk, so that 4 bytes lie
// before every end.
struct RowChunk {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t row_bytes;  // F * N: bytes between consecutive samples
    uint32_t last;       // unaligned: offset of the range's last 4 bytes
    uint32_t lead;       // bytes before the chunk
    int t_begin, t_end;
};

template <bool kAligned>
__device__ __forceinline__ RowChunk open_chunk(const CorrArgs &a, int f, int t_begin, int t_end) {
    RowChunk c;
    const int64_t first = ((int64_t)t_begin * a.F + f) * a.N;   // the chunk's first byte
    const int64_t row = (int64_t)a.F * a.N;
    int64_t extent = (int64_t)(t_end - t_begin - 1) * row + a.N;
    c.lead = 0;
    if (!kAligned) {
        c.lead = first < 3 ? (uint32_t)first : 3u;
        const int64_t left = (int64_t)a.T * row - first;
        extent = (int64_t)c.lead + (extent + 3 < left ? extent + 3 : left);
    }
    const uint64_t base = (uint64_t)(uintptr_t)(a.packed + first - c.lead);
    const uint64_t p = ((uint64_t)uniform((uint32_t)(base >> 32)) << 32) | uniform((uint32_t)base);
    const uint32_t n = uniform((uint32_t)extent);
    c.rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(uintptr_t)p, (short)0, (int)n, 0x00020000);
    c.row_bytes = uniform((uint32_t)row);
    c.last = n - 4;
    c.t_begin = t_begin;
    c.t_end = t_end;
    return c;
}

// The whole byte offset goes into the vector offset, which the hardware
// checks against the resource's range; the scalar offset stays 0.  Offsets
// stay below 2^31 (the host bounds a chunk, its lookahead included).
template <bool kAligned, int UPT>
__device__ __forceinline__ void issue_loads(const RowChunk &ch, int tb, const Unit (&u)[UPT],
                                            Prefetch<UPT> &p) {
    const uint32_t step_off = (uint32_t)(tb - ch.t_begin) * ch.row_bytes + ch.lead;
#pragma unroll
    for (int r = 0; r < UPT; ++r) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t off = u[r].voff + step_off + (uint32_t)e * ch.row_bytes;
            if (!kAligned && off > ch.last) off = ch.last;
            p.d[r][e] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(ch.rsrc, (int)off, 0, 0);
        }
    }
}
// the bytes of dwords that were cut off at the frame's end, into place (of
// loads past the chunk the result does not matter)
template <bool kAligned, int UPT>
__device__ __forceinline__ void shift_cut(const RowChunk &ch, int tb, const Unit (&u)[UPT],
                                          Prefetch<UPT> &p) {
    if (kAligned) return;
    const uint32_t step_off = (uint32_t)(tb - ch.t_begin) * ch.row_bytes + ch.lead;
    // (uniform) every row of the step, two 32-sample steps in the halves
    // geometry, ends before the range does
    if (step_off + (2 * kStep + 1) * ch.row_bytes <= ch.last) return;
#pragma unroll
    for (int r = 0; r < UPT; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t off = (uint32_t)keep_late((int)u[r].voff) + step_off +
                                 (uint32_t)e * ch.row_bytes;
            if (off > ch.last) p.d[r][e] >>= (8 * (off - ch.last)) & 31;
        }
}

// Decode one prefetched step into LDS (validity words vb0 for its units, vb1
// for the odd-step units of the halves geometry).  Per input, from the
// masked nibbles
// A' = a + 8 and B' = b + 8 (4 samples per dword):
//   Xr = (a | b)             a = (A' + 0x78) ^ 0x80
//   Xs = (a + b | b - a)     a + b = (A' + B' + 0x70) ^ 0x80,
//                            b - a = ((B' | 0x80) - A') ^ 0x80
// all per byte without carries or borrows; Xs only for diagonal groups.
// A unit writes bytes 8h .. 8h+7 of its inputs' chunks (h = sq & 1).
template <bool kXs, bool kSmall, int UPT>
__device__ __forceinline__ void commit(const Unit (&u)[UPT], const Prefetch<UPT> &p,
                                       uint32_t vb0, uint32_t vb1, uint8_t *buf,
                                       int slot_bytes) {
#pragma unroll
    for (int r = 0; r < UPT; ++r) {
        uint32_t L[4];
        transpose4(p.d[r], L);
        const uint32_t vbits = kSmall && u[r].hi ? vb1 : vb0;
        const uint32_t vq = u[r].act ? (vbits >> (4 * u[r].sq)) & 15u : 0u;
        const uint32_t m = bits_to_bytes(vq);
        const int o = u[r].sq >> 1, h = u[r].sq & 1;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            uint32_t Lm = (L[c] & m) | (0x88888888u & ~m);
            uint32_t an = (Lm >> 4) & 0x0f0f0f0fu, bn = Lm & 0x0f0f0f0fu;
            uint8_t *dst = buf + chunk_off(slot_bytes, u[r].s, 0, o >> 1,
                                           (o & 1) * 32 + 4 * u[r].q + c) + 8 * h;
            v2u xr = {nib_to_s8(an), nib_to_s8(bn)};
            *(v2u *)dst = xr;
            if (kXs) {
                v2u xs = {(an + bn + 0x70707070u) ^ 0x80808080u,
                          ((bn | 0x80808080u) - an) ^ 0x80808080u};
                *(v2u *)(dst + kFragBytes) = xs;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// the tiles of one wave
// ---------------------------------------------------------------------------

// Three tile shapes (see plan.hpp), 16 MFMAs per 32-sample step each:
//   kRect: row block s0 x column blocks c0 .. c0+3 (4 off-diagonal tiles);
//   kTriA: of the 4 blocks s0 .. s0+3, the diagonal tiles of blocks 0 and 1
//          (as Q) and the pairs (0,1) (0,2) (0,3);
//   kTriB: the diagonal tiles of blocks 2 and 3 and the pairs (1,2) (1,3)
//          (2,3).
enum Shape { kRect = 0, kTriA = 1, kTriB = 2 };

template <int SHAPE>
struct Tiles;

template <>
struct Tiles<kRect> {
    static constexpr int NQ = 0, NO = 4, NT = 4, NXP = 1;
    __device__ static constexpr int qb(int) { return 0; }
    __device__ static constexpr int row(int) { return 0; }
    __device__ static constexpr int col(int t) { return t; }
    __device__ static constexpr int xpi(int) { return 0; }  // Xp index of a row
};

template <>
struct Tiles<kTriA> {
    static constexpr int NQ = 2, NO = 3, NT = 5, NXP = 1;
    __device__ static constexpr int qb(int k) { return k; }
    __device__ static constexpr int row(int) { return 0; }
    __device__ static constexpr int col(int t) { return t + 1; }
    __device__ static constexpr int xpi(int) { return 0; }
};

template <>
struct Tiles<kTriB> {
    static constexpr int NQ = 2, NO = 3, NT = 5, NXP = 2;
    __device__ static constexpr int qb(int k) { return 2 + k; }
    __device__ static constexpr int row(int t) { return t < 2 ? 1 : 2; }
    __device__ static constexpr int col(int t) { return t < 2 ? t + 2 : 3; }
    __device__ static constexpr int xpi(int i) { return i - 1; }
};

template <int SHAPE>
struct Acc {
    using T = Tiles<SHAPE>;
    v16i q[T::NQ > 0 ? T::NQ : 1];
    v16i re[T::NO], im[T::NO];
};

// Operand fragments of one 16-sample sub-step.  kRect: x[0] = the row
// block, y[j] = column block c0 + j.  kTriA/B: x[i] = block s0 + i (the
// ones the shape uses), xs[k] = Xs of its k-th diagonal block.
template <int SHAPE>
struct Ops {
    static constexpr bool kTri = SHAPE != kRect;
    v4i x[kTri ? 4 : 1];
    v4i y[kTri ? 1 : 4];
    v4i xs[kTri ? 2 : 1];
};

template <int SHAPE>
__device__ __forceinline__ void read_ops(const uint8_t *buf, int slot_bytes, int s0, int c0,
                                         int sub, Ops<SHAPE> &o) {
    const int lane = threadIdx.x & 63;
    auto frag = [&](int s, int op) {
        return *(const v4i *)(buf + chunk_off(slot_bytes, s, op, sub, lane));
    };
    if (SHAPE == kRect) {
        o.x[0] = frag(s0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) o.y[j] = frag(c0 + j, 0);
    } else {
#pragma unroll
        for (int i = SHAPE == kTriA ? 0 : 1; i < 4; ++i) o.x[i] = frag(s0 + i, 0);
#pragma unroll
        for (int k = 0; k < 2; ++k) o.xs[k] = frag(s0 + Tiles<SHAPE>::qb(k), 1);
    }
}

// One loop step: the 16 MFMAs of step s, with the decode of step s + 2
// woven into them and the operands of the next sub-steps read ahead
// (kMma = false: the decode only, for the rectangle waves of the halves
// geometry, whose tiles would pair different time steps).
//   * (s, sub 0) operands arrive in `o`, read during the previous step;
//     (s, sub 1) operands are read at the start; (s + 1, sub 0) operands
//     are read into `o` once the sub-0 MFMAs have taken theirs, so the next
//     step starts its MFMAs as soon as it passes the barrier.
//   * the decode of step s + 2 comes in small pieces (a 4x4 transpose, or
//     the decode and LDS write of one input) between MFMAs, spread over the
//     first 14 of them so the last LDS write lands before the barrier.  A
//     piece's VALU work issues while the MFMA before it occupies the matrix
//     core; scheduling barriers keep the order.
template <int SHAPE, bool kXs, int UPT, bool kMma, bool kSmall>
__device__ __forceinline__ void pipelined_step(const uint8_t *cur, const uint8_t *next,
                                               uint8_t *dec, int slot_bytes, int s0, int c0,
                                               Acc<SHAPE> &acc, const Unit (&u)[UPT],
                                               const Prefetch<UPT> &p, uint32_t vb0,
                                               uint32_t vb1, Ops<SHAPE> &o) {
    // 5 pieces: the transposes of all units, then input c of all units;
    // the units' chains are independent, so a piece has UPT-fold ILP
    constexpr int kPieces = 5;
    constexpr int kSpan = 14;
    using TL = Tiles<SHAPE>;
    Ops<SHAPE> o1;
    if (kMma) read_ops(cur, slot_bytes, s0, c0, 1, o1);
    // decode state
    uint32_t L[UPT][4];
    uint32_t msk[UPT];
    auto piece = [&](int k) {
        const int c = k - 1;
        if (c < 0) {
#pragma unroll
            for (int r = 0; r < UPT; ++r) {
                transpose4(p.d[r], L[r]);
                const uint32_t vbits = kSmall && u[r].hi ? vb1 : vb0;
                const uint32_t vq = u[r].act ? (vbits >> (4 * u[r].sq)) & 15u : 0u;
                msk[r] = bits_to_bytes(vq);
            }
        } else {
#pragma unroll
            for (int r = 0; r < UPT; ++r) {
                const int oo = u[r].sq >> 1, h = u[r].sq & 1;
                uint32_t Lm = (L[r][c] & msk[r]) | (0x88888888u & ~msk[r]);
                uint32_t an = (Lm >> 4) & 0x0f0f0f0fu, bn = Lm & 0x0f0f0f0fu;
                uint8_t *dst = dec + chunk_off(slot_bytes, u[r].s, 0, oo >> 1,
                                               (oo & 1) * 32 + 4 * u[r].q + c) + 8 * h;
                v2u xr = {nib_to_s8(an), nib_to_s8(bn)};
                *(v2u *)dst = xr;
                if (kXs) {
                    v2u v = {(an + bn + 0x70707070u) ^ 0x80808080u,
                             ((bn | 0x80808080u) - an) ^ 0x80808080u};
                    *(v2u *)(dst + kFragBytes) = v;
                }
            }
        }
    };
    v4i xp[TL::NXP];
    auto rows_xp = [&](const Ops<SHAPE> &q) {
        if (SHAPE == kRect) {
            xp[0] = make_xp(q.x[0]);
        } else {
#pragma unroll
            for (int i = 0; i < TL::NXP; ++i) xp[i] = make_xp(q.x[TL::row(2 * i)]);
        }
    };
    // MFMA k (0..7) of a sub-step
    auto mfma_op = [&](const Ops<SHAPE> &q, int k) {
        if (SHAPE == kRect) {
            const int t = k / 2;
            if (k % 2 == 0)
                acc.re[t] = mfma(q.x[0], q.y[t], acc.re[t]);
            else
                acc.im[t] = mfma(xp[0], q.y[t], acc.im[t]);
        } else if (k < 2) {
            acc.q[k] = mfma(q.xs[k], q.x[TL::qb(k)], acc.q[k]);
        } else {
            const int t = (k - 2) / 2;
            const int i = TL::row(t), j = TL::col(t);
            if (k % 2 == 0)
                acc.re[t] = mfma(q.x[i], q.x[j], acc.re[t]);
            else
                acc.im[t] = mfma(xp[TL::xpi(i)], q.x[j], acc.im[t]);
        }
    };

    if (kMma) rows_xp(o);
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        if (kMma) {
            if (m == 8) rows_xp(o1);
            if (m == 9) read_ops(next, slot_bytes, s0, c0, 0, o);
            if (m < 8)
                mfma_op(o, m);
            else
                mfma_op(o1, m - 8);
        }
#pragma unroll
        for (int q = 0; q < kPieces; ++q)
            if (q * kSpan / kPieces == m) piece(q);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Where the tiles of a wave lie: tile k < NQ is the diagonal tile of block
// qb(k), the others pair a row block with a column block.  Element v of a
// tile held by `lane` is (i, j) = (8 (v/4) + 4 (lane/32) + v%4, lane%32)
// within the tile (the output layout of v_mfma_i32_32x32x32_i8).
template <int SHAPE>
struct TileMap {
    Group g;
    bool small;
    int s0, c0, N;
    __device__ void rc(int k, int &rs, int &cs) const {
        using TL = Tiles<SHAPE>;
        if (k < TL::NQ) {
            rs = cs = s0 + TL::qb(k);
        } else if (SHAPE == kRect) {
            rs = s0;
            cs = c0 + TL::col(k - TL::NQ);
        } else {
            rs = s0 + TL::row(k - TL::NQ);
            cs = s0 + TL::col(k - TL::NQ);
        }
    }
    // byte offset of the element in the channel's packed triangle, out of
    // range when it lies below the diagonal or past N
    __device__ uint32_t elem(int k, int v, int lane) const {
        int rs, cs;
        rc(k, rs, cs);
        const int i = slot_input(g, small, rs) + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        const int j = slot_input(g, small, cs) + (lane & 31);
        return i > j || j >= N ? kNowhere : tri_bytes(N, i, j);
    }
};

// The role of wave `wave` in a tile group: its staging share, tile shape and
// first row / column slot.  Waves w and w + 4 share a SIMD: each SIMD gets
// one rectangle and (diagonal group) one half triangle.
template <int NSLOT_, int SHAPE_, int UPT_, bool kMma_ = true, bool kSmall_ = false>
struct Role {
    static constexpr int NSLOT = NSLOT_, SHAPE = SHAPE_, UPT = UPT_;
    static constexpr bool kMma = kMma_;     // runs MFMAs (else stages only)
    static constexpr bool kSmall = kSmall_;  // the halves geometry
};

template <class Fn>
__device__ __forceinline__ void with_role(const Group &g, bool small, int wave, Fn &&fn) {
    if (small) {
        // halves geometry: the rectangle waves stage only; waves 4, 5 take
        // the triangle of slots 0..3 (even steps), waves 6, 7 of 4..7 (odd)
        if (wave < 4)
            fn(Role<8, kRect, 1, false, true>{}, wave, 4);
        else if ((wave & 1) == 0)
            fn(Role<8, kTriA, 1, true, true>{}, 2 * (wave - 4), 0);
        else
            fn(Role<8, kTriB, 1, true, true>{}, 2 * (wave - 5), 0);
    } else if (g.diag) {
        if (wave < 4)  // row block `wave` x columns 4..7
            fn(Role<8, kRect, 1>{}, wave, 4);
        else if ((wave & 1) == 0)  // triangle of blocks 0..3 (wave 4) or 4..7 (wave 6)
            fn(Role<8, kTriA, 1>{}, 2 * (wave - 4), 0);
        else
            fn(Role<8, kTriB, 1>{}, 2 * (wave - 5), 0);
    } else {
        // row slot wave % 4 x column slots 4 + 4 (wave / 4) .. + 3
        if (wave < 4)
            fn(Role<12, kRect, 2>{}, wave, 4);
        else
            fn(Role<12, kRect, 1>{}, wave - 4, 8);
    }
}

// Q of a diagonal tile -> (Re, Im) = ((Q + Q^T) / 2, (Q - Q^T) / 2), exact
// (Q + Q^T = 2 Re is even; a short chunk's Q stays below 2^20).  The transpose
// goes through LDS (32 x 33 int32 per wave, padded against bank conflicts).
__device__ __forceinline__ void split_q(const v16i &q, int32_t *tbuf, v16i &re, v16i &im) {
    const int lane = threadIdx.x & 63;
    const int col = lane & 31;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        int row = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        tbuf[row * 33 + col] = q[v];
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's LDS writes landed
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        int row = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        const int qij = q[v], qji = tbuf[col * 33 + row];
        re[v] = (qij + qji) >> 1;
        im[v] = (qij - qji) >> 1;
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
}

// UPT = staging units per lane and step (wave-rounds of 64 units): the
// 16 (diagonal) or 24 (off-diagonal) wave-rounds of a step are dealt to the
// 8 waves as x = r * 8 + wave.
template <bool kAligned, bool kOverwrite, int NSLOT, int SHAPE, int UPT, bool kMma, bool kSmall>
__device__ __forceinline__ void run_wave(const CorrArgs &a, const Group &g, int f, int gid,
                                         int split, int s0, int c0, uint8_t *lds,
                                         uint32_t *mwords) {
    using TL = Tiles<SHAPE>;
    constexpr bool kDiagGroup = NSLOT == 8;
    constexpr int SLOT = kDiagGroup ? 2 * kFragBytes : kFragBytes;
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;

    const int t_begin = split * a.steps_per_split * kStep;
    int t_end = t_begin + a.steps_per_split * kStep;
    if (t_end > a.T) t_end = a.T;
    // 32-sample steps of the chunk, and loop steps: one 32-sample step, or
    // a pair of them in the halves geometry
    const int nsteps32 = (t_end - t_begin + kStep - 1) / kStep;
    constexpr int pair = kSmall ? 2 : 1;
    const int nsteps = (nsteps32 + pair - 1) / pair;
    constexpr int step_samples = pair * kStep;

    const RowChunk ch = open_chunk<kAligned>(a, f, t_begin, t_end);
    Unit u[UPT];
#pragma unroll
    for (int r = 0; r < UPT; ++r) {
        const int x = r * kWaves + wave;  // wave-round: 64 units
        const int o = x / (NSLOT / 4), sg = x % (NSLOT / 4);
        const int h = (lane >> 4) & 1;
        u[r].q = lane & 7;
        u[r].s = 4 * sg + ((lane >> 3) & 1) + 2 * ((lane >> 5) & 1);
        u[r].sq = 2 * o + h;
        int n0 = slot_input(g, kSmall, u[r].s) + 4 * u[r].q;
        u[r].act = n0 < a.N;
        u[r].hi = kSmall && u[r].s >= 4;
        u[r].voff = u[r].act ? (uint32_t)(4 * u[r].sq + (u[r].hi ? kStep : 0)) * ch.row_bytes +
                                   (uint32_t)n0
                             : 0x80000000u;
    }

    Acc<SHAPE> acc;
#pragma unroll
    for (int k = 0; k < TL::NO; ++k) {
        acc.re[k] = (v16i){0};
        acc.im[k] = (v16i){0};
    }
#pragma unroll
    for (int k = 0; k < TL::NQ; ++k) acc.q[k] = (v16i){0};

    // pipeline, per step s:
    //   raw bytes   loaded kDepth steps ahead into a ring of register sets
    //               (set k holds steps = k mod D), loop unrolled D times so
    //               each set has fixed registers;
    //   decode      two steps ahead, into the third of three LDS buffers;
    //   MFMA        from the buffer of step s, operands read ahead.
    // Steps past the chunk are staged as zeros (the last ring is padded).
    constexpr int D = kRing;
    static_assert(D >= 3, "the ring must hold the step being decoded and two in flight");
    // one validity word per 32-sample step: each lane keeps one, read out with
    // readlane
    fill_words<kThreads>(a, f, t_begin, t_end, kShortSteps, mwords);
    Prefetch<UPT> pf[D];
#pragma unroll
    for (int k = 0; k < D; ++k) issue_loads<kAligned>(ch, t_begin + k * step_samples, u, pf[k]);
    __syncthreads();
    const uint32_t mcache = mwords[lane];
    auto vbits_of = [&](int j32) -> uint32_t {
        return j32 < nsteps32 ? (uint32_t)__builtin_amdgcn_readlane((int)mcache, j32) : 0u;
    };
    shift_cut<kAligned>(ch, t_begin, u, pf[0]);
    shift_cut<kAligned>(ch, t_begin + step_samples, u, pf[1]);
    commit<kDiagGroup, kSmall>(u, pf[0], vbits_of(0), vbits_of(pair - 1), lds, SLOT);
    commit<kDiagGroup, kSmall>(u, pf[1], vbits_of(pair), vbits_of(2 * pair - 1),
                               lds + kBufBytes, SLOT);
    __syncthreads();
    Ops<SHAPE> ops;
    if (kMma) read_ops(lds, SLOT, s0, c0, 0, ops);
    int b_cur = 0, b_next = kBufBytes, b_dec = 2 * kBufBytes;  // LDS byte offsets
    const int npad = (nsteps + D - 1) / D * D;
    for (int sb = 0; sb < npad; sb += D) {
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const int s = sb + k;
            const int j = s + 2;   // step decoded now
            const int j32 = pair * j;
            const uint32_t vb0 = vbits_of(j32), vb1 = kSmall ? vbits_of(j32 + 1) : vb0;
            issue_loads<kAligned>(ch, t_begin + (s + D) * step_samples, u, pf[k]);
            shift_cut<kAligned>(ch, t_begin + j * step_samples, u, pf[(k + 2) % D]);
            pipelined_step<SHAPE, kDiagGroup, UPT, kMma, kSmall>(
                lds + b_cur, lds + b_next, lds + b_dec, SLOT, s0, c0, acc, u, pf[(k + 2) % D], vb0,
                vb1, ops);
            __syncthreads();
            const int t = b_cur;
            b_cur = b_next;
            b_next = b_dec;
            b_dec = t;
        }
    }

    // the channel's valid samples (an unchunked frame's: one word per lane)
    if (a.count && gid == 0 && wave == 0) {
        int n = __popc(mcache);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
        if (lane == 0) a.count[f] = a.overwrite ? n : a.count[f] + n;
    }

    // ---- epilogue, one tile at a time -----------------------------------
    // Halves geometry: waves 6 and 7 (odd steps) hand their sums to waves 4
    // and 5 (even steps, the same tiles and layout) through LDS, which is
    // free after the loop's last barrier; only waves 4 and 5 write.
    if (kSmall) {
        int32_t *cb = (int32_t *)lds + (wave & 1) * (8 * 16 * 64);
        auto each = [&](auto fn) {
            int m = 0;
#pragma unroll
            for (int k = 0; k < TL::NQ; ++k) fn(acc.q[k], m++);
#pragma unroll
            for (int k = 0; k < TL::NO; ++k) {
                fn(acc.re[k], m++);
                fn(acc.im[k], m++);
            }
        };
        if (kMma && wave >= 6)
            each([&](v16i &x, int m) {
#pragma unroll
                for (int v = 0; v < 16; ++v) cb[(m * 16 + v) * 64 + lane] = x[v];
            });
        __syncthreads();
        if (kMma && (wave == 4 || wave == 5))
            each([&](v16i &x, int m) {
#pragma unroll
                for (int v = 0; v < 16; ++v) x[v] += cb[(m * 16 + v) * 64 + lane];
            });
        __syncthreads();
        if (!(kMma && (wave == 4 || wave == 5))) return;
    }
    constexpr int NT = TL::NT;
    int32_t *tbuf = (int32_t *)lds + wave * (32 * 33);  // staging buffers are free now
    const TileMap<SHAPE> map{g, kSmall, s0, c0, a.N};
    auto tile = [&](int k, v16i &re, v16i &im) {
        if (k < TL::NQ) {
            split_q(acc.q[k < TL::NQ ? k : 0], tbuf, re, im);
        } else {
            re = acc.re[k - TL::NQ];
            im = acc.im[k - TL::NQ];
        }
    };
    const Dest d = make_dest(a, f, split, true);
    const int at = keep_late(lane);   // (addresses computed below, not before the loop)
#pragma unroll
    for (int k = 0; k < NT; ++k) {
        v2i x[16];
        // previous contents first, all loads before any store
        if (!kOverwrite && d.add) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                x[v] = __builtin_amdgcn_raw_buffer_load_b64(d.rsrc, (int)map.elem(k, v, at), 0, 0);
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) x[v] = (v2i){0, 0};
        }
        v16i re, im;
        tile(k, re, im);
#pragma unroll
        for (int v = 0; v < 16; ++v)
            __builtin_amdgcn_raw_buffer_store_b64(x[v] + (v2i){re[v], im[v]}, d.rsrc,
                                                  (int)map.elem(k, v, at), 0, 0);
    }
}

// One work item: tile group gid of channel f over time chunk `split`.
// Every wave runs the same number of steps and barriers; the tile pattern is
// fixed per group kind (blocks past N are staged as zeros).
template <bool kAligned, bool kOverwrite>
__device__ __forceinline__ void run_item(const CorrArgs &a, int f, int gid, int split,
                                         bool small, uint8_t *lds, uint32_t *mwords) {
    const Group g = make_group(a.nb, gid);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    with_role(g, small, wave, [&](auto role, int s0, int c0) {
        using R = decltype(role);
        run_wave<kAligned, kOverwrite, R::NSLOT, R::SHAPE, R::UPT, R::kMma, R::kSmall>(
            a, g, f, gid, split, s0, c0, lds, mwords);
    });
}

// One frame: workgroup -> (channel, group, chunk), groups of a channel
// and chunks of a (channel, group) numbered next to each other.
template <bool kAligned, bool kOverwrite>
__global__ __launch_bounds__(kThreads, 1) void corr_kernel(CorrArgs a, int small) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[3 * kBufBytes];
    __shared__ uint32_t mwords[kShortSteps];

    const int G = a.groups;
    const int64_t total = (int64_t)a.F * G * a.splits;
    int64_t w = xcd_local_index(blockIdx.x, total);
    const int gid = (int)(w % G);
    w /= G;
    const int split = (int)(w % a.splits);
    const int f = (int)(w / a.splits);
    run_item<kAligned, kOverwrite>(a, f, gid, split, small != 0, lds, mwords);
}

}  // namespace brief
}  // namespace xe
