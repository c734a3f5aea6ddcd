// flag_kernels.hpp -- gfx950 kernels for per-input flags (Sec. II-C).
//
// The F-engine flags single data points (range or sampling faults).  Flagged
// points are zeroed before correlation, so baseline (i, j) of channel f
// integrates
//     n_ij = count_f - c_i - c_j + d_ij
// samples: count_f valid samples of the channel, c_i of them with input i
// flagged, d_ij with both flagged (d_ii = c_i).  The method keeps c and d on
// the host, listing the flagged inputs of every sample, O(E^2) per sample.
// Here d, diagonal included, is one 0/1 Gram matrix per channel,
//     D = A A^T over valid samples,  A[i][t] = flag bit of input i at t,
// on the matrix cores: exact, and its cost does not grow with the number of
// points a sample flags.
//
// Flags arrive as bit-fields flags[f][t][w], W = ceil(N/32) words, bit i % 32
// of word i / 32 = input i.  A workgroup of eight waves takes one channel,
// 8 or 10 tiles of 32 x 32 counts (a unit: the triangle of a 128-input group,
// or half a group's rows against another group) and one chunk of time; its
// waves take the chunk's K-steps of 64 samples in turn and never wait for
// each other:
//   1. a wave loads the unit's 4 or 6 words of a sample per lane (0 for lost
//      samples, samples past the chunk and inputs past N), a batch of
//      four K-steps ahead; a K-step without a flag on both sides of its tiles
//      ends there, the counterpart of the method's test of whole 32-bit words
//      before extracting bits;
//   2. a word with a flag becomes a matrix operand: its 64 lanes' 32 x 32 bits
//      (two halves) are transposed across the lanes in five exchange steps,
//      after which lane l holds 32 samples of input l % 32 in one dword, and
//      seven vector instructions expand that into 4-bit codes (code 2 is 1.0);
//   3. v_mfma_f32_32x32x64_f8f6f4 counts 64 samples of every tile whose two
//      words both hold a flag.  The counts stay in registers: float32 is
//      exact up to 2^24, a chunk has at most 32,768 samples;
//   4. at the chunk's end the waves' counts are added in LDS (16 bits each,
//      four per word), and the nonzero ones into d with integer atomics: other
//      chunks, and calls on other streams, may add to the same counts, and the
//      order does not matter.
// What bounds it: 256 inputs, 64 channels and 16,384 samples (33.6 MB) with
// bursts over 0.1% of the points take 14.7 us and 8.7 without a flag, the time
// of a launch; without the LDS additions they take 12.4, without the flagged
// K-steps, a serial chain of transposes and tests, 9.0.  Scattered flags (5%)
// cost the vector instructions of the transposes: 512 inputs, 32 channels, 8,192
// samples take 53 us, where adding the counts of every 32-sample step into LDS
// on their own took 449 us, the LDS atomics' rate.  The units are this small,
// although their words are loaded and transposed 2.5 times, because a channel's
// counts then come from one chunk: with 36 tiles to a workgroup and four chunks
// to a channel the global atomics took 34 of 59 us (256 dense inputs).  Many
// inputs: see flag_wide_kernels.hpp and use_wide_flags() in plan.hpp.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace xe {
namespace flag {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kWindow = 1024;       // validity words per chunk: chunks <= 32768 samples
constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kBatch = 4;           // K-steps a wave loads at once

struct Args {
    const uint32_t *flags;   // [F][T][W]
    const uint8_t *mask;     // [F][nblk], may be null
    int32_t *d;              // [F][P]
    int N, F, T, B, W, nblk;
    int groups;              // 128-input groups, ceil(N / 128)
    int ns;                  // super blocks, ceil(N / 256)
    int chunks;              // time chunks per (channel, unit or pair)
    int chunk_samples;       // samples per chunk, a multiple of 32, <= 32 kWindow
    uint64_t b_magic;        // ceil(2^40 / B) when B <= 2^16, else 0
};

// t / B for 0 <= t < 2^24: (t * ceil(2^40 / B)) >> 40 is exact when B <= 2^16
// (the rounding adds less than 2^-16 to t / B, whose fraction is at most
// 1 - 1/B); larger B divides.
__device__ __forceinline__ int block_of(const Args &a, int t) {
    return a.b_magic ? (int)(((uint64_t)(uint32_t)t * a.b_magic) >> 40) : t / a.B;
}

// Counts of the chunk in LDS as four 16-bit fields per 64-bit word (no field
// carries into the next): tile k, column j, rows 4 Q .. 4 Q + 3 at
// acc[k * kTile + j * kPitch + Q], row 4 Q in the low field.  The odd pitch
// spreads lanes along j over the banks.
constexpr int kPitch = 9, kTile = 32 * kPitch, kMaxTiles = 10;
struct Lds {
    uint64_t acc[kMaxTiles * kTile];
    uint32_t valid[kWindow];        // bit k of word s: sample 32 s + k of the chunk
};

__device__ __forceinline__ uint32_t uniform(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
    return __builtin_amdgcn_perm(hi, lo, sel);
}

__device__ __forceinline__ int64_t tri(int64_t N, int64_t i, int64_t j) {
    return i * N - i * (i - 1) / 2 + (j - i);
}

// A 32 x 32 bit transpose in each half-wave (lane = sample, bit = input before,
// lane = input, bit = sample after) exchanges every bit of the lane number
// with one of the bit number, five steps of 14 vector instructions in all.  A
// step pairs lanes that cross-lane moves reach without the LDS: l and l ^ 16,
// 8, 7, 2, 1.  With 7 in place of 4 the lane's number in the steps is
// l ^ 3 where bit 2 is set: lane l ends up with input shuffled(l).
__device__ __forceinline__ int shuffled(int l) { return l ^ ((l & 4) != 0 ? 3 : 0); }

struct Transpose {
    uint32_t sel16, sel8, by4, keep4, by2, keep2, by1, keep1;

    __device__ __forceinline__ explicit Transpose(int lane) {
        const int n = shuffled(lane);
        sel16 = n & 16 ? 0x03020706u : 0x01000504u;
        sel8 = n & 8 ? 0x07030501u : 0x02060004u;
        by4 = n & 4 ? 4 : 28;
        keep4 = n & 4 ? 0xf0f0f0f0u : 0x0f0f0f0fu;
        by2 = n & 2 ? 2 : 30;
        keep2 = n & 2 ? 0xccccccccu : 0x33333333u;
        by1 = n & 1 ? 1 : 31;
        keep1 = n & 1 ? 0xaaaaaaaau : 0x55555555u;
    }
    // the other lane's bits into the places that `keep` leaves
    template <int DPP>
    __device__ __forceinline__ static uint32_t step(uint32_t x, uint32_t by, uint32_t keep) {
        const uint32_t y = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, DPP, 0xf, 0xf, true);
        return (x & keep) | (__builtin_amdgcn_alignbit(y, y, by) & ~keep);
    }
    __device__ __forceinline__ uint32_t operator()(uint32_t x) const {
        // the even rows of 16 lanes twice, and the odd ones
        const auto s = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        x = perm(s[0], s[1], sel16);
        const uint32_t y = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x128, 0xf, 0xf, true);   // + 8
        x = perm(x, y, sel8);
        x = step<0x141>(x, by4, keep4);         // half rows mirrored: l ^ 7
        x = step<0x4e>(x, by2, keep2);          // quads 2 3 0 1
        return step<0xb1>(x, by1, keep1);       // 1 0 3 2
    }
};

// 32 flag bits as 4-bit codes: 2 (1.0) for a flag.  The samples' order inside
// K is the same for every operand.
__device__ __forceinline__ v4i expand(uint32_t x) {
    return (v4i){(int)((x << 1) & 0x22222222u), (int)(x & 0x22222222u),
                 (int)((x >> 1) & 0x22222222u), (int)((x >> 2) & 0x22222222u)};
}
__device__ __forceinline__ v16f mfma(v4i a, v4i b, v16f c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
        __builtin_shufflevector(a, a, 0, 1, 2, 3, -1, -1, -1, -1),
        __builtin_shufflevector(b, b, 0, 1, 2, 3, -1, -1, -1, -1), c, 4, 4, 0, 0, 0, 0);
}

// Tile k of a unit pairs its words row(k) and col(k).  A triangle's words are
// the four blocks of its group; a rectangle's two blocks of rows, then four
// of columns.
template <bool kTri>
struct Unit {
    static constexpr int kWords = kTri ? 4 : 6, kTiles = kTri ? 10 : 8;
    __device__ static constexpr int row(int k) {
        return !kTri ? k >> 2 : k < 4 ? 0 : k < 7 ? 1 : k < 9 ? 2 : 3;
    }
    __device__ static constexpr int col(int k) {
        return !kTri ? 2 + (k & 3) : k < 4 ? k : k < 7 ? k - 3 : k < 9 ? k - 5 : 3;
    }
};

// Validity of the chunk's samples, one bit each, in LDS: 1 inside the chunk
// and outside lost blocks.  All threads take part; a barrier must follow.
template <int kThreads>
__device__ __forceinline__ void fill_window(const Args &a, uint32_t *valid, int f, int t_begin,
                                            int t_end, int tid) {
    const int words = (t_end - t_begin + 31) >> 5;
    for (int s = tid; s < words; s += kThreads) {
        const int t = t_begin + 32 * s;
        const int n = min(32, t_end - t);
        uint32_t bits = n == 32 ? 0xffffffffu : (1u << n) - 1u;
        if (a.mask) {
            // the blocks touching the word's samples, eight loads at a time,
            // all issued before the first is used (indices clamped)
            const uint8_t *row = a.mask + (int64_t)f * a.nblk;
            const int first = block_of(a, t), last = block_of(a, t + n - 1);
            for (int b0 = first; b0 <= last; b0 += 8) {
                uint32_t v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = row[min(b0 + q, last)];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int b = b0 + q;
                    if (b > last || v[q] == 0u) continue;
                    const int lo = max(t, b * a.B) - t;
                    const int hi = min(t + n, (b + 1) * a.B) - t;    // exclusive
                    const uint64_t span = ((1ull << hi) - 1ull) & ~((1ull << lo) - 1ull);
                    bits &= ~(uint32_t)span;
                }
            }
        }
        valid[s] = bits;
    }
}

// Workgroup b runs on XCD b % 8; consecutive work items (the chunks of one
// channel and pair) are numbered onto one XCD so they share its L2.
__device__ __forceinline__ int64_t xcd_local(int64_t b, int64_t total) {
    const int64_t per = total / 8, rem = total % 8;
    const int64_t x = b % 8, idx = b / 8;
    return x * per + (x < rem ? x : rem) + idx;
}

template <bool kTri>
struct Wave {
    using U = Unit<kTri>;
    Lds &L;
    Transpose transpose;
    __amdgpu_buffer_rsrc_t rsrc;
    int lane, wave, samples;
    uint32_t row_bytes, at, at_rows;   // byte offsets of the lane's words in K-step `wave`
    v4i pad;                           // the bits of inputs < N of the column words
    v4i raw[kBatch];                   // column words of the next batch
    v2i raw_rows[kBatch];              // row words (rectangle)
    v4i now[kBatch];                   // of this one, masked
    uint32_t row0[kBatch], row1[kBatch];
    v4i op[U::kWords];
    v16f acc[U::kTiles];
    uint32_t counted;                  // tiles with a count

    // sample of K-step q of batch b, lane 0 (ascending; a batch is one K-step
    // of every wave, kBatch times)
    __device__ __forceinline__ int sample(int b, int q) const {
        return 64 * (wave + kWaves * (kBatch * b + q));
    }
    template <int Q>
    __device__ __forceinline__ void load(int b) {
        if constexpr (Q < kBatch) {
            const uint32_t o = (uint32_t)(64 * kWaves * (kBatch * b + Q)) * row_bytes;
            raw[Q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(at + o), 0, 0);
            if constexpr (!kTri)
                raw_rows[Q] = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(at_rows + o), 0, 0);
            load<Q + 1>(b);
        }
    }
    // masks K-step Q's words; bit Q of the result: its tiles have a flag to count
    template <int Q>
    __device__ __forceinline__ uint32_t look(int b) {
        if constexpr (Q < kBatch) {
            const int t = sample(b, Q) + lane;
            // (past the chunk the words are 0)
            const uint32_t valid = L.valid[(t >> 5) & (kWindow - 1)];
            const int keep = -(int)((valid >> (t & 31)) & 1u);
            const v4i w = raw[Q] & pad & (v4i){keep, keep, keep, keep};
            now[Q] = w;
            bool some = __ballot((w.x | w.y | w.z | w.w) != 0) != 0;
            if constexpr (!kTri) {
                const v2i y = raw_rows[Q];
                row0[Q] = (uint32_t)(y.x & keep);
                row1[Q] = (uint32_t)(y.y & keep);
                some = some && __ballot((row0[Q] | row1[Q]) != 0u) != 0;
            }
            return (some ? 1u << Q : 0u) | look<Q + 1>(b);
        } else {
            return 0u;
        }
    }
    template <int Q>
    __device__ __forceinline__ void take(uint32_t (&w)[U::kWords], int q) const {
        if constexpr (Q < kBatch) {
            if (q == Q) {
                // (The asm differs between branches: else the compiler merges
                // their loads into one from a chosen address, and everything
                // stays in memory.)
                v4i c = now[Q];
                asm volatile("; step %1" : "+v"(c) : "i"(Q));
                if constexpr (!kTri) {
                    uint32_t x = row0[Q], y = row1[Q];
                    asm volatile("; step %2" : "+v"(x), "+v"(y) : "i"(Q));
                    w[0] = x;
                    w[1] = y;
                }
                w[U::kWords - 4] = (uint32_t)c.x;
                w[U::kWords - 3] = (uint32_t)c.y;
                w[U::kWords - 2] = (uint32_t)c.z;
                w[U::kWords - 1] = (uint32_t)c.w;
            } else {
                take<Q + 1>(w, q);
            }
        }
    }
    template <int I>
    __device__ __forceinline__ uint32_t operands(const uint32_t (&w)[U::kWords]) {
        if constexpr (I < U::kWords) {
            uint32_t flagged = 0;
            if (__ballot(w[I] != 0u) != 0) {
                op[I] = expand(transpose(w[I]));
                flagged = 1u << I;
            }
            return flagged | operands<I + 1>(w);
        } else {
            return 0u;
        }
    }
    template <int K>
    __device__ __forceinline__ void count(uint32_t flagged) {
        if constexpr (K < U::kTiles) {
            constexpr uint32_t both = 1u << U::row(K) | 1u << U::col(K);
            if ((flagged & both) == both) {
                acc[K] = mfma(op[U::row(K)], op[U::col(K)], acc[K]);
                counted |= 1u << K;
            }
            count<K + 1>(flagged);
        }
    }
    // batch b: its words have been requested; those of the next one are
    __device__ __forceinline__ void batch(int b) {
        uint32_t todo = uniform(look<0>(b));
        load<0>(b + 1);
#pragma clang loop unroll(disable)
        while (todo != 0) {
            const int q = __builtin_ctz(todo);
            todo &= todo - 1;
            uint32_t w[U::kWords];
            take<0>(w, q);
            count<0>(uniform(operands<0>(w)));
        }
    }
    // Adds the wave's counts into LDS: element v of a tile is at row
    // 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32, both of shuffled inputs.
    template <int K>
    __device__ __forceinline__ void add_tiles() {
        if constexpr (K < U::kTiles) {
            if ((counted >> K) & 1u) {
                uint64_t *t = L.acc + K * kTile + shuffled(lane & 31) * kPitch + (lane >> 5);
                const bool odd = lane >= 32;   // rows 4 .. 7 of 8: in reverse
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const uint32_t x0 = (uint32_t)acc[K][4 * g], x1 = (uint32_t)acc[K][4 * g + 1];
                    const uint32_t x2 = (uint32_t)acc[K][4 * g + 2], x3 = (uint32_t)acc[K][4 * g + 3];
                    const uint32_t lo = odd ? x3 | x2 << 16 : x0 | x1 << 16;
                    const uint32_t hi = odd ? x1 | x0 << 16 : x2 | x3 << 16;
                    atomicAdd((unsigned long long *)(t + 2 * g),
                              (unsigned long long)(lo | ((uint64_t)hi << 32)));
                }
            }
            add_tiles<K + 1>();
        }
    }
};

// A unit: first word of its rows and of its columns (a triangle: the same).
template <bool kTri>
__device__ __forceinline__ void run_unit(const Args &a, Lds &L, int f, int row_word, int col_word,
                                         int t_begin, int t_end) {
    using U = Unit<kTri>;
    const int tid = threadIdx.x;
    Wave<kTri> w = {L, Transpose(tid & 63)};
    w.lane = tid & 63;
    w.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    w.samples = t_end - t_begin;
    w.counted = 0;
    // the chunk's rows of this channel's flags through a buffer resource
    // whose range ends at the chunk's last sample: dwords past it read 0
    // without a memory access
    w.row_bytes = 4u * (uint32_t)a.W;
    const uint64_t base = (uint64_t)(uintptr_t)(a.flags + ((int64_t)f * a.T + t_begin) * a.W);
    const uint64_t p = ((uint64_t)uniform((uint32_t)(base >> 32)) << 32) | uniform((uint32_t)base);
    w.rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(uintptr_t)p, (short)0,
                                               (int)uniform((uint32_t)w.samples * w.row_bytes),
                                               0x00020000);
    // The four column words' 16 bytes may reach into the next row, whose bits
    // `pad` masks; the loads need no alignment.
    auto pad = [&](int r) {
        const int left = a.N - (col_word + r) * 32;
        return left >= 32 ? -1 : left > 0 ? (int)((1u << left) - 1u) : 0;
    };
    w.pad = (v4i){pad(0), pad(1), pad(2), pad(3)};
    w.at = (uint32_t)(64 * w.wave + w.lane) * w.row_bytes + 4u * (uint32_t)col_word;
    w.at_rows = (uint32_t)(64 * w.wave + w.lane) * w.row_bytes + 4u * (uint32_t)row_word;
    w.template load<0>(0);
    for (int e = tid; e < U::kTiles * kTile; e += kThreads) L.acc[e] = 0;
    fill_window<kThreads>(a, L.valid, f, t_begin, t_end, tid);
#pragma unroll
    for (int k = 0; k < U::kTiles; ++k) w.acc[k] = (v16f){0};
#pragma unroll
    for (int k = 0; k < U::kWords; ++k) w.op[k] = (v4i){0, 0, 0, 0};
    __syncthreads();   // counts cleared, validity window visible
#pragma clang loop unroll(disable)
    for (int b = 0; w.sample(b, 0) < w.samples; ++b) w.batch(b);
    w.counted = uniform(w.counted);
    w.template add_tiles<0>();
    __syncthreads();   // every wave's counts added

    // the nonzero counts into d
    int32_t *dst = a.d + (int64_t)f * a.N * (a.N + 1) / 2;
#pragma clang loop unroll(disable)
    for (int e = tid; e < U::kTiles * 256; e += kThreads) {
        const int k = e >> 8, Q = (e >> 5) & 7, j = e & 31;
        const uint64_t word = L.acc[k * kTile + j * kPitch + Q];
        if (word == 0u) continue;
        const int gi = (row_word + U::row(k)) * 32 + 4 * Q;
        const int gj = (col_word + U::col(k) - (kTri ? 0 : 2)) * 32 + j;
        if (gj >= a.N) continue;
        int32_t *x = dst + tri(a.N, gi, gj);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int cnt = (int)((word >> (16 * r)) & 0xffffu);
            if (cnt != 0 && gi + r <= gj) atomicAdd(x, cnt);
            x += a.N - 1 - gi - r;
        }
    }
}

// Units of a channel: the triangles of its groups, then for every pair of
// groups g < h the two halves of g's rows against h, row by row.
__global__ __launch_bounds__(kThreads, 2) void gram_kernel(Args a) {
    __shared__ __attribute__((aligned(16))) Lds L;
    const int units = a.groups * a.groups;
    const int64_t w = xcd_local(blockIdx.x, (int64_t)a.F * units * a.chunks);
    const int u = (int)(w % units);
    const int64_t rest = w / units;
    const int chunk = (int)(rest % a.chunks);
    const int f = (int)(rest / a.chunks);
    const int t_begin = chunk * a.chunk_samples;
    const int t_end = min(a.T, t_begin + a.chunk_samples);
    if (u < a.groups) {
        run_unit<true>(a, L, f, 4 * u, 4 * u, t_begin, t_end);
    } else {
        int rem = (u - a.groups) >> 1, g = 0;
        while (rem >= a.groups - 1 - g) {
            rem -= a.groups - 1 - g;
            ++g;
        }
        run_unit<false>(a, L, f, 4 * g + 2 * ((u - a.groups) & 1), 4 * (g + 1 + rem), t_begin,
                        t_end);
    }
}

// Zero flagged points in place: byte 0x88 is 0 + 0i.  One thread per flag
// word; a word without flags touches nothing else.  When N % 32 == 0 the 32
// bytes of a word are rewritten with two 16-byte accesses.
template <bool kVec>
__global__ void apply_kernel(uint8_t *packed, const uint32_t *flags, int N, int F, int T, int W) {
    const int64_t total = (int64_t)F * T * W;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += stride) {
        uint32_t word = flags[e];
        const int w = (int)(e % W);
        const int64_t ft = e / W;
        const int t = (int)(ft % T), f = (int)(ft / T);
        const int rest = N - w * 32;
        if (rest < 32) word &= (1u << rest) - 1u;
        if (word == 0u) continue;
        uint8_t *row = packed + ((int64_t)t * F + f) * N + w * 32;
        if (kVec) {
            uint4 *p = (uint4 *)row;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                uint4 v = p[half];
                uint32_t *d = (uint32_t *)&v;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t b4 = (word >> (16 * half + 4 * q)) & 15u;
                    uint32_t m = (b4 * 0x00204081u) & 0x01010101u;  // bit k -> byte k
                    m = (m << 8) - m;                                // -> 0xff bytes
                    d[q] = (d[q] & ~m) | (0x88888888u & m);
                }
                p[half] = v;
            }
        } else {
            for (int b = 0; b < 32; ++b)
                if ((word >> b) & 1u) row[b] = 0x88;
        }
    }
}

// out[f][p] = vis / n_ij, n_ij = count_f - d_ii - d_jj + d_ij, in double
// rounded once to float, 0 where n_ij == 0; n_out (optional) = n_ij.  A
// workgroup takes rows i and N - 1 - i, N + 1 baselines, together; the
// workgroups of a channel share its row pairs, with the channel's d_ii in LDS:
// they lie a row apart in d.  Found from the baseline's number by a square
// root, with d_jj fetched for every baseline, the rows took 394 us at 2048
// inputs x 16 channels, 32 at 512 x 32 and 17.0 at 256 x 64, with n_out, and
// take 251, 24 and 15.0 (344 and 16.4 without n_out: 187 and 13.8).
//
// The quotients of a pair share one reciprocal: r = 1 / n and q = v r, both
// rounded, and q + r (v - n q) with fused products is off by less than 2^-104
// of v / n before its own rounding, while a quotient of integers below 2^31
// and 2^50 that is no double lies at least 2^-103 of itself from any tie of two
// doubles: the same doubles as division gives.
constexpr int kNormThreads = 256;

__device__ __forceinline__ float quotient(int v, double n, double r) {
    const double x = (double)v, q = x * r;
    return (float)__builtin_fma(__builtin_fma(-q, n, x), r, q);
}

__global__ __launch_bounds__(kNormThreads) void normalize_kernel(const int32_t *vis,
                                                                 const int64_t *count,
                                                                 const int32_t *d, float *out,
                                                                 int32_t *n_out, int N,
                                                                 int per_channel) {
    extern __shared__ int32_t diag[];   // [N]
    const int f = (int)(blockIdx.x / per_channel), b = (int)(blockIdx.x % per_channel);
    const int64_t P = (int64_t)N * (N + 1) / 2;
    const int32_t *df = d + f * P;
    for (int i = threadIdx.x; i < N; i += kNormThreads) diag[i] = df[tri(N, i, i)];
    __syncthreads();
    const int64_t total = count[f];
    const int2 *v = (const int2 *)vis + f * P;
    float2 *o = (float2 *)out + f * P;
    for (int i = b; 2 * i < N; i += per_channel) {
        const int i2 = N - 1 - i, first = N - i;
        const int len = i2 == i ? first : N + 1;
        const int64_t s1 = tri(N, i, i), s2 = tri(N, i2, i2) - first;
#pragma unroll 4
        for (int k = threadIdx.x; k < len; k += kNormThreads) {
            const bool one = k < first;
            const int row = one ? i : i2, j = one ? i + k : i2 + k - first;
            const int64_t p = (one ? s1 : s2) + k;
            const int64_t n =
                total - (int64_t)diag[row] - (int64_t)diag[j] + (int64_t)df[p];
            const int2 x = v[p];
            const double dn = (double)n, r = 1.0 / dn;
            float2 y;
            y.x = n == 0 ? 0.0f : quotient(x.x, dn, r);
            y.y = n == 0 ? 0.0f : quotient(x.y, dn, r);
            o[p] = y;
            if (n_out) n_out[f * P + p] = (int32_t)n;
        }
    }
}

// The same for N <= kFewInputs, whose row pairs would leave half of a
// workgroup's threads idle: one thread per baseline of all channels, (i, j)
// from p by inverting the row starts s(i) = i N - i (i - 1) / 2.  64 inputs x
// 1000 channels take 16 us so and 20 by row pairs, 100 x 500 18 and 19, 129 x
// 1000 56 and 60, 140 x 1000 68 and 68, 132 x 2000 172 and 143, 180 x 300 34 and
// 31.
constexpr int kFewInputs = 128;

__global__ void normalize_few_kernel(const int32_t *vis, const int64_t *count, const int32_t *d,
                                 float *out, int32_t *n_out, int N, int F) {
    const int64_t P = (int64_t)N * (N + 1) / 2;
    const int64_t total = P * F;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += stride) {
        const int64_t f = e / P, p = e % P;
        const double b = 2.0 * N + 1.0;
        int64_t i = (int64_t)((b - sqrt(b * b - 8.0 * (double)p)) * 0.5);
        if (i < 0) i = 0;
        if (i > N - 1) i = N - 1;
        while (i > 0 && tri(N, i, i) > p) --i;
        while (i + 1 < N && tri(N, i + 1, i + 1) <= p) ++i;
        const int64_t j = i + (p - tri(N, i, i));
        const int32_t *df = d + f * P;
        const int64_t n = count[f] - (int64_t)df[tri(N, i, i)] - (int64_t)df[tri(N, j, j)] +
                          (int64_t)df[p];
        const int2 v = *(const int2 *)(vis + 2 * e);
        float2 o;
        const double dn = (double)n, r = 1.0 / dn;
        o.x = n == 0 ? 0.0f : quotient(v.x, dn, r);
        o.y = n == 0 ? 0.0f : quotient(v.y, dn, r);
        *(float2 *)(out + 2 * e) = o;
        if (n_out) n_out[e] = (int32_t)n;
    }
}

}  // namespace flag
}  // namespace xe
