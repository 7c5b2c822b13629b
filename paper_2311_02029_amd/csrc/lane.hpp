// Seeding with one lane per read: the device code shared by the fused
// classification and the containment search.
//
// A wavefront takes 64 reads.  Every lane turns its read into a 2-bit stream in
// LDS and then goes along it base by base: the k-mer is rolled, hashed and put
// into the window minimum, so no step needs another lane and every lane is busy
// whatever the number of k-mers, windows or minimizers of a read.  With a
// wavefront per read (the other kernel), 130 k-mers filled 3 rounds of 64, 120
// windows 2 and 21 minimizers a third of one, and each read paid the loop and
// list overhead of every step by itself.
//
// Window minima: a k-mer's key is the top KEY_BITS bits of its hash and, below
// them, its position, so the minimum of a window is one unsigned minimum per
// comparison and its position comes with it, leftmost first.  Keys decide like
// the full (hash, position) order unless two different positions of a
// comparison share the hash bits; each comparison checks that (x ^ y below
// 2^POS_BITS), and a read with such a tie goes to the wavefront-per-read kernel,
// which compares whole hashes (equal k-mers in a window are ties; else about
// one read in 25,000).  The minima of the W last keys take three comparisons a
// position: blocks of W positions, suffix minima of the block before, prefix
// minimum of the current one.  The block is unrolled, its keys in registers,
// so W is a template argument.
#pragma once

#include <type_traits>

#include "device.hpp"
#include "runtime.hpp"

namespace mt {

constexpr int LN_TPB = 256;                  // threads (reads) per block
constexpr int LN_MAX_M = 320;                // longest read a lane takes
constexpr int LN_SHORT_M = 192;              // ... of the instance for short reads, whose LDS holds more wavefronts
// Minimizer windows with an instance: those measured (1M reads of 150 bases, a
// wavefront each and lanes, the windows in lanes faster throughout: 4 1.67 and 1.27 ms,
// 13 1.76 and 0.64, 16 1.81 and 0.58, 20 1.87 and 0.54).
constexpr int LN_MIN_W = 4, LN_MAX_W = 20;
constexpr u32 POS_BITS = 9, POS_MASK = (1u << POS_BITS) - 1;
static_assert(LN_MAX_M < (int)POS_MASK, "a position fits the key, and none makes a key of all ones");

// A wavefront's reads: word-major, so the lanes' accesses to the same word fall
// into different banks.
// MAXM: longest read, a multiple of 32.
template <int MAXM>
struct LaneReads {
    u32 stream[MAXM / 16 + 2][64];  // base j at bits 30 - 2 (j mod 16) of word j / 16; two words of padding
    u32 picks[MAXM / 32][64];       // first 1 for an N or a position past the end; then 1 for a minimizer
};

struct LaneRead {
    int m;  // bases (0 for a lane without a read)
    bool bad, has_n;  // a byte is no base; a base is N
};

// Largest value of the wavefront, in a scalar register.
__device__ inline int wave_max(int v) {
#pragma unroll
    for (int o = 32; o; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
    return __builtin_amdgcn_readfirstlane(v);
}

// Decodes the lane's read (m bytes at seq + beg, m <= max_m <= MAXM) into L:
// 16 bases per load, the 2-bit word from four byte dot products.
template <int MAXM>
__device__ __attribute__((always_inline)) inline LaneRead lane_decode(const u8 *__restrict__ seq, u64 beg, int m,
                                                                      u64 total, int lane, int max_m,
                                                                      LaneReads<MAXM> &L) {
    LaneRead rd{m, false, false};
    for (int g = 0; 32 * g < max_m; g++) {
        u32 other = 0;  // bases of this group that are N or past the end
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int cnt = min(16, m - 32 * g - 16 * h);
            const u64 at = beg + 32 * (u64)g + 16 * h;
            u32 word = 0, not_base = 0xFFFFu;
            if (cnt > 0) {
                u32 v[4] = {0, 0, 0, 0}, x[4], d[4];
                if (at + 16 <= total) {
                    load16(seq + at, v);
                } else {
#pragma unroll
                    for (int i = 0; i < 16; i++)
                        if (i < cnt) v[i >> 2] |= (u32)seq[at + i] << (8 * (i & 3));
                }
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    base_codes4(v[j], &x[j], &d[j]);
                    word = (word << 8) | __builtin_amdgcn_udot4(x[j] & 0x03030303u, 0x01041040u, 0u, false);
                }
                not_base = 0xFFFFu & ~((1u << cnt) - 1u);
                if (d[0] | d[1] | d[2] | d[3]) {
                    const u32 nz = nonzero_bytes16(d) & ~not_base;
                    if (nz) {
                        rd.has_n = true;
                        rd.bad |= (nz & ~n_bytes16(v)) != 0;
                        not_base |= nz;
                    }
                }
            }
            L.stream[2 * g + h][lane] = word;
            other |= not_base << (16 * h);
        }
        L.picks[g][lane] = other;
    }
    return rd;
}

// k-mer value at position i of the lane's stream.
template <int MAXM>
__device__ inline u64 lane_kmer(const LaneReads<MAXM> &L, int lane, int i, u32 k) {
    const int w = i >> 4;
    const u32 s = 2u * (u32)(i & 15);
    const u64 hi = ((u64)L.stream[w][lane] << 32) | L.stream[w + 1][lane];
    const u64 y = (hi << s) | (((u64)L.stream[w + 2][lane] << s) >> 32);
    return y >> (64 - 2 * k);
}

// The top 32 bits of mix64(x), but for its last step, which changes only lower
// bits than those a key keeps: (z ^ z >> 31) leaves the top 31 bits of z.
__device__ inline u32 hash_top(u64 z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return (u32)(z >> 32);
}

// The minimum of two keys of different positions; *tie gets below 2^POS_BITS
// when their hash bits are equal.  (x ^ y) - 1 is all ones for two keys of all
// ones (no k-mer), which is no tie.
__device__ inline u32 key_min(u32 x, u32 y, u32 *tie) {
    *tie = min(*tie, (x ^ y) - 1u);
    return min(x, y);
}

// Marks the minimizers of the lane's read in L.picks and returns whether its
// keys decided them (false: a tie).  kMask: some lane's read has an N or another
// length than the rest, so positions are checked one by one.
template <int W, bool kMask, int MAXM>
__device__ __attribute__((always_inline)) inline bool lane_minimizers(LaneReads<MAXM> &L, int lane, int m, int max_m,
                                                                      u32 k) {
    const int nk = m - (int)k + 1, max_nk = max_m - (int)k + 1;
    u32 *picks = &L.picks[0][lane];
    // the k - 1 bases before the first k-mer ends
    const u64 y = ((u64)L.stream[0][lane] << 32) | L.stream[1][lane];
    u64 x = k > 1 ? y >> (64 - 2 * (k - 1)) : 0ull;
    const u64 xmask = (1ull << (2 * k)) - 1;
    u32 run = 0;     // valid bases up to here (kMask)
    u32 nword = 0;   // N and end bits of 32 positions (kMask)
    if constexpr (kMask) {
        const u32 n0 = picks[0] & ((1u << (k - 1)) - 1u);
        run = n0 ? k - 2 - (31 - (u32)__builtin_clz(n0)) : k - 1;
        nword = picks[0];
    }
    picks[0] = 0;
    u32 cur = L.stream[(k - 1) >> 4][lane];
    u32 key[W], tie = ~0u;
#pragma unroll
    for (int t = 0; t < W; t++) key[t] = ~0u;  // the block before the first: no minimum
    for (int i0 = 0; i0 < max_nk; i0 += W) {
        u32 prefix = ~0u;
#pragma unroll
        for (int b = 0; b < W; b++) {
            const int i = i0 + b;
            if (i < max_nk) {
                const int j = i + (int)k - 1;  // the base entering the k-mer
                if ((j & 15) == 0) cur = L.stream[j >> 4][lane];
                if ((j & 31) == 0 && j) {  // the mask's word is read before its bits become picks
                    if constexpr (kMask) nword = picks[(j >> 5) * 64];
                    picks[(j >> 5) * 64] = 0;
                }
                x = ((x << 2) | ((cur >> (30 - 2 * (j & 15))) & 3u)) & xmask;
                u32 kv = (hash_top(x) & ~POS_MASK) | (u32)i;
                if constexpr (kMask) {
                    run = (nword >> (j & 31)) & 1u ? 0u : run + 1;
                    kv = run >= k ? kv : ~0u;
                }
                prefix = b ? key_min(prefix, kv, &tie) : kv;
                const u32 best = b + 1 < W ? key_min(prefix, key[b + 1], &tie) : prefix;
                key[b] = kv;
                // windows of W k-mers end from position W - 1 on; a read with
                // fewer k-mers has one window, ending with the last
                bool emit = best != ~0u;
                if constexpr (kMask) emit = emit && i < nk && (i >= W - 1 || i == nk - 1);
                else emit = emit && (i >= W - 1 || i == max_nk - 1);
                if (emit) {
                    const u32 p = best & POS_MASK;
                    atomicOr(&picks[(p >> 5) * 64], 1u << (p & 31));
                }
            }
        }
        if (i0 + W < max_nk) {
#pragma unroll
            for (int t = W - 2; t >= 0; t--) key[t] = key_min(key[t], key[t + 1], &tie);
        }
    }
    return tie >= POS_MASK;
}

// Goes through the marked positions of the lane's read in order.
template <int MAXM>
struct PickIter {
    int word, words;  // words: those that hold positions of the wavefront's reads
    u32 bits;
    __device__ PickIter(const LaneReads<MAXM> &L, int lane, int max_nk)
        : word(0), words(max_nk > 0 ? (max_nk + 31) / 32 : 0), bits(max_nk > 0 ? L.picks[0][lane] : 0u) {}
    // the next position, or -1 when there is none left
    __device__ int next(const LaneReads<MAXM> &L, int lane) {
        while (bits == 0) {
            if (++word >= words) return -1;
            bits = L.picks[word][lane];
        }
        const int p = 32 * word + (int)__builtin_ctz(bits);
        bits &= bits - 1;
        return p;
    }
};

// Calls f with the minimizer window's instance as an integral constant.
template <class F>
inline void with_window(u32 w, F &&f) {
    switch (w) {
#define MT_W(W)                              \
    case W:                                  \
        f(std::integral_constant<int, W>{}); \
        return;
        MT_W(4) MT_W(5) MT_W(6) MT_W(7) MT_W(8) MT_W(9) MT_W(10) MT_W(11) MT_W(12) MT_W(13) MT_W(14) MT_W(15)
        MT_W(16) MT_W(17) MT_W(18) MT_W(19) MT_W(20)
#undef MT_W
    default:
        throw Error(MT_EINTERNAL, "no lane kernel for this minimizer window");
    }
}

}  // namespace mt
