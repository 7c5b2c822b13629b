// Packing sequences into bit planes and tiled minimizer extraction
// (seeding, Fig. 1 steps 2a and 2b).
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <mutex>

#include "seq.hpp"

namespace mt {

// Small results (counts, flags, a call's summary) are written by a kernel into
// pinned memory and read after the wait: a copy to pageable
// memory goes through the runtime's staging and is waited for there as well (16 reads
// classified and taken to the host 131 us, 116 us so; 1M explicit pairs, with three
// such waits, 243 and 208 us).  Bound by latency.
// The library has one block of WORD_SLOTS places, for as many calls waiting at once;
// the next one copies.  (A place per host thread cost a program that starts a thread
// for each call an allocation each: 0.21 ms a call of 16 reads, 0.15 so; and its release
// at the thread's end waits for the whole device.)
constexpr u32 READ_WORDS = 256, WORD_SLOTS = 64;

static struct {
    std::mutex mu;
    u32 *p = nullptr;
    u64 used = 0;  // bit i: place i
} g_words;

// A free place, or null when there is none.
static u32 *take_words() {
    std::lock_guard<std::mutex> g(g_words.mu);
    if (!g_words.p && hipHostMalloc((void **)&g_words.p, WORD_SLOTS * READ_WORDS * sizeof(u32),
                                    hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        g_words.p = nullptr;
    }
    if (!g_words.p || g_words.used == ~0ull) return nullptr;
    const int i = __builtin_ctzll(~g_words.used);
    g_words.used |= 1ull << i;
    return g_words.p + i * READ_WORDS;
}

static void give_words(u32 *w) {
    std::lock_guard<std::mutex> g(g_words.mu);
    g_words.used &= ~(1ull << ((w - g_words.p) / READ_WORDS));
}

void trim_host_words() {
    std::lock_guard<std::mutex> g(g_words.mu);
    if (!g_words.p || g_words.used) return;
    (void)hipHostFree(g_words.p);
    g_words.p = nullptr;
}

__global__ void k_read_back(const u32 *__restrict__ dev, u32 n, u32 *__restrict__ host) {
    if (threadIdx.x < n) __hip_atomic_store(&host[threadIdx.x], dev[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

void read_back(hipStream_t s, const void *dev, void *host, size_t bytes) {
    static_assert(WORD_SLOTS == 64, "a bit of a word each");
    const bool small = bytes && bytes <= READ_WORDS * sizeof(u32) && bytes % sizeof(u32) == 0 &&
                       (uintptr_t)dev % sizeof(u32) == 0;
    u32 *words = small ? take_words() : nullptr;
    if (!words) {
        MT_HIP(hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, s));
        MT_HIP(hipStreamSynchronize(s));
        return;
    }
    // (a place whose kernel is not known to have ended is not given back)
    k_read_back<<<1, READ_WORDS, 0, s>>>((const u32 *)dev, (u32)(bytes / sizeof(u32)), words);
    MT_HIP(hipGetLastError());
    MT_HIP(hipStreamSynchronize(s));
    std::memcpy(host, words, bytes);
    give_words(words);
}

// ------------------------------------------------------------------ packing --

// Blocks per sequence: ceil(len / 64) + 1 (the last one is padding).  Also
// checks the offsets: 0 first, never decreasing, `total` last; and leaves the longest
// length above NOTED_LEN in flags[1], an atomic a block (an atomic a wavefront on that
// one word took 35 us for 300k reads; one a block, for short reads too, 5).
constexpr int SB_TPB = 1024, SB_BLOCKS = 512;

__global__ __launch_bounds__(SB_TPB) void k_seq_blocks(const u64 *__restrict__ off, u64 n, u64 total, u64 len_limit,
                                                       u32 len_flag, u64 *__restrict__ nblk, u32 *__restrict__ flags) {
    __shared__ u32 longest;
    if (threadIdx.x == 0) longest = 0;
    __syncthreads();
    u32 mine = 0;
    for (u64 s = (u64)blockIdx.x * SB_TPB + threadIdx.x; s < n; s += (u64)gridDim.x * SB_TPB) {
        const u64 a = off[s], b = off[s + 1];
        u32 f = 0;
        if (b < a || b > total || (s == 0 && a != 0) || (s == n - 1 && b != total)) f |= ERR_OFFSETS;
        u64 len = b >= a ? b - a : 0;
        if (len > len_limit) f |= len_flag;
        if (f) {
            atomicOr(flags, f);
            len = 0;
        }
        mine = max(mine, (u32)len);  // (lengths that pass stay below 2^32)
        nblk[s] = (len + 63) / 64 + 1;
    }
#pragma unroll
    for (int o = 32; o; o >>= 1) mine = max(mine, (u32)__shfl_xor((int)mine, o, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(&longest, mine);
    __syncthreads();
    if (threadIdx.x == 0 && longest > NOTED_LEN) atomicMax(flags + 1, longest);
}

// Four lanes per 64-base block, 16 bytes each in one load (a byte at a time
// where 16 would pass the end of the set), turned into plane bits four bases at
// a time; the quad's first lane joins the four 16-bit pieces and stores the
// block.  Bound by the bytes in and out once the per-base work is gone: 500k
// reads of 150 bases 171 -> 44 us, 500 Mbp of genomes 637 -> 205 us against one
// thread per block going base by base.
__global__ __launch_bounds__(256) void k_pack(const u8 *__restrict__ seq, const u64 *__restrict__ off,
                                              const u64 *__restrict__ src, const u64 *__restrict__ blk_off, u64 n,
                                              u64 total, u64 cap,
                                              const u32 *__restrict__ map, u64x2 *__restrict__ lohi,
                                              u64 *__restrict__ nbp, u32 *__restrict__ flags,
                                              u8 *__restrict__ has_n) {
    const u64 t = wide_block() * 256 + threadIdx.x;
    const u64 b = t >> 2;
    const u32 quarter = (u32)t & 3u;
    if (b >= blk_off[n] || b >= cap) return;  // whole quads leave
    const u32 s = map[b];
    const u64 first = src ? src[s] : off[s];
    const u64 beg = first + 64 * (b - blk_off[s]) + 16 * quarter, end = first + (off[s + 1] - off[s]);
    u32 lo = 0, hi = 0, nb = 0xFFFFu;
    if (beg < end) {
        const u32 cnt = end - beg < 16 ? (u32)(end - beg) : 16u;
        const u32 valid = (1u << cnt) - 1u;
        u32 v[4] = {0, 0, 0, 0};
        if (beg + 16 <= total) {
            load16(seq + beg, v);
        } else {
#pragma unroll
            for (u32 i = 0; i < 16; i++)
                if (i < cnt) v[i >> 2] |= (u32)seq[beg + i] << (8 * (i & 3));
        }
        u32 other;
        plane_bits16(v, &lo, &hi, &other);
        other &= valid;
        lo &= valid & ~other;
        hi &= valid & ~other;
        nb = (0xFFFFu & ~valid) | other;
        if (other) {
            if (other & ~n_bytes16(v)) atomicOr(flags, ERR_BAD_BYTE);
            if (has_n) has_n[s] = 1;
        }
    }
    // lane 0 of the quad: its piece and lane 1's, then lanes 2 and 3's
    const u32 lo2 = lo | (u32)__builtin_amdgcn_mov_dpp((int)lo, 0xF5, 0xF, 0xF, true) << 16;  // quad_perm 1,1,3,3
    const u32 hi2 = hi | (u32)__builtin_amdgcn_mov_dpp((int)hi, 0xF5, 0xF, 0xF, true) << 16;
    const u32 nb2 = nb | (u32)__builtin_amdgcn_mov_dpp((int)nb, 0xF5, 0xF, 0xF, true) << 16;
    const u32 lo3 = (u32)__builtin_amdgcn_mov_dpp((int)lo2, 0xAA, 0xF, 0xF, true);  // quad_perm 2,2,2,2
    const u32 hi3 = (u32)__builtin_amdgcn_mov_dpp((int)hi2, 0xAA, 0xF, 0xF, true);
    const u32 nb3 = (u32)__builtin_amdgcn_mov_dpp((int)nb2, 0xAA, 0xF, 0xF, true);
    if (quarter == 0) {
        lohi[b] = u64x2{((u64)lo3 << 32) | lo2, ((u64)hi3 << 32) | hi2};
        nbp[b] = ((u64)nb3 << 32) | nb2;
    }
}

void pack_sequences(const mt_seqs &in, u64 len_limit, u32 len_flag, const char *len_message, PackedSeqs &out,
                    u32 *d_flags, u8 *has_n, hipStream_t s, const u64 *src, u64 src_total) {
    out.n = in.n;
    out.max_len = src ? ~0u : 0u;
    out.blk_off.alloc(in.n + 1);
    out.blocks_cap = in.total / 64 + 2 * in.n + 1;
    out.lohi.alloc(out.blocks_cap);
    out.nb.alloc(out.blocks_cap);
    if (in.n == 0) {
        MT_HIP(hipMemsetAsync(out.blk_off.p, 0, sizeof(u64), s));
        return;
    }
    DBuf<u64> nblk(in.n);
    const unsigned sb = (unsigned)std::min<u64>(SB_BLOCKS, (in.n + SB_TPB - 1) / SB_TPB);
    k_seq_blocks<<<sb, SB_TPB, 0, s>>>(in.offsets, in.n, in.total, len_limit, len_flag, nblk.p, d_flags);
    MT_HIP(hipGetLastError());
    if (!src) {
        // The offsets decide every later address: refuse bad ones before any
        // kernel reads sequence bytes through them.
        u32 f[2] = {0, 0};
        read_back(s, d_flags, f, sizeof f);
        if (f[0] & len_flag) throw Error(MT_EINVAL, len_message);
        check_flags(f[0]);
        out.max_len = f[1];
    }
    scan_u64(nblk.p, out.blk_off.p, in.n, s);
    DBuf<u32> map(out.blocks_cap);
    segment_map(out.blk_off.p, in.n, map.p, out.blocks_cap, s);
    k_pack<<<wide_grid(out.blocks_cap, 64, 256), 256, 0, s>>>((const u8 *)in.seq, in.offsets, src, out.blk_off.p, in.n,
                                                              src ? src_total : in.total, out.blocks_cap, map.p,
                                                              out.lohi.p, out.nb.p, d_flags, has_n);
    MT_HIP(hipGetLastError());
}

// --------------------------------------------------------------- minimizers --

constexpr int MAX_HALO = 254;  // w - 1 for w <= 255

// Tiles per sequence: ceil(nk / tile) with nk = len - k + 1 k-mer starts.
__global__ void k_seq_tiles(const u64 *__restrict__ off, u64 n, u32 k, u64 tile, u64 *__restrict__ ntile) {
    u64 s = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    i64 len = (i64)(off[s + 1] - off[s]);
    i64 nk = len - (i64)k + 1;
    ntile[s] = nk > 0 ? ((u64)nk + tile - 1) / tile : 0;
}

// Leftmost smallest of the W hashes sh[i..i + W) (an invalid k-mer reads as
// ~0, which no valid k-mer hashes to: the hash is a bijection and the preimage
// of ~0 is above every 62-bit k-mer value); -1 when the window has no valid
// k-mer.  All W hashes are read before the compare chain.
template <int W>
__device__ inline int lds_window_argmin(const u64 *sh, int i) {
    u64 v[W];
#pragma unroll
    for (int t = 0; t < W; t++) v[t] = sh[i + t];
    u64 bh = ~0ull;
    int bt = -1;
#pragma unroll
    for (int t = 0; t < W; t++)
        if (v[t] < bh) {
            bh = v[t];
            bt = t;
        }
    return bt < 0 ? -1 : i + bt;
}

__device__ inline int lds_window_argmin_any(const u64 *sh, int i, int win) {
    switch (win) {
#define MT_WIN(W) \
    case W:       \
        return lds_window_argmin<W>(sh, i);
        MT_WIN(1) MT_WIN(2) MT_WIN(3) MT_WIN(4) MT_WIN(5) MT_WIN(6) MT_WIN(7) MT_WIN(8)
        MT_WIN(9) MT_WIN(10) MT_WIN(11) MT_WIN(12)
#undef MT_WIN
    default: {
        u64 bh = ~0ull;
        int best = -1;
        for (int t = 0; t < win; t++)
            if (sh[i + t] < bh) {
                bh = sh[i + t];
                best = i + t;
            }
        return best;
    }
    }
}

// MIN_RUN windows of W starts, the first at sh[i]: calls f(q, t) for each window q
// with a valid k-mer, t its leftmost smallest hash's place from i.  The W - 4
// hashes that all five windows have are compared once, with the suffix minima of
// the four before them and the prefix minima of the four after: W + 9 comparisons
// and W + 4 LDS reads for the five, 5 (W - 1) and 5 W one window at a time.
constexpr int MIN_RUN = 5;

struct MinHash {
    u64 h;
    int t;
    // the smaller of this and one to the right of it
    __device__ MinHash or_right(const MinHash &o) const {
        const bool r = o.h < h;
        return MinHash{r ? o.h : h, r ? o.t : t};
    }
};

template <int W, class F>
__device__ inline void lds_window_run(const u64 *sh, int i, F &&f) {
    static_assert(W >= MIN_RUN && MIN_RUN == 5, "the windows have a start in common");
    u64 v[W + 4];
#pragma unroll
    for (int t = 0; t < W + 4; t++) v[t] = sh[i + t];
    MinHash mid{v[4], 4};
#pragma unroll
    for (int t = 5; t < W; t++) mid = mid.or_right(MinHash{v[t], t});
    MinHash win[MIN_RUN];
    win[4] = mid;
    MinHash left{v[3], 3};
    win[3] = left.or_right(mid);
#pragma unroll
    for (int q = 2; q >= 0; q--) {
        left = MinHash{v[q], q}.or_right(left);
        win[q] = left.or_right(mid);
    }
    MinHash right{v[W], W};
    win[1] = win[1].or_right(right);
#pragma unroll
    for (int q = 2; q < MIN_RUN; q++) {
        right = right.or_right(MinHash{v[W + q - 1], W + q - 1});
        win[q] = win[q].or_right(right);
    }
#pragma unroll
    for (int q = 0; q < MIN_RUN; q++)
        if (win[q].h != ~0ull) f(q, win[q].t);
}

template <class F>
__device__ inline void lds_window_run_any(const u64 *sh, int i, int n, int win, F &&f) {
    switch (win) {
#define MT_W(W)                      \
    case W:                          \
        lds_window_run<W>(sh, i, f); \
        break;
        MT_W(5) MT_W(6) MT_W(7) MT_W(8) MT_W(9) MT_W(10) MT_W(11) MT_W(12) MT_W(13) MT_W(14) MT_W(15) MT_W(16)
        MT_W(17) MT_W(18) MT_W(19) MT_W(20)
#undef MT_W
    default:
        for (int q = 0; q < n; q++) {
            const int best = lds_window_argmin_any(sh, i + q, win);
            if (best >= 0) f(q, best - i);
        }
    }
}

// One block per tile of TILE consecutive k-mer starts of one sequence.  The
// hashes of the tile plus a halo of w - 1 starts on each side go to LDS; every
// window that overlaps the tile picks its smallest (hash, position) among the
// valid k-mers, and picks inside the tile are marked.  The marks leave as one
// 64-bit word per 64 starts (tile_bits, TILE / 64 words per tile) with their
// count in tile_count.
// Bound by VALU issue.  A thread takes MIN_RUN windows in a row (in LDS their
// first hashes are 10 banks apart, so that 32 lanes read 32 pairs of banks), and
// the tile with the halo of usual windows is just under TPB * MIN_RUN starts.
// 500 Mbp at k = 21, w = 11: 1.95 ms with a window per thread, tiles of 1,024 and a
// byte per start for the marks, 1.16 ms so.
template <int TPB, int TILE>
__global__ __launch_bounds__(TPB) void k_min_tiles(const u64x2 *__restrict__ lohi, const u64 *__restrict__ nbp,
                                                   const u64 *__restrict__ blk_off, const u64 *__restrict__ off,
                                                   const u64 *__restrict__ tile_off, const u32 *__restrict__ tile_map,
                                                   u64 n, u32 k, u32 w, u32 *__restrict__ tile_count,
                                                   u64 *__restrict__ tile_bits) {
    static_assert(TILE % 64 == 0 && TILE / 64 <= 64 && TPB % 64 == 0, "a lane of one wavefront for each word of marks");
    static_assert((TILE + 2 * MAX_HALO) / TPB + 1 + 31 <= 64, "a thread's starts and k-mers fit its 64-base window");
    constexpr int SPAN = TILE + 2 * MAX_HALO, WORDS = TILE / 64;
    __shared__ u64 sh_h[SPAN + MIN_RUN];  // the last thread's windows past the last one read on
    __shared__ u32 marks[2 * WORDS];
    const u64 t = wide_block();
    if (t >= tile_off[n]) return;
    const u32 s = tile_map[t];
    const i64 lt = (i64)(t - tile_off[s]);
    const i64 len = (i64)(off[s + 1] - off[s]);
    const i64 nk = len - (i64)k + 1;
    const i64 win = nk < (i64)w ? nk : (i64)w;
    const i64 t0 = lt * TILE, t1 = t0 + TILE < nk ? t0 + TILE : nk;
    const i64 h0 = t0 - win + 1 > 0 ? t0 - win + 1 : 0;
    const i64 h1 = t1 + win - 1 < nk ? t1 + win - 1 : nk;
    const u64x2 *ql = lohi + blk_off[s];
    const u64 *qn = nbp + blk_off[s];
    // Each thread hashes a run of consecutive starts: the first k-mer value
    // from its 64-base window, the next ones rolled in one base at a time.
    const u64 kmask = (1ull << k) - 1, xmask = (1ull << (2 * k)) - 1;
    const int span = (int)(h1 - h0);
    const int run = (span + TPB - 1) / TPB;  // at most (TILE + 2 * MAX_HALO) / TPB + 1 <= 64 - 31
    const int c0 = (int)threadIdx.x * run;
    if (c0 < span) {
        const Bits64 b = fetch_planes(ql, qn, h0 + c0);
        u64 x = kmer_value(b.lo, b.hi, k);
        const int cn = min(run, span - c0);
        for (int j = 0; j < cn; j++) {
            if (j > 0) {
                const u32 t = (u32)j + k - 1;  // the base entering the k-mer
                x = ((x << 2) | (((b.hi >> t) & 1ull) << 1) | ((b.lo >> t) & 1ull)) & xmask;
            }
            sh_h[c0 + j] = ((b.nb >> j) & kmask) == 0 ? mix64(x) : ~0ull;
        }
    }
    for (int i = threadIdx.x; i < 2 * WORDS; i += TPB) marks[i] = 0;
    __syncthreads();
    // windows from h0 to the last that starts in the tile and ends in the sequence
    const int nw = (int)((t1 - 1 < nk - win ? t1 - 1 : nk - win) - h0) + 1, lead = (int)(t0 - h0);
    for (int w0 = (int)threadIdx.x * MIN_RUN; w0 < nw; w0 += TPB * MIN_RUN) {
        const int cnt = min(MIN_RUN, nw - w0);
        int last = -1;  // a pick is marked once for the windows in a row that share it
        lds_window_run_any(sh_h, w0, cnt, (int)win, [&](int q, int b) {
            const int p = w0 + b - lead;
            if (q < cnt && b != last && p >= 0 && p < TILE) atomicOr(&marks[p >> 5], 1u << (p & 31));
            last = b;
        });
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const int i = (int)threadIdx.x;
        u64 m = 0;
        if (i < WORDS) {
            m = (u64)marks[2 * i] | (u64)marks[2 * i + 1] << 32;
            tile_bits[t * WORDS + i] = m;
        }
        u32 total = (u32)__popcll(m);
#pragma unroll
        for (int o = 32; o; o >>= 1) total += __shfl_xor(total, o, 64);
        if (i == 0) tile_count[t] = total;
    }
}

// One wavefront per tile: the marked starts are first listed in LDS, then
// their k-mer values computed 64 at a time (one lane per start) and written in
// start order at the tile's output offset with sequence and position (each
// of those two outputs may be null).
constexpr int EMIT_WPB = 4;

template <int TILE>
__global__ __launch_bounds__(64 * EMIT_WPB) void k_min_emit(const u64x2 *__restrict__ lohi,
                                                            const u64 *__restrict__ nbp,
                                                            const u64 *__restrict__ blk_off,
                                                            const u64 *__restrict__ tile_off,
                                                            const u32 *__restrict__ tile_map, u64 n, u32 k,
                                                            const u64 *__restrict__ tile_bits,
                                                            const u64 *__restrict__ min_off, u64 *__restrict__ out_x,
                                                            u32 *__restrict__ out_seq, u32 *__restrict__ out_pos) {
    static_assert(TILE <= 65536, "starts within a tile fit 16 bits");
    __shared__ u16 list_all[EMIT_WPB][TILE];
    const u32 lane = threadIdx.x & 63;
    const u32 wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u64 t = wide_block() * EMIT_WPB + wid;
    if (t >= tile_off[n]) return;
    u16 *list = list_all[wid];
    const u32 s = tile_map[t];
    const i64 t0 = (i64)(t - tile_off[s]) * TILE;
    const u64 below = lane ? (~0ull) >> (64 - lane) : 0ull;
    u32 nl = 0;
    static_assert(TILE / 64 <= 64, "a lane for each word of marks");
    const u64 mine = lane < TILE / 64 ? tile_bits[t * (TILE / 64) + lane] : 0;
#pragma unroll 1
    for (int q = 0; q < TILE / 64; q++) {
        const u64 m = ((u64)(u32)__builtin_amdgcn_readlane((int)(mine >> 32), q) << 32) |
                      (u32)__builtin_amdgcn_readlane((int)mine, q);
        if ((m >> lane) & 1) list[nl + (u32)__popcll(m & below)] = (u16)(64 * q + lane);
        nl += (u32)__popcll(m);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const u64x2 *ql = lohi + blk_off[s];
    const u64 *qn = nbp + blk_off[s];
    const u64 o = min_off[t];
#pragma unroll 1
    for (u32 b = 0; b < nl; b += 64) {
        if (b + lane < nl) {
            const i64 i = t0 + list[b + lane];
            const Bits64 bits = fetch_planes(ql, qn, i);
            out_x[o + b + lane] = kmer_value(bits.lo, bits.hi, k);
            if (out_seq) out_seq[o + b + lane] = s;
            if (out_pos) out_pos[o + b + lane] = (u32)i;
        }
    }
}

template <int TPB, int TILE>
static void launch_tiles(const mt_seqs &in, const PackedSeqs &ps, u32 k, u32 w, MinimizerPlan &mp, hipStream_t s) {
    k_min_tiles<TPB, TILE><<<wide_grid(mp.tiles_cap, 1, TPB), TPB, 0, s>>>(ps.lohi.p, ps.nb.p, ps.blk_off.p, in.offsets,
                                                                      mp.tile_off.p, mp.tile_map.p, in.n, k, w,
                                                                      mp.tile_count.p, mp.tile_bits.p);
    MT_HIP(hipGetLastError());
}

template <int TILE>
static void launch_emit(const mt_seqs &in, const PackedSeqs &ps, u32 k, MinimizerPlan &mp, u64 *out_x,
                        u32 *out_seq, u32 *out_pos, hipStream_t s) {
    k_min_emit<TILE><<<wide_grid(mp.tiles_cap, EMIT_WPB, 64 * EMIT_WPB), 64 * EMIT_WPB, 0, s>>>(
        ps.lohi.p, ps.nb.p, ps.blk_off.p, mp.tile_off.p, mp.tile_map.p, in.n, k, mp.tile_bits.p, mp.min_off.p, out_x,
        out_seq, out_pos);
    MT_HIP(hipGetLastError());
}

void minimizer_plan(const mt_seqs &in, const PackedSeqs &ps, u32 k, u32 w, int tile, MinimizerPlan &mp,
                    hipStream_t s) {
    mp.tile = tile;
    mp.tiles_cap = in.total / (u64)tile + in.n + 1;
    mp.tile_off.alloc(in.n + 1);
    mp.tile_map.alloc(mp.tiles_cap);
    mp.tile_count.alloc(mp.tiles_cap);
    mp.min_off.alloc(mp.tiles_cap + 1);
    mp.tile_bits.alloc(mp.tiles_cap * (u64)(tile / 64));
    if (tile != MIN_TILE_SHORT && tile != MIN_TILE) throw Error(MT_EINTERNAL, "unsupported minimizer tile");
    if (in.n == 0) {  // no tiles: every offset is 0 (callers read min_off[tiles_cap])
        MT_HIP(hipMemsetAsync(mp.tile_off.p, 0, sizeof(u64), s));
        MT_HIP(hipMemsetAsync(mp.min_off.p, 0, (mp.tiles_cap + 1) * sizeof(u64), s));
        return;
    }
    DBuf<u64> ntile(in.n);
    k_seq_tiles<<<grid_for(in.n, 256), 256, 0, s>>>(in.offsets, in.n, k, (u64)tile, ntile.p);
    MT_HIP(hipGetLastError());
    scan_u64(ntile.p, mp.tile_off.p, in.n, s);
    segment_map(mp.tile_off.p, in.n, mp.tile_map.p, mp.tiles_cap, s);
    MT_HIP(hipMemsetAsync(mp.tile_count.p, 0, mp.tiles_cap * sizeof(u32), s));
    if (tile == MIN_TILE)
        launch_tiles<256, MIN_TILE>(in, ps, k, w, mp, s);
    else
        launch_tiles<64, MIN_TILE_SHORT>(in, ps, k, w, mp, s);
    // min_off over the full tile bound: tiles past the real count hold 0.
    scan_u32(mp.tile_count.p, mp.min_off.p, mp.tiles_cap, s);
}

void minimizer_emit(const mt_seqs &in, const PackedSeqs &ps, u32 k, u32 w, MinimizerPlan &mp, u64 *out_x,
                    u32 *out_seq, u32 *out_pos, hipStream_t s) {
    (void)w;
    if (in.n == 0) return;
    if (mp.tile == MIN_TILE)
        launch_emit<MIN_TILE>(in, ps, k, mp, out_x, out_seq, out_pos, s);
    else
        launch_emit<MIN_TILE_SHORT>(in, ps, k, mp, out_x, out_seq, out_pos, s);
}

}  // namespace mt
