// The obstacle-count filter over explicit pair lists (Fig. 1 step 2d), used by
// the per-stage form, by the fused form's fallback and by mt_filter_pairs.
//
// Pairs are bucketed by their threshold E, and long pairs by the LDS they
// need, so that each bucket gets the kernel shaped for it (uneven batching):
//   E <= 31  one lane per pair, the rows as the bits of one or two words; groups of G
//            lanes per pair, one band row per lane, for longer reads (see far_len; G = 16
//            for E <= 7, 32 for E <= 15, else 64), or for all (G = 32 or 64 for
//            E <= 7, 64 for E <= 15)
//   E > 31   long reads, four bins by the 64-base blocks of read plus
//            reference window they stage in LDS (<= 96, 192, 384, 768): 1, 2, 4
//            or 8 pairs per wavefront, the rows as the bits of words dealt to the
//            pair's lanes;
//            or the rows-in-lanes kernel reading the window from global memory
//   larger   the rows-in-lanes kernel.
// The variant of each bucket (lane or G, pairs per wavefront, layout) is chosen by the autotuner
// (mt_autotune) or set by mt_tune_set; every variant gives the same result.
#include <algorithm>
#include <mutex>
#include <string>

#include "classify.hpp"

namespace mt {

constexpr int N_BUCKETS = 8;  // E<=7, E<=15, E<=31, four long bins, general
constexpr int CLS_LONG = 3, LONG_BINS = 4, CLS_GENERAL = 7;
// Classes are the buckets, and the long bins twice more: for the pairs with an N
// in read or window, or a window past a genome end, which stage and compare a
// third plane (CLS_LONG_N), and for bands too wide to stage in segments
// (CLS_LONG_WIDE); and the short ones once more, for reads past far_len (CLS_FAR).
constexpr int CLS_LONG_N = N_BUCKETS, CLS_LONG_WIDE = CLS_LONG_N + LONG_BINS, CLS_FAR = CLS_LONG_WIDE + LONG_BINS;
constexpr int N_CLASSES = CLS_FAR + CLS_LONG;
__host__ __device__ inline int class_bucket(int c) {
    return c < N_BUCKETS ? c : c >= CLS_FAR ? c - CLS_FAR : CLS_LONG + (c - N_BUCKETS) % LONG_BINS;
}
constexpr int LONG_CAP[LONG_BINS] = {96, 192, 384, 768};  // 64-base blocks staged per wavefront
constexpr int LDS_BLOCK_BYTES = 24;                        // {lo, hi} + nb of one 64-base block
constexpr int LONG_LDS_MAX = 64 * 1024;                    // per workgroup
// A pair of the long kernel holds LONG_TILE blocks in LDS, or LONG_TILE_N with the N
// planes (the same bytes), a segment of its columns at a time; bands up to
// LONG_MAX_E, or LONG_MAX_E_N, leave at least 1,000 columns for a segment.
constexpr int LONG_TILE = 81, LONG_TILE_N = 54, LONG_MAX_E = 1440, LONG_MAX_E_N = 600;

__device__ inline void pair_fields(const FilterArgs &a, u64 p, u32 &r, u32 &g, int &E, bool &ok, u32 &err) {
    r = a.pair_read[p];
    g = a.pair_genome[p];
    ok = true;
    err = 0;
    if (r >= a.n_reads || g >= a.n_genomes) {
        ok = false;
        err = ERR_PAIR_RANGE;
        E = 0;
        return;
    }
    E = a.pair_E ? a.pair_E[p] : a.read_E[r];
    if (E > 65534) {
        ok = false;
        err = ERR_E_TOO_LARGE;
    }
}

__device__ inline i64 pair_diag(const FilterArgs &a, u64 p) { return near_diag(a.pair_diag[p]); }

__device__ inline int read_len(const FilterArgs &a, u32 r) { return (int)(a.read_off[r + 1] - a.read_off[r]); }

// Blocks the long kernel stages for a pair: the read's (with its padding
// block) and the reference window from diag - E, long enough for a 128-base
// fetch at any column < m of any row.
__device__ inline void long_blocks(int m, int E, int &nrb, int &nwb) {
    nrb = (m + 63) / 64 + 1;
    nwb = ((m + 2 * E + 190) >> 6) + 2;
}

// Whether any compared column of a pair can meet an N or a position outside the
// genome.
__device__ inline bool pair_with_n(const FilterArgs &a, u32 r, const GenomeMeta &gm, i64 diag, int m, int E) {
    return meta_has_n(gm) || !window_inside(diag, m, E, (i64)gm.len) || a.read_has_n[r];
}

__device__ inline u8 pair_class(const FilterArgs &a, u64 p) {
    u32 r, g, err;
    int E;
    bool ok;
    pair_fields(a, p, r, g, E, ok, err);
    if (!ok) return CLS_GENERAL;  // the general kernel reports the error
    if (E <= 31) {
        const int b = E <= 7 ? 0 : E <= 15 ? 1 : 2;
        return (u8)(a.max_len > (u32)a.far_len && read_len(a, r) > a.far_len ? CLS_FAR + b : b);
    }
    int nrb, nwb;
    const int m = read_len(a, r);
    long_blocks(m, E, nrb, nwb);
    for (int b = 0; b < LONG_BINS; b++)
        if (nrb + nwb <= LONG_CAP[b])
        {
            const bool with_n = pair_with_n(a, r, a.meta[g], pair_diag(a, p), m, E);
            return (u8)((E > (with_n ? LONG_MAX_E_N : LONG_MAX_E) ? CLS_LONG_WIDE : with_n ? CLS_LONG_N : CLS_LONG) + b);
        }
    return CLS_GENERAL;
}

// Bucketing without shared counters: block b of both passes takes the same
// contiguous range of pairs; the first pass leaves the block's count of every
// class, k_pair_offsets turns the counts (class-major) into places, and the
// second pass fills them.  With global cursors, one atomic per wavefront and
// class on a handful of words, each pass took 180 us for 1M pairs, waiting on
// those words; now each takes 8 us (2M pairs of mixed classes).
constexpr int CL_TPB = 256, CL_MAX_BLOCKS = 512;

struct PairRange {
    u64 lo, hi;
};
__device__ inline PairRange block_range(u64 n) {
    const u64 per = ((n + gridDim.x - 1) / gridDim.x + CL_TPB - 1) / CL_TPB * CL_TPB;
    const u64 lo = min((u64)blockIdx.x * per, n);
    return PairRange{lo, min(lo + per, n)};
}

// Pairs to filter: the device count when there is one (bounded by the
// launch's capacity), else the host count.
__device__ inline u64 pair_count(const FilterArgs &a, u64 n_cap) {
    const u64 n = a.n_dev ? *a.n_dev : a.n_host;
    return n < n_cap ? n : n_cap;
}

__global__ __launch_bounds__(CL_TPB) void k_pair_class(FilterArgs a, u64 n_cap, u32 *__restrict__ blk_count,
                                                       u8 *__restrict__ cls) {
    __shared__ u32 cnt[N_CLASSES];
    if (threadIdx.x < N_CLASSES) cnt[threadIdx.x] = 0;
    __syncthreads();
    const PairRange range = block_range(pair_count(a, n_cap));
    const int lane = threadIdx.x & 63;
    u32 mine = 0;  // lane k of a wavefront counts class k
    for (u64 p0 = range.lo; p0 < range.hi; p0 += CL_TPB) {
        const u64 p = p0 + threadIdx.x;
        u8 c = 0xFF;
        if (p < range.hi) {
            c = pair_class(a, p);
            cls[p] = c;
        }
#pragma unroll
        for (int k = 0; k < N_CLASSES; k++) {
            const u64 m = __ballot(c == k);
            if (lane == k) mine += (u32)__popcll(m);
        }
    }
    if (lane < N_CLASSES && mine) atomicAdd(&cnt[lane], mine);
    __syncthreads();
    if (threadIdx.x < N_CLASSES) blk_count[(u64)threadIdx.x * gridDim.x + blockIdx.x] = cnt[threadIdx.x];
}

// One block: exclusive offsets of the N_CLASSES * nb counts in class-major
// order, and every class's total.
constexpr int OFF_TPB = 1024, OFF_ITEMS = (N_CLASSES * CL_MAX_BLOCKS + OFF_TPB - 1) / OFF_TPB;
__global__ __launch_bounds__(OFF_TPB) void k_pair_offsets(u32 *__restrict__ blk_count, u32 nb,
                                                          u32 *__restrict__ total) {
    __shared__ u32 begin[N_CLASSES + 1];
    const u32 n = N_CLASSES * nb, i0 = threadIdx.x * OFF_ITEMS;
    u32 v[OFF_ITEMS], t = 0;
#pragma unroll
    for (int i = 0; i < OFF_ITEMS; i++) {
        v[i] = i0 + i < n ? blk_count[i0 + i] : 0;
        t += v[i];
    }
    u32 all;
    u32 run = block_exclusive_sum<OFF_TPB, u32>(t, &all);
#pragma unroll
    for (int i = 0; i < OFF_ITEMS; i++) {
        if (i0 + i < n) {
            blk_count[i0 + i] = run;
            if ((i0 + i) % nb == 0) begin[(i0 + i) / nb] = run;
        }
        run += v[i];
    }
    if (threadIdx.x == 0) begin[N_CLASSES] = all;
    __syncthreads();
    if (threadIdx.x < N_CLASSES) total[threadIdx.x] = begin[threadIdx.x + 1] - begin[threadIdx.x];
}

__global__ __launch_bounds__(CL_TPB) void k_pair_scatter(FilterArgs a, u64 n_cap, const u8 *__restrict__ cls,
                                                         const u32 *__restrict__ blk_off, u32 *__restrict__ idx) {
    __shared__ u32 cursor[N_CLASSES];
    if (threadIdx.x < N_CLASSES) cursor[threadIdx.x] = blk_off[(u64)threadIdx.x * gridDim.x + blockIdx.x];
    __syncthreads();
    const PairRange range = block_range(pair_count(a, n_cap));
    const int lane = threadIdx.x & 63;
    for (u64 p0 = range.lo; p0 < range.hi; p0 += CL_TPB) {
        const u64 p = p0 + threadIdx.x;
        const u8 c = p < range.hi ? cls[p] : (u8)0xFF;
#pragma unroll
        for (int k = 0; k < N_CLASSES; k++) {
            const u64 m = __ballot(c == k);
            if (!m) continue;
            const int leader = __builtin_ctzll(m);
            u32 first = 0;
            if (lane == leader) first = atomicAdd(&cursor[k], (u32)__builtin_popcountll(m));
            first = __shfl(first, leader, 64);
            if (c == k) idx[first + __builtin_popcountll(m & ((1ull << lane) - 1))] = (u32)p;
        }
    }
}

// The obstacle walk of one pair by a group of G lanes with one band row per
// lane (2E + 1 <= G) for a read of at most 64 NW bases: lane l builds row
// d = l - E in NW registers (rows past 2E + 1 read as all obstacles and never
// lead), then every step is a run length per lane from its registers and a
// maximum over the group.  Returns min(count, E + 1).
template <int G, int NW>
__device__ inline int walk_in_registers(const PairView &v, int E, int lane) {
    const int nwr = (v.m + 63) / 64 + 1;  // the read's blocks, its padding block included
    u64 row[NW];
    if (lane < 2 * E + 1) {
        auto qword = [&](int w) {
            Bits64 q;
            if (w < nwr) {
                const u64x2 x = v.qlohi[w];
                q.lo = x.lo;
                q.hi = x.hi;
                q.nb = v.qnb[w];
            } else {
                q.lo = q.hi = 0;
                q.nb = ~0ull;
            }
            return q;
        };
        band_row<NW>(qword, v.rlohi, v.rnb, v.L, v.has_n, v.diag + (lane - E), row);
    } else {
#pragma unroll
        for (int w = 0; w < NW; w++) row[w] = ~0ull;
    }
    int j = 0, c = 0;
    for (;;) {
        j += group_max<G>(reg_run<NW>(row, j));
        if (j >= v.m) break;
        c += 1;
        if (c > E) break;
        j += 1;
    }
    return c < E + 1 ? c : E + 1;
}

// G lanes per pair over the bucket idx[0, n), or over pairs [0, n) when idx is
// null (n then also bounded by the pairs there are).
template <int G>
__global__ __launch_bounds__(256) void k_filter(FilterArgs a, const u32 *__restrict__ idx, u64 n) {
    u64 tid = wide_block() * blockDim.x + threadIdx.x;
    u64 t = tid / G;
    int lane = (int)(tid % G);
    if (t >= (idx ? n : pair_count(a, n))) return;
    u64 p = idx ? idx[t] : t;
    u32 r, g, err;
    int E;
    bool ok;
    pair_fields(a, p, r, g, E, ok, err);
    if (!ok) {
        if (lane == 0) {
            atomicOr(a.flags, err);
            a.approx[p] = 0xFFFF;
            a.accept[p] = 0;
        }
        return;
    }
    PairView v;
    v.qlohi = a.read_lohi + a.read_blk[r];
    v.qnb = a.read_nb + a.read_blk[r];
    v.m = read_len(a, r);
    GenomeMeta gm = a.meta[g];
    v.rlohi = a.ref_lohi + gm.blk;
    v.rnb = a.ref_nb + gm.blk;
    v.L = (i64)gm.len;
    v.has_n = meta_has_n(gm);
    v.diag = pair_diag(a, p);
    const int rows = 2 * E + 1;
    int approx;
    // One band row per lane and reads of up to 256 bases (the E <= 7 / 15 / 31
    // buckets but their reads of 257+ bases): the row's mismatch words are
    // built once, from one fetch of each reference block it spans, and the
    // walk runs on registers.  The branch is uniform over the group.  (A
    // five-word path for reads up to 320 bases took the kernel from 69 to 81
    // registers and 7 to 5 wavefronts per SIMD.)
    if (rows <= G && v.m <= 256)
        approx = walk_in_registers<G, 4>(v, E, lane);
    else
        approx = obstacle_walk<G>(v, E, lane);
    if (lane == 0) {
        a.approx[p] = (u16)approx;
        a.accept[p] = approx <= E;
    }
}

__device__ inline void lds_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Longest read of a short E whose pair takes one lane, of n pairs.  A lane's time goes
// with the read and hardly with the number of pairs (1 kbp at E = 7, 2,000 pairs to
// 120,000: 0.14 to 0.19 ms the whole call), that of groups with the number of pairs and
// hardly with the read (0.09 to 0.18 ms), so they meet at a ratio, about 90 pairs a base
// for E = 7 and 50 for E = 31.  Lanes and groups at E = 7 (E = 31): 300 bases, 2,000
// pairs 0.10 and 0.09 ms (0.13, 0.10), 400,000 0.17 and 0.36 (0.26, 1.44); 1 kbp, 2,000
// 0.19 and 0.10 (0.29, 0.10), 120,000 0.24 and 0.25 (0.36, 0.62); 2 kbp, 60,000 0.41 and
// 0.21 (0.73, 0.45); 10 kbp, 12,000 3.3 and 0.16.  Reads up to 256 bases keep to lanes;
// past 1 kbp too few pairs fit a wavefront's LDS at once.
constexpr int FAR_LEAST = 256, FAR_MOST = 1024;
static_assert(FAR_LEAST >= (int)NOTED_LEN, "the longest length is known from there on");
constexpr u64 FAR_PAIRS = 64;  // pairs a base
static int far_len(u64 n) {
    return (int)std::min<u64>(std::max<u64>(n / FAR_PAIRS, FAR_LEAST), FAR_MOST);
}

// One lane per pair, E <= 31.  The walk is a serial chain of a few steps, each
// over the 2E+1 rows; here a lane takes a pair's whole step with the rows as
// the bits of R 32-bit words.  Column t of all rows at once: the window's planes
// from column j, shifted by t, against the read's base t (a mask of ones or
// zeros per plane), two three-input bit operations a word.  A row stays alive
// while its columns match, so after NC columns (few rows match that far by
// chance: rows / 4^NC) either no row is alive and the longest run is the number
// of columns that left one, or the few survivors' runs are measured 64 columns
// at a time.  Bound by VALU issue: rows in lanes (k_filter) spends a group of
// 16 to 64 lanes on a step of the same length.
// 1M pairs of 150 bases at E = 7, half of them wrong places: 298 us with 16
// lanes a pair, 58 us here.
//
// The pair's read and window planes are staged in LDS: every step reads them at
// places of its own per lane, which the vector cache serves one line at a time.
// A wavefront's 64 pairs share LANE_DW dwords (a pair of 150 bases takes 24 to
// 28, with the N planes 42); longer pairs go in several batches.  The whole read is
// staged, by its lane, however soon the walk ends, so longer reads (past far_len) are
// left to the groups of lanes, which read what a step touches.
constexpr int LANE_TPB = 256, LANE_DW = 2552, LANE_PAD = 8;  // 40 KB a block: four blocks a CU

// A pair's planes in LDS as dwords of 32 bases: the read's from its first base, the
// window's from its first staged block.
struct LdsPair {
    const u32 *ql, *qh, *qn, *wl, *wh, *wn;
    __device__ LdsPair(const u32 *Q, int nbr, const u32 *W, int nbw)
        : ql(Q), qh(Q + 2 * nbr), qn(Q + 4 * nbr), wl(W), wh(W + 2 * nbw), wn(W + 4 * nbw) {}
};

// 32 bits of a plane from bit p.
__device__ inline u32 plane_at(const u32 *d, int p) {
    return __builtin_amdgcn_alignbit(d[(p >> 5) + 1], d[p >> 5], (u32)p & 31u);
}

// Run of the row whose column j lies at window position pw, known to match for
// `run` columns, 64 columns at a time (past the read's end it counts whatever
// lies there: the caller cuts it).
template <bool kN>
__device__ inline int long_run(const LdsPair &P, int j, int pw, int m, int run) {
    while (j + run < m) {
        const int cq = j + run, cw = pw + run;
        const int k = cq >> 5, kk = cw >> 5;
        const u32 s = (u32)cq & 31u, ss = (u32)cw & 31u;
        const u32 q1 = P.ql[k + 1], h1 = P.qh[k + 1], w1 = P.wl[kk + 1], v1 = P.wh[kk + 1];
        u32 m0 = (__builtin_amdgcn_alignbit(q1, P.ql[k], s) ^ __builtin_amdgcn_alignbit(w1, P.wl[kk], ss)) |
                 (__builtin_amdgcn_alignbit(h1, P.qh[k], s) ^ __builtin_amdgcn_alignbit(v1, P.wh[kk], ss));
        u32 m1 = (__builtin_amdgcn_alignbit(P.ql[k + 2], q1, s) ^ __builtin_amdgcn_alignbit(P.wl[kk + 2], w1, ss)) |
                 (__builtin_amdgcn_alignbit(P.qh[k + 2], h1, s) ^ __builtin_amdgcn_alignbit(P.wh[kk + 2], v1, ss));
        if constexpr (kN) {
            m0 |= plane_at(P.qn, cq) | plane_at(P.wn, cw);
            m1 |= plane_at(P.qn, cq + 32) | plane_at(P.wn, cw + 32);
        }
        if (m0 | m1) return run + (m0 ? (int)__builtin_ctz(m0) : 32 + (int)__builtin_ctz(m1));
        run += 64;
    }
    return run;
}

// One step from column j for the 32 W rows whose first lies at window position pw
// (rows: those of them that exist): the longest run, found column by column with
// the rows as bits.
template <int W, int NC, bool kN>
__device__ inline int rows_step(const LdsPair &P, u32 ql, u32 qh, u32 qn, int j, int pw, int m, int rows) {
    const int kw = pw >> 5;
    const u32 sw = (u32)pw & 31u;
    u32 xl[W + 1], xh[W + 1], xn[W + 1], alive[W], any = 0;
#pragma unroll
    for (int i = 0; i <= W; i++) {
        xl[i] = __builtin_amdgcn_alignbit(P.wl[kw + i + 1], P.wl[kw + i], sw);
        xh[i] = __builtin_amdgcn_alignbit(P.wh[kw + i + 1], P.wh[kw + i], sw);
        xn[i] = kN ? __builtin_amdgcn_alignbit(P.wn[kw + i + 1], P.wn[kw + i], sw) : 0u;
    }
    int best = 0;
#pragma unroll
    for (int i = 0; i < W; i++)
        alive[i] = rows >= 32 * (i + 1) ? ~0u : rows > 32 * i ? (1u << (rows - 32 * i)) - 1u : 0u;
#pragma unroll
    for (int t = 0; t < NC; t++) {
        const u32 a = (u32)((int)(ql << (31 - t)) >> 31), b = (u32)((int)(qh << (31 - t)) >> 31);
        const u32 n = kN ? (u32)((int)(qn << (31 - t)) >> 31) : 0u;
        any = 0;
#pragma unroll
        for (int i = 0; i < W; i++) {
            // truth table 0x90 takes (x, y, z) to x & ~(y ^ z)
            const u32 wl = t ? __builtin_amdgcn_alignbit(xl[i + 1], xl[i], t) : xl[i];
            const u32 wh = t ? __builtin_amdgcn_alignbit(xh[i + 1], xh[i], t) : xh[i];
            u32 v = __builtin_amdgcn_bitop3_b32(alive[i], wl, a, 0x90);
            v = __builtin_amdgcn_bitop3_b32(v, wh, b, 0x90);
            if constexpr (kN) v &= ~((t ? __builtin_amdgcn_alignbit(xn[i + 1], xn[i], t) : xn[i]) | n);
            alive[i] = v;
            any |= v;
        }
        best += any != 0;
    }
    if (any) {
        static_assert(W <= 4, "the survivors of up to 128 rows");
        u64 al = alive[0], more = 0;
        if (W > 1) al |= (u64)alive[W > 1 ? 1 : 0] << 32;
        if (W > 2) more = alive[W > 2 ? 2 : 0] | (W > 3 ? (u64)alive[W > 3 ? 3 : 0] << 32 : 0ull);
        int base = 0;
        while (al | more) {
            if (W > 2 && al == 0) {
                al = more;
                more = 0;
                base = 64;
            }
            const int row = base + (int)__builtin_ctzll(al);
            al &= al - 1;
            best = max(best, long_run<kN>(P, j, pw + row, m, NC));
        }
    }
    return best;
}

template <int R, int NC, bool kN>
__device__ inline int lane_walk(const LdsPair &P, int wofs, int m, int E) {
    int j = 0, c = 0;
    for (;;) {
        const u32 qn = kN ? plane_at(P.qn, j) : 0u;
        const int best = rows_step<R, NC, kN>(P, plane_at(P.ql, j), plane_at(P.qh, j), qn, j, wofs + j, m, 2 * E + 1);
        j += min(best, m - j);  // columns past the read's end count for nothing
        if (j >= m) break;
        c += 1;
        if (c > E) break;
        j += 1;
    }
    return c;
}

// Planes of 64 bases of ASCII (nb of a byte past the wanted ones is whatever lies
// there).
__device__ inline Bits64 ascii_planes(const u32 (&v)[4][4]) {
    u32 lo[4], hi[4], nb[4];
#pragma unroll
    for (int i = 0; i < 4; i++) plane_bits16(v[i], &lo[i], &hi[i], &nb[i]);
    return Bits64{lo[0] | lo[1] << 16 | (u64)(lo[2] | lo[3] << 16) << 32,
                  hi[0] | hi[1] << 16 | (u64)(hi[2] | hi[3] << 16) << 32,
                  nb[0] | nb[1] << 16 | (u64)(nb[2] | nb[3] << 16) << 32};
}

// The planes of cnt bases from byte at, 16 bytes to a load as long as they lie in
// the set.
__device__ inline Bits64 ascii_block(const FilterArgs &a, u64 at, int cnt) {
    u32 v[4][4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int c = min(16, cnt - 16 * i);
        v[i][0] = v[i][1] = v[i][2] = v[i][3] = 0;
        if (c <= 0) continue;
        if (at + 16 * i + 16 <= a.seq_total) {
            load16(a.seq + at + 16 * i, v[i]);
        } else {
#pragma unroll
            for (int t = 0; t < 16; t++)
                if (t < c) v[i][t >> 2] |= (u32)a.seq[at + 16 * i + t] << (8 * (t & 3));
        }
    }
    return ascii_planes(v);
}

// Block b of a read, from block rb of the planes or byte rb of the ASCII.
template <bool kAscii>
__device__ inline Bits64 read_block(const FilterArgs &a, u64 rb, int b, int m) {
    if constexpr (kAscii) {
        return ascii_block(a, rb + 64 * (u64)b, m - 64 * b);
    } else {
        const u64x2 x = a.read_lohi[rb + b];
        return Bits64{x.lo, x.hi, a.read_nb[rb + b]};
    }
}

// Stages the lane's pair (nbr read blocks, from block rb of the planes or byte
// rb of the ASCII; nbw window blocks from b0 of its genome) at S.  kAhead: the
// window's and the read's first blocks are all requested before any is waited for.
// Block by block, a wavefront spent most of its life in seven round trips to
// memory (1M pairs of the fused form: 153 us, 91 us ahead); SHD, whose words take
// the registers that this needs, is better off without (36 against 40 us).
template <bool kN, bool kAscii, bool kAhead>
__device__ inline LdsPair stage_pair(const FilterArgs &a, u32 *S, u64 rb, int nbr, const GenomeMeta &gm, i64 b0,
                                     int nbw, int m) {
    constexpr int AHEAD_W = kAhead && !kN ? 5 : 0, AHEAD_Q = !kAhead ? 0 : kAscii ? 3 : kN ? 0 : 4;
    u64 *q = (u64 *)S, *w = q + (kN ? 3 : 2) * nbr;
    const u64x2 *rl = a.ref_lohi + gm.blk;
    const u64 *rn = a.ref_nb + gm.blk;
    u64x2 wv[AHEAD_W ? AHEAD_W : 1];
#pragma unroll
    for (int b = 0; b < AHEAD_W; b++)
        if (b < nbw) wv[b] = rl[b0 + b];
    auto put_read = [&](int b, const Bits64 &x) {
        q[b] = x.lo;
        q[nbr + b] = x.hi;
        if (kN) q[2 * nbr + b] = x.nb;
    };
    // The window, requested first, is put away before the read is decoded (after it,
    // its registers spilled 56 bytes a pair: 27M pairs of strains 1.86 against 1.81 ms).
    auto put_window = [&] {
#pragma unroll
        for (int b = 0; b < AHEAD_W; b++)
            if (b < nbw) {
                w[b] = wv[b].lo;
                w[nbw + b] = wv[b].hi;
            }
    };
    int done = 0;  // read blocks staged
    if constexpr (kAscii && kAhead) {
        if (rb + 64 * (u64)nbr <= a.seq_total) {  // whole blocks lie in the set (all but its last reads)
            u32 t[AHEAD_Q][4][4];
#pragma unroll
            for (int b = 0; b < AHEAD_Q; b++)
                if (b < nbr)
#pragma unroll
                    for (int i = 0; i < 4; i++) load16(a.seq + rb + 64 * b + 16 * i, t[b][i]);
            put_window();
#pragma unroll
            for (int b = 0; b < AHEAD_Q; b++)
                if (b < nbr) put_read(b, ascii_planes(t[b]));
            done = AHEAD_Q;
        } else {
            put_window();
        }
    } else if constexpr (kAhead && !kN) {
        u64x2 t[AHEAD_Q];
#pragma unroll
        for (int b = 0; b < AHEAD_Q; b++)
            if (b < nbr) t[b] = a.read_lohi[rb + b];
        put_window();
#pragma unroll
        for (int b = 0; b < AHEAD_Q; b++)
            if (b < nbr) put_read(b, Bits64{t[b].lo, t[b].hi, 0});
        done = AHEAD_Q;
    }
    for (int b = done; b < nbr; b++) {
        if constexpr (kAscii || kN) {
            put_read(b, read_block<kAscii>(a, rb, b, m));
        } else {
            const u64x2 x = a.read_lohi[rb + b];
            put_read(b, Bits64{x.lo, x.hi, 0});
        }
    }
    for (int b = AHEAD_W; b < nbw; b++) {
        if constexpr (kN) {
            const Bits64 x = ref_block(rl, rn, (i64)gm.len, meta_has_n(gm), b0 + b);
            w[b] = x.lo;
            w[nbw + b] = x.hi;
            w[2 * nbw + b] = x.nb;
        } else {  // the whole window lies inside a genome without N
            const u64x2 x = rl[b0 + b];
            w[b] = x.lo;
            w[nbw + b] = x.hi;
        }
    }
    return LdsPair(S, nbr, (const u32 *)w, nbw);
}

// A filter that k_filter_lane runs on a staged pair: the obstacle walk with its
// rows in R words, surviving NC columns ...
template <int R, int NC>
struct WalkFilter {
    static constexpr int MAX_M = FAR_MOST, MAX_DW = LANE_DW;
    static constexpr bool AHEAD = true, ALL_FIT = true;
    template <bool kN>
    __device__ static int value(const LdsPair &P, int wofs, int m, int E) {
        return lane_walk<R, NC, kN>(P, wofs, m, E);
    }
};

// kAscii: the fused form's pairs, reads of at most 320 bases as ASCII.  F::ALL_FIT: by
// their class, all pairs fit in LDS.  per_wave: pairs a wavefront takes, 64 where all fit.
template <class F, bool kAscii>
__global__ __launch_bounds__(LANE_TPB) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_filter_lane(FilterArgs a, const u32 *__restrict__ idx, u64 n, u32 per_wave) {
    __shared__ __align__(16) u32 lds[LANE_TPB / 64][LANE_DW + LANE_PAD];
    const int lane = threadIdx.x & 63;
    u32 *S = lds[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)];
    const u32 P = kAscii || F::ALL_FIT ? 64u : per_wave;
    const u64 t0 = (wide_block() * (LANE_TPB / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * P, t = t0 + lane;
    // the pair's fields are requested along with the number of pairs (n bounds
    // their arrays) and looked at after it
    const bool inside = (u32)lane < P && t < n;
    const u64 p = !inside ? 0 : idx ? idx[t] : t;
    const u32 gate = kAscii ? *a.gate : 0u;
    const u64 np = idx ? n : pair_count(a, n);
    u32 r = 0, g = 0;
    i64 diag = 0;
    if (inside) {
        r = a.pair_read[p];
        g = a.pair_genome[p];
        diag = pair_diag(a, p);
    }
    if (gate || t0 >= np) return;  // malformed offsets; the whole wavefront is past the end
    const bool in = inside && t < np;
    u32 err = 0;
    int E = 0, m = 0, nbr = 0, nbw = 0, wofs = 0;
    bool ok = false, with_n = false;
    u64 rb = 0;
    i64 b0 = 0;
    GenomeMeta gm{};
    if (in) {
        if (r >= a.n_reads || g >= a.n_genomes) {
            err = ERR_PAIR_RANGE;
        } else {
            E = a.pair_E ? a.pair_E[p] : a.read_E[r];
            const u64 o = a.read_off[r];
            m = (int)(a.read_off[r + 1] - o);
            rb = kAscii ? o : a.read_blk[r];
            gm = a.meta[g];
            const bool read_n = a.read_has_n[r] != 0;
            ok = E <= 65534;
            err = ok ? 0u : (u32)ERR_E_TOO_LARGE;
            b0 = (diag - E) >> 6;  // floor: the window starts left of the genome for some
            wofs = (int)(diag - E - 64 * b0);
            nbr = (m + 63) / 64;
            nbw = (wofs + 2 * E + m + 63) / 64;
            with_n = ok && (read_n || meta_has_n(gm) || !window_inside(diag, m, E, (i64)gm.len));
        }
    }
    int c = 0;
    const u64 any_n = __ballot(with_n);
    const int need = (any_n ? 6 : 4) * (nbr + nbw);
    const bool fits = need <= F::MAX_DW && m <= F::MAX_M;
    u64 todo = __ballot(ok && m > 0 && fits);
    while (todo) {
        int end = ((todo >> lane) & 1) ? need : 0;  // inclusive prefix sum of the lanes left
        const int mine = end;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(end, o, 64);
            if (lane >= o) end += y;
        }
        const bool now = mine && end <= LANE_DW;
        if (now) {
            u32 *at = S + (end - mine);
            if (any_n)
                c = F::template value<true>(stage_pair<true, kAscii, F::AHEAD>(a, at, rb, nbr, gm, b0, nbw, m), wofs, m,
                                            E);
            else
                c = F::template value<false>(stage_pair<false, kAscii, F::AHEAD>(a, at, rb, nbr, gm, b0, nbw, m), wofs,
                                             m, E);
        }
        todo &= ~__ballot(now);
        lds_wave_sync();
    }
    if constexpr (kAscii || F::ALL_FIT) {
        if (ok && !fits) {
            ok = false;
            err = ERR_INTERNAL;
        }
    } else {
        // The pairs that do not fit, a lane per 64-base word of the read: as many pairs at
        // once as have words for the lanes.  One pair at a time left most lanes without a
        // word (100,000 pairs of 400 bases at E = 7: 1.12 ms, 0.21 so; 40,000 of 1 kbp
        // at E = 50: 4.9 ms, 1.39).
        u64 big = __ballot(ok && !fits);
        u32 *owner = S, *count = S + 64;
        while (big) {
            int end = ((big >> lane) & 1) ? max(1, min((m + 63) / 64, 64)) : 0;
            const int mine = end;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(end, o, 64);
                if (lane >= o) end += y;
            }
            const u64 now = __ballot(mine && end <= 64);  // the first of those left at least
            const bool me = (now >> lane) & 1;
            if (me)
                for (int i = end - mine; i < end; i++) owner[i] = (u32)lane;
            count[lane] = 0;
            const int used = __shfl(end, 63 - __builtin_clzll(now), 64);
            lds_wave_sync();
            const int l = lane < used ? (int)owner[lane] : __builtin_ctzll(now);
            const u32 wr = __shfl(r, l, 64), wg = __shfl(g, l, 64);
            const i64 wdiag = __shfl(diag, l, 64);
            const int wE = __shfl(E, l, 64), first = __shfl(end - mine, l, 64);
            const GenomeMeta wm = a.meta[wg];
            const PairView v{a.read_lohi + a.read_blk[wr], a.read_nb + a.read_blk[wr], read_len(a, wr),
                             a.ref_lohi + wm.blk, a.ref_nb + wm.blk, (i64)wm.len, meta_has_n(wm), wdiag};
            // a pair of more words than lanes is alone and takes turns
            const int turns = __popcll(now) == 1 ? max(1, (v.m + 4095) / 4096) : 1;
            int wc = 0;
            for (int t = 0; t < turns; t++) {
                if (lane < used) wc += F::word(v, wE, lane - first + 64 * t);
                if (t + 1 < turns) {
                    int all = wc;
#pragma unroll
                    for (int o = 32; o; o >>= 1) all += __shfl_xor(all, o, 64);
                    if (all > wE) break;
                }
            }
            if (lane < used) atomicAdd(&count[l], (u32)wc);
            lds_wave_sync();
            if (me) c = (int)count[lane];
            big &= ~now;
            lds_wave_sync();
        }
    }
    if (!in) return;
    if (!ok) atomicOr(a.flags, err);
    const int ap = min(c, E + 1);
    a.approx[p] = ok ? (u16)ap : (u16)0xFFFF;
    a.accept[p] = ok && ap <= E;
}

// Long reads / large E: P = 64 / G pairs per wavefront (and block), each by a group
// of G lanes with its planes in LDS (`tile` 64-base blocks a pair), the rows as
// bits: the words of 32 rows are dealt to the lanes in strips, a step is rows_step
// on a lane's words and a maximum over the group.  A group that is done with its
// pair takes its next one at once, so pairs of one wavefront need not be alike.
// The planes are staged a segment of columns at a time, the next one from the
// current column on when fewer than LONG_AHEAD columns are left: whole reads of 10
// kbp took 25 KB for four pairs, six wavefronts a CU.  A run that leaves the
// segment is measured from global memory.
// Bound by VALU issue.  With the rows in lanes (16 of them each, 32 columns
// compared per row) a step took a whole wavefront for one pair; a step here is
// about as long, for P pairs.  kN: the classes with N planes.
// 300k pairs of 1-10 kbp at E = 5%: 21.1 ms in the three bins before, 8.7 ms now.
template <int G>
__device__ inline int long_group_max(int v) {
    if constexpr (G == 8) {
        v = max(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
        v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
        return max(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false));  // row_half_mirror
    } else {
        return group_max<G>(v);
    }
}

constexpr int LONG_PAD = 16;  // dwords: a step may read a few words past the last plane
constexpr int LONG_AHEAD = 256;

// Pairs idx[0, n) (pairs [0, n) when idx is null) by block `block` of `blocks`.
template <int G, bool kN>
__device__ inline void filter_long(const FilterArgs &a, const u32 *__restrict__ idx, u64 n, int tile, u32 block,
                                   u32 blocks, u32 *lds) {
    constexpr int P = 64 / G, PLANES = kN ? 3 : 2;
    const int lane = threadIdx.x, lg = lane % G;
    u64 *S = (u64 *)(lds + (lane / G) * tile * 2 * PLANES);
    u64 t = (u64)block * P + lane / G, p = 0;
    bool live = false, stage = false;
    u32 r = 0, g = 0;
    int m = 0, E = 0, j = 0, c = 0, wofs = 0, strip = 0;
    int sb = 0, nbr = 0, nbw = 0, end = 0;  // segment: first block, blocks of read and window, end column
    i64 b0 = 0;
    while (__ballot(live || t < n)) {
        if (!live && t < n) {  // the group's next pair (bucketed pairs are valid)
            p = idx ? idx[t] : t;
            t += (u64)blocks * P;
            u32 err;
            bool ok;
            pair_fields(a, p, r, g, E, ok, err);
            m = read_len(a, r);
            const i64 from = pair_diag(a, p) - E;
            b0 = from >> 6;  // first window block (floor)
            wofs = (int)(from - 64 * b0);
            strip = ((2 * E + 32) / 32 + G - 1) / G;  // words of 32 rows per lane
            j = c = 0;
            live = stage = true;
        }
        if (stage) {
            sb = j >> 6;
            const int extra = (2 * E + 126) / 64;  // window blocks beyond the read's
            nbr = min((m + 63) / 64 - sb, (tile - extra) / 2);
            nbw = min((wofs + 2 * E + m + 63) / 64 - sb, nbr + extra);
            end = min(m, 64 * (sb + nbr));
            const u64 rb = a.read_blk[r] + sb;
            const GenomeMeta gm = a.meta[g];
            for (int b = lg; b < nbr; b += G) {
                const u64x2 x = a.read_lohi[rb + b];
                S[b] = x.lo;
                S[nbr + b] = x.hi;
                if (kN) S[2 * nbr + b] = a.read_nb[rb + b];
            }
            u64 *w = S + PLANES * nbr;
            const u64x2 *rl = a.ref_lohi + gm.blk;
            const i64 wb = b0 + sb;
            for (int b = lg; b < nbw; b += G) {
                if constexpr (kN) {
                    const Bits64 x = ref_block(rl, a.ref_nb + gm.blk, (i64)gm.len, meta_has_n(gm), wb + b);
                    w[b] = x.lo;
                    w[nbw + b] = x.hi;
                    w[2 * nbw + b] = x.nb;
                } else {  // the whole window lies inside a genome without N
                    const u64x2 x = rl[wb + b];
                    w[b] = x.lo;
                    w[nbw + b] = x.hi;
                }
            }
            stage = false;
        }
        lds_wave_sync();
        const bool wide = __ballot(live && strip > 2) != 0;  // some group's strips pass two words
        // (Alone in its wavefront, a pair steps on until it is done or its segment is:
        // one pair of 8-10 kbp takes 0.37 ms so, 0.42 with the staging asked at each step.)
        if (live) do {
            const LdsPair L((const u32 *)S, nbr, (const u32 *)(S + PLANES * nbr), nbw);
            const int jl = j - 64 * sb, left = end - j;  // column in the segment; columns left of it
            int best = 0;
            if (left > 0) {
                const u32 ql = plane_at(L.ql, jl), qh = plane_at(L.qh, jl), qn = kN ? plane_at(L.qn, jl) : 0u;
                const int rows = min(2 * E + 1, 32 * strip * (lg + 1));  // the lane's rows end here
                int r0 = 32 * strip * lg;
                if (wide)
                    for (; r0 < rows; r0 += 128)
                        best = max(best, rows_step<4, 6, kN>(L, ql, qh, qn, jl, wofs + jl + r0, jl + left, rows - r0));
                else if (G == 64 && strip == 1) {  // (one pair a wavefront: uniform)
                    if (r0 < rows) best = rows_step<1, 6, kN>(L, ql, qh, qn, jl, wofs + jl + r0, jl + left, rows - r0);
                } else if (r0 < rows)
                    best = rows_step<2, 6, kN>(L, ql, qh, qn, jl, wofs + jl + r0, jl + left, rows - r0);
            }
            best = long_group_max<G>(best);
            if (best >= left && end < m) {  // a run leaves the segment
                const GenomeMeta gm = a.meta[g];
                const PairView v{a.read_lohi + a.read_blk[r], a.read_nb + a.read_blk[r], m, a.ref_lohi + gm.blk,
                                 a.ref_nb + gm.blk, (i64)gm.len, meta_has_n(gm), pair_diag(a, p)};
                best = 0;
                for (int row = lg; row <= 2 * E; row += G) best = max(best, row_run(v, row - E, j));
                best = long_group_max<G>(best);
            }
            j += min(best, m - j);
            if (j < m) {
                c += 1;
                j += 1;
            }
            stage = j + LONG_AHEAD > end && end < m;
            if (j >= m || c > E) {
                live = stage = false;
                if (lg == 0) {
                    const int ap = min(c, E + 1);
                    a.approx[p] = (u16)ap;
                    a.accept[p] = ap <= E;
                }
            }
        } while (G == 64 && live && !stage);
        lds_wave_sync();  // a group's planes are read before its next ones come in
    }
}

// The first blocks_n blocks take the n_n pairs with N planes at idx_n (few, as a
// rule, and as long as the others: they run beside them), the rest the n pairs at
// idx.
template <int G>
__global__ __launch_bounds__(64) void k_filter_long(FilterArgs a, const u32 *__restrict__ idx, u64 n, int tile,
                                                    const u32 *__restrict__ idx_n, u64 n_n, int tile_n,
                                                    u32 blocks_n) {
    extern __shared__ __align__(16) u32 lds[];
    if (blockIdx.x < blocks_n) filter_long<G, true>(a, idx_n, n_n, tile_n, blockIdx.x, blocks_n, lds);
    else filter_long<G, false>(a, idx, n, tile, blockIdx.x - blocks_n, gridDim.x - blocks_n, lds);
}

// ------------------------------------------------------------- variants --

namespace {

struct BucketDesc {
    const char *name;
    int n_variants;
    const char *variants[6];
};

// Variant 0 of a short bucket is one lane per pair; it keeps the name of the
// narrowest group, which it replaces, so that saved selections go on loading.
// Variant v of a long bin: v < 4 -> pairs in LDS, up to 8 per wavefront for the
// default variant and half as many with each below it (long_lanes); v == 4 -> rows in
// lanes from global memory.  (The names count the wavefronts that shared a block when a pair took a
// whole wavefront and its whole planes; their limits stay, so that the same
// selections are taken and refused as ever.)
const BucketDesc BUCKETS[N_BUCKETS] = {
    {"E<=7", 3, {"g16", "g32", "g64"}},
    {"E<=15", 2, {"g32", "g64"}},
    {"E<=31", 1, {"g64"}},
    {"long<=96", 5, {"lds_w1", "lds_w2", "lds_w4", "lds_w8", "global"}},
    {"long<=192", 5, {"lds_w1", "lds_w2", "lds_w4", "lds_w8", "global"}},
    {"long<=384", 5, {"lds_w1", "lds_w2", "lds_w4", "lds_w8", "global"}},
    {"long<=768", 5, {"lds_w1", "lds_w2", "lds_w4", "lds_w8", "global"}},
    {"general", 1, {"global"}},
};

// Defaults: a lane per pair for short E, eight pairs per wavefront for the long bins.
const int DEFAULT_VARIANT[N_BUCKETS] = {0, 0, 0, 3, 3, 2, 1, 0};

std::mutex g_tune_mu;
int g_variant[N_BUCKETS] = {0, 0, 0, 3, 3, 2, 1, 0};
float g_tune_ms[N_BUCKETS][6];
u64 g_tune_pairs[N_BUCKETS];

bool variant_ok(int bucket, int v) {
    if (v < 0 || v >= BUCKETS[bucket].n_variants) return false;
    if (bucket >= CLS_LONG && bucket < CLS_LONG + LONG_BINS && v < 4)
        return (1 << v) * LONG_CAP[bucket - CLS_LONG] * LDS_BLOCK_BYTES <= LONG_LDS_MAX;
    return true;
}

int current_variant(int bucket) {
    std::lock_guard<std::mutex> g(g_tune_mu);
    return g_variant[bucket];
}

}  // namespace

// Lanes for each of so many pairs of a long bin, by one of its variants in LDS.  A few
// pairs leave the chip idle whatever their layout: more lanes each make a step shorter
// (1,024 pairs of 4-5 kbp: 0.29 ms with 64 lanes, 0.35 with 32, 0.36 with 8; 1,024 of
// 8-10 kbp: 0.58 ms with 32 lanes, 0.75 with 8; 4,096: 0.71 with 16, 0.81 with 32, 0.86
// with 8; 16,384: 1.16 and 1.19 with 16 and 8; 40,000: 2.54 and 2.30).  A variant below
// the default, which is the last that fits, doubles them: a selection tuned on a few
// pairs and used for many is then a step from the default at most, as the tuner times
// no second variant with the same lanes.
static int long_lanes(int bucket, int v, u64 pairs) {
    const int few = pairs <= 1024 ? 3 : pairs <= 2048 ? 2 : pairs <= 8192 ? 1 : 0;
    return 8 << std::min(few + std::max(DEFAULT_VARIANT[bucket] - v, 0), 3);
}

// Blocks for cnt pairs of the long kernel: up to four pairs to a group once there
// are blocks for every CU, so that groups with short pairs go on while others finish.
static u32 long_blocks_for(u64 cnt, int G) {
    const u64 one = (cnt * G + 63) / 64, four = (cnt * G + 255) / 256;
    return (u32)std::min<u64>(std::max<u64>(four, std::min<u64>(one, 4096)), 1u << 20);
}

template <int G>
static void launch_long(const FilterArgs &a, const u32 *idx, u64 cnt, int tile, const u32 *idx_n, u64 cnt_n,
                        int tile_n, hipStream_t s) {
    const u32 blocks = long_blocks_for(cnt, G), blocks_n = long_blocks_for(cnt_n, G);
    if (blocks + blocks_n == 0) return;
    const size_t bytes = (size_t)(64 / G) * std::max(cnt ? tile * 16 : 0, cnt_n ? tile_n * 24 : 0) + LONG_PAD * 4;
    k_filter_long<G><<<blocks + blocks_n, 64, bytes, s>>>(a, idx, cnt, tile, idx_n, cnt_n, tile_n, blocks_n);
}

// A bucket's pairs, class by class: places in idx (or pairs [0, count) of the one
// class there is, idx null) and counts.
struct Buckets {
    const u32 *idx;
    const u32 *count, *at;  // per class
    const u32 *of(int cls) const { return idx ? idx + at[cls] : nullptr; }
};

// Launches the pairs of a short bucket or the general one.  far: of reads past far_len.
static void launch_short(const FilterArgs &a, const u32 *idx, u64 cnt, int bucket, int v, bool far, hipStream_t s) {
    if (cnt == 0) return;
    if (bucket == 0 && v == 0 && far) {
        k_filter<16><<<wide_grid(cnt, 16, 256), 256, 0, s>>>(a, idx, cnt);
    } else if (bucket < CLS_LONG && v == 0 && !far) {
        const dim3 blocks = wide_grid(cnt, LANE_TPB, LANE_TPB);
        if (bucket < 2) k_filter_lane<WalkFilter<1, 6>, false><<<blocks, LANE_TPB, 0, s>>>(a, idx, cnt, 64);
        else k_filter_lane<WalkFilter<2, 7>, false><<<blocks, LANE_TPB, 0, s>>>(a, idx, cnt, 64);
    } else if ((bucket == 0 && v == 1) || (bucket == 1 && v == 0)) {
        k_filter<32><<<wide_grid(cnt, 8, 256), 256, 0, s>>>(a, idx, cnt);
    } else {
        k_filter<64><<<wide_grid(cnt, 4, 256), 256, 0, s>>>(a, idx, cnt);
    }
    MT_HIP(hipGetLastError());
}

// Launches the pairs of one bucket with one of its variants.
static void launch_bucket(const FilterArgs &a, const Buckets &B, int bucket, int v, hipStream_t s) {
    const u64 cnt = B.count[bucket];
    const u32 *idx = B.of(bucket);
    if (bucket >= CLS_LONG && bucket < CLS_LONG + LONG_BINS) {
        const int b = bucket - CLS_LONG, cn = CLS_LONG_N + b, cw = CLS_LONG_WIDE + b;
        const int lanes = long_lanes(bucket, v, cnt + B.count[cn]);
        if (v == 4) {
            for (int c : {bucket, cn, cw})
                if (B.count[c])
                    k_filter<64><<<wide_grid(B.count[c], 4, 256), 256, 0, s>>>(a, B.of(c), B.count[c]);
        } else {
            if (lanes == 8)
                launch_long<8>(a, idx, cnt, LONG_TILE, B.of(cn), B.count[cn], LONG_TILE_N, s);
            else if (lanes == 16)
                launch_long<16>(a, idx, cnt, LONG_TILE, B.of(cn), B.count[cn], LONG_TILE_N, s);
            else if (lanes == 32)
                launch_long<32>(a, idx, cnt, LONG_TILE, B.of(cn), B.count[cn], LONG_TILE_N, s);
            else
                launch_long<64>(a, idx, cnt, LONG_TILE, B.of(cn), B.count[cn], LONG_TILE_N, s);
            launch_long<32>(a, nullptr, 0, 0, B.of(cw), B.count[cw], LONG_CAP[b], s);
        }
        MT_HIP(hipGetLastError());
    } else {
        launch_short(a, idx, cnt, bucket, v, false, s);
        if (bucket < CLS_LONG) launch_short(a, B.of(CLS_FAR + bucket), B.count[CLS_FAR + bucket], bucket, v, true, s);
    }
}

// Buckets the pairs (one synchronization for the bucket sizes); idx / counts
// receive the bucketed pair indices and the per-bucket counts and offsets.
// When one bucket holds every pair there is nothing to place: idx stays empty
// (its pointer null) and the bucket is pairs [0, count).
static void bucket_pairs(const FilterArgs &a, u64 n_cap, DBuf<u32> &idx, u32 hc[N_CLASSES], u32 hb[N_CLASSES],
                         hipStream_t s) {
    const unsigned nb = (unsigned)std::min<u64>(grid_for(n_cap, CL_TPB), CL_MAX_BLOCKS);
    DBuf<u32> blk(N_CLASSES * (u64)nb), total(N_CLASSES);
    DBuf<u8> cls(n_cap);
    k_pair_class<<<nb, CL_TPB, 0, s>>>(a, n_cap, blk.p, cls.p);
    MT_HIP(hipGetLastError());
    k_pair_offsets<<<1, OFF_TPB, 0, s>>>(blk.p, nb, total.p);
    MT_HIP(hipGetLastError());
    read_back(s, total.p, hc, N_CLASSES * sizeof(u32));
    u32 acc = 0;
    int populated = 0;
    for (int c = 0; c < N_CLASSES; c++) {
        hb[c] = acc;
        acc += hc[c];
        populated += hc[c] != 0;
    }
    if (populated <= 1) {
        for (int c = 0; c < N_CLASSES; c++) hb[c] = 0;
        return;
    }
    idx.alloc(n_cap);
    k_pair_scatter<<<nb, CL_TPB, 0, s>>>(a, n_cap, cls.p, blk.p, idx.p);
    MT_HIP(hipGetLastError());
}

// Table 1's single-row and base-frequency filters on explicit pairs, one
// thread per pair over the read's 64-base words.  Kind 1 (Hamming distance)
// counts the mismatch bits of row 0 of the band, the diagonal alone; kind 2
// (base counting) compares the counts of A, C, G and T in the read and in the
// reference window [diag, diag + m) (N and positions outside the genome are no
// base) and reports ceil(L1 / 2).  Both saturate at E + 1.
template <int KIND, bool kAscii>
__global__ void k_filter_simple(FilterArgs a, u64 n_cap) {
    const u64 p = wide_block() * blockDim.x + threadIdx.x;
    if (kAscii && *a.gate) return;
    if (p >= pair_count(a, n_cap)) return;
    u32 r, g, err;
    int E;
    bool ok;
    pair_fields(a, p, r, g, E, ok, err);
    if (!ok) {
        atomicOr(a.flags, err);
        a.approx[p] = 0xFFFF;
        a.accept[p] = 0;
        return;
    }
    const int m = read_len(a, r);
    const u64 rb = kAscii ? a.read_off[r] : a.read_blk[r];
    const GenomeMeta gm = a.meta[g];
    const u64x2 *rl = a.ref_lohi + gm.blk;
    const u64 *rn = a.ref_nb + gm.blk;
    const i64 L = (i64)gm.len;
    const bool hn = meta_has_n(gm);
    const i64 diag = pair_diag(a, p);
    int c = 0;
    int dA = 0, dC = 0, dG = 0, dT = 0;  // read count minus window count per base
    for (int w0 = 0; w0 < m; w0 += 64) {
        const Bits64 q = read_block<kAscii>(a, rb, w0 >> 6, m);
        const u64 qn = q.nb;
        const int left = m - w0;
        const u64 vm = left >= 64 ? ~0ull : (1ull << left) - 1;
        const Bits64 wb = fetch_ref(rl, rn, L, hn, diag + w0);
        if constexpr (KIND == 1) {
            c += __popcll(((q.lo ^ wb.lo) | (q.hi ^ wb.hi) | qn | wb.nb) & vm);
            if (c > E) break;
        } else {
            const u64 qv = ~qn & vm, wv = ~wb.nb & vm;
            dA += __popcll(~q.lo & ~q.hi & qv) - __popcll(~wb.lo & ~wb.hi & wv);
            dC += __popcll(q.lo & ~q.hi & qv) - __popcll(wb.lo & ~wb.hi & wv);
            dG += __popcll(~q.lo & q.hi & qv) - __popcll(~wb.lo & wb.hi & wv);
            dT += __popcll(q.lo & q.hi & qv) - __popcll(wb.lo & wb.hi & wv);
        }
    }
    if constexpr (KIND == 2) c = (abs(dA) + abs(dC) + abs(dG) + abs(dT) + 1) / 2;
    const int v = c < E + 1 ? c : E + 1;
    a.approx[p] = (u16)v;
    a.accept[p] = v <= E;
}

// Table 1's q-gram filter (q = QG_Q), one wavefront per pair: the q-grams of
// the reference window [diag - E, diag + m + E) free of N and of positions
// outside the genome are counted in a per-wavefront LDS table of 4^q
// counters; each of the read's q-grams then takes one count (an atomic
// decrement that found it positive), so the number taken is the size of the
// multiset intersection.  Value: ceil((m - q + 1 - shared) / q), 0 for m < q,
// saturated at E + 1.
constexpr int QG_Q = 5;
constexpr int QG_WPB = 4;

template <bool kAscii>
__global__ __launch_bounds__(64 * QG_WPB) void k_filter_qgram(FilterArgs a, u64 n_cap) {
    if (kAscii && *a.gate) return;
    const u64 n = pair_count(a, n_cap);
    __shared__ int cnt_all[QG_WPB][1 << (2 * QG_Q)];
    const int lane = threadIdx.x & 63;
    const u32 wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int *cnt = cnt_all[wid];
    constexpr u64 QMASK = (1ull << QG_Q) - 1;
    for (u64 p = (u64)blockIdx.x * QG_WPB + wid; p < n; p += (u64)gridDim.x * QG_WPB) {
        u32 r, g, err;
        int E;
        bool ok;
        pair_fields(a, p, r, g, E, ok, err);
        if (!ok) {
            if (lane == 0) {
                atomicOr(a.flags, err);
                a.approx[p] = 0xFFFF;
                a.accept[p] = 0;
            }
            continue;
        }
        const int m = read_len(a, r);
        if (m < QG_Q) {
            if (lane == 0) {
                a.approx[p] = 0;
                a.accept[p] = 1;
            }
            continue;
        }
        for (int i = lane; i < (1 << (2 * QG_Q)); i += 64) cnt[i] = 0;
        lds_wave_sync();
        const GenomeMeta gm = a.meta[g];
        const u64x2 *rl = a.ref_lohi + gm.blk;
        const u64 *rn = a.ref_nb + gm.blk;
        const i64 L = (i64)gm.len;
        const bool hn = meta_has_n(gm);
        const i64 w0 = pair_diag(a, p) - E;
        const i64 nwq = (i64)m + 2 * (i64)E - QG_Q + 1;
        for (i64 t = lane; t < nwq; t += 64) {
            const Bits64 b = fetch_ref(rl, rn, L, hn, w0 + t);
            if ((b.nb & QMASK) == 0) atomicAdd(&cnt[kmer_value(b.lo, b.hi, QG_Q)], 1);
        }
        lds_wave_sync();
        const u64 rb = kAscii ? a.read_off[r] : a.read_blk[r];
        int shared = 0;
        for (int j0 = 0; j0 <= m - QG_Q; j0 += 64) {
            const int j = j0 + lane;
            bool took = false;
            if (j <= m - QG_Q) {
                Bits64 b;
                if constexpr (kAscii) b = ascii_block(a, rb + j, min(QG_Q, 16));
                else b = fetch_planes(a.read_lohi + rb, a.read_nb + rb, j);
                if ((b.nb & QMASK) == 0) took = atomicSub(&cnt[kmer_value(b.lo, b.hi, QG_Q)], 1) > 0;
            }
            shared += __popcll(__ballot(took));
        }
        const int missing = m - QG_Q + 1 - shared;
        const int v = min((missing + QG_Q - 1) / QG_Q, E + 1);
        if (lane == 0) {
            a.approx[p] = (u16)v;
            a.accept[p] = v <= E;
        }
        lds_wave_sync();  // the next pair clears the counters
    }
}

// Shifted Hamming distance (Table 1's SHD).  Row d's mismatch word w covers
// columns 64w .. 64w+63 (zero at columns >= m); in each row, a run of one or two
// zeros with a one on both sides (inside the read) becomes ones; the value is the
// number of columns where every amended row is one, saturated at E + 1.
// Word x of a row with its neighbours xp (columns before) and xn (after),
// short zero runs between ones set.
__device__ inline u64 shd_amend(u64 xp, u64 x, u64 xn) {
    const u64 l1 = (x << 1) | (xp >> 63), l2 = (x << 2) | (xp >> 62);  // bit i: x[i - 1], x[i - 2]
    const u64 r1 = (x >> 1) | (xn << 63), r2 = (x >> 2) | (xn << 62);  // bit i: x[i + 1], x[i + 2]
    const u64 one = ~x & l1 & r1;            // 1 0 1
    const u64 first = ~x & ~r1 & l1 & r2;    // 1 [0] 0 1
    const u64 second = ~x & ~l1 & l2 & r1;   // 1 0 [0] 1
    return x | one | first | second;
}

// ... and SHD, for k_filter_lane: rows outer, the read's words in registers.  Bound
// by VALU issue (about 25 operations a row and word); 250k pairs of 100 bases at
// E = 5: 74 us with each row word fetched from global memory, 32 us staged.
struct ShdFilter {
    // MAX_DW: with fewer than 16 pairs at once in LDS, a lane for each word does more
    // (40,000 pairs of 150 bases at E = 3,000, three at once: 9.5 ms and 3.1)
    static constexpr int WORDS = 5, MAX_M = 64 * WORDS, MAX_DW = LANE_DW / 16;
    static constexpr bool AHEAD = false, ALL_FIT = false;
    template <bool kN>
    __device__ static int value(const LdsPair &P, int wofs, int m, int E) {
        u64 acc[WORDS];
#pragma unroll
        for (int w = 0; w < WORDS; w++) {
            const int left = m - 64 * w;
            acc[w] = left >= 64 ? ~0ull : left > 0 ? (1ull << left) - 1 : 0ull;
        }
        const u64 *ql = (const u64 *)P.ql, *qh = (const u64 *)P.qh, *qn = (const u64 *)P.qn;
        for (int row = 0; row <= 2 * E; row++) {
            u64 x[WORDS];
#pragma unroll
            for (int w = 0; w < WORDS; w++) {
                const int left = m - 64 * w;
                x[w] = 0;
                if (left <= 0) continue;
                const int p = wofs + row + 64 * w, k = p >> 5;
                const u32 sh = (u32)p & 31u;
                u64 v = ql[w] ^ word_at(P.wl, k, sh);
                v |= qh[w] ^ word_at(P.wh, k, sh);
                if constexpr (kN) v |= qn[w] | word_at(P.wn, k, sh);
                x[w] = left >= 64 ? v : v & ((1ull << left) - 1);
            }
            u64 any = 0;
#pragma unroll
            for (int w = 0; w < WORDS; w++) {
                acc[w] &= shd_amend(w ? x[w - 1] : 0ull, x[w], w + 1 < WORDS ? x[w + 1] : 0ull);
                any |= acc[w];
            }
            if (any == 0) break;
        }
        int c = 0;
#pragma unroll
        for (int w = 0; w < WORDS; w++) c += __popcll(acc[w]);
        return c;
    }
    // 64 bits of a plane from bit sh of dword k
    __device__ static u64 word_at(const u32 *d, int k, u32 sh) {
        const u32 mid = d[k + 1];
        return (u64)__builtin_amdgcn_alignbit(d[k + 2], mid, sh) << 32 | __builtin_amdgcn_alignbit(mid, d[k], sh);
    }
    // a word of a longer read, each row word with its neighbours
    __device__ static u64 row_word(const PairView &v, int d, int w) {
        const int left = v.m - 64 * w;
        if (w < 0 || left <= 0) return 0;
        const u64x2 q = v.qlohi[w];
        const Bits64 r = fetch_ref(v.rlohi, v.rnb, v.L, v.has_n, v.diag + d + 64 * (i64)w);
        const u64 x = (q.lo ^ r.lo) | (q.hi ^ r.hi) | v.qnb[w] | r.nb;
        return left >= 64 ? x : x & ((1ull << left) - 1);
    }
    __device__ static int word(const PairView &v, int E, int w) {
        const int left = v.m - 64 * w;
        u64 acc = left >= 64 ? ~0ull : left > 0 ? (1ull << left) - 1 : 0ull;
        for (int d = -E; d <= E && acc; d++)
            acc &= shd_amend(row_word(v, d, w - 1), row_word(v, d, w), row_word(v, d, w + 1));
        return __popcll(acc);
    }
};

// Pairs of long reads keep a wavefront for several rounds of words, so a few of them
// are spread over wavefronts for the whole chip (at least 4 each; 40,000 pairs of 1 kbp
// at E = 50: 1.39 ms with 64 a wavefront, 0.74 so).
static void launch_shd(const FilterArgs &a, u64 n, hipStream_t s) {
    constexpr u64 CHIP_WAVES = 4096;
    const u32 per = a.max_len <= (u32)ShdFilter::MAX_M ? 64u : (u32)std::min<u64>(std::max<u64>(n / CHIP_WAVES, 4), 64);
    k_filter_lane<ShdFilter, false><<<wide_grid(n, (u64)per * (LANE_TPB / 64), LANE_TPB), LANE_TPB, 0, s>>>(a, nullptr, n,
                                                                                                           per);
}

void launch_filter_simple(const FilterArgs &a, u64 n, u32 kind, hipStream_t s) {
    if (n == 0) return;  // n: the capacity; the kernels read the count itself
    if (kind == MT_FILTER_HAMMING)
        k_filter_simple<1, false><<<wide_grid(n, 256, 256), 256, 0, s>>>(a, n);
    else if (kind == MT_FILTER_BASE_COUNT)
        k_filter_simple<2, false><<<wide_grid(n, 256, 256), 256, 0, s>>>(a, n);
    else if (kind == MT_FILTER_SHD)
        launch_shd(a, n, s);
    else if (kind == MT_FILTER_QGRAM)
        k_filter_qgram<false><<<(unsigned)std::min<u64>(grid_for(n, QG_WPB), 65536), 64 * QG_WPB, 0, s>>>(a, n);
    else
        throw Error(MT_EINVAL, "unknown filter kind");
    MT_HIP(hipGetLastError());
}

// Pairs of a bucket's classes.
static u64 bucket_count(const u32 *count, int bucket) {
    u64 n = 0;
    for (int c = 0; c < N_CLASSES; c++) n += class_bucket(c) == bucket ? count[c] : 0;
    return n;
}

// Stage names of the per-bucket timing marks.
static const char *const BUCKET_MARKS[N_BUCKETS] = {"filter E<=7",     "filter E<=15",    "filter E<=31",
                                                    "filter long<=96", "filter long<=192", "filter long<=384",
                                                    "filter long<=768", "filter general"};

void launch_filter(const FilterArgs &args, u64 n_cap, int fixed_E, hipStream_t s, Timer *tm) {
    if (n_cap == 0) return;
    FilterArgs a = args;
    a.far_len = far_len(n_cap);
    const bool near = a.max_len <= (u32)a.far_len;
    if (fixed_E >= 0 && fixed_E <= 31 && (near || a.far_len == FAR_LEAST)) {
        // one class, known without looking at the pairs: no bucketing and no
        // synchronization (pairs out of range are reported by every kernel; a few pairs
        // are not worth telling long reads from short ones either)
        const int c = fixed_E <= 7 ? 0 : fixed_E <= 15 ? 1 : 2;
        launch_short(a, nullptr, n_cap, c, current_variant(c), !near, s);
        if (tm) tm->mark(BUCKET_MARKS[c]);
        return;
    }
    DBuf<u32> idx;
    u32 hc[N_CLASSES], hb[N_CLASSES];
    bucket_pairs(a, n_cap, idx, hc, hb, s);
    if (tm) tm->mark("filter buckets");
    for (int b = 0; b < N_BUCKETS; b++) {
        if (bucket_count(hc, b) == 0) continue;
        launch_bucket(a, Buckets{idx.p, hc, hb}, b, current_variant(b), s);
        if (tm) tm->mark(BUCKET_MARKS[b]);
    }
}

void launch_filter_fused(const FilterArgs &a, u64 cap, int max_E, u32 kind, hipStream_t s) {
    if (cap == 0) return;
    const dim3 blocks = wide_grid(cap, LANE_TPB, LANE_TPB);
    static_assert(LANE_TPB == 256, "the simple filters share the grid");
    switch (kind) {
    case MT_FILTER_OBSTACLE:
        if (max_E <= 15) k_filter_lane<WalkFilter<1, 6>, true><<<blocks, LANE_TPB, 0, s>>>(a, nullptr, cap, 64);
        else k_filter_lane<WalkFilter<2, 7>, true><<<blocks, LANE_TPB, 0, s>>>(a, nullptr, cap, 64);
        break;
    case MT_FILTER_HAMMING:
        k_filter_simple<1, true><<<blocks, LANE_TPB, 0, s>>>(a, cap);
        break;
    case MT_FILTER_BASE_COUNT:
        k_filter_simple<2, true><<<blocks, LANE_TPB, 0, s>>>(a, cap);
        break;
    case MT_FILTER_SHD:
        k_filter_lane<ShdFilter, true><<<blocks, LANE_TPB, 0, s>>>(a, nullptr, cap, 64);
        break;
    case MT_FILTER_QGRAM:
        k_filter_qgram<true><<<(unsigned)std::min<u64>(grid_for(cap, QG_WPB), 65536), 64 * QG_WPB, 0, s>>>(a, cap);
        break;
    default:
        throw Error(MT_EINVAL, "unknown filter kind");
    }
    MT_HIP(hipGetLastError());
}

// Whether a variant's launch is that of a variant nearer the default, for the pairs
// of the bucket.
static bool same_launch(const u32 *count, int bucket, int v) {
    if (bucket < CLS_LONG || bucket >= CLS_LONG + LONG_BINS || v >= DEFAULT_VARIANT[bucket]) return false;
    const int b = bucket - CLS_LONG;
    const u64 pairs = (u64)count[bucket] + count[CLS_LONG_N + b];
    return long_lanes(bucket, v, pairs) == long_lanes(bucket, v + 1, pairs);
}

// Times the variants of every bucket that holds pairs (best of `reps`
// launches each, after one untimed launch) and keeps the fastest.  A variant whose
// launch is another's is not timed: noise would choose between them.
void autotune_filter(const FilterArgs &args, u64 n_pairs, u32 reps, hipStream_t s) {
    if (n_pairs == 0) return;
    FilterArgs a = args;
    a.far_len = far_len(n_pairs);
    DBuf<u32> idx;
    u32 hc[N_CLASSES], hb[N_CLASSES];
    bucket_pairs(a, n_pairs, idx, hc, hb, s);
    hipEvent_t e0, e1;
    MT_HIP(hipEventCreate(&e0));
    MT_HIP(hipEventCreate(&e1));
    try {
        for (int c = 0; c < N_BUCKETS; c++) {
            const u64 pairs = bucket_count(hc, c);
            if (pairs == 0) continue;
            auto launch = [&](int v) { launch_bucket(a, Buckets{idx.p, hc, hb}, c, v, s); };
            float best_ms = 0;
            int best = -1;
            float ms_v[6] = {0, 0, 0, 0, 0, 0};
            for (int v = 0; v < BUCKETS[c].n_variants; v++) {
                if (!variant_ok(c, v) || same_launch(hc, c, v)) continue;
                launch(v);
                float mn = 0;
                for (u32 r = 0; r < (reps ? reps : 1); r++) {
                    MT_HIP(hipEventRecord(e0, s));
                    launch(v);
                    MT_HIP(hipEventRecord(e1, s));
                    MT_HIP(hipEventSynchronize(e1));
                    float ms = 0;
                    MT_HIP(hipEventElapsedTime(&ms, e0, e1));
                    if (r == 0 || ms < mn) mn = ms;
                }
                ms_v[v] = mn;
                if (best < 0 || mn < best_ms) {
                    best_ms = mn;
                    best = v;
                }
            }
            std::lock_guard<std::mutex> g(g_tune_mu);
            if (best >= 0) g_variant[c] = best;
            for (int v = 0; v < 6; v++) g_tune_ms[c][v] = ms_v[v];
            g_tune_pairs[c] = pairs;
        }
    } catch (...) {
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        throw;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
}

int tune_buckets() { return N_BUCKETS; }

void tune_info(int bucket, mt_tune_bucket &out) {
    MT_REQUIRE(bucket >= 0 && bucket < N_BUCKETS, "no such filter bucket");
    std::lock_guard<std::mutex> g(g_tune_mu);
    const BucketDesc &d = BUCKETS[bucket];
    out.name = d.name;
    out.n_variants = (u32)d.n_variants;
    out.current = (u32)g_variant[bucket];
    for (int v = 0; v < 6; v++) {
        out.variant_names[v] = v < d.n_variants ? d.variants[v] : nullptr;
        out.ms[v] = g_tune_ms[bucket][v];
    }
    out.pairs = g_tune_pairs[bucket];
}

void tune_set(int bucket, int variant) {
    MT_REQUIRE(bucket >= 0 && bucket < N_BUCKETS, "no such filter bucket");
    MT_REQUIRE(variant_ok(bucket, variant), "variant not available for this bucket");
    std::lock_guard<std::mutex> g(g_tune_mu);
    g_variant[bucket] = variant;
}

void tune_reset() {
    std::lock_guard<std::mutex> g(g_tune_mu);
    for (int c = 0; c < N_BUCKETS; c++) {
        g_variant[c] = DEFAULT_VARIANT[c];
        for (int v = 0; v < 6; v++) g_tune_ms[c][v] = 0;
        g_tune_pairs[c] = 0;
    }
}

}  // namespace mt
