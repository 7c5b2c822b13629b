// The obstacle-count filter over explicit pair lists (Fig. 1 step 2d), used by
// the per-stage form, by the fused form's fallback and by mt_filter_pairs.
//
// Pairs are bucketed by their threshold E, and long pairs by the LDS they
// need, so that each bucket gets the kernel shaped for it (uneven batching):
//   E <= 31  one lane per pair, the rows as the bits of one or two words; or
//            groups of G lanes per pair, one band row per lane (G = 32 or 64 for
//            E <= 7, 64 for E <= 15)
//   E > 31   long reads, four bins by the 64-base blocks of read plus
//            reference window they stage in LDS (<= 96, 192, 384, 768): one
//            pair per wavefront, each lane owning a contiguous strip of the
//            2E+1 rows, compared 32 columns at a time from three window
//            dwords per chunk of 32 rows, with the bin's LDS tile and W
//            wavefronts per block;
//            or the rows-in-lanes kernel reading the window from global memory
//   larger   the rows-in-lanes kernel.
// The variant of each bucket (lane or G, W, layout) is chosen by the autotuner
// (mt_autotune) or set by mt_tune_set; every variant gives the same result.
#include <mutex>
#include <string>

#include "classify.hpp"

namespace mt {

constexpr int N_CLASSES = 8;  // E<=7, E<=15, E<=31, four long bins, general
constexpr int CLS_LONG = 3, LONG_BINS = 4, CLS_GENERAL = 7;
constexpr int LONG_CAP[LONG_BINS] = {96, 192, 384, 768};  // 64-base blocks staged per wavefront
constexpr int LDS_BLOCK_BYTES = 24;                        // {lo, hi} + nb of one 64-base block
constexpr int LONG_LDS_MAX = 64 * 1024;                    // per workgroup

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

__device__ inline int read_len(const FilterArgs &a, u32 r) { return (int)(a.read_off[r + 1] - a.read_off[r]); }

// Blocks the long kernel stages for a pair: the read's (with its padding
// block) and the reference window from diag - E, long enough for a 128-base
// fetch at any column < m of any row.
__device__ inline void long_blocks(int m, int E, int &nrb, int &nwb) {
    nrb = (m + 63) / 64 + 1;
    nwb = ((m + 2 * E + 190) >> 6) + 2;
}

// Class of pair p (0..3: the bucket kernels; 4: the general kernel).
__device__ inline u8 pair_class(const FilterArgs &a, u64 p) {
    u32 r, g, err;
    int E;
    bool ok;
    pair_fields(a, p, r, g, E, ok, err);
    if (!ok) return CLS_GENERAL;  // the general kernel reports the error
    if (E <= 7) return 0;
    if (E <= 15) return 1;
    if (E <= 31) return 2;
    int nrb, nwb;
    long_blocks(read_len(a, r), E, nrb, nwb);
    for (int b = 0; b < LONG_BINS; b++)
        if (nrb + nwb <= LONG_CAP[b]) return (u8)(CLS_LONG + b);
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
    u64 tid = (u64)blockIdx.x * blockDim.x + threadIdx.x;
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
    v.diag = a.pair_diag[p];
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

// 64 bases from position p of planes staged in LDS (p >= 0, block p/64 + 1
// staged); kWithN = false reads the N plane as zero.
template <bool kWithN = true>
__device__ inline Bits64 lds_bits(const u64x2 *lohi, const u64 *nb, i64 p) {
    u64 b = (u64)p >> 6;
    u32 s = (u32)p & 63u;
    u64x2 x0 = lohi[b], x1 = lohi[b + 1];
    Bits64 r;
    r.lo = funnel(x0.lo, x1.lo, s);
    r.hi = funnel(x0.hi, x1.hi, s);
    r.nb = kWithN ? funnel(nb[b], nb[b + 1], s) : 0ull;
    return r;
}

// Dword k (bases 32k .. 32k+31) of the lo (pl = 0) or hi (pl = 1) plane of
// {lo, hi} blocks staged in LDS, and of the nb plane.
__device__ inline u32 plane_dw(const u64x2 *lohi, int pl, u32 k) {
    return reinterpret_cast<const u32 *>(lohi)[(k >> 1) * 4 + pl * 2 + (k & 1)];
}
__device__ inline u32 nb_dw(const u64 *nb, u32 k) { return reinterpret_cast<const u32 *>(nb)[k]; }

// One chunk of a lane's rows in the long walk, without branches (a divergent
// branch costs scalar exec-mask instructions): row i's 32 window bases are
// bits [i, i + 32) of (x1:x0) per plane.  The trip count is the wave's rows
// per chunk (uniform); with kTail, rows past the lane's cnt repeat its last
// row, which leaves the maximum unchanged.  bmax gets the largest run (all
// ones for a row whose 32 columns match: the find-first-one value for 0), and
// full the rows whose 32 columns all match, to be continued by the caller.
template <bool kWithN, bool kTail>
__device__ inline void chunk_rows(u32 xl0, u32 xl1, u32 xh0, u32 xh1, u32 xn0, u32 xn1, u32 ql, u32 qh, u32 qn,
                                  int SC, int cnt, u32 &full, u32 &bmax) {
#pragma unroll 4
    for (int i = 0; i < SC; i++) {
        const u32 ie = kTail ? (u32)min(i, cnt - 1) : (u32)i;
        const u32 wl = __builtin_amdgcn_alignbit(xl1, xl0, ie);
        const u32 wh = __builtin_amdgcn_alignbit(xh1, xh0, ie);
        const u32 wn = kWithN ? __builtin_amdgcn_alignbit(xn1, xn0, ie) : 0u;
        // (ql ^ wl) | (qh ^ wh) | qn | wn in two (three with the window's N
        // plane) 3-input bit operations: truth table 0xde takes (x, z, y) to
        // (x ^ y) | z
        const u32 t = __builtin_amdgcn_bitop3_b32(ql, kWithN ? (qn | wn) : qn, wl, 0xde);
        const u32 mm = __builtin_amdgcn_bitop3_b32(qh, t, wh, 0xde);
        const u32 run = mm ? (u32)__builtin_ctz(mm) : ~0u;
        full |= (run >> 31) << i;
        bmax = max(bmax, run);
    }
    if (kTail) full &= cnt >= 32 ? ~0u : (1u << cnt) - 1u;  // the repeated rows are not continued
}

// The obstacle walk of one pair over planes staged in LDS (read at L / NB,
// window at WL / WN, row 0 and column 0 at window offset wbase), rows in
// contiguous strips per lane; returns the obstacle count.  kWithN = false
// leaves the window's N plane out: only for pairs whose compared window lies
// inside a genome without N, where that plane is zero.
template <bool kWithN>
__device__ inline int long_walk(const u64x2 *L, const u64 *NB, const u64x2 *WL, const u64 *WN, i64 wbase, int m,
                                int E, int lane) {
    // lane owns the contiguous rows [r0, r1); per step each chunk of 32 of
    // them is compared over 32 columns from three window dwords per plane
    // (one alignbit per plane and row), and only a row with no obstacle
    // in those columns continues 64 columns at a time
    const int rows = 2 * E + 1;
    const int S = (rows + 63) / 64;
    // every lane takes S rows; the last lanes repeat the band's last rows,
    // which leaves the maximum unchanged
    const int r0 = min(lane * S, rows - S), r1 = r0 + S;
    const int SC = min(32, S);
    int j = 0, c = 0;
    for (;;) {
        // 32 read bases from j (one alignbit per plane)
        const u32 kq = (u32)j >> 5, sq = (u32)j & 31u;
        const u32 ql = __builtin_amdgcn_alignbit(plane_dw(L, 0, kq + 1), plane_dw(L, 0, kq), sq);
        const u32 qh = __builtin_amdgcn_alignbit(plane_dw(L, 1, kq + 1), plane_dw(L, 1, kq), sq);
        const u32 qn = __builtin_amdgcn_alignbit(nb_dw(NB, kq + 1), nb_dw(NB, kq), sq);
        const int left = m - j;
        int best = 0;
        for (int s0 = r0; s0 < r1; s0 += 32) {  // chunks of <= 32 rows
            // window bases of rows s0.. at column j start at p0; three
            // dwords per plane cover every row of the chunk
            const i64 p0 = wbase + (s0 - E) + j;
            const u32 k0 = (u32)((u64)p0 >> 5), sh0 = (u32)p0 & 31u;
            const u32 l0 = plane_dw(WL, 0, k0), l1 = plane_dw(WL, 0, k0 + 1), l2 = plane_dw(WL, 0, k0 + 2);
            const u32 h0 = plane_dw(WL, 1, k0), h1 = plane_dw(WL, 1, k0 + 1), h2 = plane_dw(WL, 1, k0 + 2);
            u32 n0 = 0, n1 = 0, n2 = 0;
            if constexpr (kWithN) {
                n0 = nb_dw(WN, k0);
                n1 = nb_dw(WN, k0 + 1);
                n2 = nb_dw(WN, k0 + 2);
            }
            const int cnt = min(32, r1 - s0);
            // Bits [sh0, sh0 + 64) of the three dwords: row i's 32 window
            // bases are bits [i, i + 32) of them, one alignbit per plane.
            const u32 xl0 = __builtin_amdgcn_alignbit(l1, l0, sh0), xl1 = __builtin_amdgcn_alignbit(l2, l1, sh0);
            const u32 xh0 = __builtin_amdgcn_alignbit(h1, h0, sh0), xh1 = __builtin_amdgcn_alignbit(h2, h1, sh0);
            u32 xn0 = 0, xn1 = 0;
            if constexpr (kWithN) {
                xn0 = __builtin_amdgcn_alignbit(n1, n0, sh0);
                xn1 = __builtin_amdgcn_alignbit(n2, n1, sh0);
            }
            u32 full = 0, bmax = 0;
            if (S <= 32)  // every chunk row is the lane's own: no tail to mask
                chunk_rows<kWithN, false>(xl0, xl1, xh0, xh1, xn0, xn1, ql, qh, qn, SC, cnt, full, bmax);
            else
                chunk_rows<kWithN, true>(xl0, xl1, xh0, xh1, xn0, xn1, ql, qh, qn, SC, cnt, full, bmax);
            best = max(best, min((int)min(bmax, 32u), left));
            // 32 matching columns: continue 64 at a time
            while (full) {
                const int i = (int)__builtin_ctz(full);
                full &= full - 1;
                int run = 32;
                const i64 pos = p0 + i;
                while (j + run < m) {
                    const u64 m2 = mismatch(lds_bits(L, NB, j + run), lds_bits<kWithN>(WL, WN, pos + run));
                    if (m2) {
                        run += (int)__builtin_ctzll(m2);
                        break;
                    }
                    run += 64;
                }
                best = max(best, min(run, left));
            }
        }
        best = group_max<64>(best);
        j += best;
        if (j >= m) break;
        c += 1;
        if (c > E) break;
        j += 1;
    }
    return c;
}

// Long reads / large E: one wavefront per pair, planes in LDS (`tile` blocks
// per wavefront, at least the pairs' nrb + nwb; blockDim.x / 64 wavefronts).
__global__ __launch_bounds__(512) void k_filter_long(FilterArgs a, const u32 *__restrict__ idx, u64 n, int tile) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int wpb = blockDim.x >> 6;
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    u64x2 *L = (u64x2 *)(lds + (size_t)wid * tile * LDS_BLOCK_BYTES);
    u64 *NB = (u64 *)(lds + (size_t)wid * tile * LDS_BLOCK_BYTES + (size_t)tile * 16);
    for (u64 t = (u64)blockIdx.x * wpb + wid; t < n; t += (u64)gridDim.x * wpb) {
        const u64 p = idx ? idx[t] : t;
        u32 r, g, err;
        int E;
        bool ok;
        pair_fields(a, p, r, g, E, ok, err);  // bucketed pairs are valid
        const int m = read_len(a, r);
        const i64 diag = a.pair_diag[p];
        const GenomeMeta gm = a.meta[g];
        int nrb, nwb;
        long_blocks(m, E, nrb, nwb);
        const i64 b0 = (diag - E) >> 6;  // first window block (floor)
        const i64 gblocks = ((i64)gm.len + 63) / 64 + 1;
        const u64 rb = a.read_blk[r];
        const bool with_n = meta_has_n(gm) || diag - E < 0 || diag + m + E > (i64)gm.len;
        for (int b = lane; b < nrb; b += 64) {
            L[b] = a.read_lohi[rb + b];
            NB[b] = a.read_nb[rb + b];
        }
        for (int b = lane; b < nwb; b += 64) {
            const i64 gb = b0 + b;
            u64x2 v{0ull, 0ull};
            u64 nbv = ~0ull;
            if (gb >= 0 && gb < gblocks) {
                v = a.ref_lohi[gm.blk + (u64)gb];
                nbv = with_n ? a.ref_nb[gm.blk + (u64)gb] : 0ull;
            }
            L[nrb + b] = v;
            NB[nrb + b] = nbv;
        }
        lds_wave_sync();
        const u64x2 *WL = L + nrb;
        const u64 *WN = NB + nrb;
        const i64 wbase = diag - 64 * b0;  // window offset of (row 0, column 0)
        // every compared window position inside a genome without N: no N plane
        const int c = with_n ? long_walk<true>(L, NB, WL, WN, wbase, m, E, lane)
                             : long_walk<false>(L, NB, WL, WN, wbase, m, E, lane);
        const int ap = c < E + 1 ? c : E + 1;
        if (lane == 0) {
            a.approx[p] = (u16)ap;
            a.accept[p] = ap <= E;
        }
        lds_wave_sync();
    }
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
// lanes a pair, 79 us here.
//
// The pair's read and window planes are staged in LDS: every step reads them at
// places of its own per lane, which the vector cache serves one line at a time.
// A wavefront's 64 pairs share LANE_DW dwords (a pair of 150 bases takes 24 to
// 28, with the N planes 42); longer pairs go in several batches, and one that
// does not fit at all (reads past 20 kbp) takes the whole wavefront.
constexpr int LANE_TPB = 256, LANE_DW = 2552, LANE_PAD = 8;  // 40 KB a block: four blocks a CU

template <int R, int NC, bool kN>
__device__ inline int lane_walk(const u32 *Q, int nbr, const u32 *W, int nbw, int wofs, int m, int E) {
    const u32 *ql_ = Q, *qh_ = Q + 2 * nbr, *qn_ = Q + 4 * nbr;
    const u32 *wl_ = W, *wh_ = W + 2 * nbw, *wn_ = W + 4 * nbw;
    const int rows = 2 * E + 1;
    u32 mask[R];
#pragma unroll
    for (int i = 0; i < R; i++) mask[i] = rows >= 32 * (i + 1) ? ~0u : rows > 32 * i ? (1u << (rows - 32 * i)) - 1u : 0u;
    int j = 0, c = 0;
    for (;;) {
        const int kq = j >> 5;
        const u32 sq = (u32)j & 31u;
        const u32 ql = __builtin_amdgcn_alignbit(ql_[kq + 1], ql_[kq], sq);
        const u32 qh = __builtin_amdgcn_alignbit(qh_[kq + 1], qh_[kq], sq);
        const u32 qn = kN ? __builtin_amdgcn_alignbit(qn_[kq + 1], qn_[kq], sq) : 0u;
        const int pw = wofs + j, kw = pw >> 5;
        const u32 sw = (u32)pw & 31u;
        u32 xl[R + 1], xh[R + 1], xn[R + 1];
#pragma unroll
        for (int i = 0; i <= R; i++) {
            xl[i] = __builtin_amdgcn_alignbit(wl_[kw + i + 1], wl_[kw + i], sw);
            xh[i] = __builtin_amdgcn_alignbit(wh_[kw + i + 1], wh_[kw + i], sw);
            xn[i] = kN ? __builtin_amdgcn_alignbit(wn_[kw + i + 1], wn_[kw + i], sw) : 0u;
        }
        u32 alive[R], any = 0;
        int best = 0;
#pragma unroll
        for (int i = 0; i < R; i++) alive[i] = mask[i];
#pragma unroll
        for (int t = 0; t < NC; t++) {
            const u32 a = (u32)((int)(ql << (31 - t)) >> 31), b = (u32)((int)(qh << (31 - t)) >> 31);
            const u32 n = kN ? (u32)((int)(qn << (31 - t)) >> 31) : 0u;
            any = 0;
#pragma unroll
            for (int i = 0; i < R; i++) {
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
            u64 al = alive[0];
            if (R > 1) al |= (u64)alive[R - 1] << 32;
            while (al) {
                const int row = (int)__builtin_ctzll(al);
                al &= al - 1;
                int run = NC;
                while (j + run < m) {
                    const int cq = j + run, cw = pw + row + run;
                    const int k = cq >> 5, kk = cw >> 5;
                    const u32 s = (u32)cq & 31u, ss = (u32)cw & 31u;
                    const u32 q1 = ql_[k + 1], h1 = qh_[k + 1], w1 = wl_[kk + 1], v1 = wh_[kk + 1];
                    u32 m0 = (__builtin_amdgcn_alignbit(q1, ql_[k], s) ^ __builtin_amdgcn_alignbit(w1, wl_[kk], ss)) |
                             (__builtin_amdgcn_alignbit(h1, qh_[k], s) ^ __builtin_amdgcn_alignbit(v1, wh_[kk], ss));
                    u32 m1 = (__builtin_amdgcn_alignbit(ql_[k + 2], q1, s) ^
                              __builtin_amdgcn_alignbit(wl_[kk + 2], w1, ss)) |
                             (__builtin_amdgcn_alignbit(qh_[k + 2], h1, s) ^
                              __builtin_amdgcn_alignbit(wh_[kk + 2], v1, ss));
                    if constexpr (kN) {
                        m0 |= __builtin_amdgcn_alignbit(qn_[k + 1], qn_[k], s) |
                              __builtin_amdgcn_alignbit(wn_[kk + 1], wn_[kk], ss);
                        m1 |= __builtin_amdgcn_alignbit(qn_[k + 2], qn_[k + 1], s) |
                              __builtin_amdgcn_alignbit(wn_[kk + 2], wn_[kk + 1], ss);
                    }
                    if (m0 | m1) {
                        run += m0 ? (int)__builtin_ctz(m0) : 32 + (int)__builtin_ctz(m1);
                        break;
                    }
                    run += 64;
                }
                best = max(best, run);
            }
        }
        j += min(best, m - j);  // columns past the read's end count for nothing
        if (j >= m) break;
        c += 1;
        if (c > E) break;
        j += 1;
    }
    return c;
}

// One 64-base block of a read's planes from its ASCII (cnt bases from byte at).
__device__ inline Bits64 ascii_block(const FilterArgs &a, u64 at, int cnt) {
    u32 lo[4], hi[4], nb[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        u32 v[4] = {0, 0, 0, 0};
        const int c = min(16, cnt - 16 * i);
        lo[i] = hi[i] = 0;
        nb[i] = 0xFFFFu;
        if (c > 0) {
            if (at + 16 * i + 16 <= a.seq_total) {
                load16(a.seq + at + 16 * i, v);
            } else {
#pragma unroll
                for (int t = 0; t < 16; t++)
                    if (t < c) v[t >> 2] |= (u32)a.seq[at + 16 * i + t] << (8 * (t & 3));
            }
            plane_bits16(v, &lo[i], &hi[i], &nb[i]);
        }
    }
    return Bits64{lo[0] | lo[1] << 16 | (u64)(lo[2] | lo[3] << 16) << 32,
                  hi[0] | hi[1] << 16 | (u64)(hi[2] | hi[3] << 16) << 32,
                  nb[0] | nb[1] << 16 | (u64)(nb[2] | nb[3] << 16) << 32};
}

// Stages the lane's pair (nbr read blocks, from block rb of the planes or byte
// rb of the ASCII; nbw window blocks from b0 of its genome) at S and walks it.
template <int R, int NC, bool kN, bool kAscii>
__device__ inline int lane_pair(const FilterArgs &a, u32 *S, u64 rb, int nbr, const GenomeMeta &gm, i64 b0, int nbw,
                                int wofs, int m, int E) {
    u64 *q = (u64 *)S;
    for (int b = 0; b < nbr; b++) {
        if constexpr (kAscii) {
            const Bits64 x = ascii_block(a, rb + 64 * (u64)b, m - 64 * b);
            q[b] = x.lo;
            q[nbr + b] = x.hi;
            if (kN) q[2 * nbr + b] = x.nb;
        } else {
            const u64x2 x = a.read_lohi[rb + b];
            q[b] = x.lo;
            q[nbr + b] = x.hi;
            if (kN) q[2 * nbr + b] = a.read_nb[rb + b];
        }
    }
    u64 *w = q + (kN ? 3 : 2) * nbr;
    const u64x2 *rl = a.ref_lohi + gm.blk;
    const u64 *rn = a.ref_nb + gm.blk;
    for (int b = 0; b < nbw; b++) {
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
    return lane_walk<R, NC, kN>(S, nbr, (const u32 *)w, nbw, wofs, m, E);
}

// kAscii: the fused form's pairs, reads of at most 320 bases as ASCII (no pair
// is too long for the LDS).
template <int R, int NC, bool kAscii>
__global__ __launch_bounds__(LANE_TPB) void k_filter_lane(FilterArgs a, const u32 *__restrict__ idx, u64 n) {
    __shared__ __align__(16) u32 lds[LANE_TPB / 64][LANE_DW + LANE_PAD];
    if (kAscii && *a.gate) return;
    const u64 np = idx ? n : pair_count(a, n);
    const u64 t = (u64)blockIdx.x * LANE_TPB + threadIdx.x;
    if (t - (threadIdx.x & 63) >= np) return;  // the whole wavefront is past the end
    const int lane = threadIdx.x & 63;
    u32 *S = lds[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)];
    const bool in = t < np;
    const u64 p = !in ? 0 : idx ? idx[t] : t;
    u32 r = 0, g = 0, err = 0;
    int E = 0, m = 0, nbr = 0, nbw = 0, wofs = 0;
    bool ok = false, with_n = false;
    u64 rb = 0;
    i64 diag = 0, b0 = 0;
    GenomeMeta gm{};
    if (in) {
        pair_fields(a, p, r, g, E, ok, err);
        if (ok) {
            m = read_len(a, r);
            rb = kAscii ? a.read_off[r] : a.read_blk[r];
            diag = a.pair_diag[p];
            gm = a.meta[g];
            b0 = (diag - E) >> 6;  // floor: the window starts left of the genome for some
            wofs = (int)(diag - E - 64 * b0);
            nbr = (m + 63) / 64;
            nbw = (wofs + 2 * E + m + 63) / 64;
            with_n = meta_has_n(gm) || diag - E < 0 || diag + m + E > (i64)gm.len;
            if constexpr (kAscii) {
                with_n |= a.read_n[r] != 0;
            } else {
                for (int w = 0; w < nbr && !with_n; w++) {
                    const int left = m - 64 * w;
                    with_n = (a.read_nb[rb + w] & (left >= 64 ? ~0ull : (1ull << left) - 1)) != 0;
                }
            }
        }
    }
    int c = 0;
    const u64 any_n = __ballot(with_n);
    const int need = (any_n ? 6 : 4) * (nbr + nbw);
    u64 todo = __ballot(ok && m > 0 && need <= LANE_DW);
    u64 big = __ballot(ok && need > LANE_DW);
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
            if (any_n)
                c = lane_pair<R, NC, true, kAscii>(a, S + (end - mine), rb, nbr, gm, b0, nbw, wofs, m, E);
            else
                c = lane_pair<R, NC, false, kAscii>(a, S + (end - mine), rb, nbr, gm, b0, nbw, wofs, m, E);
        }
        todo &= ~__ballot(now);
        lds_wave_sync();
    }
    while (!kAscii && big) {
        const int l = __builtin_ctzll(big);
        big &= big - 1;
        const u32 wr = __shfl(r, l, 64), wg = __shfl(g, l, 64);
        const GenomeMeta wm = a.meta[wg];
        PairView v;
        v.qlohi = a.read_lohi + a.read_blk[wr];
        v.qnb = a.read_nb + a.read_blk[wr];
        v.m = read_len(a, wr);
        v.rlohi = a.ref_lohi + wm.blk;
        v.rnb = a.ref_nb + wm.blk;
        v.L = (i64)wm.len;
        v.has_n = meta_has_n(wm);
        v.diag = __shfl(diag, l, 64);
        const int wc = obstacle_walk<64>(v, __shfl(E, l, 64), lane);
        if (lane == l) c = wc;
    }
    if (!in) return;
    if (!ok) atomicOr(a.flags, err);
    const int ap = min(c, E + 1);
    a.approx[p] = ok ? (u16)ap : (u16)0xFFFF;
    a.accept[p] = ok && ap <= E;
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
// Variant v of a long bin: v < 4 -> strips in LDS with 1 << v wavefronts per
// block (if its LDS fits a workgroup), v == 4 -> rows in lanes from global memory.
const BucketDesc BUCKETS[N_CLASSES] = {
    {"E<=7", 3, {"g16", "g32", "g64"}},
    {"E<=15", 2, {"g32", "g64"}},
    {"E<=31", 1, {"g64"}},
    {"long<=96", 5, {"lds_w1", "lds_w2", "lds_w4", "lds_w8", "global"}},
    {"long<=192", 5, {"lds_w1", "lds_w2", "lds_w4", "lds_w8", "global"}},
    {"long<=384", 5, {"lds_w1", "lds_w2", "lds_w4", "lds_w8", "global"}},
    {"long<=768", 5, {"lds_w1", "lds_w2", "lds_w4", "lds_w8", "global"}},
    {"general", 1, {"global"}},
};

// Defaults: a lane per pair for short E, the most wavefronts per block whose LDS
// fits 64 KB for the long bins.
const int DEFAULT_VARIANT[N_CLASSES] = {0, 0, 0, 3, 3, 2, 1, 0};

std::mutex g_tune_mu;
int g_variant[N_CLASSES] = {0, 0, 0, 3, 3, 2, 1, 0};
float g_tune_ms[N_CLASSES][6];
u64 g_tune_pairs[N_CLASSES];

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

// Launches the pairs idx[0, cnt) of one bucket with one of its variants.
static void launch_bucket(const FilterArgs &a, const u32 *idx, u64 cnt, int bucket, int v, hipStream_t s) {
    if (cnt == 0) return;
    if (bucket < CLS_LONG && v == 0) {
        const unsigned blocks = grid_for(cnt, LANE_TPB);
        if (bucket < 2) k_filter_lane<1, 6, false><<<blocks, LANE_TPB, 0, s>>>(a, idx, cnt);
        else k_filter_lane<2, 7, false><<<blocks, LANE_TPB, 0, s>>>(a, idx, cnt);
    } else if (bucket == 0 && v == 1) {
        k_filter<32><<<grid_for(cnt * 32, 256), 256, 0, s>>>(a, idx, cnt);
    } else if (bucket >= CLS_LONG && bucket < CLS_LONG + LONG_BINS && v < 4) {
        const int tile = LONG_CAP[bucket - CLS_LONG], wpb = 1 << v;
        u64 blocks = (cnt + wpb - 1) / wpb;
        if (blocks > 16384) blocks = 16384;
        k_filter_long<<<(unsigned)blocks, 64 * wpb, (size_t)wpb * tile * LDS_BLOCK_BYTES, s>>>(a, idx, cnt, tile);
    } else {
        k_filter<64><<<grid_for(cnt * 64, 256), 256, 0, s>>>(a, idx, cnt);
    }
    MT_HIP(hipGetLastError());
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
template <int KIND>
__global__ void k_filter_simple(FilterArgs a, u64 n_cap) {
    const u64 p = (u64)blockIdx.x * blockDim.x + threadIdx.x;
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
    const u64 rb = a.read_blk[r];
    const GenomeMeta gm = a.meta[g];
    const u64x2 *rl = a.ref_lohi + gm.blk;
    const u64 *rn = a.ref_nb + gm.blk;
    const i64 L = (i64)gm.len;
    const bool hn = meta_has_n(gm);
    const i64 diag = a.pair_diag[p];
    int c = 0;
    int dA = 0, dC = 0, dG = 0, dT = 0;  // read count minus window count per base
    for (int w0 = 0; w0 < m; w0 += 64) {
        const u64x2 q = a.read_lohi[rb + (u64)(w0 >> 6)];
        const u64 qn = a.read_nb[rb + (u64)(w0 >> 6)];
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

__global__ __launch_bounds__(64 * QG_WPB) void k_filter_qgram(FilterArgs a, u64 n_cap) {
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
        const i64 w0 = a.pair_diag[p] - E;
        const i64 nwq = (i64)m + 2 * (i64)E - QG_Q + 1;
        for (i64 t = lane; t < nwq; t += 64) {
            const Bits64 b = fetch_ref(rl, rn, L, hn, w0 + t);
            if ((b.nb & QMASK) == 0) atomicAdd(&cnt[kmer_value(b.lo, b.hi, QG_Q)], 1);
        }
        lds_wave_sync();
        const u64 rb = a.read_blk[r];
        int shared = 0;
        for (int j0 = 0; j0 <= m - QG_Q; j0 += 64) {
            const int j = j0 + lane;
            bool took = false;
            if (j <= m - QG_Q) {
                const Bits64 b = fetch_planes(a.read_lohi + rb, a.read_nb + rb, j);
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

// Shifted Hamming distance (Table 1's SHD), one thread per pair.  Row d's
// mismatch word w covers columns 64w .. 64w+63 (zero at columns >= m); in
// each row, a run of one or two zeros with a one on both sides (inside the
// read) becomes ones; the value is the number of columns where every amended
// row is one, saturated at E + 1.
__device__ inline u64 shd_word(const FilterArgs &a, u64 rb, int m, const u64x2 *rl, const u64 *rn, i64 L, bool hn,
                               i64 diag, int d, int w) {
    if (w < 0 || 64 * w >= m) return 0;
    const u64x2 q = a.read_lohi[rb + (u64)w];
    const u64 qn = a.read_nb[rb + (u64)w];
    const Bits64 r = fetch_ref(rl, rn, L, hn, diag + d + 64 * (i64)w);
    const int left = m - 64 * w;
    const u64 vm = left >= 64 ? ~0ull : (1ull << left) - 1;
    return ((q.lo ^ r.lo) | (q.hi ^ r.hi) | qn | r.nb) & vm;
}

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

__global__ void k_filter_shd(FilterArgs a, u64 n_cap) {
    const u64 p = (u64)blockIdx.x * blockDim.x + threadIdx.x;
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
    const u64 rb = a.read_blk[r];
    const GenomeMeta gm = a.meta[g];
    const u64x2 *rl = a.ref_lohi + gm.blk;
    const u64 *rn = a.ref_nb + gm.blk;
    const i64 L = (i64)gm.len;
    const bool hn = meta_has_n(gm);
    const i64 diag = a.pair_diag[p];
    int c = 0;
    if (m <= 256) {  // the whole read in four words: rows outer, four accumulators
        u64 acc[4];
#pragma unroll
        for (int w = 0; w < 4; w++) {
            const int left = m - 64 * w;
            acc[w] = left >= 64 ? ~0ull : left > 0 ? (1ull << left) - 1 : 0ull;
        }
        for (int d = -E; d <= E && (acc[0] | acc[1] | acc[2] | acc[3]); d++) {
            u64 x[4];
#pragma unroll
            for (int w = 0; w < 4; w++) x[w] = shd_word(a, rb, m, rl, rn, L, hn, diag, d, w);
#pragma unroll
            for (int w = 0; w < 4; w++) acc[w] &= shd_amend(w ? x[w - 1] : 0ull, x[w], w < 3 ? x[w + 1] : 0ull);
        }
        c = __popcll(acc[0]) + __popcll(acc[1]) + __popcll(acc[2]) + __popcll(acc[3]);
    } else {  // longer reads: words outer, each row word with its neighbours
        const int nw = (m + 63) / 64;
        for (int w = 0; w < nw && c <= E; w++) {
            const int left = m - 64 * w;
            u64 acc = left >= 64 ? ~0ull : (1ull << left) - 1;
            for (int d = -E; d <= E && acc; d++)
                acc &= shd_amend(shd_word(a, rb, m, rl, rn, L, hn, diag, d, w - 1),
                                 shd_word(a, rb, m, rl, rn, L, hn, diag, d, w),
                                 shd_word(a, rb, m, rl, rn, L, hn, diag, d, w + 1));
            c += __popcll(acc);
        }
    }
    const int v = c < E + 1 ? c : E + 1;
    a.approx[p] = (u16)v;
    a.accept[p] = v <= E;
}

void launch_filter_simple(const FilterArgs &a, u64 n, u32 kind, hipStream_t s) {
    if (n == 0) return;  // n: the capacity; the kernels read the count itself
    if (kind == MT_FILTER_HAMMING)
        k_filter_simple<1><<<grid_for(n, 256), 256, 0, s>>>(a, n);
    else if (kind == MT_FILTER_BASE_COUNT)
        k_filter_simple<2><<<grid_for(n, 256), 256, 0, s>>>(a, n);
    else if (kind == MT_FILTER_SHD)
        k_filter_shd<<<grid_for(n, 256), 256, 0, s>>>(a, n);
    else if (kind == MT_FILTER_QGRAM)
        k_filter_qgram<<<(unsigned)std::min<u64>(grid_for(n, QG_WPB), 65536), 64 * QG_WPB, 0, s>>>(a, n);
    else
        throw Error(MT_EINVAL, "unknown filter kind");
    MT_HIP(hipGetLastError());
}

// Stage names of the per-bucket timing marks.
static const char *const BUCKET_MARKS[N_CLASSES] = {"filter E<=7",     "filter E<=15",    "filter E<=31",
                                                    "filter long<=96", "filter long<=192", "filter long<=384",
                                                    "filter long<=768", "filter general"};

void launch_filter(const FilterArgs &a, u64 n_cap, int fixed_E, hipStream_t s, Timer *tm) {
    if (n_cap == 0) return;
    if (fixed_E >= 0 && fixed_E <= 31) {
        // one class, known without looking at the pairs: no bucketing and no
        // synchronization (pairs out of range are reported by every kernel)
        const int c = fixed_E <= 7 ? 0 : fixed_E <= 15 ? 1 : 2;
        launch_bucket(a, nullptr, n_cap, c, current_variant(c), s);
        if (tm) tm->mark(BUCKET_MARKS[c]);
        return;
    }
    DBuf<u32> idx;
    u32 hc[N_CLASSES], hb[N_CLASSES];
    bucket_pairs(a, n_cap, idx, hc, hb, s);
    if (tm) tm->mark("filter buckets");
    for (int c = 0; c < N_CLASSES; c++) {
        if (hc[c] == 0) continue;
        launch_bucket(a, idx.p ? idx.p + hb[c] : nullptr, hc[c], c, current_variant(c), s);
        if (tm) tm->mark(BUCKET_MARKS[c]);
    }
}

void launch_filter_fused(const FilterArgs &a, u64 cap, int max_E, hipStream_t s) {
    if (cap == 0) return;
    const unsigned blocks = grid_for(cap, LANE_TPB);
    if (max_E <= 15) k_filter_lane<1, 6, true><<<blocks, LANE_TPB, 0, s>>>(a, nullptr, cap);
    else k_filter_lane<2, 7, true><<<blocks, LANE_TPB, 0, s>>>(a, nullptr, cap);
    MT_HIP(hipGetLastError());
}

// Times every variant of every bucket that holds pairs (best of `reps`
// launches each, after one untimed launch) and keeps the fastest.
void autotune_filter(const FilterArgs &a, u64 n_pairs, u32 reps, hipStream_t s) {
    if (n_pairs == 0) return;
    DBuf<u32> idx;
    u32 hc[N_CLASSES], hb[N_CLASSES];
    bucket_pairs(a, n_pairs, idx, hc, hb, s);
    hipEvent_t e0, e1;
    MT_HIP(hipEventCreate(&e0));
    MT_HIP(hipEventCreate(&e1));
    try {
        for (int c = 0; c < N_CLASSES; c++) {
            if (hc[c] == 0) continue;
            float best_ms = 0;
            int best = -1;
            float ms_v[6] = {0, 0, 0, 0, 0, 0};
            for (int v = 0; v < BUCKETS[c].n_variants; v++) {
                if (!variant_ok(c, v)) continue;
                launch_bucket(a, idx.p ? idx.p + hb[c] : nullptr, hc[c], c, v, s);
                float mn = 0;
                for (u32 r = 0; r < (reps ? reps : 1); r++) {
                    MT_HIP(hipEventRecord(e0, s));
                    launch_bucket(a, idx.p ? idx.p + hb[c] : nullptr, hc[c], c, v, s);
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
            g_tune_pairs[c] = hc[c];
        }
    } catch (...) {
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        throw;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
}

int tune_buckets() { return N_CLASSES; }

void tune_info(int bucket, mt_tune_bucket &out) {
    MT_REQUIRE(bucket >= 0 && bucket < N_CLASSES, "no such filter bucket");
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
    MT_REQUIRE(bucket >= 0 && bucket < N_CLASSES, "no such filter bucket");
    MT_REQUIRE(variant_ok(bucket, variant), "variant not available for this bucket");
    std::lock_guard<std::mutex> g(g_tune_mu);
    g_variant[bucket] = variant;
}

void tune_reset() {
    std::lock_guard<std::mutex> g(g_tune_mu);
    for (int c = 0; c < N_CLASSES; c++) {
        g_variant[c] = DEFAULT_VARIANT[c];
        for (int v = 0; v < 6; v++) g_tune_ms[c][v] = 0;
        g_tune_pairs[c] = 0;
    }
}

}  // namespace mt
