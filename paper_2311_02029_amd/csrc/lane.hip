// The lane-per-read kernels of one minimizer window, MT_WINDOW (a macro of the
// build, which compiles this file once for each window with an instance).
#include "fused.hpp"

namespace mt {

static_assert(MT_WINDOW >= LN_MIN_W && MT_WINDOW <= LN_MAX_W, "with_window reaches it");

// One lane per read.  MAXD: locations a lane's list holds; MAXM: longest read.  The list is searched
// from its front for every hit; the first location, usually the only one, stays
// in registers.
// Bound by the random table lines of the probes: 1M reads of 150 bases on 500 Mbp
// take 0.65 ms (20.8M probes, 32 G/s; the per-stage lookup, which does nothing
// else, reaches 36 G/s), 10M on 4 Gbp of strains 13.4 ms with 52M occurrence
// lists (208M probes, 16 G/s; the lookup alone reaches 19 G/s on that table of
// 24 GB).  k_seed_wave takes 1.57 and 18.6 ms on the same reads.
template <int W, int MAXD, int MAXM>
__global__ __launch_bounds__(LN_TPB) void k_seed_lane(SeedArgs a) {
    __shared__ LaneReads<MAXM> sh_reads[LN_TPB / 64];
    __shared__ u64 sh_key[LN_TPB / 64][MAXD][64];
    __shared__ u16 sh_cnt[LN_TPB / 64][MAXD][64];
    __shared__ u32 sh_stats[ST_COUNT];
    if (*a.gate) return;  // malformed offsets: nothing may be read through them
    if (threadIdx.x < ST_COUNT) sh_stats[threadIdx.x] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    LaneReads<MAXM> &L = sh_reads[wid];
    u64 *keys = &sh_key[wid][0][lane];
    u16 *cnts = &sh_cnt[wid][0][lane];
    const u32 k = a.k, T = a.min_hits ? a.min_hits : 1u, N = a.ncap;
    const u64 r = (u64)blockIdx.x * LN_TPB + threadIdx.x;
    const bool in = r < a.n;
    u64 beg = 0;
    int m = 0, E = 0;
    u32 wflags = 0;
    bool fall = false, slow = false;
    if (in) {
        beg = a.off[r];
        m = (int)(a.off[r + 1] - beg);
        E = read_threshold(a, m, &wflags);
        a.read_E[r] = (u16)E;
        fall = m > LN_MAX_M || E > F_MAX_E;
        slow = !fall && m > MAXM;
    }
    const bool take = in && !fall && !slow;
    const int length = m;
    if (!take) m = 0;
    const int max_m = wave_max(m);
    const LaneRead rd = lane_decode(a.seq, beg, m, a.total, lane, max_m, L);
    if (rd.bad) wflags |= ERR_BAD_BYTE;  // the call fails; its codes are in range all the same
    const bool mixed = ballot64(rd.has_n || m != max_m) != 0;
    const bool sure = mixed ? lane_minimizers<W, true>(L, lane, m, max_m, k)
                            : lane_minimizers<W, false>(L, lane, m, max_m, k);
    slow |= take && !sure;

    // one probe per minimizer; every occurrence is a hit on its location
    int H = 0, nd = 0, nmin = 0, nocc = 0;
    bool many = false;
    u64 key0 = ~0ull;
    u32 cnt0 = 0;
    auto hit = [&](u64 key) {
        if (key == key0) {
            cnt0++;
            return;
        }
        if (nd == 0) {
            key0 = key;
            cnt0 = 1;
            nd = 1;
            return;
        }
        int e = 1;
        while (e < nd && keys[e * 64] != key) e++;
        if (e < nd) {
            cnts[e * 64] += 1;
        } else if (nd < MAXD) {
            keys[e * 64] = key;
            cnts[e * 64] = 1;
            nd++;
        } else {
            many = true;
        }
    };
    if (take && !slow) {
        PickIter<MAXM> it(L, lane, max_m - (int)k + 1);
        // the next minimizer's bucket is requested before this one's is looked at
        Probe cur, nxt;
        int pn = it.next(L, lane);
        if (pn >= 0) nxt.request(a.table, a.nbuckets, lane_kmer(L, lane, pn, k));
        while (pn >= 0) {
            const int p = pn;
            cur = nxt;
            pn = it.next(L, lane);
            if (pn >= 0) nxt.request(a.table, a.nbuckets, lane_kmer(L, lane, pn, k));
            const u64 v = cur.find(a.table, a.nbuckets);
            nmin++;
            if (v == SLOT_NONE) continue;
            const u32 c = slot_count(v);  // 0 for a k-mer above max_occ
            H += (int)min(c, (u32)F_HIT_CAP + 1u);
            if (H > F_HIT_CAP) {
                fall = true;
                break;
            }
            if (!(v & SLOT_MULTI)) {
                hit(cand_key((u32)(v >> 32), (i64)(u32)v - p));
            } else {  // four occurrences in flight at a time
                const u64 st = slot_start(v);
                nocc += (int)c;
                for (u32 u0 = 0; u0 < c; u0 += 4) {
                    u64 gp[4];
#pragma unroll
                    for (int t = 0; t < 4; t++) gp[t] = u0 + t < c ? a.occ[st + u0 + t] : 0ull;
#pragma unroll
                    for (int t = 0; t < 4; t++)
                        if (u0 + t < c) hit(cand_key((u32)(gp[t] >> 32), (i64)(u32)gp[t] - p));
                }
            }
            if (many) break;
        }
    }
    if (many) slow = true;

    // the locations with >= min_hits hits, each to its rank
    int nc = 0;
    if (take && !slow && !fall && nd) {
        keys[0] = key0;
        cnts[0] = (u16)cnt0;
        u32 C = 0;
        for (int e = 0; e < nd; e++) C += cnts[e * 64] >= T;
        if (a.top_n == 0 && C > N) {
            fall = true;  // keep-all with more candidates than staging slots
        } else {
            nc = (int)min(C, N);
            for (int e = 0; e < nd; e++) {
                const u32 he = cnts[e * 64];
                if (he < T) continue;
                const u64 ke = keys[e * 64];
                u32 rank = 0;
                for (int b = 0; b < nd; b++) {
                    const u32 hb = cnts[b * 64];
                    rank += hb > he || (hb == he && keys[b * 64] < ke);
                }
                if (rank < N) {
                    a.st_key[(u64)rank * a.n + r] = ke;
                    a.st_hits[(u64)rank * a.n + r] = he;
                }
            }
        }
    }
    if (in) {
        a.ncand[r] = (u32)nc;
        a.read_n[r] = rd.has_n;
    }
    list_append(in && slow && !fall, r, lane, a.slow_list, a.slow_count);
    list_append(in && fall, r, lane, a.fb_list, a.fb_count);
    if (wflags) atomicOr(a.flags, wflags);
    // work counts: one record per block, summed by k_fused_summary
    const bool done = take && !slow && !fall;
    const u32 st[ST_COUNT] = {done, done ? (u32)m : 0u, done ? (u32)nmin : 0u,
                              (u32)nc * (u32)((m + 2 * E + 63) / 64), (u32)nc, done ? (u32)nocc : 0u,
                              done ? (u32)H : 0u, in && fall ? (u32)length : 0u};
#pragma unroll
    for (u32 i = 0; i < ST_COUNT; i++) {
        const u32 t = wave_sum(st[i]);
        if (lane == 0) atomicAdd(&sh_stats[i], t);
    }
    __syncthreads();
    if (threadIdx.x < ST_COUNT) a.stats_part[(u64)blockIdx.x * ST_COUNT + threadIdx.x] = sh_stats[threadIdx.x];
}
// One lane per read, grid-stride so that a block's counters are flushed once.
// Bound by the probes' random table lines: 1M reads of 150 bases on 500 Mbp,
// 0.60 ms (k_contain_wave on the same reads 1.09 ms).
template <int W, int MAXM>
__global__ __launch_bounds__(LN_TPB) void k_contain_lane(ContainArgs a) {
    __shared__ LaneReads<MAXM> sh_reads[LN_TPB / 64];
    extern __shared__ unsigned long long cnt[];  // one counter per genome when they fit (sized at launch)
    if (*a.gate) return;  // malformed offsets: the whole grid leaves
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    LaneReads<MAXM> &L = sh_reads[wid];
    const bool in_lds = a.n_genomes <= CF_LDS_GENOMES;  // uniform over the grid
    unsigned long long *dst = in_lds ? cnt : a.hits;
    if (in_lds)
        for (u64 g = threadIdx.x; g < a.n_genomes; g += LN_TPB) cnt[g] = 0;
    __syncthreads();
    const u32 k = a.k;
    u32 wflags = 0;
    for (u64 r0 = (u64)blockIdx.x * LN_TPB + 64 * wid; r0 < a.n; r0 += (u64)gridDim.x * LN_TPB) {
        const u64 r = r0 + lane;
        const bool in = r < a.n;
        u64 beg = 0;
        int m = 0;
        if (in) {
            beg = a.off[r];
            m = (int)(a.off[r + 1] - beg);
        }
        const bool fall = m > LN_MAX_M;
        bool slow = !fall && m > MAXM;
        const bool take = in && !fall && !slow;
        const int length = m;
        if (!take) m = 0;
        const int max_m = wave_max(m);
        const LaneRead rd = lane_decode(a.seq, beg, m, a.total, lane, max_m, L);
        if (rd.bad) wflags |= ERR_BAD_BYTE;  // the call fails; its codes are in range all the same
        const bool mixed = ballot64(rd.has_n || m != max_m) != 0;
        const bool sure = mixed ? lane_minimizers<W, true>(L, lane, m, max_m, k)
                                : lane_minimizers<W, false>(L, lane, m, max_m, k);
        slow |= take && !sure;
        if (take && !slow) {
            PickIter<MAXM> it(L, lane, max_m - (int)k + 1);
            Probe cur, nxt;
            int pn = it.next(L, lane);
            if (pn >= 0) nxt.request(a.table, a.nbuckets, lane_kmer(L, lane, pn, k));
            while (pn >= 0) {
                cur = nxt;
                pn = it.next(L, lane);
                if (pn >= 0) nxt.request(a.table, a.nbuckets, lane_kmer(L, lane, pn, k));
                count_genomes(a.occ, cur.find(a.table, a.nbuckets), dst);
            }
        }
        list_append(in && slow, r, lane, a.slow_list, a.slow_count);
        list_append(in && fall, r, length, lane, a.fb_list, a.fb_count, a.fb_bases);
    }
    if (wflags) atomicOr(a.flags, wflags);
    if (in_lds) {
        __syncthreads();
        for (u64 g = threadIdx.x; g < a.n_genomes; g += LN_TPB)
            if (cnt[g]) atomicAdd(&a.hits[g], cnt[g]);
    }
}

template <int W>
void launch_seed_lane(const SeedArgs &a, bool rep, unsigned blocks, hipStream_t s) {
    // Reads that are short on average take the instance whose LDS holds half
    // as many wavefronts again (1M reads of 150 bases: 0.67 against 0.75 ms); its
    // longer reads go to k_seed_wave.
    const bool brief = a.total / a.n <= 160;
    if (rep) {
        if (brief) k_seed_lane<W, 12, LN_SHORT_M><<<blocks, LN_TPB, 0, s>>>(a);
        else k_seed_lane<W, 12, LN_MAX_M><<<blocks, LN_TPB, 0, s>>>(a);
    } else {
        if (brief) k_seed_lane<W, 6, LN_SHORT_M><<<blocks, LN_TPB, 0, s>>>(a);
        else k_seed_lane<W, 6, LN_MAX_M><<<blocks, LN_TPB, 0, s>>>(a);
    }
    MT_HIP(hipGetLastError());
}

template <int W>
void launch_contain_lane(const ContainArgs &a, unsigned blocks, size_t lds, hipStream_t s) {
    if (a.total / a.n <= 160) k_contain_lane<W, LN_SHORT_M><<<blocks, LN_TPB, lds, s>>>(a);
    else k_contain_lane<W, LN_MAX_M><<<blocks, LN_TPB, lds, s>>>(a);
    MT_HIP(hipGetLastError());
}

template void launch_seed_lane<MT_WINDOW>(const SeedArgs &, bool, unsigned, hipStream_t);
template void launch_contain_lane<MT_WINDOW>(const ContainArgs &, unsigned, size_t, hipStream_t);

}  // namespace mt
