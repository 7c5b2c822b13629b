// Fused seeding for short reads (Fig. 1 steps 2b-2c in one kernel), then the
// filter and the taxon step over its candidates (2d, 3a).
//   k_seed_lane   one lane per read (lane.hip): 2-bit stream, k-mers and window
//                 minima base by base, then one table probe per minimizer; the
//                 read's locations are counted in a short per-lane list, and the
//                 ones with >= min_hits hits ranked in (hits desc, genome,
//                 diagonal) order and cut to the top_n;
//   k_seed_wave   one wavefront per read: the reads whose lane met a tie of
//                 minimizer keys or more locations than its list holds, small
//                 read sets (which would leave most of the chip idle with 64
//                 reads a wavefront) and minimizer windows without a lane instance;
//   k_compact_seeds   candidates to their places in the result;
//   k_filter_lane     the obstacle walk, one lane per pair (filter.hip), or the
//                     kernel of the query's other filter;
//   k_reduce          accept flag and taxon counts per read (classify.hip).
// The launches follow one another without the host.  Reads beyond the kernels'
// limits (longer than 320 bases; E above 31; more than 256 seed hits; more than 8
// candidates when every candidate is kept) are queued and finished by the per-stage
// kernels, so every read gets the same result as
// in per-stage mode; top_n above 8 runs per stage throughout.
#include <algorithm>

#include "fused.hpp"

namespace mt {

constexpr int F_WPB = 4;         // wavefronts per block
constexpr int F_MAX_M = LN_MAX_M;  // longest read of k_seed_wave
static_assert(F_MAX_M == FUSED_MAX_M, "the forms are told apart by it");
constexpr int F_ROUNDS = F_MAX_M / 64;  // of 64 positions; a read takes those it reaches
constexpr int F_TSLOTS = 256;    // per-read LDS hash table of locations
constexpr int F_MAX_TOPN = 8;    // staged candidates per read (top_n = 0 keeps up to this many)
constexpr int F_WORDS = F_MAX_M / 16 + 2;  // 2-bit stream words (16 bases per word) + padding

// Fewest reads for the lane kernels (see lane_least): 64 reads a wavefront fill the chip late, and a
// lane's chain of k-mers and probes has a latency of its own of about 80 us.
// 32k reads of 150 bases: 88 us in lanes, 63 with a wavefront each; 64k: 101
// against 119.
constexpr u64 LANE_MIN_READS = 48 * 1024;

// Slot of a location key in the per-read LDS table.
__device__ inline u32 tslot(u64 key) {
    u32 x = (u32)key ^ (u32)(key >> 29);
    return (x * 0x9E3779B1u) >> 24;
}

// Counts one seed hit of `key` in the per-read LDS table (linear probing; the
// table never holds more than F_HIT_CAP <= F_TSLOTS distinct keys).  A key's
// first hit also lists its slot (tlist, count *tn), so that the candidate
// scan visits only the slots in use.
__device__ inline void table_add(u64 *tkey, u32 *tcnt, u8 *tlist, u32 *tn, u64 key) {
    u32 s = tslot(key);
    for (int probe = 0; probe < F_TSLOTS; probe++, s = (s + 1) & (F_TSLOTS - 1)) {
        u64 cur = tkey[s];
        if (cur == ~0ull) {
            cur = atomicCAS((unsigned long long *)&tkey[s], ~0ull, (unsigned long long)key);
            if (cur == ~0ull) {
                cur = key;
                tlist[atomicAdd(tn, 1u)] = (u8)s;
            }
        }
        if (cur == key) {
            atomicAdd(&tcnt[s], 1u);
            return;
        }
    }
}

// k-mer value at position i from the big-endian 2-bit stream (base j at bits
// 30 - 2(j mod 16) of word j / 16): bits [2i, 2i + 2k) of the stream.
__device__ inline u64 stream_kmer(const u32 *st, int i, u32 k) {
    int w = i >> 4;
    u32 s = 2u * (u32)(i & 15);
    u64 hi = ((u64)st[w] << 32) | st[w + 1];
    u64 y = (hi << s) | (((u64)st[w + 2] << s) >> 32);
    return y >> (64 - 2 * k);
}

// Smallest hash of window [ws, ws + W) (leftmost on ties), all W hashes read
// before the compare chain; -1 when every hash reads ~0 (no valid k-mer in
// the window).  Unrolled for W <= 12 (the usual minimizer windows); wider
// windows take a loop.
template <int W>
__device__ inline int window_argmin(const u64 *hh, int ws) {
    u64 v[W];
#pragma unroll
    for (int t = 0; t < W; t++) v[t] = hh[ws + t];
    u64 bh = ~0ull;
    int bt = -1;  // offset of the best so far (a constant per step)
#pragma unroll
    for (int t = 0; t < W; t++)
        if (v[t] < bh) {
            bh = v[t];
            bt = t;
        }
    return bt < 0 ? -1 : ws + bt;
}

__device__ inline int window_argmin_any(const u64 *hh, int ws, int win) {
    switch (win) {
#define MT_WIN(W) \
    case W:       \
        return window_argmin<W>(hh, ws);
        MT_WIN(1) MT_WIN(2) MT_WIN(3) MT_WIN(4) MT_WIN(5) MT_WIN(6) MT_WIN(7) MT_WIN(8)
        MT_WIN(9) MT_WIN(10) MT_WIN(11) MT_WIN(12)
#undef MT_WIN
    default: {
        u64 bh = ~0ull;
        int best = -1;
        for (int t = 0; t < win; t++) {
            u64 hv = hh[ws + t];
            if (hv < bh) {
                bh = hv;
                best = ws + t;
            }
        }
        return best;
    }
    }
}

// The bytes of one read, one per lane for each 64-base round (reads longer
// than the kernel takes are not loaded).
struct ReadBytes {
    u64 beg;
    int m;
    u32 b[F_ROUNDS];
};

__device__ inline void issue_read_bytes(const SeedArgs &a, u64 r, int lane, ReadBytes &rb) {
    rb.beg = a.off[r];
    rb.m = (int)(a.off[r + 1] - rb.beg);
#pragma unroll
    for (int q = 0; q < F_ROUNDS; q++) {
        int i = 64 * q + lane;
        rb.b[q] = 'N';
        if (64 * q < rb.m && rb.m <= F_MAX_M && i < rb.m) rb.b[q] = (u32)a.seq[rb.beg + i];
    }
}

// One wavefront per read: reads list[0, *list_n), or all of them when list is null.
//   1. the read's bytes, one per lane and requested while the previous read was
//      counted, become an N plane (ballots) and a big-endian 2-bit stream in LDS;
//   2. lane i hashes the k-mer at position i (per 64-position round);
//   3. lane s scans window s for its smallest valid (hash, position); picks are
//      marked in LDS and compacted with ballot + popcount;
//   4. each minimizer lane probes one table bucket; a read's hits are counted in
//      registers, one ballot per distinct location, when they fit one lane each,
//      and in a per-read LDS hash table otherwise;
//   5. the locations with >= min_hits hits are ranked and staged.
// A read left to the per-stage kernels costs one atomic, for its place in the list; its
// bases are summed with the work counts (a second atomic on that line took as long as
// the rest: 300,000 reads on families of 50 strains, 126,000 left, 3.04 ms, 1.55 so).
// blk0: first record of stats_part.
__global__ __launch_bounds__(64 * F_WPB) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_seed_wave(
    SeedArgs a, const u32 *__restrict__ list, const u32 *__restrict__ list_n, u32 blk0) {
    __shared__ u64 sh_h[F_WPB][F_MAX_M];     // k-mer hashes (~0 when invalid); later candidate keys
    __shared__ u64 sh_tkey[F_WPB][F_TSLOTS]; // per-read hash table of (genome, diagonal) keys
    __shared__ u32 sh_tcnt[F_WPB][F_TSLOTS]; // ... and their seed-hit counts
    __shared__ u16 sh_pos[F_WPB][F_MAX_M];   // minimizer positions; later candidate hit counts
    __shared__ u8 sh_pick[F_WPB][F_MAX_M];   // window picks
    __shared__ u32 sh_st[F_WPB][F_WORDS];    // big-endian 2-bit stream of the read
    __shared__ u64 sh_nb[F_WPB][F_ROUNDS];          // N plane (1 past the end)
    __shared__ u64 sh_stats[F_WPB][ST_COUNT];
    __shared__ u8 sh_tlist[F_WPB][F_TSLOTS];  // slots of the per-read table in use
    __shared__ u32 sh_tn[F_WPB];             // ... and their number

    // wid is wave-uniform; saying so keeps every per-read value (read index,
    // length, E, loop bounds) in scalar registers.
    if (*a.gate) return;  // malformed offsets: nothing may be read through them
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    u64 *hh = sh_h[wid];
    u64 *tkey = sh_tkey[wid];
    u32 *tcnt = sh_tcnt[wid];
    u16 *ccnt = sh_pos[wid];  // candidate hit counts reuse the minimizer positions (dead after the probes)
    u16 *mpos = sh_pos[wid];
    u8 *pick = sh_pick[wid];
    u32 *stream = sh_st[wid];
    u64 *nbp = sh_nb[wid];
    u64 *wst = sh_stats[wid];
    u8 *tlist = sh_tlist[wid];
    u32 *tn = &sh_tn[wid];
    if (lane < (int)ST_COUNT) wst[lane] = 0;
    if (lane == 0) *tn = 0;
    // the table starts empty and every read leaves it empty
    for (int t = lane; t < F_TSLOTS; t += 64) {
        tkey[t] = ~0ull;
        tcnt[t] = 0;
    }

    const u32 k = a.k, T = a.min_hits ? a.min_hits : 1u, N = a.ncap;
    const u64 kmask = (1ull << k) - 1;
    const u64 stride = (u64)gridDim.x * F_WPB;
    u32 wflags = 0;
    const u64 n = list ? *list_n : a.n;
    u64 i = (u64)blockIdx.x * F_WPB + wid;
    u64 r = 0;
    ReadBytes cur;
    if (i < n) {
        r = list ? list[i] : i;
        issue_read_bytes(a, r, lane, cur);
    }
    for (u64 rn = 0; i < n; i += stride, r = rn) {
        const bool more = i + stride < n;
        rn = !more ? 0 : list ? list[i + stride] : i + stride;  // the next read
        const int m = cur.m;
        const int E = read_threshold(a, m, &wflags);
        if (lane == 0) a.read_E[r] = (u16)E;
        if (m > F_MAX_M || E > F_MAX_E) {
            if (lane == 0) {
                a.fb_list[atomicAdd(a.fb_count, 1u)] = (u32)r;
                wst[ST_FB_BASES] += (u64)m;
                a.ncand[r] = 0;  // until the per-stage kernels fill it in
                a.read_n[r] = 0;
            }
            if (more) issue_read_bytes(a, rn, lane, cur);
            continue;
        }

        // 1. N plane of the read (bases past m are N) and its big-endian 2-bit stream
        if (lane < F_WORDS) stream[lane] = 0;
        bool bad = false, has_n = false;
        // the next read's offsets, its start in even lanes and its end in odd
        // ones: requested before the planes are built and read after them, so
        // the planes hide the load (a wave-uniform load would be waited for at
        // once, to move it to scalar registers)
        u64 noff = 0;
        if (more) noff = a.off[rn + (u64)(lane & 1)];
        wave_sync();
#pragma unroll
        for (int q = 0; q < F_ROUNDS; q++) {
            u64 nb = ~0ull;
            if (64 * q < m) {  // (wave-uniform)
                int i = 64 * q + lane;
                u32 c = i < m ? base_code(cur.b[q]) : 4u;
                bad |= c == 5;
                nb = ballot64(c >= 4);
                has_n |= i < m && c == 4;
                if (c < 4 && c > 0) atomicOr(&stream[i >> 4], c << (30 - 2 * (i & 15)));
            }
            if (lane == 0) nbp[q] = nb;
        }
        // (the next read's bytes are requested after the probes)
        const u64 nbeg = readlane64(noff, 0), nend = readlane64(noff, 1);
        if (ballot64(bad)) {
            wflags |= ERR_BAD_BYTE;
            if (lane == 0) {  // the call fails; its compaction still runs
                a.ncand[r] = 0;
                a.read_n[r] = 0;
            }
            if (more) issue_read_bytes(a, rn, lane, cur);
            continue;
        }
        has_n = ballot64(has_n) != 0;
        wave_sync();

        // 2. k-mer hashes (~0 for k-mers with an N)
        const int nk = m - (int)k + 1;
#pragma unroll
        for (int q = 0; q < F_ROUNDS; q++) {
            if (64 * q >= nk) continue;
            int i = 64 * q + lane;
            if (i < nk) {
                u64 nb = funnel(nbp[q], q + 1 < F_ROUNDS ? nbp[q + 1] : ~0ull, (u32)lane);
                hh[i] = (nb & kmask) == 0 ? mix64(stream_kmer(stream, i, k)) : ~0ull;
            }
            pick[i] = 0;
        }
        wave_sync();

        // 3. window minima: an invalid k-mer reads as ~0, a hash no valid k-mer
        // has (the hash is a bijection and the preimage of ~0 lies above every
        // 62-bit k-mer value), so a window of ~0 alone has no minimizer.
        int nmin = 0;
        if (nk > 0) {
            const int win = nk < (int)a.w ? nk : (int)a.w;
            const int nws = nk - win + 1;
#pragma unroll 1
            for (int q = 0; q < F_ROUNDS; q++) {
                if (64 * q >= nws) break;
                int ws = 64 * q + lane;
                if (ws < nws) {
                    const int best = window_argmin_any(hh, ws, win);
                    if (best >= 0) pick[best] = 1;
                }
            }
            wave_sync();
#pragma unroll
            for (int q = 0; q < F_ROUNDS; q++) {
                if (64 * q >= nk) continue;
                int i = 64 * q + lane;
                bool chosen = i < nk && pick[i];
                u64 cm = ballot64(chosen);
                if (chosen) mpos[nmin + lanes_below(cm, lane)] = (u16)i;
                nmin += __popcll(cm);
            }
            wave_sync();
        }

        // 4. table probes -> seed hits.  When every minimizer fits one round
        // and the hits fit one lane each (at most 64 of them, at most 15 per
        // probe), they are counted in registers: one ballot per distinct
        // location; otherwise they go through the per-read LDS table.  With
        // one occurrence per probe (the usual case) a probe's lane holds its
        // hit; otherwise every probe lists its hits in the (empty) table at
        // its prefix offset and lane h takes hit h, the occurrences of all
        // probes being read in one round trip.
        int H = 0, C = 0, nocc = 0;  // nocc: entries read from the multi-occurrence array
        bool overflow = false, counted = false;
        for (int t0 = 0; t0 < nmin; t0 += 64) {
            int j = t0 + lane;
            u64 v = SLOT_NONE;
            int p = 0;
            u32 cnt = 0;
            if (j < nmin) {
                p = mpos[j];
                v = table_lookup(a.table, a.nbuckets, stream_kmer(stream, p, k));
                cnt = v == SLOT_NONE ? 0u : slot_count(v);
            }
            const bool single = cnt == 1 && !(v & SLOT_MULTI);
            const u64 sm = ballot64(single);
            const u64 mm = ballot64(cnt != 0 && !single);  // probes with several occurrences
            bool inreg = false;
            u64 key = 0, hm = 0;  // this lane's hit and the lanes holding one
            if (t0 == 0 && nmin <= 64 && mm == 0) {
                key = single ? cand_key((u32)(v >> 32), (i64)(u32)v - p) : 0ull;
                hm = sm;
                H = __popcll(sm);
                inreg = true;
            } else if (t0 == 0 && nmin <= 64 && ballot64(cnt > 15u) == 0) {
                // exclusive prefix sum of cnt over the lanes, bit by bit
                u32 off = 0, tot = 0;
#pragma unroll
                for (int b = 0; b < 4; b++) {
                    const u64 bm = ballot64((cnt >> b) & 1u);
                    off += lanes_below(bm, lane) << b;
                    tot += (u32)__popcll(bm) << b;
                }
                if (tot <= 64) {
                    // per hit: the slot value (one occurrence) or the index of
                    // the occurrence, and the minimizer position with bit 16
                    // marking an index
                    for (u32 u = 0; u < cnt; u++) {
                        tkey[off + u] = single ? v : slot_start(v) + u;
                        tcnt[off + u] = (u32)p | (single ? 0u : 0x10000u);
                    }
                    wave_sync();
                    const bool has = lane < (int)tot;
                    u64 gv = has ? tkey[lane] : 0ull;
                    const u32 f = has ? tcnt[lane] : 0u;
                    if (has) {  // the table is left empty again
                        tkey[lane] = ~0ull;
                        tcnt[lane] = 0;
                    }
                    if (f & 0x10000u) gv = a.occ[gv];
                    key = has ? cand_key((u32)(gv >> 32), (i64)(u32)gv - (i64)(f & 0xffffu)) : 0ull;
                    hm = ballot64(has);
                    H = (int)tot;
                    nocc += (int)tot - __popcll(sm);
                    inreg = true;
                }
            }
            if (inreg) {
                const bool mine = (hm >> lane) & 1u;
                for (u64 rem = hm; rem;) {
                    const int ld = __builtin_amdgcn_readfirstlane(__builtin_ctzll(rem));
                    const u64 kl = readlane64(key, ld);
                    const u64 eq = ballot64(mine && key == kl);
                    const u32 c = (u32)__popcll(eq);
                    if (c >= T) {
                        if (lane == 0) {
                            hh[C] = kl;
                            ccnt[C] = (u16)c;
                        }
                        C++;
                    }
                    rem &= ~eq;
                }
                counted = true;
                break;
            }
            u32 tot = (u32)__popcll(sm);
            for (u64 rem = mm; rem; rem &= rem - 1)
                tot += __builtin_amdgcn_readlane(cnt, __builtin_amdgcn_readfirstlane(__builtin_ctzll(rem)));
            nocc += (int)(tot - (u32)__popcll(sm));
            if (H + (int)tot > F_HIT_CAP) {
                overflow = true;
                break;
            }
            if (cnt) {
                if (!(v & SLOT_MULTI)) {
                    table_add(tkey, tcnt, tlist, tn, cand_key((u32)(v >> 32), (i64)(u32)v - p));
                } else {  // several occurrences: four loads in flight at a time
                    const u64 st = slot_start(v);
                    for (u32 u0 = 0; u0 < cnt; u0 += 4) {
                        u64 gp[4];
#pragma unroll
                        for (int t = 0; t < 4; t++) gp[t] = u0 + t < cnt ? a.occ[st + u0 + t] : 0ull;
#pragma unroll
                        for (int t = 0; t < 4; t++)
                            if (u0 + t < cnt) table_add(tkey, tcnt, tlist, tn, cand_key((u32)(gp[t] >> 32), (i64)(u32)gp[t] - p));
                    }
                }
            }
            H += (int)tot;
        }
        // the next read's bytes arrive while this one is counted and filtered
        ReadBytes nxt;
        if (more) {
            nxt.beg = nbeg;
            nxt.m = (int)(nend - nbeg);
#pragma unroll
            for (int q = 0; q < F_ROUNDS; q++) {
                int i = 64 * q + lane;
                nxt.b[q] = 'N';
                if (64 * q < nxt.m && nxt.m <= F_MAX_M && i < nxt.m) nxt.b[q] = (u32)a.seq[nbeg + i];
            }
        }
        wave_sync();
        if (overflow) {
            for (int t = lane; t < F_TSLOTS; t += 64) {
                tkey[t] = ~0ull;
                tcnt[t] = 0;
            }
            if (lane == 0) {
                *tn = 0;
                a.fb_list[atomicAdd(a.fb_count, 1u)] = (u32)r;
                wst[ST_FB_BASES] += (u64)m;
                a.ncand[r] = 0;
                a.read_n[r] = has_n;
            }
            cur = nxt;
            wave_sync();
            continue;
        }

        // 5. locations with >= min_hits hits become candidates (the table is
        // emptied as it is read), then top_n by rank
        if (!counted && H > 0) {
            const int nd = (int)*tn;  // distinct keys: the listed slots
            for (int q0 = 0; q0 < nd; q0 += 64) {
                const bool in = q0 + lane < nd;
                const int t = in ? tlist[q0 + lane] : 0;
                const u64 key = in ? tkey[t] : ~0ull;
                const u32 c = in ? tcnt[t] : 0u;
                const bool is_c = key != ~0ull && c >= T;
                if (in) {
                    tkey[t] = ~0ull;
                    tcnt[t] = 0;
                }
                const u64 cm = ballot64(is_c);
                if (is_c) {
                    const int s2 = C + (int)lanes_below(cm, lane);
                    hh[s2] = key;
                    ccnt[s2] = (u16)c;
                }
                C += __popcll(cm);
            }
        }
        wave_sync();
        if (lane == 0) *tn = 0;
        if (a.top_n == 0 && C > (int)N) {
            // keep-all with more candidates than staging slots: per-stage finish
            if (lane == 0) {
                a.fb_list[atomicAdd(a.fb_count, 1u)] = (u32)r;
                wst[ST_FB_BASES] += (u64)m;
                a.ncand[r] = 0;
                a.read_n[r] = has_n;
            }
            cur = nxt;
            wave_sync();
            continue;
        }
        const int nc = C < (int)N ? C : (int)N;
        for (int t0 = 0; t0 < C; t0 += 64) {
            int cidx = t0 + lane;
            if (cidx < C) {
                u64 kc = hh[cidx];
                u32 hc = ccnt[cidx];
                int rank = 0;
#pragma unroll 4
                for (int b = 0; b < C; b++) {
                    u32 hb = ccnt[b];
                    rank += hb > hc || (hb == hc && hh[b] < kc);
                }
                if (rank < nc) {
                    a.st_key[(u64)rank * a.n + r] = kc;
                    a.st_hits[(u64)rank * a.n + r] = hc;
                }
            }
        }
        if (lane == 0) {
            a.ncand[r] = (u32)nc;
            a.read_n[r] = has_n;
        }
        if (lane == 0) {  // work counts, kept in LDS to spare registers
            wst[ST_READS] += 1;
            wst[ST_BASES] += (u64)m;
            wst[ST_MINS] += (u64)nmin;
            wst[ST_CANDS] += (u64)nc;
            wst[ST_WBLOCKS] += (u64)nc * (u64)((m + 2 * E + 63) / 64);
            wst[ST_OCC] += (u64)nocc;
            wst[ST_HITS] += (u64)H;
        }
        cur = nxt;
        wave_sync();
    }
    if (lane == 0 && wflags) atomicOr(a.flags, wflags);
    // work counts: one record per block, summed by k_fused_summary
    __syncthreads();
    if (threadIdx.x < ST_COUNT) {
        u64 t = 0;
        for (int w = 0; w < F_WPB; w++) t += sh_stats[w][threadIdx.x];
        a.stats_part[(u64)(blk0 + blockIdx.x) * ST_COUNT + threadIdx.x] = t;
    }
}

// Control words of one fused call: [0] offsets check, [1] run flags,
// [2] reads for the per-stage kernels, [3] reads for k_seed_wave, [4..5] bases of
// the former (containment; the classification sums them with its work counts).
constexpr int CTL_GATE = 0, CTL_FLAGS = 1, CTL_FB = 2, CTL_SLOW = 3, CTL_FB_BASES = 4, CTL_WORDS = 6;

// Host-visible summary of one fused call, read back with a single copy.
struct FusedSummary {
    u32 gate, flags, nfb, pad;
    u64 n_cands;
    u64 stats[ST_COUNT];
};

// Clears the control words and n counters.
__global__ void k_fused_init(u32 *__restrict__ ctl, u64 *__restrict__ counters, u64 n) {
    const u64 t = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < CTL_WORDS) ctl[t] = 0;
    for (u64 i = t; i < n; i += (u64)gridDim.x * blockDim.x) counters[i] = 0;
}

// Block s < ST_COUNT sums work count s over the kernel's blocks; block 0
// also copies the control words and the candidate total.
constexpr int SUM_TPB = 1024;
__global__ __launch_bounds__(SUM_TPB) void k_fused_summary(const u32 *__restrict__ ctl,
                                                           const u64 *__restrict__ cand_end,
                                                           const u64 *__restrict__ stats_part, u32 blocks,
                                                           FusedSummary *__restrict__ out) {
    __shared__ u64 part[SUM_TPB / 64];
    const int st = blockIdx.x, t = threadIdx.x;
    u64 acc = 0;
    if (!ctl[CTL_GATE])
        for (u32 b = t; b < blocks; b += SUM_TPB) acc += stats_part[(u64)b * ST_COUNT + st];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if ((t & 63) == 0) part[t >> 6] = acc;
    __syncthreads();
    if (t == 0) {
        u64 v = 0;
        for (int i = 0; i < SUM_TPB / 64; i++) v += part[i];
        out->stats[st] = v;
        if (st == 0) {
            out->gate = ctl[CTL_GATE];
            out->flags = ctl[CTL_FLAGS];
            out->nfb = ctl[CTL_FB];
            out->pad = 0;
            out->n_cands = ctl[CTL_GATE] ? 0 : *cand_end;
        }
    }
}

// Offsets check for the fused path (it reads the ASCII bytes directly): the
// error flags of read r.
__device__ inline u32 check_read(const u64 *__restrict__ off, u64 r, u64 n, u64 total) {
    const u64 a = off[r], b = off[r + 1];
    if (b < a || b > total || (r == 0 && a != 0) || (r == n - 1 && b != total)) return ERR_OFFSETS;
    return b - a > 65535 ? (u32)ERR_READ_TOO_LONG : 0u;
}

__global__ void k_check_reads(const u64 *__restrict__ off, u64 n, u64 total, u32 *__restrict__ flags) {
    const u64 r = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const u32 f = check_read(off, r, n, total);
    if (f) atomicOr(flags, f);
}

// k_fused_init and k_check_reads in one launch, by one block: for small read sets,
// where a launch costs more than the block's few rounds.
constexpr int BEGIN_TPB = 1024;
constexpr u64 BEGIN_MAX = 16 * BEGIN_TPB;  // reads and counters
__global__ __launch_bounds__(BEGIN_TPB) void k_fused_begin(const u64 *__restrict__ off, u64 n, u64 total,
                                                           u32 *__restrict__ ctl, u64 *__restrict__ counters,
                                                           u64 n_counters) {
    __shared__ u32 gate;
    if (threadIdx.x == 0) gate = 0;
    __syncthreads();
    u32 f = 0;
    for (u64 r = threadIdx.x; r < n; r += BEGIN_TPB) f |= check_read(off, r, n, total);
    for (u64 i = threadIdx.x; i < n_counters; i += BEGIN_TPB) counters[i] = 0;
    if (f) atomicOr(&gate, f);
    __syncthreads();
    if (threadIdx.x < CTL_WORDS) ctl[threadIdx.x] = threadIdx.x == CTL_GATE ? gate : 0;
}

static void enqueue_begin(const u64 *off, u64 n, u64 total, u32 *ctl, u64 *counters, u64 n_counters, hipStream_t s) {
    if (n <= BEGIN_MAX && n_counters <= BEGIN_MAX) {
        k_fused_begin<<<1, BEGIN_TPB, 0, s>>>(off, n, total, ctl, counters, n_counters);
    } else {
        const unsigned blocks = (unsigned)std::min<u64>(grid_for(n_counters, 1024), 1024);
        k_fused_init<<<blocks, 1024, 0, s>>>(ctl, counters, n_counters);
        k_check_reads<<<grid_for(n, 256), 256, 0, s>>>(off, n, total, ctl + CTL_GATE);
    }
    MT_HIP(hipGetLastError());
}

// Lengths and first bytes of a subset of the reads (the fallback list).
__global__ void k_subset(const u64 *__restrict__ off, const u32 *__restrict__ list, u64 n, u64 *__restrict__ len,
                         u64 *__restrict__ src) {
    u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    src[i] = off[list[i]];
    len[i] = off[list[i] + 1] - src[i];
}

// The subset as a read set that shares the bytes: off its lengths' offsets, src its
// reads' first bytes.
struct Subset {
    DBuf<u64> off, src;
    mt_seqs seqs;
    Subset(const mt_seqs &reads, const u32 *list, u64 n, u64 bases, hipStream_t s)
        : off(n + 1), src(n), seqs{reads.seq, off.p, n, bases} {
        DBuf<u64> len(n);
        k_subset<<<grid_for(n, 256), 256, 0, s>>>(reads.offsets, list, n, len.p, src.p);
        MT_HIP(hipGetLastError());
        scan_u64(len.p, off.p, n, s);
    }
};

// Counts and accept flags of the per-stage finished reads.
__global__ void k_subset_counts(const u32 *__restrict__ list, u64 n, const u64 *__restrict__ sub_off,
                                const u8 *__restrict__ sub_acc, u32 *__restrict__ ncand,
                                u8 *__restrict__ read_accepted) {
    const u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    ncand[list[i]] = (u32)(sub_off[i + 1] - sub_off[i]);
    read_accepted[list[i]] = sub_acc[i];
}

// Filtered candidates of the fused reads from their places without the
// per-stage finished reads (which had none) to those with them.
__global__ void k_move_cands(const u64 *__restrict__ from, const u64 *__restrict__ to, u64 n,
                             const u32 *__restrict__ sg, const i64 *__restrict__ sd, const u32 *__restrict__ sh,
                             const u16 *__restrict__ sa, const u8 *__restrict__ sc, u32 *__restrict__ genome,
                             i64 *__restrict__ diag, u32 *__restrict__ hits, u16 *__restrict__ approx,
                             u8 *__restrict__ accept) {
    const u64 r = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const u64 o = to[r];
    for (u64 c = from[r], e = from[r + 1], d = o; c < e; c++, d++) {
        genome[d] = sg[c];
        diag[d] = sd[c];
        hits[d] = sh[c];
        approx[d] = sa[c];
        accept[d] = sc[c];
    }
}

// Candidates of the per-stage finished reads.
__global__ void k_subset_place(const u32 *__restrict__ list, u64 n, const u64 *__restrict__ sub_off,
                               const u32 *__restrict__ sg, const i64 *__restrict__ sd, const u32 *__restrict__ sh,
                               const u16 *__restrict__ sa, const u8 *__restrict__ sc,
                               const u64 *__restrict__ cand_off, u32 *__restrict__ genome,
                               i64 *__restrict__ diag, u32 *__restrict__ hits, u16 *__restrict__ approx,
                               u8 *__restrict__ accept) {
    u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const u64 b = sub_off[i], e = sub_off[i + 1], o = cand_off[list[i]];
    for (u64 c = b; c < e; c++) {
        genome[o + c - b] = sg[c];
        diag[o + c - b] = sd[c];
        hits[o + c - b] = sh[c];
        approx[o + c - b] = sa[c];
        accept[o + c - b] = sc[c];
    }
}

__global__ void k_add_u64(unsigned long long *__restrict__ dst, const u64 *__restrict__ src, u64 n, u64 less) {
    u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] += src[i] - less;
}

// Staged candidates to their places (cap: room in the result's arrays).
__global__ void k_compact_seeds(const u32 *__restrict__ gate, const u64 *__restrict__ cand_off, u64 n, u32 N, u64 cap,
                                const u64 *__restrict__ st_key, const u32 *__restrict__ st_hits,
                                u32 *__restrict__ genome, i64 *__restrict__ diag, u32 *__restrict__ hits,
                                u32 *__restrict__ pair_read) {
    const u64 r = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n || *gate) return;
    const u64 o = cand_off[r];
    u64 c = cand_off[r + 1] - o;
    if (c > N) c = N;
    if (o > cap || c > cap - o) return;  // never past the candidate capacity
    for (u64 i = 0; i < c; i++) {
        const u64 key = st_key[i * n + r];
        genome[o + i] = key_genome(key);
        diag[o + i] = key_diag(key);
        hits[o + i] = st_hits[i * n + r];
        pair_read[o + i] = (u32)r;
    }
}

// The launches of one fused call once its buffers exist: no host
// synchronization and no memset, so the sequence can also be captured and
// replayed as one HIP graph.
struct FusedLaunch {
    SeedArgs a;
    const mt_index *ix;
    u32 filter;
    u32 *ctl;
    u32 *pair_read;
    unsigned lane_blocks, wave_blocks;  // lane_blocks 0: every read in k_seed_wave
    mt_result *res;
    FusedSummary *sum;
    bool rep;  // repetitive index: room for more locations per read in the lane kernel
};

static void enqueue_fused(const FusedLaunch &L, Timer *tm, hipStream_t s) {
    const SeedArgs &a = L.a;
    mt_result &res = *L.res;
    enqueue_begin(a.off, a.n, a.total, L.ctl, res.uniq.p, res.n_counters(), s);
    if (tm) tm->mark("check");
    if (L.lane_blocks) {
        with_window(a.w, [&](auto w) { launch_seed_lane<decltype(w)::value>(a, L.rep, L.lane_blocks, s); });
        k_seed_wave<<<L.wave_blocks, 64 * F_WPB, 0, s>>>(a, a.slow_list, a.slow_count, L.lane_blocks);
    } else {
        k_seed_wave<<<L.wave_blocks, 64 * F_WPB, 0, s>>>(a, nullptr, nullptr, 0);
    }
    MT_HIP(hipGetLastError());
    if (tm) tm->mark("fused");
    scan_u32(a.ncand, res.cand_off.p, a.n, s);
    k_compact_seeds<<<grid_for(a.n, 256), 256, 0, s>>>(a.gate, res.cand_off.p, a.n, a.ncap, res.cap, a.st_key,
                                                       a.st_hits, res.genome.p, res.diag.p, res.hits.p, L.pair_read);
    MT_HIP(hipGetLastError());
    if (tm) tm->mark("compact");
    FilterArgs fa{};
    fa.pair_read = L.pair_read;
    fa.pair_genome = res.genome.p;
    fa.pair_diag = res.diag.p;
    fa.read_E = a.read_E;
    fa.n_dev = res.cand_off.p + a.n;
    fa.n_host = res.cap;
    fa.n_reads = a.n;
    fa.read_off = a.off;
    fa.n_genomes = L.ix->n_genomes;
    fa.meta = L.ix->meta.p;
    fa.ref_lohi = L.ix->ref.lohi.p;
    fa.ref_nb = L.ix->ref.nb.p;
    fa.approx = res.approx.p;
    fa.accept = res.accept.p;
    fa.flags = a.flags;
    fa.seq = a.seq;
    fa.seq_total = a.total;
    fa.read_has_n = a.read_n;
    fa.gate = a.gate;
    // the largest E a fused read can have: E is fixed, or grows with the length
    const u64 maxE = a.e_mode == MT_E_FIXED           ? a.e_value
                     : a.e_mode == MT_E_CEIL_PERMILLE ? ((u64)LN_MAX_M * a.e_value + 999) / 1000
                                                      : ((u64)LN_MAX_M * a.e_value) / 1000;
    launch_filter_fused(fa, res.cap, (int)std::min<u64>(maxE, F_MAX_E), L.filter, s);
    if (tm) tm->mark("filter");
    launch_reduce(res, *L.ix, a.read_E, a.gate, s);
    k_fused_summary<<<ST_COUNT, SUM_TPB, 0, s>>>(L.ctl, res.cand_off.p + a.n, a.stats_part,
                                                 L.lane_blocks + L.wave_blocks, L.sum);
    MT_HIP(hipGetLastError());
    if (tm) tm->mark("reduce");
}

// One executable graph per host thread, updated in place when a new capture
// has the same shape (only kernel arguments differ) and rebuilt otherwise.
struct GraphCache {
    hipGraphExec_t exec = nullptr;
    ~GraphCache() {
        if (exec) (void)hipGraphExecDestroy(exec);
    }
};
static thread_local GraphCache g_graph;

static void launch_fused_graph(const FusedLaunch &L, hipStream_t s) {
    if (s == nullptr) throw Error(MT_EINVAL, "the graph form needs a stream other than the null stream");
    hipGraph_t graph = nullptr;
    MT_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeRelaxed));
    try {
        enqueue_fused(L, nullptr, s);
    } catch (...) {
        (void)hipStreamEndCapture(s, &graph);
        if (graph) (void)hipGraphDestroy(graph);
        throw;
    }
    MT_HIP(hipStreamEndCapture(s, &graph));
    bool updated = false;
    if (g_graph.exec) {
        hipGraphNode_t err_node = nullptr;
        hipGraphExecUpdateResult ur;
        updated = hipGraphExecUpdate(g_graph.exec, graph, &err_node, &ur) == hipSuccess &&
                  ur == hipGraphExecUpdateSuccess;
        if (!updated) {
            (void)hipGetLastError();
            (void)hipGraphExecDestroy(g_graph.exec);
            g_graph.exec = nullptr;
        }
    }
    hipError_t e = hipSuccess;
    if (!updated) e = hipGraphInstantiate(&g_graph.exec, graph, nullptr, nullptr, 0);
    if (e == hipSuccess) e = hipGraphLaunch(g_graph.exec, s);
    (void)hipGraphDestroy(graph);
    MT_HIP(e);
}

// Hits of a read of the mean length beyond one for each of its minimizers.
static double extra_hits(const mt_index &ix, const mt_seqs &reads) {
    return ix.hits_of(reads.total / reads.n) * (1 - 1 / ix.hits);
}

// Fewest reads for k_seed_lane: LANE_MIN_READS, more on repetitive databases, where a
// lane goes through a read's extra hits one after the other, and none at all where the
// locations of a read pass its list.  Lanes and a wavefront each, 150 bases, k = 21:
//   families of 5 (20 extra hits)   60k 0.28, 0.21 ms; 120k 0.33, 0.34; 1M 1.47, 2.10
//   of 8 (36)                       120k 0.42, 0.38; 300k 0.76, 0.79; 1M 1.99, 2.33
//   of 10 (44)                      300k 0.90, 0.84; 1M 2.40, 2.50
//   of 12 (50; 12 locations)        1M 2.86, 2.63
//   of 20 (89)                      300k 2.47, 1.49
//   k = 13, unrelated (12; 13 locations)   300k 1.16, 0.68
static u64 lane_least(const mt_index &ix, const mt_seqs &reads) {
    if (!ix.repetitive()) return LANE_MIN_READS;
    const double extra = extra_hits(ix, reads), x = extra / 16;
    if ((ix.scattered() ? 1 + extra : ix.locations) > 10) return ~0ull;
    return (u64)((double)LANE_MIN_READS * (1 + x * x));
}

void classify_fused(const mt_index &ix, const mt_query_params &q, const mt_seqs &reads, ReadBatch &rb,
                    mt_result &res, Timer &tm, hipStream_t s, bool graph) {
    // the two-strand read set comes back here; a served batch may not be for the fused form
    if (q.strands == 2 || (q.filter != MT_FILTER_OBSTACLE && !takes_fused(ix, q, reads))) {
        classify_staged(ix, q, reads, rb, res, tm, s);
        return;
    }
    const u64 n = reads.n;
    // staging slots per read: top_n, or F_MAX_TOPN for keep-all (top_n = 0;
    // reads with more candidates are finished per stage)
    const u32 N = q.top_n ? q.top_n : (u32)F_MAX_TOPN;
    if (q.top_n > (u32)F_MAX_TOPN) {
        // Long candidate lists: the per-stage kernels handle them.
        rb.prepare(reads, q.e_mode, q.e_value, s);
        MT_HIP(hipMemcpyAsync(res.read_E.p, rb.read_E.p, (n ? n : 1) * sizeof(u16), hipMemcpyDeviceToDevice, s));
        tm.mark("pack");
        classify_per_stage(ix, q, reads, rb, res, tm, s);
        u32 f = 0;
        read_back(s, rb.flags.p, &f, sizeof f);
        check_flags(f);
        read_back(s, res.cand_off.p + n, &res.n_cands, sizeof(u64));
        return;
    }
    rb.n = n;
    if (n == 0) {
        zero_counters(res, s);
        res.n_cands = 0;
        return;
    }

    int dev = 0, cus = 0;
    MT_HIP(hipGetDevice(&dev));
    MT_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    const bool lanes = ix.w >= (u32)LN_MIN_W && ix.w <= (u32)LN_MAX_W && n >= lane_least(ix, reads);
    const u64 lane_blocks = lanes ? grid_for(n, LN_TPB) : 0;
    // k_seed_wave: many short blocks, so that resident blocks finish together; a
    // list of slow reads, whose length only the device knows, takes fewer
    u64 wave_blocks = std::min<u64>((n + F_WPB - 1) / F_WPB, (u64)cus * (lanes ? 8 : 64));

    DBuf<u64> st_key(n * N);
    DBuf<u32> st_hits(n * N), ncand(n), fb_list(n), slow_list(lanes ? n : 0), ctl(CTL_WORDS), pair_read(n * N);
    DBuf<u8> read_n(n);
    DBuf<u64> stats_part((lane_blocks + wave_blocks) * ST_COUNT);
    DBuf<FusedSummary> sum(1);
    res.alloc_cands(n * N);

    FusedLaunch L{};
    SeedArgs &a = L.a;
    a.seq = (const u8 *)reads.seq;
    a.off = reads.offsets;
    a.n = n;
    a.total = reads.total;
    a.k = ix.k;
    a.w = ix.w;
    a.min_hits = q.min_hits;
    a.top_n = q.top_n;
    a.ncap = N;
    a.e_mode = q.e_mode;
    a.e_value = q.e_value;
    a.table = ix.table.p;
    a.nbuckets = ix.nbuckets;
    a.occ = ix.occ.p;
    a.st_key = st_key.p;
    a.st_hits = st_hits.p;
    a.ncand = ncand.p;
    a.read_E = res.read_E.p;
    a.read_n = read_n.p;
    a.slow_list = slow_list.p;
    a.slow_count = ctl.p + CTL_SLOW;
    a.fb_list = fb_list.p;
    a.fb_count = ctl.p + CTL_FB;
    a.flags = ctl.p + CTL_FLAGS;
    a.gate = ctl.p + CTL_GATE;
    a.stats_part = stats_part.p;
    L.ix = &ix;
    L.filter = q.filter;
    L.ctl = ctl.p;
    L.pair_read = pair_read.p;
    L.lane_blocks = (unsigned)lane_blocks;
    L.wave_blocks = (unsigned)wave_blocks;
    L.res = &res;
    L.sum = sum.p;
    L.rep = ix.repetitive();

    if (graph) {
        launch_fused_graph(L, s);
        tm.mark("graph");
    } else {
        enqueue_fused(L, &tm, s);
    }
    FusedSummary h{};
    read_back(s, sum.p, &h, sizeof h);
    check_flags(h.gate | h.flags);
    mt_stats &ls = last_stats();
    ls.fused_reads += h.stats[ST_READS];
    ls.fused_bases += h.stats[ST_BASES];
    ls.fused_minimizers += h.stats[ST_MINS];
    ls.fused_window_blocks += h.stats[ST_WBLOCKS];
    ls.fused_cands += h.stats[ST_CANDS];
    ls.fused_occ += h.stats[ST_OCC];
    ls.n_minimizers += h.stats[ST_MINS];
    ls.n_hits += h.stats[ST_HITS];
    // Every read's count is at most N (the seed kernels write one per read), so
    // the total fits the staged capacity; a result never claims more
    // candidates than its arrays hold.
    if (h.n_cands > res.cap) throw Error(MT_EINTERNAL, "fused candidate count exceeds the staged capacity");
    res.n_cands = h.n_cands;
    const u32 nfb = h.nfb;
    if (nfb == 0) return;

    // Reads past the fused kernels' limits: finish them per stage, as a subset
    // that shares the bytes, and make room for their candidates among the others'.
    const Subset sub(reads, fb_list.p, nfb, h.stats[ST_FB_BASES], s);
    mt_result tmp;
    mt_result_init(tmp, nfb, ix.n_taxa, s);
    ReadBatch srb;
    srb.prepare(sub.seqs, q.e_mode, q.e_value, s, sub.src.p, reads.total);
    classify_per_stage(ix, q, sub.seqs, srb, tmp, tm, s);
    k_subset_counts<<<grid_for(nfb, 256), 256, 0, s>>>(fb_list.p, nfb, tmp.cand_off.p, tmp.read_accepted.p, ncand.p,
                                                       res.read_accepted.p);
    MT_HIP(hipGetLastError());
    if (ix.n_taxa) {
        k_add_u64<<<grid_for(ix.n_taxa, 256), 256, 0, s>>>((unsigned long long *)res.uniq.p, tmp.uniq.p, ix.n_taxa, 0);
        k_add_u64<<<grid_for(ix.n_taxa, 256), 256, 0, s>>>((unsigned long long *)res.multi.p, tmp.multi.p,
                                                           ix.n_taxa, 0);
    }
    // these reads counted as unmapped while they had no candidates
    k_add_u64<<<1, 64, 0, s>>>((unsigned long long *)res.unmapped.p, tmp.unmapped.p, 1, nfb);
    MT_HIP(hipGetLastError());
    DBuf<u64> old_off(n + 1);
    MT_HIP(hipMemcpyAsync(old_off.p, res.cand_off.p, (n + 1) * sizeof(u64), hipMemcpyDeviceToDevice, s));
    const DBuf<u8> old_cands(std::move(res.cands_block));
    const auto old_genome = res.genome, old_hits = res.hits;
    const auto old_diag = res.diag;
    const auto old_approx = res.approx;
    const auto old_accept = res.accept;
    scan_u32(ncand.p, res.cand_off.p, n, s);
    u32 f2 = 0;
    u64 total = 0;
    MT_HIP(hipMemcpyAsync(&f2, srb.flags.p, sizeof f2, hipMemcpyDeviceToHost, s));
    read_back(s, res.cand_off.p + n, &total, sizeof total);
    check_flags(f2);
    res.alloc_cands(total);
    k_move_cands<<<grid_for(n, 256), 256, 0, s>>>(old_off.p, res.cand_off.p, n, old_genome.p, old_diag.p, old_hits.p,
                                                  old_approx.p, old_accept.p, res.genome.p, res.diag.p, res.hits.p,
                                                  res.approx.p, res.accept.p);
    MT_HIP(hipGetLastError());
    k_subset_place<<<grid_for(nfb, 256), 256, 0, s>>>(fb_list.p, nfb, tmp.cand_off.p, tmp.genome.p, tmp.diag.p,
                                                      tmp.hits.p, tmp.approx.p, tmp.accept.p, res.cand_off.p,
                                                      res.genome.p, res.diag.p, res.hits.p, res.approx.p,
                                                      res.accept.p);
    MT_HIP(hipGetLastError());
    res.n_cands = total;
    tm.mark("fallback");
}

// ------------------------------------------------------ containment search --

// Containment search (Fig. 1 steps 1a-1c): minimizers as in the classification,
// then one table probe each, adding one hit to the genome of every occurrence.
// Up to CF_LDS_GENOMES genomes a block counts in LDS and adds its nonzero
// counters to the global ones when it ends; with more genomes the hits go to
// the global counters directly.  k_contain_lane takes a lane per read,
// k_contain_wave a wavefront (k_seed_lane and k_seed_wave divide the reads the
// same way); reads beyond both are listed for the per-stage chain.

// One wavefront per read: reads list[0, *list_n), or all of them when list is null.
__global__ __launch_bounds__(64 * F_WPB) void k_contain_wave(ContainArgs a, const u32 *__restrict__ list,
                                                             const u32 *__restrict__ list_n) {
    __shared__ u64 sh_h[F_WPB][F_MAX_M];
    __shared__ u16 sh_pos[F_WPB][F_MAX_M];
    __shared__ u8 sh_pick[F_WPB][F_MAX_M];
    __shared__ u32 sh_st[F_WPB][F_WORDS];
    __shared__ u64 sh_nb[F_WPB][F_ROUNDS];
    extern __shared__ unsigned long long cnt[];  // one counter per genome when they fit (sized at launch)
    if (*a.gate) return;  // malformed offsets: the whole grid leaves
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    u64 *hh = sh_h[wid];
    u16 *mpos = sh_pos[wid];
    u8 *pick = sh_pick[wid];
    u32 *stream = sh_st[wid];
    u64 *nbp = sh_nb[wid];
    const bool in_lds = a.n_genomes <= CF_LDS_GENOMES;  // uniform over the grid
    unsigned long long *dst = in_lds ? cnt : a.hits;
    if (in_lds)
        for (u64 g = threadIdx.x; g < a.n_genomes; g += blockDim.x) cnt[g] = 0;
    __syncthreads();
    const u32 k = a.k;
    const u64 kmask = (1ull << k) - 1;
    u32 wflags = 0;
    u64 fb_bases = 0;
    const u64 stride = (u64)gridDim.x * F_WPB;
    const u64 n = list ? *list_n : a.n;
    u64 i = (u64)blockIdx.x * F_WPB + wid;
    u64 r = i >= n ? 0 : list ? list[i] : i;
    // the read in hand: its length and its bytes, one per lane per 64-base
    // round (the next read's are requested while this one is probed)
    int m = 0;
    u32 b[F_ROUNDS];
    if (i < n) {
        const u64 beg = a.off[r];
        m = (int)(a.off[r + 1] - beg);
#pragma unroll
        for (int q = 0; q < F_ROUNDS; q++) {
            const int i = 64 * q + lane;
            b[q] = (m <= F_MAX_M && i < m) ? (u32)a.seq[beg + i] : (u32)'N';
        }
    }
    for (u64 rn = 0; i < n; i += stride, r = rn) {
        const bool more = i + stride < n;
        rn = !more ? 0 : list ? list[i + stride] : i + stride;  // the next read
        // the next read's offsets, its start in even lanes and its end in odd
        // ones (read after the minimizers; a wave-uniform load would be waited
        // for at once)
        u64 noff = 0;
        if (more) noff = a.off[rn + (u64)(lane & 1)];
        if (m > F_MAX_M) {
            if (lane == 0) a.fb_list[atomicAdd(a.fb_count, 1u)] = (u32)r;
            fb_bases += (u64)m;
            const u64 nbeg = readlane64(noff, 0);
            m = (int)(readlane64(noff, 1) - nbeg);
#pragma unroll
            for (int q = 0; q < F_ROUNDS; q++) {
                const int i = 64 * q + lane;
                b[q] = (more && m <= F_MAX_M && i < m) ? (u32)a.seq[nbeg + i] : (u32)'N';
            }
            continue;
        }
        // 1. N plane and big-endian 2-bit stream
        if (lane < F_WORDS) stream[lane] = 0;
        wave_sync();
        bool bad = false;
#pragma unroll
        for (int q = 0; q < F_ROUNDS; q++) {
            u64 nb = ~0ull;
            if (64 * q < m) {  // (wave-uniform)
                const int i = 64 * q + lane;
                const u32 c = i < m ? base_code(b[q]) : 4u;
                bad |= c == 5;
                nb = ballot64(c >= 4);
                if (c < 4 && c > 0) atomicOr(&stream[i >> 4], c << (30 - 2 * (i & 15)));
            }
            if (lane == 0) nbp[q] = nb;
        }
        if (ballot64(bad)) {
            wflags |= ERR_BAD_BYTE;  // the call fails; the grid still reads no further bytes
            wave_sync();
            break;
        }
        wave_sync();
        // 2. k-mer hashes (~0 for k-mers with an N)
        const int nk = m - (int)k + 1;
#pragma unroll
        for (int q = 0; q < F_ROUNDS; q++) {
            if (64 * q >= nk) continue;
            const int i = 64 * q + lane;
            if (i < nk) {
                const u64 nb = funnel(nbp[q], q + 1 < F_ROUNDS ? nbp[q + 1] : ~0ull, (u32)lane);
                hh[i] = (nb & kmask) == 0 ? mix64(stream_kmer(stream, i, k)) : ~0ull;
            }
            pick[i] = 0;
        }
        wave_sync();
        // 3. window minima (~0 marks an invalid k-mer, as in k_seed_wave) and their
        // positions in order
        int nmin = 0;
        if (nk > 0) {
            const int win = nk < (int)a.w ? nk : (int)a.w;
            const int nws = nk - win + 1;
#pragma unroll 1
            for (int q = 0; q < F_ROUNDS; q++) {
                if (64 * q >= nws) break;
                const int ws = 64 * q + lane;
                if (ws < nws) {
                    const int best = window_argmin_any(hh, ws, win);
                    if (best >= 0) pick[best] = 1;
                }
            }
            wave_sync();
#pragma unroll
            for (int q = 0; q < F_ROUNDS; q++) {
                if (64 * q >= nk) continue;
                const int i = 64 * q + lane;
                const bool chosen = i < nk && pick[i];
                const u64 cm = ballot64(chosen);
                if (chosen) mpos[nmin + lanes_below(cm, lane)] = (u16)i;
                nmin += __popcll(cm);
            }
            wave_sync();
        }
        // the next read's bytes, requested ahead of the probes
        {
            const u64 nbeg = readlane64(noff, 0);
            const int nm = (int)(readlane64(noff, 1) - nbeg);
#pragma unroll
            for (int q = 0; q < F_ROUNDS; q++) {
                const int i = 64 * q + lane;
                b[q] = (more && nm <= F_MAX_M && i < nm) ? (u32)a.seq[nbeg + i] : (u32)'N';
            }
            m = more ? nm : 0;
        }
        // 4. one probe per minimizer; one hit per occurrence to its genome
        for (int t0 = 0; t0 < nmin; t0 += 64) {
            const int j = t0 + lane;
            if (j >= nmin) continue;
            const u64 v = table_lookup(a.table, a.nbuckets, stream_kmer(stream, mpos[j], k));
            count_genomes(a.occ, v, dst);
        }
        wave_sync();  // the next read reuses the wavefront's LDS
    }
    if (lane == 0 && wflags) atomicOr(a.flags, wflags);
    if (lane == 0 && fb_bases) atomicAdd(a.fb_bases, (unsigned long long)fb_bases);
    if (in_lds) {
        __syncthreads();
        for (u64 g = threadIdx.x; g < a.n_genomes; g += blockDim.x)
            if (cnt[g]) atomicAdd(&a.hits[g], cnt[g]);
    }
}

void containment(const mt_index &ix, const mt_seqs &reads, u64 *hits, hipStream_t s) {
    const u64 n = reads.n;
    if (ix.n_genomes == 0) return;
    if (n == 0) {
        MT_HIP(hipMemsetAsync(hits, 0, ix.n_genomes * sizeof(u64), s));
        return;
    }
    // A lane adds the occurrences of a k-mer one after the other; where they are many and
    // go to global counters, a wavefront per read has more of them on their way (300,000
    // reads, 3,000 genomes: strains 0.87 ms in lanes and 0.66, random ones 0.42 and 0.48).
    // In LDS they matter less than to the classification (60,000, 120,000 and 300,000
    // reads, lanes and a wavefront each: families of 10 0.15, 0.18; 0.19, 0.26 and 0.34,
    // 0.50 ms; of 50 0.31, 0.26; 0.37, 0.42 and 0.66, 0.90; k = 13, unrelated, 0.29, 0.24;
    // 0.37, 0.31 and 0.65, 0.65).
    const double x = ix.repetitive() ? extra_hits(ix, reads) / (ix.scattered() ? 10 : 200) : 0;
    const bool lanes = ix.w >= (u32)LN_MIN_W && ix.w <= (u32)LN_MAX_W &&
                       n >= (u64)((double)LANE_MIN_READS * (1 + x)) &&
                       (ix.n_genomes <= CF_LDS_GENOMES || !ix.repetitive());
    DBuf<u32> ctl(CTL_WORDS), fb_list(n), slow_list(lanes ? n : 0);
    enqueue_begin(reads.offsets, n, reads.total, ctl.p, hits, ix.n_genomes, s);
    int dev = 0, cus = 0;
    MT_HIP(hipGetDevice(&dev));
    MT_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    // the genome counters take only the LDS the index needs, so more blocks fit
    // a CU (eight wavefronts per SIMD for a few hundred genomes); enough blocks
    // to fill them
    const size_t lds = ix.n_genomes <= CF_LDS_GENOMES ? ix.n_genomes * sizeof(unsigned long long) : 0;
    const ContainArgs a{(const u8 *)reads.seq, reads.offsets, n, reads.total, ix.k, ix.w, ix.table.p, ix.nbuckets,
                        ix.occ.p, ix.n_genomes, (unsigned long long *)hits, slow_list.p, ctl.p + CTL_SLOW, fb_list.p,
                        ctl.p + CTL_FB, (unsigned long long *)(ctl.p + CTL_FB_BASES), ctl.p + CTL_FLAGS,
                        ctl.p + CTL_GATE};
    const u64 wave_blocks = std::min<u64>(grid_for(n, F_WPB), (u64)std::max(cus, 1) * (lanes ? 8 : 32));
    if (lanes) {
        const unsigned blocks = (unsigned)std::min<u64>(grid_for(n, LN_TPB), (u64)std::max(cus, 1) * 16);
        with_window(ix.w, [&](auto w) { launch_contain_lane<decltype(w)::value>(a, blocks, lds, s); });
        k_contain_wave<<<(unsigned)wave_blocks, 64 * F_WPB, lds, s>>>(a, a.slow_list, a.slow_count);
    } else {
        k_contain_wave<<<(unsigned)wave_blocks, 64 * F_WPB, lds, s>>>(a, nullptr, nullptr);
    }
    MT_HIP(hipGetLastError());
    u32 h[CTL_WORDS];
    read_back(s, ctl.p, h, sizeof h);
    check_flags(h[CTL_GATE] | h[CTL_FLAGS]);
    const u32 nfb = h[CTL_FB];
    if (nfb == 0) return;
    // longer reads: the per-stage chain, adding to hits
    const u64 bases = h[CTL_FB_BASES] | (u64)h[CTL_FB_BASES + 1] << 32;
    const Subset sub(reads, fb_list.p, nfb, bases, s);
    containment_per_stage(ix, sub.seqs, sub.src.p, reads.total, hits, s);
}

}  // namespace mt
