// Seed index over the reference genomes (Fig. 1 step 2a; "Reference Database
// Organisation and Index Construction & Querying").
//
// Built entirely on the device:
//   1. the genomes are packed into bit planes (kept: the filter reads its
//      reference windows from them);
//   2. every genome's minimizers (the same k, w and hash as the reads) are
//      extracted tile by tile;
//   3. each minimizer's k-mer is inserted into a bucketed open-addressing
//      table (4 slots of {k-mer, value} = one 64-byte line per bucket), a large
//      one a region of buckets at a time; k-mers occurring once keep their
//      (genome, position) inline in the slot, so the common lookup costs one
//      random 64-byte line;
//   4. the minimizers whose k-mer was there already are listed and counted per
//      slot: k-mers occurring several times point into an occurrence array,
//      k-mers occurring more than max_occ times are marked as never seeding.
// The table is sized for a load of at most 1/2 of its slots, so a lookup
// nearly always ends in its first bucket.  Buckets come from a second,
// salted hash of the k-mer (see bucket_of).
#include <algorithm>
#include <cstring>
#include <vector>

#include "index.hpp"
#include "seq.hpp"

namespace mt {

__global__ void k_genome_meta(const u64 *__restrict__ off, u64 n, const u64 *__restrict__ blk_off,
                              const u8 *__restrict__ has_n, const u32 *__restrict__ taxon, u64 *__restrict__ glen,
                              GenomeMeta *__restrict__ meta) {
    u64 g = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    u64 len = off[g + 1] - off[g];
    glen[g] = len;
    meta[g] = GenomeMeta{blk_off[g], (u32)len, taxon[g] | (has_n[g] ? 0x80000000u : 0u)};
}

// Puts k-mer x, unless it is there already, into the first empty slot from bucket
// b on.  The bucket's four keys are read together; a key never changes once set,
// so only an empty slot needs the swap.  False: x was there, in *slot.
__device__ inline bool place_kmer(u64x2 *table, u64 nbuckets, u64 b, u64 x, u64 occ, u64 *slot) {
    for (;;) {
        u64x2 *bk = table + b * 4;
        u64 key[4];
#pragma unroll
        for (int s = 0; s < 4; s++) key[s] = __hip_atomic_load(&bk[s].lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int s = 0; s < 4; s++) {
            u64 cur = key[s];
            if (cur == SLOT_EMPTY_KEY) {
                cur = atomicCAS((unsigned long long *)&bk[s].lo, (unsigned long long)SLOT_EMPTY_KEY,
                                (unsigned long long)x);
                if (cur == SLOT_EMPTY_KEY) {
                    bk[s].hi = occ;
                    return true;
                }
            }
            if (cur == x) {
                *slot = b * 4 + s;
                return false;
            }
        }
        b = (b + 1 == nbuckets) ? 0 : b + 1;
    }
}

// Every minimizer claims its k-mer's slot: the thread that brings a k-mer first
// writes its (genome, position) into the slot, later ones of the same k-mer go
// on the duplicate list (slot and occurrence).  The list takes one atomic per
// block of INS_ITEMS * INS_TPB minimizers and the number of distinct k-mers is
// what is not on it: a counter that every first insertion adds to serialises
// the whole kernel on one address (500 Mbp, 83M minimizers: 84.8 ms with that
// counter, 7.3 ms without).  Bound by the random table lines: a read and a
// compare-and-swap of one 64-byte bucket each.
constexpr int INS_TPB = 256, INS_ITEMS = 4;

__global__ __launch_bounds__(INS_TPB) void k_insert(const u64 *__restrict__ xs, const u32 *__restrict__ gs,
                                                    const u32 *__restrict__ ps, u64 n, u64x2 *table, u64 nbuckets,
                                                    u64 *__restrict__ dup_slot, u64 *__restrict__ dup_occ,
                                                    unsigned long long *__restrict__ n_dups) {
    __shared__ u64 first;
    u64 slot[INS_ITEMS];
    u32 mine = 0;
    const u64 base = (u64)blockIdx.x * (INS_TPB * INS_ITEMS) + threadIdx.x;
#pragma unroll
    for (int it = 0; it < INS_ITEMS; it++) {
        const u64 i = base + (u64)it * INS_TPB;
        slot[it] = ~0ull;
        if (i >= n) continue;
        const u64 x = xs[i];
        if (!place_kmer(table, nbuckets, bucket_of(x, nbuckets), x, ((u64)gs[i] << 32) | ps[i], &slot[it])) mine++;
    }
    u32 tot;
    const u32 pre = block_exclusive_sum<INS_TPB, u32>(mine, &tot);
    if (tot == 0) return;
    if (threadIdx.x == 0) first = atomicAdd(n_dups, (unsigned long long)tot);
    __syncthreads();
    u64 o = first + pre;
#pragma unroll
    for (int it = 0; it < INS_ITEMS; it++) {
        if (slot[it] == ~0ull) continue;
        const u64 i = base + (u64)it * INS_TPB;
        dup_slot[o] = slot[it];
        dup_occ[o] = ((u64)gs[i] << 32) | ps[i];
        o++;
    }
}

// Large tables are built a region of REGION buckets at a time in LDS.  k_insert
// works the table in random order: a line read, swapped into and written back
// for each minimizer, 83M of them in 7.3 ms and 0.5 ms for the table's fill.
// Here the minimizers are first brought into the order of their regions, by two
// passes of a partition (up to PART_DIGITS ways each), and a block inserts those
// of one region into LDS and writes its 32 KB out once: 3.1 ms in all (count 0.2, move
// 0.9, count 0.2, move 0.8, build 0.9 ms, which is the copy rate).  A region
// of 512 buckets leaves five blocks to a compute unit.
constexpr u32 REGION_LOG = 9, REGION = 1u << REGION_LOG, PART_DIGITS = 1024;
constexpr int PART_TPB = 1024, PART_ITEMS = 6, PART_CHUNK = PART_TPB * PART_ITEMS;
constexpr int REG_TPB = 256, REG_ITEMS = 4;

// One partition pass: the minimizers of each segment, by a digit of their region.
// A chunk (of one segment) is a block's work; counts and their prefix sums lie
// segment by segment, digit by digit, chunk by chunk.
struct PartPass {
    const u64 *seg_start, *chunk_off;  // n_seg + 1 each
    u32 n_seg, shift, mask, digits;    // digit = (region >> shift) & mask, below digits
    u64 nbuckets;
};

struct PartChunk {
    u64 at;      // of the chunk's first count
    u64 stride;  // from a digit's count to the next one's: the segment's chunks
    u64 first;   // minimizer
    u32 n;       // minimizers (0: no such chunk)
};

__device__ inline u32 part_digit(const PartPass &a, u64 x) {
    return (u32)(bucket_of(x, a.nbuckets) >> (REGION_LOG + a.shift)) & a.mask;
}

__device__ inline PartChunk part_chunk(const PartPass &a) {
    const u64 c = blockIdx.x;
    PartChunk r{0, 0, 0, 0};
    if (c >= a.chunk_off[a.n_seg]) return r;
    u32 lo = 0, hi = a.n_seg;  // the last segment with chunk_off <= c (and, so, with chunks)
    while (hi - lo > 1) {
        const u32 mid = (lo + hi) / 2;
        if (a.chunk_off[mid] <= c) lo = mid; else hi = mid;
    }
    const u64 c0 = a.chunk_off[lo], e = a.seg_start[lo + 1];
    r.stride = a.chunk_off[lo + 1] - c0;
    r.at = c0 * a.digits + (c - c0);
    r.first = a.seg_start[lo] + (c - c0) * PART_CHUNK;
    r.n = (u32)(e - r.first < (u64)PART_CHUNK ? e - r.first : (u64)PART_CHUNK);
    return r;
}

// Starts of the segments (every stride-th of scanned; one segment if it is null)
// and the chunks before each.
__global__ __launch_bounds__(PART_DIGITS) void k_part_segments(const u64 *__restrict__ scanned, u64 stride, u32 n_seg,
                                                               u64 n, u64 *__restrict__ seg_start,
                                                               u64 *__restrict__ chunk_off) {
    const u32 d = threadIdx.x;
    u64 a = 0, chunks = 0;
    if (d < n_seg) {
        a = scanned ? scanned[d * stride] : 0;
        const u64 e = d + 1 < n_seg ? scanned[(d + 1) * stride] : n;
        chunks = (e - a + PART_CHUNK - 1) / PART_CHUNK;
    }
    u64 tot;
    const u64 before = block_exclusive_sum<PART_DIGITS, u64>(chunks, &tot);
    if (d < n_seg) {
        seg_start[d] = a;
        chunk_off[d] = before;
    }
    if (d == 0) {
        seg_start[n_seg] = n;
        chunk_off[n_seg] = tot;
    }
}

__global__ __launch_bounds__(PART_TPB) void k_part_count(PartPass a, const u64 *__restrict__ xs,
                                                         u32 *__restrict__ count) {
    __shared__ u32 h[PART_DIGITS];
    const PartChunk c = part_chunk(a);
    if (c.n == 0) return;
    h[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < PART_ITEMS; it++) {
        const u32 i = it * PART_TPB + threadIdx.x;
        if (i < c.n) atomicAdd(&h[part_digit(a, xs[c.first + i])], 1u);
    }
    __syncthreads();
    if (threadIdx.x < a.digits) count[c.at + threadIdx.x * c.stride] = h[threadIdx.x];
}

// A chunk is put in the order of its digits in LDS first, so that it leaves in
// runs (6,144 minimizers on 636 digits: 77 bytes each) and not one by one.
// kPair: the occurrences come as two arrays, genomes and positions.
template <bool kPair>
__global__ __launch_bounds__(PART_TPB) void k_part_move(PartPass a, const u64 *__restrict__ scanned,
                                                        const u64 *__restrict__ xs, const u64 *__restrict__ occ,
                                                        const u32 *__restrict__ gs, const u32 *__restrict__ ps,
                                                        u64 *__restrict__ out_x, u64 *__restrict__ out_occ) {
    static_assert(PART_TPB == PART_DIGITS, "a thread for each digit");
    __shared__ u64 buf[PART_CHUNK];
    __shared__ u64 delta[PART_DIGITS];  // from a place in the chunk to the one in the output
    __shared__ u32 h[PART_DIGITS];
    const PartChunk c = part_chunk(a);
    if (c.n == 0) return;
    const u32 tid = threadIdx.x;
    h[tid] = 0;
    __syncthreads();
    u64 v[PART_ITEMS];
    u32 pos[PART_ITEMS], dig[PART_ITEMS];
#pragma unroll
    for (int it = 0; it < PART_ITEMS; it++) {
        const u32 i = it * PART_TPB + tid;
        if (i < c.n) v[it] = xs[c.first + i];
    }
#pragma unroll
    for (int it = 0; it < PART_ITEMS; it++) {
        const u32 i = it * PART_TPB + tid;
        dig[it] = i < c.n ? part_digit(a, v[it]) : 0u;
        pos[it] = i < c.n ? atomicAdd(&h[dig[it]], 1u) : 0u;
    }
    __syncthreads();
    u32 tot;
    const u32 st = block_exclusive_sum<PART_DIGITS, u32>(h[tid], &tot);
    if (tid < a.digits) delta[tid] = scanned[c.at + tid * c.stride] - st;
    __syncthreads();
    h[tid] = st;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < PART_ITEMS; it++) {
        const u32 i = it * PART_TPB + tid;
        pos[it] += h[dig[it]];
        if (i < c.n) buf[pos[it]] = v[it];
    }
    __syncthreads();
    u64 to[PART_ITEMS];
#pragma unroll
    for (int it = 0; it < PART_ITEMS; it++) {
        const u32 i = it * PART_TPB + tid;
        to[it] = 0;
        if (i < c.n) {
            const u64 x = buf[i];
            to[it] = delta[part_digit(a, x)] + i;
            out_x[to[it]] = x;
            if constexpr (kPair) v[it] = ((u64)gs[c.first + i] << 32) | ps[c.first + i];
            else v[it] = occ[c.first + i];
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < PART_ITEMS; it++) {
        const u32 i = it * PART_TPB + tid;
        if (i < c.n) buf[pos[it]] = v[it];
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < PART_ITEMS; it++) {
        const u32 i = it * PART_TPB + tid;
        if (i < c.n) out_occ[to[it]] = buf[i];
    }
}

// A block builds one region.  Its duplicates go to the front of the region's own
// range of (out_x, out_occ), as slot and occurrence, and the minimizers that
// pass its last bucket to the end of that range, as they came; no counter is
// shared by blocks.
__global__ __launch_bounds__(REG_TPB) void k_build_regions(PartPass a, const u64 *__restrict__ scanned, u32 n_regions,
                                                           u32 sub_log, const u64 *__restrict__ xs,
                                                           const u64 *__restrict__ occ, u64x2 *__restrict__ table,
                                                           u64 *__restrict__ out_x, u64 *__restrict__ out_occ,
                                                           u64 *__restrict__ region_start, u32 *__restrict__ dups,
                                                           u32 *__restrict__ spills) {
    __shared__ u64 key[REGION * 4], val[REGION * 4];
    __shared__ u32 n_dup, n_spill;
    const u32 r = blockIdx.x, g = r >> sub_log, d = r & ((1u << sub_log) - 1);
    const u64 c0 = a.chunk_off[g], nch = a.chunk_off[g + 1] - c0;
    const u64 start = scanned[c0 * a.digits + d * nch], end = scanned[c0 * a.digits + (d + 1) * nch];
    const u64 b0 = (u64)r * REGION;
    const u32 nb = (u32)(a.nbuckets - b0 < (u64)REGION ? a.nbuckets - b0 : (u64)REGION);
    for (u32 i = threadIdx.x; i < REGION * 4; i += REG_TPB) key[i] = val[i] = ~0ull;
    if (threadIdx.x == 0) n_dup = n_spill = 0;
    __syncthreads();
    const u32 lane = threadIdx.x & 63;
    for (u64 j0 = start; j0 < end; j0 += REG_TPB * REG_ITEMS) {
        u64 x[REG_ITEMS], o[REG_ITEMS];
#pragma unroll
        for (int it = 0; it < REG_ITEMS; it++) {
            const u64 j = j0 + (u64)it * REG_TPB + threadIdx.x;
            x[it] = j < end ? xs[j] : SLOT_EMPTY_KEY;
            o[it] = j < end ? occ[j] : 0;
        }
#pragma unroll
        for (int it = 0; it < REG_ITEMS; it++) {
            u32 slot = 0;
            bool placed = x[it] == SLOT_EMPTY_KEY, dup = false;
            u32 b = placed ? nb : (u32)(bucket_of(x[it], a.nbuckets) - b0);
            for (; !placed && b < nb; b++) {
#pragma unroll
                for (u32 q = 0; q < 4; q++) {
                    if (placed) continue;
                    u64 cur = __hip_atomic_load(&key[b * 4 + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (cur == SLOT_EMPTY_KEY) {
                        cur = atomicCAS((unsigned long long *)&key[b * 4 + q], (unsigned long long)SLOT_EMPTY_KEY,
                                        (unsigned long long)x[it]);
                        if (cur == SLOT_EMPTY_KEY) {
                            val[b * 4 + q] = o[it];
                            placed = true;
                        }
                    }
                    if (cur == x[it]) {
                        slot = b * 4 + q;
                        dup = placed = true;
                    }
                }
            }
            const bool spill = !placed;
            for (int kind = 0; kind < 2; kind++) {
                const bool mine = kind ? spill : dup;
                const u64 m = __ballot(mine);
                if (m == 0) continue;
                const u32 head = (u32)__ffsll((unsigned long long)m) - 1;
                u32 at = 0;
                if (lane == head) at = atomicAdd(kind ? &n_spill : &n_dup, (u32)__popcll(m));
                at = __shfl(at, (int)head, 64) + (u32)__popcll(m & ((1ull << lane) - 1));
                if (mine) {
                    const u64 w = kind ? end - 1 - at : start + at;
                    out_x[w] = kind ? x[it] : b0 * 4 + slot;
                    out_occ[w] = o[it];
                }
            }
        }
    }
    __syncthreads();
    for (u32 i = threadIdx.x; i < nb * 4; i += REG_TPB) table[b0 * 4 + i] = u64x2{key[i], val[i]};
    if (threadIdx.x == 0) {
        region_start[r] = start;
        if (r + 1 == n_regions) region_start[n_regions] = end;
        dups[r] = n_dup;
        spills[r] = n_spill;
    }
}

// What passed the end of each region goes on in the buckets after it (a thread
// per region: one region in ten has one or two of them).  A duplicate joins those
// of its region: the front of the range grows no faster than its end is read.
__global__ void k_place_spills(u32 n_regions, u64 nbuckets, u64x2 *table, const u64 *__restrict__ region_start,
                               u64 *__restrict__ xs, u64 *__restrict__ occ, u32 *__restrict__ dups,
                               const u32 *__restrict__ spills) {
    const u32 r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_regions || spills[r] == 0) return;
    const u64 start = region_start[r], end = region_start[r + 1], after = (u64)(r + 1) * REGION;
    u64 nd = start + dups[r];
    for (u64 j = end - spills[r]; j < end; j++) {
        const u64 x = xs[j], o = occ[j];
        u64 slot;
        if (!place_kmer(table, nbuckets, after < nbuckets ? after : 0, x, o, &slot)) {
            xs[nd] = slot;
            occ[nd] = o;
            nd++;
        }
    }
    dups[r] = (u32)(nd - start);
}

// The regions' duplicates side by side: a wavefront per region.
__global__ __launch_bounds__(256) void k_gather_dups(u32 n_regions, const u64 *__restrict__ region_start,
                                                     const u64 *__restrict__ dup_off, const u64 *__restrict__ xs,
                                                     const u64 *__restrict__ occ, u64 *__restrict__ dup_slot,
                                                     u64 *__restrict__ dup_occ) {
    const u32 r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= n_regions) return;
    const u64 o = dup_off[r], n = dup_off[r + 1] - o, st = region_start[r];
    for (u64 j = threadIdx.x & 63; j < n; j += 64) {
        dup_slot[o + j] = xs[st + j];
        dup_occ[o + j] = occ[st + j];
    }
}

// A table that stays in the caches is inserted into as fast as it is partitioned,
// and with fewer launches (whole build, direct and by regions: 1.7M minimizers
// 0.36 and 0.37 ms, 3.3M 0.55 and 0.54, 6.7M 1.11 and 0.72, 667M of near-identical
// strains 121 and 93).  Two passes reach 2^20 regions.
static bool by_regions(u64 n, u64 nbuckets) {
    return n >= 3 * (1ull << 20) && nbuckets <= (1ull << 20) * REGION;
}

// Builds ix.table from the n minimizers (x, genome, position) by regions and
// returns the number of duplicates, which are left in (x, occ).  occ holds the n
// genomes and then the n positions; (tx, tocc) is room for n of each.
static u64 insert_by_regions(mt_index &ix, u64 n, u64 *x, u64 *occ, u64 *tx, u64 *tocc, hipStream_t s) {
    const u64 nbuckets = ix.nbuckets;
    const u32 n_regions = (u32)((nbuckets + REGION - 1) >> REGION_LOG);
    u32 sub_log = 0;
    while (((u64)(n_regions - 1) >> sub_log) >= PART_DIGITS || (1ull << (2 * sub_log + 2)) <= n_regions) sub_log++;
    const u32 bins = ((n_regions - 1) >> sub_log) + 1, sub = 1u << sub_log;
    DBuf<u64> region_start((u64)n_regions + 1), dup_off((u64)n_regions + 1);
    DBuf<u32> dups(n_regions), spills(n_regions);
    DBuf<u64> seg(2 * (PART_DIGITS + 1)), chunk(2 * (PART_DIGITS + 1)), scanned;
    u64 *seg2 = seg.p + PART_DIGITS + 1, *chunk2 = chunk.p + PART_DIGITS + 1;
    const u64 chunks1 = (n + PART_CHUNK - 1) / PART_CHUNK, chunks2 = n / PART_CHUNK + bins;
    const PartPass p1{seg.p, chunk.p, 1, sub_log, ~0u, bins, nbuckets};
    const PartPass p2{seg2, chunk2, bins, 0, sub - 1, sub, nbuckets};
    DBuf<u32> count(std::max(chunks1 * bins, chunks2 * sub));
    scanned.alloc(std::max(chunks1 * bins, chunks2 * sub) + 1);
    k_part_segments<<<1, PART_DIGITS, 0, s>>>(nullptr, 0, 1, n, seg.p, chunk.p);
    MT_HIP(hipGetLastError());
    k_part_count<<<grid_for(chunks1, 1), PART_TPB, 0, s>>>(p1, x, count.p);
    MT_HIP(hipGetLastError());
    scan_u32(count.p, scanned.p, chunks1 * bins, s);
    k_part_move<true><<<grid_for(chunks1, 1), PART_TPB, 0, s>>>(p1, scanned.p, x, nullptr, (const u32 *)occ,
                                                               (const u32 *)occ + n, tx, tocc);
    MT_HIP(hipGetLastError());
    k_part_segments<<<1, PART_DIGITS, 0, s>>>(scanned.p, chunks1, bins, n, seg2, chunk2);
    MT_HIP(hipGetLastError());
    MT_HIP(hipMemsetAsync(count.p, 0, chunks2 * sub * sizeof(u32), s));  // there may be fewer chunks
    k_part_count<<<grid_for(chunks2, 1), PART_TPB, 0, s>>>(p2, tx, count.p);
    MT_HIP(hipGetLastError());
    scan_u32(count.p, scanned.p, chunks2 * sub, s);
    k_part_move<false><<<grid_for(chunks2, 1), PART_TPB, 0, s>>>(p2, scanned.p, tx, tocc, nullptr, nullptr, x, occ);
    MT_HIP(hipGetLastError());
    k_build_regions<<<n_regions, REG_TPB, 0, s>>>(p2, scanned.p, n_regions, sub_log, x, occ, ix.table.p, tx, tocc,
                                                 region_start.p, dups.p, spills.p);
    MT_HIP(hipGetLastError());
    k_place_spills<<<grid_for(n_regions, 256), 256, 0, s>>>(n_regions, nbuckets, ix.table.p, region_start.p, tx, tocc,
                                                           dups.p, spills.p);
    MT_HIP(hipGetLastError());
    scan_u32(dups.p, dup_off.p, n_regions, s);
    u64 nd = 0;
    read_back(s, dup_off.p + n_regions, &nd, sizeof(u64));
    if (nd) {
        k_gather_dups<<<grid_for(n_regions, 4), 256, 0, s>>>(n_regions, region_start.p, dup_off.p, tx, tocc, x, occ);
        MT_HIP(hipGetLastError());
    }
    return nd;
}

// The duplicates of a slot are numbered in the order of their atomics.
__global__ void k_dup_rank(const u64 *__restrict__ dup_slot, u64 n_dups, u32 *__restrict__ cnt,
                           u32 *__restrict__ rank) {
    const u64 d = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (d < n_dups) rank[d] = atomicAdd(&cnt[dup_slot[d]], 1u);
}

// Length of the occurrence list of each repeated k-mer, at its first duplicate
// (0 at the others); a k-mer above max_occ gets none.
__global__ void k_dup_sizes(const u64 *__restrict__ dup_slot, const u32 *__restrict__ rank, u64 n_dups,
                            const u32 *__restrict__ cnt, u32 max_occ, u32 *__restrict__ size,
                            u32 *__restrict__ flags) {
    const u64 d = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= n_dups) return;
    u32 sz = 0;
    if (rank[d] == 0) {
        const u32 c = cnt[dup_slot[d]] + 1;
        if (!max_occ || c <= max_occ) {
            if (c > MAX_KEY_OCC) atomicOr(flags, ERR_KEY_OVERFLOW);
            sz = c;
        }
    }
    size[d] = sz;
}

// The first duplicate moves the slot's inline occurrence to the front of the
// k-mer's list and points the slot at the list (count 0 marks a k-mer above
// max_occ: never a seed).
__global__ void k_dup_heads(const u64 *__restrict__ dup_slot, const u32 *__restrict__ rank,
                            const u64 *__restrict__ start, u64 n_dups, u64x2 *__restrict__ table,
                            u64 *__restrict__ occ) {
    const u64 d = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= n_dups || rank[d] != 0) return;
    const u64 st = start[d], sz = start[d + 1] - st, s = dup_slot[d];
    if (sz) occ[st] = table[s].hi;
    table[s].hi = sz ? SLOT_MULTI | (sz << 40) | st : SLOT_MULTI;
}

__global__ void k_dup_place(const u64 *__restrict__ dup_slot, const u64 *__restrict__ dup_occ,
                            const u32 *__restrict__ rank, u64 n_dups, const u64x2 *__restrict__ table,
                            u64 *__restrict__ occ) {
    const u64 d = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= n_dups) return;
    const u64 v = table[dup_slot[d]].hi;
    if (slot_count(v)) occ[slot_start(v) + 1 + rank[d]] = dup_occ[d];
}

// How repetitive the database is, as a read of it meets it: SAMPLES runs of SAMPLE_RUN
// minimizers in a row, from tiles spread over the genomes; out receives the sums of
// their locations (genome, diagonal), of their hits, and of the minimizers.  A
// wavefront per run, which stops at SAMPLE_MOST locations and occurrences of one k-mer.
constexpr int SAMPLES = 512, SAMPLE_RUN = mt_index::SAMPLE_RUN, SAMPLE_MOST = 32, SAMPLE_SLOTS = 128, SAMPLE_WPB = 4;

__global__ __launch_bounds__(64 * SAMPLE_WPB) void k_sample_locations(
    const u64x2 *__restrict__ lohi, const u64 *__restrict__ nbp, const u64 *__restrict__ blk_off,
    const u64 *__restrict__ tile_off, const u32 *__restrict__ tile_map, u64 n, u32 k,
    const u64 *__restrict__ tile_bits, const u64x2 *__restrict__ table, u64 nbuckets, const u64 *__restrict__ occ,
    unsigned long long *__restrict__ out) {
    __shared__ u64 key_all[SAMPLE_WPB][SAMPLE_SLOTS];
    __shared__ u16 list_all[SAMPLE_WPB][SAMPLE_RUN];
    __shared__ u32 found_all[SAMPLE_WPB];
    const u32 lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    u64 *key = key_all[wid];
    for (int i = (int)lane; i < SAMPLE_SLOTS; i += 64) key[i] = ~0ull;
    if (lane == 0) found_all[wid] = 0;
    const u64 tiles = tile_off[n];
    const u64 t = tiles * ((u64)blockIdx.x * SAMPLE_WPB + wid) / SAMPLES;
    u32 nl = 0, s = 0;
    if (tiles) {
        s = tile_map[t];
        constexpr int WORDS = MIN_TILE / 64;
        for (int q = 0; q < WORDS && nl < (u32)SAMPLE_RUN; q++) {
            const u64 m = tile_bits[t * WORDS + q];
            const u32 at = nl + (u32)__popcll(m & ((1ull << lane) - 1));
            if (((m >> lane) & 1) && at < (u32)SAMPLE_RUN) list_all[wid][at] = (u16)(64 * q + lane);
            nl += (u32)__popcll(m);
        }
    }
    if (nl > (u32)SAMPLE_RUN) nl = SAMPLE_RUN;
    __syncthreads();
    u32 hits = 0;
    if (lane < nl) {
        const i64 p = (i64)(t - tile_off[s]) * MIN_TILE + list_all[wid][lane];
        const Bits64 bits = fetch_planes(lohi + blk_off[s], nbp + blk_off[s], p);
        const u64 v = table_lookup(table, nbuckets, kmer_value(bits.lo, bits.hi, k));
        if (v != SLOT_NONE) hits = slot_count(v) < (u32)SAMPLE_MOST ? slot_count(v) : (u32)SAMPLE_MOST;
        for (u32 u = 0; u < hits; u++) {
            // (the lanes pass the bound by one each at most, far from filling the slots)
            if (__hip_atomic_load(&found_all[wid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= (u32)SAMPLE_MOST) break;
            const u64 gp = (v & SLOT_MULTI) ? occ[slot_start(v) + u] : v;
            const u64 x = cand_key((u32)(gp >> 32), (i64)(u32)gp - p);
            for (u32 sl = (u32)(mix64(x) % SAMPLE_SLOTS);; sl = (sl + 1) % SAMPLE_SLOTS) {
                const u64 cur = atomicCAS((unsigned long long *)&key[sl], ~0ull, (unsigned long long)x);
                if (cur == ~0ull) atomicAdd(&found_all[wid], 1u);
                if (cur == ~0ull || cur == x) break;
            }
        }
    }
#pragma unroll
    for (int o = 32; o; o >>= 1) hits += __shfl_xor(hits, o, 64);
    __syncthreads();
    if (lane == 0 && nl) {
        atomicAdd(&out[0], (unsigned long long)found_all[wid]);
        atomicAdd(&out[1], (unsigned long long)hits);
        atomicAdd(&out[2], (unsigned long long)nl);
    }
}

void build_index(mt_index &ix, const mt_index_params &p, const mt_seqs &g, const uint32_t *taxon, uint32_t n_taxa,
                 hipStream_t s) {
    Timer tm;
    tm.begin(s);
    MT_REQUIRE(p.k >= 1 && p.k <= 31, "k must be in 1..31");
    MT_REQUIRE(p.w >= 1 && p.w <= 255, "w must be in 1..255");
    MT_REQUIRE(p.reserved == 0, "reserved field must be 0");
    MT_REQUIRE(g.n < (1ull << 31), "at most 2^31 - 1 genomes");
    MT_REQUIRE(n_taxa < (1u << 31), "at most 2^31 - 1 taxa");
    MT_REQUIRE(g.n == 0 || (g.seq && g.offsets), "null genome arrays");
    std::vector<u32> tax(g.n);
    for (u64 i = 0; i < g.n; i++) {
        tax[i] = taxon ? taxon[i] : (u32)i;
        MT_REQUIRE(tax[i] < n_taxa, "taxon id out of range");
    }
    ix.k = p.k;
    ix.w = p.w;
    ix.max_occ = p.max_occ;
    ix.n_taxa = n_taxa;
    ix.n_genomes = g.n;
    ix.total_bases = g.total;

    DBuf<u32> flags(8);  // the flags, the longest length, three 64-bit sums of k_sample_locations
    MT_HIP(hipMemsetAsync(flags.p, 0, 8 * sizeof(u32), s));
    ix.has_n.alloc(g.n);
    MT_HIP(hipMemsetAsync(ix.has_n.p, 0, g.n ? g.n : 1, s));
    pack_sequences(g, 4294901759ull, ERR_READ_TOO_LONG, "genome length must be below 2^32 - 2^16", ix.ref,
                   flags.p, ix.has_n.p, s);
    ix.taxon.alloc(g.n);
    if (g.n) MT_HIP(hipMemcpyAsync(ix.taxon.p, tax.data(), g.n * sizeof(u32), hipMemcpyHostToDevice, s));
    ix.glen.alloc(g.n);
    ix.meta.alloc(g.n);
    if (g.n) {
        k_genome_meta<<<grid_for(g.n, 256), 256, 0, s>>>(g.offsets, g.n, ix.ref.blk_off.p, ix.has_n.p, ix.taxon.p,
                                                          ix.glen.p, ix.meta.p);
        MT_HIP(hipGetLastError());
    }
    tm.mark("index_pack");

    MinimizerPlan mp;
    minimizer_plan(g, ix.ref, p.k, p.w, MIN_TILE, mp, s);
    u32 f0 = 0;
    read_back(s, flags.p, &f0, sizeof(u32));
    check_flags(f0);
    u64 n_min = 0;
    read_back(s, mp.min_off.p + mp.tiles_cap, &n_min, sizeof(u64));
    ix.n_minimizers = n_min;
    tm.mark("index_min_count");

    DBuf<u64> ex(n_min), eocc(n_min);  // eocc: the genomes and then the positions
    u32 *eg = (u32 *)eocc.p, *ep = eg + n_min;
    minimizer_emit(g, ix.ref, p.k, p.w, mp, ex.p, eg, ep, s);
    tm.mark("index_min_emit");

    u64 nbuckets = (n_min + 1) / 2;
    if (nbuckets < 1) nbuckets = 1;
    ix.nbuckets = nbuckets;
    u64 nslots = nbuckets * 4;
    ix.table.alloc(nslots);
    // Two pairs of arrays for the minimizers: the duplicates end up in one, and the
    // other's memory then serves the occurrence lists (nd < n_min, so rank and size fit
    // x's and the nd + 1 starts occ's).
    DBuf<u64> tx(n_min), tocc(n_min);
    u64 *dup_slot = tx.p, *dup_occ = tocc.p, *free_x = ex.p, *free_occ = eocc.p, nd = 0;
    if (by_regions(n_min, nbuckets)) {
        nd = insert_by_regions(ix, n_min, ex.p, eocc.p, tx.p, tocc.p, s);
        dup_slot = ex.p;
        dup_occ = eocc.p;
        free_x = tx.p;
        free_occ = tocc.p;
    } else {
        MT_HIP(hipMemsetAsync(ix.table.p, 0xFF, nslots * sizeof(u64x2), s));
        DBuf<unsigned long long> ndups(1);
        MT_HIP(hipMemsetAsync(ndups.p, 0, sizeof(u64), s));
        if (n_min) {
            k_insert<<<grid_for(n_min, INS_TPB * INS_ITEMS), INS_TPB, 0, s>>>(ex.p, eg, ep, n_min, ix.table.p, nbuckets,
                                                                              dup_slot, dup_occ, ndups.p);
            MT_HIP(hipGetLastError());
        }
        read_back(s, ndups.p, &nd, sizeof(u64));
    }
    ix.n_keys = n_min - nd;
    tm.mark("index_insert");
    // the occurrence lists of the k-mers that several minimizers brought; the
    // work is that of the duplicates, not of the table
    u64 n_multi = 0;
    if (nd) {
        DBuf<u32> cnt(nslots);
        u32 *rank = (u32 *)free_x, *size = rank + nd;
        u64 *start = free_occ;
        MT_HIP(hipMemsetAsync(cnt.p, 0, nslots * sizeof(u32), s));
        k_dup_rank<<<grid_for(nd, 256), 256, 0, s>>>(dup_slot, nd, cnt.p, rank);
        MT_HIP(hipGetLastError());
        k_dup_sizes<<<grid_for(nd, 256), 256, 0, s>>>(dup_slot, rank, nd, cnt.p, p.max_occ, size, flags.p);
        MT_HIP(hipGetLastError());
        scan_u32(size, start, nd, s);
        u32 f1 = 0;
        MT_HIP(hipMemcpyAsync(&f1, flags.p, sizeof(u32), hipMemcpyDeviceToHost, s));
        read_back(s, start + nd, &n_multi, sizeof(u64));
        check_flags(f1);
        tm.mark("index_sizes");
        ix.occ.alloc(n_multi);
        k_dup_heads<<<grid_for(nd, 256), 256, 0, s>>>(dup_slot, rank, start, nd, ix.table.p, ix.occ.p);
        MT_HIP(hipGetLastError());
        k_dup_place<<<grid_for(nd, 256), 256, 0, s>>>(dup_slot, dup_occ, rank, nd, ix.table.p, ix.occ.p);
        MT_HIP(hipGetLastError());
    } else {
        ix.occ.alloc(0);
    }
    ix.n_multi_occ = n_multi;
    if (ix.repetitive()) {
        auto *sums = (unsigned long long *)(flags.p + 2);
        k_sample_locations<<<SAMPLES / SAMPLE_WPB, 64 * SAMPLE_WPB, 0, s>>>(
            ix.ref.lohi.p, ix.ref.nb.p, ix.ref.blk_off.p, mp.tile_off.p, mp.tile_map.p, g.n, p.k, mp.tile_bits.p,
            ix.table.p, nbuckets, ix.occ.p, sums);
        MT_HIP(hipGetLastError());
        u64 h[3];
        read_back(s, sums, h, sizeof h);
        if (h[2]) {
            ix.locations = (double)h[0] / SAMPLES;
            ix.hits = (double)h[1] / (double)h[2];
        }
    }
    tm.mark("index_fill");
    MT_HIP(hipStreamSynchronize(s));
    tm.finish();
}

u64 index_device_bytes(const mt_index &ix) {
    return ix.ref.lohi.n * sizeof(u64x2) + ix.ref.nb.n * sizeof(u64) + ix.ref.blk_off.n * sizeof(u64) +
           ix.glen.n * sizeof(u64) + ix.has_n.n + ix.taxon.n * sizeof(u32) +
           ix.meta.n * sizeof(GenomeMeta) +
           ix.table.n * sizeof(u64x2) + ix.occ.n * sizeof(u64);
}

}  // namespace mt

// ---------------------------------------------------------------------- ABI --

using mt::Error;

extern "C" int mt_index_build(const mt_index_params *params, const mt_seqs *genomes,
                              const uint32_t *taxon_of_genome, uint32_t n_taxa, void *stream, mt_index **out) {
    if (!params || !genomes || !out) {
        mt::set_last_error("mt_index_build: null argument");
        return MT_EINVAL;
    }
    *out = nullptr;
    mt_index *ix = nullptr;
    try {
        ix = new mt_index();
        MT_HIP(hipGetDevice(&ix->device));
        {
            mt::CallScope scope((hipStream_t)stream);
            mt::build_index(*ix, *params, *genomes, taxon_of_genome, n_taxa, (hipStream_t)stream);
        }
        mt::pool_trim();  // the build's scratch (several times the index) is not needed again
        *out = ix;
        mt::set_last_error("");
        return MT_OK;
    } catch (const Error &e) {
        delete ix;
        mt::set_last_error(e.what());
        return e.status;
    } catch (const std::exception &e) {
        delete ix;
        mt::set_last_error(e.what());
        return MT_EINTERNAL;
    }
}

extern "C" int mt_index_free(mt_index *index) {
    delete index;
    return MT_OK;
}

extern "C" int mt_index_get_info(const mt_index *ix, mt_index_info *info) {
    if (!ix || !info) {
        mt::set_last_error("mt_index_get_info: null argument");
        return MT_EINVAL;
    }
    std::memset(info, 0, sizeof *info);
    info->n_genomes = ix->n_genomes;
    info->total_bases = ix->total_bases;
    info->n_minimizers = ix->n_minimizers;
    info->n_keys = ix->n_keys;
    info->n_slots = ix->nbuckets * 4;
    info->n_multi_occ = ix->n_multi_occ;
    info->device_bytes = mt::index_device_bytes(*ix);
    info->k = ix->k;
    info->w = ix->w;
    info->max_occ = ix->max_occ;
    info->n_taxa = ix->n_taxa;
    return MT_OK;
}
