// Seed index over the reference genomes (Fig. 1 step 2a; "Reference Database
// Organisation and Index Construction & Querying").
//
// Built entirely on the device:
//   1. the genomes are packed into bit planes (kept: the filter reads its
//      reference windows from them);
//   2. every genome's minimizers (the same k, w and hash as the reads) are
//      extracted tile by tile;
//   3. each minimizer's k-mer is inserted into a bucketed open-addressing
//      table (4 slots of {k-mer, value} = one 64-byte line per bucket); k-mers
//      occurring once keep their (genome, position) inline in the slot, so the
//      common lookup costs one random 64-byte line;
//   4. the minimizers whose k-mer was there already are listed and counted per
//      slot: k-mers occurring several times point into an occurrence array,
//      k-mers occurring more than max_occ times are marked as never seeding.
// The table is sized for a load of at most 1/2 of its slots, so a lookup
// nearly always ends in its first bucket.  Buckets come from a second,
// salted hash of the k-mer (see bucket_of).
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

// Every minimizer claims its k-mer's slot: the thread that brings a k-mer first
// writes its (genome, position) into the slot, later ones of the same k-mer go
// on the duplicate list (slot and occurrence).  The list takes one atomic per
// block of INS_ITEMS * INS_TPB minimizers and the number of distinct k-mers is
// what is not on it: a counter that every first insertion adds to serialises
// the whole kernel on one address (500 Mbp, 83M minimizers: 84.8 ms with that
// counter, 7.3 ms without).  Bound by the random table lines: a read and a
// compare-and-swap of one 64-byte bucket each.  The bucket's four keys are read
// together; a key never changes once set, so only an empty slot needs the swap.
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
        u64 b = bucket_of(x, nbuckets);
        for (bool placed = false; !placed;) {
            u64x2 *bk = table + b * 4;
            u64 key[4];
#pragma unroll
            for (int s = 0; s < 4; s++) key[s] = __hip_atomic_load(&bk[s].lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int s = 0; s < 4; s++) {
                if (placed) continue;
                u64 cur = key[s];
                if (cur == SLOT_EMPTY_KEY) {
                    cur = atomicCAS((unsigned long long *)&bk[s].lo, (unsigned long long)SLOT_EMPTY_KEY,
                                    (unsigned long long)x);
                    if (cur == SLOT_EMPTY_KEY) {
                        bk[s].hi = ((u64)gs[i] << 32) | ps[i];
                        placed = true;
                    }
                }
                if (cur == x) {
                    slot[it] = b * 4 + s;
                    mine++;
                    placed = true;
                }
            }
            b = (b + 1 == nbuckets) ? 0 : b + 1;
        }
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

    DBuf<u32> flags(1);
    MT_HIP(hipMemsetAsync(flags.p, 0, sizeof(u32), s));
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
    minimizer_plan(g, ix.ref, p.k, p.w, 1024, mp, s);
    u32 f0 = 0;
    read_back(s, flags.p, &f0, sizeof(u32));
    check_flags(f0);
    u64 n_min = 0;
    read_back(s, mp.min_off.p + mp.tiles_cap, &n_min, sizeof(u64));
    ix.n_minimizers = n_min;
    tm.mark("index_min_count");

    DBuf<u64> ex(n_min);
    DBuf<u32> eg(n_min), ep(n_min);
    minimizer_emit(g, ix.ref, p.k, p.w, mp, ex.p, eg.p, ep.p, s);
    tm.mark("index_min_emit");

    u64 nbuckets = (n_min + 1) / 2;
    if (nbuckets < 1) nbuckets = 1;
    ix.nbuckets = nbuckets;
    u64 nslots = nbuckets * 4;
    ix.table.alloc(nslots);
    MT_HIP(hipMemsetAsync(ix.table.p, 0xFF, nslots * sizeof(u64x2), s));
    DBuf<u64> dup_slot(n_min), dup_occ(n_min);
    DBuf<unsigned long long> ndups(1);
    MT_HIP(hipMemsetAsync(ndups.p, 0, sizeof(u64), s));
    if (n_min) {
        k_insert<<<grid_for(n_min, INS_TPB * INS_ITEMS), INS_TPB, 0, s>>>(ex.p, eg.p, ep.p, n_min, ix.table.p,
                                                                          nbuckets, dup_slot.p, dup_occ.p, ndups.p);
        MT_HIP(hipGetLastError());
    }
    u64 nd = 0;
    read_back(s, ndups.p, &nd, sizeof(u64));
    ix.n_keys = n_min - nd;
    tm.mark("index_insert");
    // the occurrence lists of the k-mers that several minimizers brought; the
    // work is that of the duplicates, not of the table
    u64 n_multi = 0;
    if (nd) {
        DBuf<u32> cnt(nslots), rank(nd), size(nd);
        DBuf<u64> start(nd + 1);
        MT_HIP(hipMemsetAsync(cnt.p, 0, nslots * sizeof(u32), s));
        k_dup_rank<<<grid_for(nd, 256), 256, 0, s>>>(dup_slot.p, nd, cnt.p, rank.p);
        MT_HIP(hipGetLastError());
        k_dup_sizes<<<grid_for(nd, 256), 256, 0, s>>>(dup_slot.p, rank.p, nd, cnt.p, p.max_occ, size.p, flags.p);
        MT_HIP(hipGetLastError());
        scan_u32(size.p, start.p, nd, s);
        u32 f1 = 0;
        MT_HIP(hipMemcpyAsync(&f1, flags.p, sizeof(u32), hipMemcpyDeviceToHost, s));
        read_back(s, start.p + nd, &n_multi, sizeof(u64));
        check_flags(f1);
        tm.mark("index_sizes");
        ix.occ.alloc(n_multi);
        k_dup_heads<<<grid_for(nd, 256), 256, 0, s>>>(dup_slot.p, rank.p, start.p, nd, ix.table.p, ix.occ.p);
        MT_HIP(hipGetLastError());
        k_dup_place<<<grid_for(nd, 256), 256, 0, s>>>(dup_slot.p, dup_occ.p, rank.p, nd, ix.table.p, ix.occ.p);
        MT_HIP(hipGetLastError());
    } else {
        ix.occ.alloc(0);
    }
    ix.n_multi_occ = n_multi;
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
