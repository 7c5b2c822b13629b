// What the fused kernels of fused.hip (a wavefront per read, and the launches) and of
// lane.hip (a lane per read) share.  lane.hip is compiled once for each minimizer
// window, each a code object of its own: the runtime loads a code object whole at its
// first launch.
#pragma once

#include "classify.hpp"
#include "lane.hpp"

namespace mt {

constexpr int F_HIT_CAP = FUSED_MAX_HITS;  // seed hits per read (distinct locations fit the table)
constexpr int F_MAX_E = FUSED_MAX_E;       // 2E + 1 rows fit two words of the filter

enum : u32 { ST_READS, ST_BASES, ST_MINS, ST_WBLOCKS, ST_CANDS, ST_OCC, ST_HITS, ST_FB_BASES, ST_COUNT };

struct SeedArgs {
    const u8 *seq;
    const u64 *off;
    u64 n, total;
    u32 k, w, min_hits, top_n, e_mode, e_value;
    u32 ncap;  // staging slots per read: top_n, or F_MAX_TOPN when top_n = 0 (keep all)
    const u64x2 *table;
    u64 nbuckets;
    const u64 *occ;
    // staging: rank-major, slot (rank, read) at rank * n + read
    u64 *st_key;
    u32 *st_hits;
    u32 *ncand;
    u16 *read_E;
    u8 *read_n;  // 1 if the read has an N
    u32 *slow_list, *slow_count;  // reads for k_seed_wave
    u32 *fb_list, *fb_count;      // reads for the per-stage kernels
    u32 *flags;
    const u32 *gate;  // offsets check result: nonzero skips the whole launch
    u64 *stats_part;  // ST_COUNT work counts per block
};

// E of a read of m bases; ERR_E_TOO_LARGE in *flags when it passes the limit.
__device__ inline int read_threshold(const SeedArgs &a, int m, u32 *flags) {
    const u64 E = a.e_mode == MT_E_FIXED           ? a.e_value
                  : a.e_mode == MT_E_CEIL_PERMILLE ? ((u64)m * a.e_value + 999) / 1000
                                                   : ((u64)m * a.e_value) / 1000;
    if (E > 65534) *flags |= ERR_E_TOO_LARGE;
    return E > 65535 ? 65535 : (int)E;
}

__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline u64 ballot64(bool p) { return __ballot(p); }

// Value of v in lane l (l wave-uniform).
__device__ inline u64 readlane64(u64 v, int l) {
    const u32 lo = __builtin_amdgcn_readlane((u32)v, l), hi = __builtin_amdgcn_readlane((u32)(v >> 32), l);
    return ((u64)hi << 32) | lo;
}

// Number of set bits of m below this lane.
__device__ inline u32 lanes_below(u64 m, int lane) {
    return (u32)__popcll(lane ? m & ((~0ull) >> (64 - lane)) : 0ull);
}

// Appends r to a list for the lanes with `add` set, one atomic per wavefront.
__device__ inline void list_append(bool add, u64 r, int lane, u32 *list, u32 *count) {
    const u64 m = ballot64(add);
    if (!m) return;
    const int leader = __builtin_ctzll(m);
    u32 first = 0;
    if (lane == leader) first = atomicAdd(count, (u32)__popcll(m));
    first = __shfl(first, leader, 64);
    if (add) list[first + lanes_below(m, lane)] = (u32)r;
}

__device__ inline u32 wave_sum(u32 v) {
#pragma unroll
    for (int o = 32; o; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// ... and their bases to *bases.
__device__ inline void list_append(bool add, u64 r, int m, int lane, u32 *list, u32 *count,
                                   unsigned long long *bases) {
    if (!ballot64(add)) return;
    list_append(add, r, lane, list, count);
    const u32 t = wave_sum(add ? (u32)m : 0u);
    if (lane == 0) atomicAdd(bases, (unsigned long long)t);
}

// Arguments of the containment kernels.
struct ContainArgs {
    const u8 *seq;
    const u64 *off;
    u64 n, total;
    u32 k, w;
    const u64x2 *table;
    u64 nbuckets;
    const u64 *occ;
    u64 n_genomes;
    unsigned long long *hits;
    u32 *slow_list, *slow_count;  // reads for k_contain_wave
    u32 *fb_list, *fb_count;
    unsigned long long *fb_bases;
    u32 *flags;
    const u32 *gate;  // offsets check result: nonzero skips the whole launch
};

constexpr u64 CF_LDS_GENOMES = 2048;  // 64-bit counters, at most 16 KB per block

// One hit per occurrence of a probed k-mer (v: its slot value).
__device__ inline void count_genomes(const u64 *__restrict__ occ, u64 v, unsigned long long *dst) {
    if (v == SLOT_NONE) return;
    if (!(v & SLOT_MULTI)) {
        atomicAdd(&dst[v >> 32], 1ull);
        return;
    }
    const u32 c = slot_count(v);  // 0 for a k-mer above max_occ
    const u64 st = slot_start(v);
    for (u32 u = 0; u < c; u++) atomicAdd(&dst[occ[st + u] >> 32], 1ull);
}

// k_seed_lane and k_contain_lane of window W (rep: a list for more locations a read;
// lds: bytes of the genome counters).
template <int W>
void launch_seed_lane(const SeedArgs &a, bool rep, unsigned blocks, hipStream_t s);
template <int W>
void launch_contain_lane(const ContainArgs &a, unsigned blocks, size_t lds, hipStream_t s);

}  // namespace mt
