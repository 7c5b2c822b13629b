// Read classification: the result handle and the per-stage / fused drivers.
#pragma once

#include "index.hpp"

namespace mt {
// One of a result's arrays, inside one of its two blocks.
template <class T>
struct Arr {
    T *p = nullptr;
};
}  // namespace mt

struct mt_result {
    mt::u64 n_reads = 0, n_cands = 0, cap = 0;
    mt::u32 n_taxa = 0;
    // One block holds the arrays whose sizes the reads and the index give, one the
    // candidate arrays (capacity cap): two allocations a result, and the counters
    // (uniq, multi, unmapped, back to back) are cleared at once.
    mt::DBuf<mt::u8> reads_block, cands_block;
    mt::Arr<mt::u64> uniq, multi;       // n_taxa
    mt::Arr<mt::u64> unmapped;          // 1
    mt::Arr<mt::u64> cand_off;          // n_reads + 1
    mt::Arr<mt::u16> read_E;            // n_reads
    mt::Arr<mt::u8> read_accepted;      // n_reads
    mt::Arr<mt::i64> diag;              // candidates
    mt::Arr<mt::u32> genome, hits;
    mt::Arr<mt::u16> approx;
    mt::Arr<mt::u8> accept;
    mt::Arr<mt::u8> strand;             // both-strand results only (else null)
    void alloc_reads(mt::u64 n, mt::u32 taxa);
    void alloc_cands(mt::u64 c, bool strands = false);
    mt::u64 n_counters() const { return 2 * (mt::u64)n_taxa + 1; }  // at uniq.p
    // Served results live in host memory (the DBufs above stay empty).
    bool on_host = false;
    struct Host {
        std::vector<mt::u64> cand_off;
        std::vector<mt::u8> read_accepted;
        std::vector<mt::u16> read_E;
        std::vector<mt::u32> genome;
        std::vector<mt::i64> diag;
        std::vector<mt::u32> hits;
        std::vector<mt::u16> approx;
        std::vector<mt::u8> accept;
        std::vector<mt::u8> strand;   // both-strand results only (else empty)
        std::vector<mt::u64> counts;  // unique[n_taxa], multi[n_taxa], unmapped
    } h;
    mt::u64 submit_ns = 0, done_ns = 0;
};

namespace mt {

// Per-call read state shared by both execution forms.
struct ReadBatch {
    u64 n = 0;
    DBuf<u32> flags;   // validation flags, longest read
    DBuf<u16> read_E;  // E per read
    DBuf<u8> has_n;    // 1 if the read has an N
    PackedSeqs planes; // read bit planes
    // src, src_total: a subset that was not gathered, see pack_sequences
    void prepare(const mt_seqs &reads, u32 e_mode, u32 e_value, hipStream_t s, const u64 *src = nullptr,
                 u64 src_total = 0);
};

// Pair lists handed to the filter kernels.
struct FilterArgs {
    const u32 *pair_read;
    const u32 *pair_genome;
    const i64 *pair_diag;
    const u16 *pair_E;   // per-pair E, or null to use read_E
    const u16 *read_E;
    const u64 *n_dev;    // pair count on the device, or null to use n_host
    u64 n_host;
    u64 n_reads;
    const u64 *read_off;  // ASCII offsets (lengths)
    const u64 *read_blk;
    const u64x2 *read_lohi;
    const u64 *read_nb;
    const u8 *read_has_n;
    u32 max_len;      // of the reads, as PackedSeqs has it
    int far_len;      // short E: reads past it take groups of lanes (set by launch_filter)
    u64 n_genomes;
    const GenomeMeta *meta;
    const u64x2 *ref_lohi;
    const u64 *ref_nb;
    u16 *approx;
    u8 *accept;
    u32 *flags;
    // the fused form: reads as ASCII instead of planes (read_off into seq, its
    // bytes seq_total), and its offsets check (nonzero: nothing is filtered)
    const u8 *seq;
    u64 seq_total;
    const u32 *gate;
};

// Filters pairs [0, n) (n = *n_dev if set, else n_host; n_cap bounds it):
// pairs are bucketed by their E (one synchronization to size the buckets),
// then each bucket runs the kernel shaped for it.  fixed_E: the E of every
// pair when the caller knows it, else -1; pairs of one short E need no buckets unless
// some of many are of long reads.
void launch_filter(const FilterArgs &a, u64 n_cap, int fixed_E, hipStream_t s, Timer *tm = nullptr);
// Pairs [0, *n_dev) of the fused form (at most cap), every E at most max_E <= 31,
// through filter kind.
void launch_filter_fused(const FilterArgs &a, u64 cap, int max_E, u32 kind, hipStream_t s);
// Pairs [0, count) through the Hamming (MT_FILTER_HAMMING), base-counting
// (MT_FILTER_BASE_COUNT), q-gram (MT_FILTER_QGRAM) or shifted Hamming (MT_FILTER_SHD)
// filter; count = *n_dev if set, else n_host, at most n.
void launch_filter_simple(const FilterArgs &a, u64 n, u32 kind, hipStream_t s);

// Filter variants per bucket (see filter.hip) and their autotuner.
void autotune_filter(const FilterArgs &a, u64 n_pairs, u32 reps, hipStream_t s);
int tune_buckets();
void tune_info(int bucket, mt_tune_bucket &out);
void tune_set(int bucket, int variant);
void tune_reset();

// Limits of the fused form: longest read, largest E, most seed hits of a read.
constexpr int FUSED_MAX_M = 320, FUSED_MAX_E = 31, FUSED_MAX_HITS = 256;
// Whether a query over these reads takes the fused form (classify.hip).
bool takes_fused(const mt_index &ix, const mt_query_params &q, const mt_seqs &reads);

void validate_query(const mt_query_params &q);
// Allocates the per-read and per-taxon arrays; the forms below clear the counters.
void mt_result_init(mt_result &res, u64 n, u32 n_taxa, hipStream_t s);
void zero_counters(mt_result &res, hipStream_t s);
void classify_per_stage(const mt_index &ix, const mt_query_params &q, const mt_seqs &reads, ReadBatch &rb,
                        mt_result &res, Timer &tm, hipStream_t s);
// Containment search: every genome's seed hits over `reads` (device, n_genomes;
// containment_per_stage adds to hits).  containment runs reads of up to 320 bases in the
// fused kernels and the rest through containment_per_stage.
void containment(const mt_index &ix, const mt_seqs &reads, u64 *hits, hipStream_t s);
void containment_per_stage(const mt_index &ix, const mt_seqs &reads, const u64 *src, u64 src_total, u64 *hits,
                           hipStream_t s);

// The per-stage form end to end: packing and validation, classify_per_stage,
// flags, candidate count.
void classify_staged(const mt_index &ix, const mt_query_params &q, const mt_seqs &reads, ReadBatch &rb,
                     mt_result &res, Timer &tm, hipStream_t s);
// Fused form.  Checks the call's flags and sets res.n_cands before it
// returns; graph = launch the sequence as one captured HIP graph.
void classify_fused(const mt_index &ix, const mt_query_params &q, const mt_seqs &reads, ReadBatch &rb,
                    mt_result &res, Timer &tm, hipStream_t s, bool graph);
// The taxon step: read_accepted and the taxon counts of res from its filtered
// candidates; gate (nullable): nonzero skips it.
void launch_reduce(mt_result &res, const mt_index &ix, const u16 *read_E, const u32 *gate, hipStream_t s);
// The taxon step of a batch that holds several requests: reads
// [slot_off[s], slot_off[s+1]) add into counts[s] = {unique[n_taxa],
// multi[n_taxa], unmapped} (device arrays; slot_off and counts on the device).
void launch_reduce_slots(const mt_result &res, const mt_index &ix, const u64 *slot_off, u32 n_slots,
                         unsigned long long *const *counts, hipStream_t s);

}  // namespace mt
