"""The lane-per-read seeding kernel, which takes read sets of 48k reads and more:
minimizer windows with and without an instance, k from 1 to 31, read lengths
around its words and its limits (192 and 320 bases), N, low-complexity reads
(equal k-mers in a window are key ties, which go to the wavefront kernel) and
databases with more locations per read than a lane lists.  Every read against
the oracle.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
N_READS = 50_000
FIELDS = ("cand_offsets", "read_accepted", "read_E", "genome", "diag", "hits", "approx", "accept", "unique", "multi")


@pytest.fixture(scope="module")
def mt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2311_02029_amd as mt_
    return mt_


@pytest.fixture(scope="module")
def db():
    """Random genomes, a family of 24 strains, and repeats: a homopolymer, a
    dinucleotide repeat and a tandem repeat of 7."""
    rng = np.random.default_rng(61)
    gen = [synth.ACGT[synth.random_codes(rng, 40_000)] for _ in range(3)]
    root = synth.random_codes(rng, 6000)
    gen += [synth.ACGT[synth.substitute(rng, root, 0.01)] for _ in range(24)]
    gen += [np.frombuffer(b"A" * 900 + b"AC" * 500 + b"ACGTTCA" * 150, np.uint8)]
    return synth.SeqSet.from_list([g.tobytes() for g in gen])


def _cut(rng, ga, n, lens, p_sub, p_n):
    """n reads of the given lengths from anywhere in the database, with errors."""
    g = rng.integers(0, ga.n, n)
    glen = ga.lengths()[g]
    lens = np.minimum(lens, glen)
    start = ga.offsets[:-1].astype(np.int64)[g] + np.floor(rng.random(n) * (glen - lens + 1)).astype(np.int64)
    offs = np.zeros(n + 1, np.uint64)
    np.cumsum(lens, out=offs[1:])
    at = np.repeat(start - offs[:-1].astype(np.int64), lens) + np.arange(int(offs[-1]))
    seq = ga.seq[at].copy()
    hit = rng.random(len(seq)) < p_sub
    seq[hit] = synth.ACGT[rng.integers(0, 4, int(hit.sum()))]
    seq[rng.random(len(seq)) < p_n] = ord("N")
    return synth.SeqSet(seq=seq, offsets=offs)


def _check(mt, ga, reads, k, w, mode=1, max_occ=0, **q):
    ix = mt.Index(ga, k, w, max_occ)
    oix = oracle.Index(ga, k, w, max_occ)
    got = ix.classify(mt.to_device(reads), mode=mode, **q).to_host()
    ref = oix.classify(reads, q.get("min_hits", 3), q.get("top_n", 3), q.get("e_mode", 0), q.get("e_value", 7),
                       strands=q.get("strands", 1))
    for f in FIELDS:
        assert np.array_equal(got[f], ref[f]), (f, k, w, q)
    assert got["unmapped"] == ref["unmapped"]
    hits = ix.containment(mt.to_device(reads)).cpu().numpy().view(np.uint64)
    assert np.array_equal(hits, oix.containment(reads)), (k, w)


@pytest.mark.parametrize("k,w", [(21, 11), (15, 10), (28, 18), (31, 20), (31, 21), (17, 3), (13, 4), (12, 5), (11, 8),
                                 (16, 16), (20, 19), (4, 12), (1, 7), (21, 60)])
def test_windows_and_kmer_lengths(mt, db, k, w):
    rng = np.random.default_rng(100 * k + w)
    reads = _cut(rng, db, N_READS, rng.integers(0, 200, N_READS), 0.01, 0.002)
    _check(mt, db, reads, k, w, max_occ=200)


@pytest.mark.parametrize("lo,hi", [(150, 150), (192, 192), (64, 64), (256, 256), (320, 320), (20, 21), (0, 340),
                                   (185, 200), (310, 330), (30, 34), (21, 21)])
def test_read_lengths(mt, db, lo, hi):
    rng = np.random.default_rng(lo + 7 * hi)
    reads = _cut(rng, db, N_READS, rng.integers(lo, hi + 1, N_READS), 0.01, 0.0 if lo == hi else 0.001)
    _check(mt, db, reads, 21, 11, max_occ=200)


@pytest.mark.parametrize("q", [dict(top_n=1), dict(top_n=8), dict(top_n=0), dict(min_hits=1), dict(e_value=0),
                               dict(e_value=15), dict(e_value=31), dict(e_mode=1, e_value=50), dict(e_mode=2, e_value=100),
                               dict(mode=2), dict(strands=2), dict(e_value=40)])
def test_queries(mt, db, q):
    rng = np.random.default_rng(5)
    reads = _cut(rng, db, N_READS, rng.integers(60, 180, N_READS), 0.02, 0.0005)
    if q.get("strands") == 2:
        reads = synth.from_reverse_strand(rng, reads, 0.5)
    _check(mt, db, reads, 21, 11, **q)


def test_low_complexity_and_whole_n_reads(mt, db):
    rng = np.random.default_rng(8)
    kinds = [b"A" * 150, b"AC" * 75, b"ACGTTCA" * 21, b"N" * 150, b"A" * 70 + b"N" * 10 + b"A" * 70, b"", b"T" * 20]
    own = [kinds[i % len(kinds)][:int(rng.integers(1, 151))] if rng.random() < 0.5 else kinds[i % len(kinds)]
           for i in range(2000)]
    reads = synth.SeqSet.concat([synth.SeqSet.from_list(own), _cut(rng, db, N_READS, np.full(N_READS, 150), 0.01, 0.0)])
    _check(mt, db, reads, 21, 11)
    _check(mt, db, reads, 5, 10, min_hits=1, max_occ=100)


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("kind", [1, 2, 3, 4])
def test_other_filters_in_every_mode(mt, db, kind, mode):
    """The filters other than the obstacle walk on reads of 0 to 340 bases (past
    the lane's length and its words), small and large read sets, one and both strands."""
    rng = np.random.default_rng(40 + kind)
    ix, oix = mt.Index(db, 21, 11, 200), oracle.Index(db, 21, 11, 200)
    for n, strands, q in ((300, 1, dict(e_value=3)), (N_READS, 1, dict(e_mode=1, e_value=50)), (5000, 2, dict(e_value=40))):
        reads = _cut(rng, db, n, rng.integers(0, 341, n), 0.02, 0.001)
        got = ix.classify(mt.to_device(reads), mode=mode, filter_kind=kind, strands=strands, **q).to_host()
        ref = oix.classify(reads, 3, 3, q.get("e_mode", 0), q["e_value"], filter_kind=kind, strands=strands)
        for f in FIELDS:
            assert np.array_equal(got[f], ref[f]), (f, n, strands)


@pytest.mark.parametrize("strands", [1, 2])
@pytest.mark.parametrize("lo,hi,q,fused", [(100, 540, dict(e_value=7), True), (100, 560, dict(e_value=7), False),
                                           (60, 140, dict(e_value=31), True), (60, 140, dict(e_value=32), False),
                                           (300, 300, dict(e_mode=1, e_value=100), True),
                                           (310, 330, dict(e_mode=2, e_value=101), False)])
def test_other_filters_go_per_stage_where_most_reads_are_left_over(mt, db, lo, hi, q, fused, strands):
    """By the mean length and its E; both routes with short and long reads among them.
    A database of many strains, whose reads have more hits than the fused form counts,
    goes per stage as well."""
    rng = np.random.default_rng(lo + hi)
    n = 1501
    db = synth.SeqSet.from_list([db.get(i) for i in range(3)])
    reads = _cut(rng, db, n, np.linspace(lo, hi, n).astype(np.int64), 0.01, 0.001)
    reads = synth.SeqSet.from_list([reads.get(i) for i in rng.permutation(n)])
    ix, oix = mt.Index(db, 21, 11, 200), oracle.Index(db, 21, 11, 200)
    for kind in range(1, 5):
        ref = oix.classify(reads, 3, 3, q.get("e_mode", 0), q["e_value"], filter_kind=kind, strands=strands)
        for mode in range(3):
            got = ix.classify(mt.to_device(reads), mode=mode, filter_kind=kind, strands=strands, **q).to_host()
            assert (mt.last_stats()["fused_reads"] > 0) == fused, (kind, mode)
            for f in FIELDS:
                assert np.array_equal(got[f], ref[f]), (f, kind, mode)
    if strands == 1 and fused:
        many = synth.SeqSet.from_list([synth.ACGT[synth.substitute(rng, synth.random_codes(np.random.default_rng(1), 6000),
                                                                   0.002)].tobytes() for _ in range(60)])
        reads = _cut(rng, many, n, np.full(n, 300), 0.01, 0.001)
        got = mt.Index(many, 21, 11).classify(mt.to_device(reads), filter_kind=4).to_host()
        assert mt.last_stats()["fused_reads"] == 0
        ref = oracle.Index(many, 21, 11).classify(reads, 3, 3, 0, 7, filter_kind=4)
        for f in FIELDS:
            assert np.array_equal(got[f], ref[f]), f


@pytest.mark.parametrize("strands", [1, 2])
@pytest.mark.parametrize("hi", [400, 1200])
def test_other_filters_served_short_and_long(mt, db, hi, strands):
    rng = np.random.default_rng(hi)
    ix, oix = mt.Index(db, 21, 11, 200), oracle.Index(db, 21, 11, 200)
    sets = [_cut(rng, db, 500, rng.integers(80, hi, 500), 0.01, 0.001) for _ in range(4)]
    with mt.Server(ix) as server:
        ids = [server.submit(s, filter_kind=1 + i, strands=strands) for i, s in enumerate(sets)]
        for i, (s, rid) in enumerate(zip(sets, ids)):
            got = server.wait(rid).to_host()
            ref = oix.classify(s, 3, 3, 0, 7, filter_kind=1 + i, strands=strands)
            for f in FIELDS:
                assert np.array_equal(got[f], ref[f]), (f, i)


@pytest.mark.parametrize("n", [400, N_READS])
def test_seed_hits_counted_in_every_form(mt, db, n):
    """Work counts: the hits of a classification are those of the containment search over
    the same reads, whatever the form, the filter or the reads left over."""
    rng = np.random.default_rng(n)
    reads = _cut(rng, db, n, rng.integers(0, 341, n), 0.01, 0.001)
    ix = mt.Index(db, 21, 11, 20)
    want = int(oracle.Index(db, 21, 11, 20).containment(reads).sum())
    dr = mt.to_device(reads)
    minimizers = set()
    for q in (dict(), dict(top_n=0), dict(min_hits=1, top_n=8), dict(top_n=9), dict(filter_kind=1), dict(filter_kind=4, e_value=40)):
        for mode in range(3):
            ix.classify(dr, mode=mode, **q).free()
            st = mt.last_stats()
            assert st["n_hits"] == want, (q, mode)
            minimizers.add(st["n_minimizers"])
    assert len(minimizers) == 1


@pytest.mark.parametrize("family", [1, 5])
@pytest.mark.parametrize("genomes", [2045, 2050])
def test_containment_around_the_counters_in_lds(mt, genomes, family):
    """On both sides of the genomes whose counters fit LDS, distinct and repetitive."""
    rng = np.random.default_rng(genomes + family)
    gen = []
    for _ in range(genomes // family):
        root = synth.random_codes(rng, 300)
        gen += [synth.ACGT[synth.substitute(rng, root, 0.02)].tobytes() for _ in range(family)]
    ga = synth.SeqSet.from_list(gen)
    reads = _cut(rng, ga, N_READS, rng.integers(0, 200, N_READS), 0.01, 0.001)
    hits = mt.Index(ga, 15, 8).containment(mt.to_device(reads)).cpu().numpy().view(np.uint64)
    assert np.array_equal(hits, oracle.Index(ga, 15, 8).containment(reads))
