"""The filter over explicit pairs at the edges of its kernels: read lengths
around the 32- and 64-base words, E around the buckets' bounds, windows that
leave either genome end, N on both sides, pair counts around the bucketing's
blocks, one bucket or several.  Every pair against the oracle.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2311_02029_amd as mt_
    return mt_


LENGTHS = [0, 1, 5, 6, 7, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 150, 191, 192, 193, 255, 256, 257, 300, 700]
ALL_E = [0, 1, 3, 7, 8, 15, 16, 31]


@pytest.fixture(scope="module")
def case(mt):
    """Reads of every length from a genome without N, one with N and a short
    one, with errors; each at its place, shifted, off both genome ends and at
    a wrong place, under every E."""
    rng = np.random.default_rng(91)
    clean = synth.ACGT[synth.random_codes(rng, 3000)]
    dirty = synth.ACGT[synth.random_codes(rng, 3000)].copy()
    dirty[rng.random(3000) < 0.01] = ord("N")
    genomes = [clean, dirty, clean[:40], np.frombuffer(b"A" * 400, np.uint8)]
    ga = synth.SeqSet.from_list([g.tobytes() for g in genomes])
    reads, pr, pg, pd, pe = [], [], [], [], []
    for m in LENGTHS:
        for g, start in ((0, 0), (0, 1500), (0, 3000 - m), (1, 700), (2, 0), (3, 100)):
            L = len(genomes[g])
            body = genomes[g][max(0, min(start, L - m)):][:m].copy()
            if len(body) < m:
                body = np.concatenate([body, synth.ACGT[rng.integers(0, 4, m - len(body))]])
            hit = rng.random(m) < rng.choice([0.0, 0.02, 0.1])
            body[hit] = synth.ACGT[rng.integers(0, 4, int(hit.sum()))]
            if rng.random() < 0.3 and m:
                body[rng.integers(0, m)] = ord("N")
            if rng.random() < 0.5 and m > 20:  # an indel
                i = int(rng.integers(5, m - 5))
                body = np.concatenate([body[:i], body[i + 1:], synth.ACGT[rng.integers(0, 4, 1)]])
            reads.append(body.tobytes())
            for E in ALL_E:
                for gg, d in ((g, start), (g, start - 3), (g, start + 20), (0, -E - m), (0, -m // 2), (0, 2990),
                              (0, 3000 + E), (2, -5), (0, int(rng.integers(0, 2500)))):
                    pr.append(len(reads) - 1)
                    pg.append(gg)
                    pd.append(d)
                    pe.append(E)
    rs = synth.SeqSet.from_list(reads)
    arr = (np.array(pr, np.uint32), np.array(pg, np.uint32), np.array(pd, np.int64), np.array(pe, np.uint16))
    oix = oracle.Index(ga, 15, 10)
    return dict(ga=ga, ix=mt.Index(ga, 15, 10), rs=rs, dr=mt.to_device(rs), pairs=arr,
                want=[oix.filter_pairs(rs, *arr, kind=kind) for kind in range(5)])


def _run(mt, case, sel, kind=0):
    import torch
    pr, pg, pd, pe = (a[sel] for a in case["pairs"])
    ap, ac = case["ix"].filter_pairs(case["dr"], torch.from_numpy(pr.view(np.int32)).cuda(),
                                     torch.from_numpy(pg.view(np.int32)).cuda(), torch.from_numpy(pd).cuda(),
                                     torch.from_numpy(pe.view(np.int16)).cuda(), kind=kind)
    return ap.cpu().numpy().view(np.uint16), ac.cpu().numpy()


@pytest.mark.parametrize("kind", range(5))
def test_every_pair_under_every_filter(mt, case, kind):
    sel = np.arange(len(case["pairs"][0]))
    ap, ac = _run(mt, case, sel, kind)
    bad = np.flatnonzero(ap != case["want"][kind][0])
    assert len(bad) == 0, [tuple(int(a[i]) for a in case["pairs"]) for i in bad[:5]]
    assert np.array_equal(ac, case["want"][kind][1])


@pytest.mark.parametrize("E", ALL_E)
def test_one_bucket(mt, case, E):
    sel = np.flatnonzero(case["pairs"][3] == E)
    np.random.default_rng(E).shuffle(sel)
    ap, ac = _run(mt, case, sel)
    assert np.array_equal(ap, case["want"][0][0][sel]) and np.array_equal(ac, case["want"][0][1][sel])


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 512, 262_143, 262_144, 262_145, 600_001])
def test_pair_counts_around_blocks(mt, case, n):
    sel = np.random.default_rng(n).integers(0, len(case["pairs"][0]), n)
    ap, ac = _run(mt, case, sel)
    assert np.array_equal(ap, case["want"][0][0][sel]) and np.array_equal(ac, case["want"][0][1][sel])


# ------------------------------------------------------------- long pairs --

@pytest.fixture(scope="module")
def long_case(mt):
    """Long reads with E above 31: exact copies (runs past every staged segment),
    reads with errors, with one N, with a long deletion; windows past both genome
    ends, wrong places, and E on both sides of the limits of the staged bands."""
    rng = np.random.default_rng(17)
    clean = synth.ACGT[synth.random_codes(rng, 30_000)]
    dirty = synth.ACGT[synth.random_codes(rng, 20_000)].copy()
    dirty[rng.integers(0, 20_000, 15)] = ord("N")
    genomes = [clean, dirty, clean[:500]]
    ga = synth.SeqSet.from_list([g.tobytes() for g in genomes])
    reads, rows = [], []
    for m in (1, 40, 300, 1000, 1900, 2500, 2600, 5000, 9000):
        for g, start in ((0, 5000), (0, 0), (0, 30_000 - m), (1, 3000)):
            for kind in ("exact", "errors", "n", "deletion"):
                body = genomes[g][start:start + m].copy()
                if kind == "errors":
                    hit = rng.random(m) < 0.05
                    body[hit] = synth.ACGT[rng.integers(0, 4, int(hit.sum()))]
                elif kind == "n":
                    body[m // 2] = ord("N")
                elif kind == "deletion" and m > 200:
                    body = np.concatenate([body[:m // 3], body[m // 3 + 30:]])
                reads.append(body.tobytes())
                Es = (32, 100, 303, 599, 600, 601, 1439, 1440, 1441) if m <= 2600 else (32, 250, 600, 601)
                for E in Es:
                    rows.append((len(reads) - 1, g, start, E))
                rows.append((len(reads) - 1, 0, int(rng.integers(0, 20_000)), 60))
                rows.append((len(reads) - 1, g, start - 40, 50))
                rows.append((len(reads) - 1, 2, -10, 45))
                rows.append((len(reads) - 1, 0, 29_990, 77))
    rs = synth.SeqSet.from_list(reads)
    r = np.array(rows, np.int64)
    arr = (r[:, 0].astype(np.uint32), r[:, 1].astype(np.uint32), r[:, 2].copy(), r[:, 3].astype(np.uint16))
    return dict(ga=ga, ix=mt.Index(ga, 15, 10), rs=rs, dr=mt.to_device(rs), pairs=arr,
                want=[oracle.Index(ga, 15, 10).filter_pairs(rs, *arr)])


@pytest.mark.parametrize("variant", range(5))
def test_long_pairs_in_segments(mt, long_case, variant):
    mt.tune_reset()
    try:
        for bucket in range(3, 7):
            try:
                mt.tune_set(bucket, variant)
            except mt.MTError:
                pass  # past the bucket's limit: the default runs
        ap, ac = _run(mt, long_case, np.arange(len(long_case["pairs"][0])))
    finally:
        mt.tune_reset()
    bad = np.flatnonzero(ap != long_case["want"][0][0])
    assert len(bad) == 0, [tuple(int(a[i]) for a in long_case["pairs"]) + (int(ap[i]),) for i in bad[:5]]
    assert np.array_equal(ac, long_case["want"][0][1])


def test_one_long_pair_per_bucket_alone(mt, long_case):
    """A single pair leaves every other group of its wavefront without one."""
    for i in range(0, len(long_case["pairs"][0]), 97):
        sel = np.array([i])
        ap, ac = _run(mt, long_case, sel)
        assert ap[0] == long_case["want"][0][0][i], i


# ---------------------------------------------------- places outside genomes --

@pytest.mark.parametrize("kind", range(5))
def test_diagonals_to_the_ends_of_64_bits(mt, kind):
    """Any diagonal is a place; one far outside the genome matches nothing there, also
    where a sum with it would wrap (the smallest value stands for "no place" in many
    programs)."""
    rng = np.random.default_rng(23)
    clean = synth.ACGT[synth.random_codes(rng, 12_000)]
    dirty = clean.copy()
    dirty[5000] = ord("N")
    ga = synth.SeqSet.from_list([clean.tobytes(), dirty.tobytes()])
    top = 2**63 - 1
    far = [-top - 1, -top, -top + 5, -top + 70_000, -2**40, -2**33, 2**32, 2**33, 2**40, 2**57 * 3, top - 140_000,
           top - 65_600, top - 9_100, top - 1000, top - 200, top - 64, top - 7, top - 1, top]
    reads, rows = [], []
    for m in (1, 40, 150, 300, 700, 2500, 9000):
        body = clean[100:100 + m].copy()
        for with_n in (False, True):
            if with_n:
                body[m // 2] = ord("N")
            reads.append(body.tobytes())
            for E in (0, 1, 7, 15, 31, 32, 60, 700, 1500):
                rows += [(len(reads) - 1, g, d, E) for g in (0, 1) for d in far + [100]]
    rs = synth.SeqSet.from_list(reads)
    r = np.array(rows, np.int64)
    pr, pg, pe = r[:, 0].astype(np.uint32), r[:, 1].astype(np.uint32), r[:, 3].astype(np.uint16)
    near = np.clip(r[:, 2], -2**33, 2**33)  # the oracle adds to it
    want = oracle.Index(ga, 15, 10).filter_pairs(rs, pr, pg, near, pe, kind=kind)
    case = dict(ix=mt.Index(ga, 15, 10), dr=mt.to_device(rs), pairs=(pr, pg, r[:, 2].copy(), pe))
    classes = [np.flatnonzero((pe > 31) == long) for long in (False, True)]
    for sel in [np.arange(len(rows)), *classes, *(np.flatnonzero(pe == E) for E in (7, 15, 31))]:
        ap, ac = _run(mt, case, sel, kind)
        bad = np.flatnonzero(ap != want[0][sel])
        assert len(bad) == 0, [rows[sel[i]] for i in bad[:5]]
        assert np.array_equal(ac, want[1][sel])


# ------------------------------------------------ short E and longer reads --

@pytest.fixture(scope="module")
def far_case(mt):
    """Reads on both sides of the lengths that go to groups of lanes at a short E (past
    256 bases of few pairs to 1,024 of many), exact, with errors, with an N, with an indel."""
    rng = np.random.default_rng(29)
    clean = synth.ACGT[synth.random_codes(rng, 40_000)]
    dirty = clean.copy()
    dirty[rng.integers(0, 40_000, 40)] = ord("N")
    ga = synth.SeqSet.from_list([clean.tobytes(), dirty.tobytes(), clean[:900].tobytes()])
    reads, rows = [], []
    for m in (150, 255, 256, 257, 258, 259, 1000, 1023, 1024, 1025, 1088, 2500, 21_000):
        for what in ("exact", "errors", "n", "indel"):
            start = int(rng.integers(100, 40_000 - m - 100))
            body = clean[start:start + m].copy()
            if what == "errors":
                hit = rng.random(m) < 0.01
                body[hit] = synth.ACGT[rng.integers(0, 4, int(hit.sum()))]
            elif what == "n":
                body[m - 3] = ord("N")
            elif what == "indel":
                body = np.concatenate([body[:m // 3], body[m // 3 + 2:], body[:2]])
            reads.append(body.tobytes())
            for E in (0, 3, 7, 8, 15, 16, 31):
                rows += [(len(reads) - 1, g, d, E) for g, d in ((0, start), (1, start - 2), (0, 200), (2, -5), (0, 39_900))]
    rs = synth.SeqSet.from_list(reads)
    r = np.array(rows, np.int64)
    arr = (r[:, 0].astype(np.uint32), r[:, 1].astype(np.uint32), r[:, 2].copy(), r[:, 3].astype(np.uint16))
    oix = oracle.Index(ga, 15, 10)
    return dict(ga=ga, ix=mt.Index(ga, 15, 10), oix=oix, rs=rs, dr=mt.to_device(rs), pairs=arr,
                want=[oix.filter_pairs(rs, *arr)])


@pytest.mark.parametrize("variant", range(3))
@pytest.mark.parametrize("n", [0, 16_384, 16_512, 65_536, 80_000])
def test_short_E_of_longer_reads(mt, far_case, n, variant):
    total = len(far_case["pairs"][0])
    sel = np.random.default_rng(n).integers(0, total, n) if n else np.arange(total)
    mt.tune_reset()
    try:
        for bucket in range(3):
            try:
                mt.tune_set(bucket, variant)
            except mt.MTError:
                pass  # past the bucket's variants: the default runs
        ap, ac = _run(mt, far_case, sel)
        one = sel[far_case["pairs"][3][sel] == 31]  # one bucket: no pair is placed
        ap1, _ = _run(mt, far_case, one)
    finally:
        mt.tune_reset()
    bad = np.flatnonzero(ap != far_case["want"][0][0][sel])
    assert len(bad) == 0, [tuple(int(a[sel[i]]) for a in far_case["pairs"]) + (int(ap[i]),) for i in bad[:5]]
    assert np.array_equal(ac, far_case["want"][0][1][sel])
    assert np.array_equal(ap1, far_case["want"][0][0][one])


@pytest.mark.parametrize("E", [7, 15, 31])
@pytest.mark.parametrize("n", [200, 12_000])
def test_classify_longer_reads_at_a_fixed_short_E(mt, far_case, n, E):
    rng = np.random.default_rng(n + E)
    genome = far_case["ga"].get(0)
    own = []
    for m in rng.choice([150, 256, 257, 1000, 1024, 1025, 1500, 3000], n):
        s = int(rng.integers(0, 40_000 - m))
        body = np.frombuffer(genome[s:s + m], np.uint8).copy()
        hit = rng.random(m) < 0.01
        body[hit] = synth.ACGT[rng.integers(0, 4, int(hit.sum()))]
        own.append(body.tobytes())
    reads = synth.SeqSet.from_list(own)
    ref = far_case["oix"].classify(reads, 3, 3, 0, E)
    for mode in (0, 1):
        got = far_case["ix"].classify(mt.to_device(reads), mode=mode, e_value=E).to_host()
        for f in ("cand_offsets", "genome", "diag", "hits", "approx", "accept", "unique", "multi"):
            assert np.array_equal(got[f], ref[f]), (f, mode)


# ----------------------------------------------------- SHD of longer reads --

@pytest.mark.parametrize("n", [1, 63, 64, 65, 700, 5000])
def test_shd_of_reads_past_the_staged_words(mt, n):
    """A lane for each 64-base word of the reads past 320 bases, several pairs to a
    wavefront: lengths around the words, more words than lanes, empty reads, bands too
    wide for LDS, short reads among them."""
    rng = np.random.default_rng(37)
    clean = synth.ACGT[synth.random_codes(rng, 20_000)]
    dirty = clean.copy()
    dirty[rng.integers(0, 20_000, 60)] = ord("N")
    ga = synth.SeqSet.from_list([clean.tobytes(), dirty.tobytes(), clean[:900].tobytes()])
    lens = [0, 1, 64, 150, 319, 320, 321, 383, 384, 385, 575, 640, 1000, 2047, 2048, 2049, 4095, 4096, 4097, 4160, 9000]
    reads, rows = [], []
    for m in lens:
        for _ in range(2):
            start = int(rng.integers(100, 20_000 - m - 50))
            body = clean[start:start + m].copy()
            hit = rng.random(m) < 0.02
            body[hit] = synth.ACGT[rng.integers(0, 4, int(hit.sum()))]
            if m and rng.random() < 0.4:
                body[rng.integers(0, m)] = ord("N")
            reads.append(body.tobytes())
            for E in (0, 5, 31, 60) + ((15_000,) if m <= 400 else ()):
                rows += [(len(reads) - 1, g, d, E) for g, d in ((0, start), (1, start + 1), (0, 3), (2, -20), (0, 19_700))]
    r = np.array(rows, np.int64)
    sel = rng.permutation(len(r)) if n == 5000 else rng.integers(0, len(r), n)
    rs = synth.SeqSet.from_list(reads)
    arr = (r[:, 0].astype(np.uint32), r[:, 1].astype(np.uint32), r[:, 2].copy(), r[:, 3].astype(np.uint16))
    want = oracle.Index(ga, 15, 10).filter_pairs(rs, *(a[sel] for a in arr), kind=4)
    ap, ac = _run(mt, dict(ix=mt.Index(ga, 15, 10), dr=mt.to_device(rs), pairs=arr), sel, 4)
    bad = np.flatnonzero(ap != want[0])
    assert len(bad) == 0, [rows[sel[i]] + (int(ap[i]), int(want[0][i])) for i in bad[:5]]
    assert np.array_equal(ac, want[1])
