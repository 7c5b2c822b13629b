"""The lane-per-read seeding kernel on the databases that it is chosen for: distinct
genomes (from 48k reads on) and small families of strains (from more reads on, by the
hits that their reads have). Databases that are more repetitive take the wavefront
kernel. Windows, k, read lengths around the kernel's words and limits, N and queries;
every read against the oracle.
"""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_lane import FIELDS, _cut

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2311_02029_amd as mt_
    return mt_


def _database(family):
    """Genomes of 240 kb in families, a repeat of 7 and a homopolymer at the end of one."""
    rng = np.random.default_rng(70 + family)
    gen = []
    for _ in range(8):
        root = synth.random_codes(rng, 30_000 // family)
        gen += [synth.ACGT[synth.substitute(rng, root, 0.03)].tobytes() if family > 1 else synth.ACGT[root].tobytes()
                for _ in range(family)]
    gen[0] += b"ACGTTCA" * 40 + b"A" * 300
    return synth.SeqSet.from_list(gen)


@pytest.fixture(scope="module")
def dbs():
    return {f: _database(f) for f in (1, 3, 6, 16)}


READS = {1: 50_000, 3: 90_000, 6: 200_000, 16: 90_000}  # past the line, or (16) never


def _check(mt, ga, reads, k, w, max_occ=0, mode=1, **q):
    ix, oix = mt.Index(ga, k, w, max_occ), oracle.Index(ga, k, w, max_occ)
    dr = mt.to_device(reads)
    got = ix.classify(dr, mode=mode, **q).to_host()
    ref = oix.classify(reads, q.get("min_hits", 3), q.get("top_n", 3), q.get("e_mode", 0), q.get("e_value", 7),
                       strands=q.get("strands", 1))
    for f in FIELDS:
        assert np.array_equal(got[f], ref[f]), (f, k, w, q)
    assert got["unmapped"] == ref["unmapped"]
    hits = ix.containment(dr).cpu().numpy().view(np.uint64)
    assert np.array_equal(hits, oix.containment(reads)), (k, w)


@pytest.mark.parametrize("k,w", [(21, 11), (15, 10), (28, 18), (31, 20), (31, 21), (17, 3), (13, 4), (16, 16), (20, 19),
                                 (12, 8), (1, 7)])
def test_windows_and_kmer_lengths(mt, dbs, k, w):
    rng = np.random.default_rng(100 * k + w)
    reads = _cut(rng, dbs[1], READS[1], rng.integers(0, 200, READS[1]), 0.01, 0.002)
    _check(mt, dbs[1], reads, k, w, max_occ=200)


@pytest.mark.parametrize("lo,hi", [(150, 150), (192, 192), (64, 64), (256, 256), (320, 320), (20, 21), (0, 340),
                                   (185, 200), (310, 330), (21, 21)])
def test_read_lengths(mt, dbs, lo, hi):
    rng = np.random.default_rng(lo + 7 * hi)
    reads = _cut(rng, dbs[1], READS[1], rng.integers(lo, hi + 1, READS[1]), 0.01, 0.0 if lo == hi else 0.001)
    _check(mt, dbs[1], reads, 21, 11, max_occ=200)


@pytest.mark.parametrize("family", [3, 6, 16])
@pytest.mark.parametrize("q", [dict(), dict(top_n=8), dict(top_n=0), dict(min_hits=1, top_n=1), dict(e_mode=1, e_value=50),
                               dict(mode=2), dict(strands=2), dict(e_value=31)])
def test_families(mt, dbs, family, q):
    rng = np.random.default_rng(5 + family)
    n = READS[family]
    reads = _cut(rng, dbs[family], n, rng.integers(60, 200, n), 0.02, 0.0005)
    if q.get("strands") == 2:
        reads = synth.from_reverse_strand(rng, reads, 0.5)
    _check(mt, dbs[family], reads, 21, 11, **q)
