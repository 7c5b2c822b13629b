"""The index build on databases around its block sizes: minimizers whose k-mer
is in the table already go on a duplicate list (one reservation per block of
1,024 minimizers), from which the occurrence lists are built.  The counts the
index reports against numpy's over the oracle's occurrences, and every
occurrence through the seed hits of reads cut from the genomes themselves.
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


def _genomes(kind):
    rng = np.random.default_rng(77)
    if kind == "no minimizers":
        return [b"ACGTACGT", b"NNNNNNNNNNNNNNNNNNNNNNNNNNNNNN"]
    if kind == "no duplicates":
        return [synth.ACGT[synth.random_codes(rng, 5000)].tobytes() for _ in range(3)]
    if kind == "one block":  # fewer than 1,024 minimizers, half of them duplicates
        g = synth.ACGT[synth.random_codes(rng, 2400)].tobytes()
        return [g, g]
    if kind == "many copies":  # 40 copies over several blocks, one of them reversed in order
        a, b = (synth.ACGT[synth.random_codes(rng, 3000)].tobytes() for _ in range(2))
        return [a + b] * 39 + [b + a]
    if kind == "one k-mer":  # homopolymers: a single k-mer, thousands of occurrences
        return [b"A" * 4000, b"A" * 3000 + b"C" * 2000]
    gen = synth.make_strain_genomes(rng, 3, 20_000, 4)
    return [gen.ascii().get(i) for i in range(gen.n)]


@pytest.mark.parametrize("max_occ", [0, 1, 3, 39])
@pytest.mark.parametrize("kind", ["no minimizers", "no duplicates", "one block", "many copies", "one k-mer", "strains"])
def test_index_lists_every_occurrence(mt, kind, max_occ):
    ga = synth.SeqSet.from_list(_genomes(kind))
    k, w = 15, 8
    ix, oix = mt.Index(ga, k, w, max_occ), oracle.Index(ga, k, w, max_occ)
    x = oix.occurrences()[0] if max_occ == 0 else oracle.Index(ga, k, w).occurrences()[0]
    keys, counts = np.unique(x, return_counts=True)
    info = ix.info()
    assert info["n_minimizers"] == len(x) and info["n_keys"] == len(keys)
    listed = (counts >= 2) & ((counts <= max_occ) if max_occ else True)
    assert info["n_multi_occ"] == int(counts[listed].sum())
    reads = synth.SeqSet.from_list([ga.get(g)[a:a + 120] for g in range(ga.n)
                                    for a in range(0, max(1, len(ga.get(g)) - 100), 90)])
    hits = ix.containment(mt.to_device(reads)).cpu().numpy().view(np.uint64)
    assert np.array_equal(hits, oix.containment(reads))
    got = ix.classify(mt.to_device(reads), min_hits=1, top_n=0, e_value=3).to_host()
    ref = oix.classify(reads, 1, 0, 0, 3)
    for f in ("cand_offsets", "genome", "diag", "hits", "approx"):
        assert np.array_equal(got[f], ref[f]), f


# Tables from 3 x 2^20 minimizers on are built by regions of 512 buckets; with
# w = 1 every start is a minimizer, so that small genomes reach them.
@pytest.mark.parametrize("kind", ["below", "at", "strains", "one region over full"])
def test_index_by_regions_lists_every_occurrence(mt, kind):
    rng = np.random.default_rng(78)
    least, k = 3 << 20, 17
    if kind == "strains":  # most k-mers several times
        gen = synth.make_strain_genomes(rng, 8, 500_000, 4)
        ga = synth.SeqSet.from_list([gen.ascii().get(i) for i in range(gen.n)])
    else:
        g = synth.ACGT[synth.random_codes(rng, least + k - 1)].tobytes()
        more = {"below": [g[:-1]], "at": [g],  # the last minimizer decides
                "one region over full": [g[:-1], b"A" * 300_000, b"ACG" * 60_000]}[kind]
        ga = synth.SeqSet.from_list(more)
    ix, oix = mt.Index(ga, k, 1), oracle.Index(ga, k, 1)
    keys, counts = np.unique(oix.occurrences()[0], return_counts=True)
    info = ix.info()
    assert info["n_minimizers"] == int(counts.sum()) and info["n_keys"] == len(keys)
    assert (info["n_minimizers"] >= least) == (kind != "below")
    assert info["n_multi_occ"] == int(counts[counts >= 2].sum())
    reads = synth.SeqSet.from_list([ga.get(0)[a:a + 5000] for a in range(0, len(ga.get(0)) - 5000, 4900)]
                                   + [ga.get(i)[:150] for i in range(ga.n)])
    if kind != "one region over full":  # every k-mer of the first genome has its occurrences
        hits = ix.containment(mt.to_device(reads)).cpu().numpy().view(np.uint64)
        assert np.array_equal(hits, oix.containment(reads))
    short = synth.SeqSet.from_list([ga.get(0)[a:a + 150] for a in range(0, len(ga.get(0)) - 150, 1501)])
    got = ix.classify(mt.to_device(short), min_hits=1, top_n=0, e_value=3).to_host()
    ref = oix.classify(short, 1, 0, 0, 3)
    for f in ("cand_offsets", "genome", "diag", "hits", "approx"):
        assert np.array_equal(got[f], ref[f]), f


# Minimizers are picked five windows to a thread, in tiles of 1,216 starts of long
# sequences and 256 of short ones: lengths around both, windows with an unrolled
# instance (5 to 20) and beside them.
@pytest.mark.parametrize("w", [4, 5, 6, 11, 20, 21, 255])
def test_minimizers_around_tiles(mt, w):
    rng = np.random.default_rng(79 + w)
    k = 15

    def seq(m):
        s = synth.random_codes(rng, m) % 4
        text = synth.ACGT[s].copy()
        if m > 400:  # a repeat, and an N now and then
            text[m // 2:m // 2 + 100] = np.tile(text[:5], 20)
            text[rng.integers(0, m, m // 300)] = ord("N")
        return text.tobytes()

    starts = [0, 1, 2, 4, 5, 6, w - 1, w, w + 1, 255, 256, 257, 320, 511, 512, 513, 1215, 1216, 1217, 1221,
              2431, 2432, 2433, 3648]
    ga = synth.SeqSet.from_list([seq(max(0, n) + k - 1) for n in starts])
    ix, oix = mt.Index(ga, k, w), oracle.Index(ga, k, w)
    x = oix.occurrences()[0]
    info = ix.info()
    assert info["n_minimizers"] == len(x) and info["n_keys"] == len(np.unique(x))
    for keep in (range(ga.n), [i for i in range(ga.n) if starts[i] < 514]):  # long tiles, short tiles
        reads = synth.SeqSet.from_list([ga.get(i) for i in keep])
        hits = ix.containment(mt.to_device(reads)).cpu().numpy().view(np.uint64)
        assert np.array_equal(hits, oix.containment(reads))


@pytest.mark.parametrize("w", [8, 1])  # inserted directly, and by regions
@pytest.mark.parametrize("copies", [1, 40])
def test_index_build_memory(mt, copies, w):
    """The build holds at most 48 bytes a minimizer beside the index, and less than half a
    byte a base, whether its k-mers are distinct or nearly all duplicates."""
    import torch
    rng = np.random.default_rng(80)
    g = synth.ACGT[synth.random_codes(rng, 6_000_000 // copies)].tobytes()
    ga = mt.to_device(synth.SeqSet.from_list([g] * copies))
    mt.Index(ga, 17, w).free()
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    info = mt.Index(ga, 17, w).info()
    peak = torch.cuda.max_memory_allocated() - before
    assert info["n_keys"] * copies <= info["n_minimizers"] + 1000 * copies
    assert peak <= info["device_bytes"] + 48 * info["n_minimizers"] + ga.total // 2 + (4 << 20)
