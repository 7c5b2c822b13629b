"""Abundance over short and long candidate lists: reads with up to four
candidates are taken together, longer lists one by one.  Taxa shared by several
genomes, counters in LDS and in global memory; against the oracle, bit for bit.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_taxa", [30, 7, 5000])
@pytest.mark.parametrize("top_n", [1, 3, 4, 5, 8, 0])
def test_lists_around_four_candidates(top_n, n_taxa):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2311_02029_amd as mt
    rng = np.random.default_rng(23)
    gen = synth.make_strain_genomes(rng, 5, 8000, 6, p_div=(0.001, 0.02))
    ga = gen.ascii()
    taxon = (np.arange(gen.n) * 7919 % n_taxa).astype(np.uint32)
    reads, _ = synth.make_reads(rng, gen, rng.integers(60, 150, 6000), 0.004, 0.0005)
    ix = mt.Index(ga, 15, 10, taxon=taxon, n_taxa=n_taxa)
    oix = oracle.Index(ga, 15, 10, taxon=taxon, n_taxa=n_taxa)
    ref = oix.classify(reads, 2, top_n, 0, 7)
    want, want_ab, want_kept = oracle.abundance(ref, taxon, n_taxa)
    for mode in (0, 1):
        res = ix.classify(mt.to_device(reads), min_hits=2, top_n=top_n, mode=mode)
        counts, ab, kept = ix.abundance(res)
        assert np.array_equal(counts.cpu().numpy().view(np.uint64), want) and kept == want_kept
        assert np.array_equal(ab.cpu().numpy(), want_ab)
