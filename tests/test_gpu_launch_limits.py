"""Read sets whose kernels take more than 2^32 threads, which one dimension of a grid
cannot hold: four lanes for each of 2^30 blocks packed, sixteen for each of 2^28 reads
turned round, a wavefront for each of 2^26 reads' minimizers and hits.  All reads but the last are empty.
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
    if torch.cuda.mem_get_info()[0] < 150 << 30:
        pytest.skip("needs 150 GB of device memory")
    import paper_2311_02029_amd as mt_
    yield mt_
    torch.cuda.empty_cache()


def _last_of(mt, n, body):
    """n reads, the last one body and the rest empty."""
    import torch
    offs = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    offs[n] = len(body)
    return mt.DeviceSeqs(torch.from_numpy(body).cuda(), offs, n, len(body))


@pytest.fixture(scope="module")
def genome():
    return synth.ACGT[synth.random_codes(np.random.default_rng(5), 5000)].copy()


def test_pairs_of_a_set_of_2_to_30_blocks(mt, genome):
    import torch
    n = 1 << 29
    body = genome[700:850].copy()
    body[[20, 90]] = ord("N")
    reads = _last_of(mt, n, body)
    ix = mt.Index(synth.SeqSet.from_list([genome.tobytes()]), 15, 10)
    pr = torch.tensor([n - 1, 0, n - 1], dtype=torch.int32, device="cuda")
    pg = torch.zeros(3, dtype=torch.int32, device="cuda")
    pd = torch.tensor([700, 0, 100], device="cuda")
    pe = torch.full((3,), 7, dtype=torch.int16, device="cuda")
    ap, ac = ix.filter_pairs(reads, pr, pg, pd, pe)
    assert ap.cpu().tolist() == [2, 0, oracle.approx(body, genome, 100, 7)] and ac.cpu().tolist() == [1, 1, 0]


def test_both_strands_of_2_to_28_reads(mt, genome):
    n = 1 << 28
    body = np.frombuffer(genome[700:850].tobytes().translate(bytes.maketrans(b"ACGT", b"TGCA"))[::-1], np.uint8).copy()
    ix = mt.Index(synth.SeqSet.from_list([genome.tobytes()]), 15, 10)
    r = ix.classify(_last_of(mt, n, body), top_n=1, mode=mt.MT_MODE_FUSED, strands=2)
    nc, (g, d, h, a, ac) = r._cands()
    assert nc == 1
    assert mt._copy_to_host(d, 1, np.int64)[0] == 700 and mt._copy_to_host(a, 1, np.uint16)[0] == 0
    assert mt._copy_to_host(ac, 1, np.uint8)[0] == 1 and mt._copy_to_host(r._strands(), 1, np.uint8)[0] == 1
    _, (u, mu, un) = r._taxa()
    assert mt._copy_to_host(un, 1, np.uint64)[0] == n - 1 and mt._copy_to_host(u, 1, np.uint64)[0] == 1


def test_per_stage_of_2_to_27_reads(mt, genome):
    n = 1 << 27
    r = mt.Index(synth.SeqSet.from_list([genome.tobytes()]), 15, 10).classify(
        _last_of(mt, n, genome[700:850].copy()), top_n=1, mode=mt.MT_MODE_PER_STAGE)
    nc, (g, d, h, a, ac) = r._cands()
    assert nc == 1 and mt._copy_to_host(d, 1, np.int64)[0] == 700 and mt._copy_to_host(a, 1, np.uint16)[0] == 0
    _, (u, mu, un) = r._taxa()
    assert mt._copy_to_host(un, 1, np.uint64)[0] == n - 1 and mt._copy_to_host(u, 1, np.uint64)[0] == 1
