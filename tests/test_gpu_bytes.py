"""Which bytes are bases: every byte value at a place of its own in a read,
through the packing step (per-stage form, pair filter, index build) and through
the kernels that read the ASCII themselves (fused form, containment).  A, C, G,
T and N in either case are taken, as the oracle takes them; every other byte
fails the call, and the next call works.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
VALID = b"ACGTNacgtn"


@pytest.fixture(scope="module")
def mt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2311_02029_amd as mt_
    return mt_


@pytest.fixture(scope="module")
def db(mt):
    rng = np.random.default_rng(3)
    g = synth.ACGT[synth.random_codes(rng, 4000)]
    ga = synth.SeqSet.from_list([g.tobytes()])
    return dict(g=g, ix=mt.Index(ga, 15, 10), oix=oracle.Index(ga, 15, 10))


CALLS = {
    "per_stage": lambda mt, ix, r: ix.classify(r, mode=mt.MT_MODE_PER_STAGE),
    "fused": lambda mt, ix, r: ix.classify(r, mode=mt.MT_MODE_FUSED),
    "containment": lambda mt, ix, r: ix.containment(r),
    "index": lambda mt, ix, r: mt.Index(r, 15, 10),
}


def _read(db, value, m, at):
    a = np.frombuffer(db["g"][500:500 + m].tobytes(), np.uint8).copy()
    a[at] = value
    return a.tobytes()


@pytest.mark.parametrize("call", CALLS)
def test_every_other_byte_is_refused(mt, db, call):
    for value in range(256):
        if bytes([value]) in VALID:
            continue
        m = (150, 64, 33, 17, 16, 7, 200, 256)[value % 8]
        reads = synth.SeqSet.from_list([_read(db, ord("A"), 40 + value % 5, 0), _read(db, value, m, (value * 37) % m)])
        with pytest.raises(mt.MTError) as e:
            CALLS[call](mt, db["ix"], mt.to_device(reads))
        assert e.value.status == mt._abi.MT_EINVAL, value
    good = synth.SeqSet.from_list([_read(db, ord("A"), 150, 0)])
    CALLS[call](mt, db["ix"], mt.to_device(good))


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_bases_in_either_case_at_every_place(mt, db, mode):
    reads = [_read(db, v, m, at) for v in VALID for m in (1, 15, 16, 17, 63, 64, 65, 130, 150, 255, 256, 257, 300)
             for at in sorted({0, m // 2, m - 1, min(m - 1, 15), min(m - 1, 16), min(m - 1, 63), min(m - 1, 64)})]
    reads += [r.lower() for r in reads[:200]]
    rs = synth.SeqSet.from_list(reads)
    got = db["ix"].classify(mt.to_device(rs), min_hits=1, mode=mode).to_host()
    ref = db["oix"].classify(rs, 1, 3, 0, 7)
    for f in ("cand_offsets", "genome", "diag", "hits", "approx", "accept", "read_accepted", "unique", "multi"):
        assert np.array_equal(got[f], ref[f]), f


def test_complements_in_either_case_at_every_length(mt, db):
    """Both strands: pieces of 16 bytes of a read and their mirror, reads of every
    length up to 70 and around 256, lower case and N among them."""
    rng = np.random.default_rng(4)
    reads = []
    for m in [*range(0, 70), 150, 255, 256, 257, 271, 272, 273, 300, 520]:
        a = db["g"][700:700 + m].copy()
        a[rng.random(m) < 0.3] |= 0x20
        if m > 30:
            a[rng.integers(0, m)] = ord("n")
        reads.append(a.tobytes())
    rs = synth.from_reverse_strand(rng, synth.SeqSet.from_list(reads * 2), 0.5)
    for mode in (0, 1):
        got = db["ix"].classify(mt.to_device(rs), min_hits=1, mode=mode, strands=2).to_host()
        ref = db["oix"].classify(rs, 1, 3, 0, 7, strands=2)
        for f in ("cand_offsets", "genome", "diag", "hits", "approx", "accept", "strand", "unique", "multi"):
            assert np.array_equal(got[f], ref[f]), f
    bad = synth.SeqSet.from_list([reads[40], b"ACGTACGTACGTACGTAC*TACGTACGTACGT"])
    with pytest.raises(mt.MTError):
        db["ix"].classify(mt.to_device(bad), mode=1, strands=2)
