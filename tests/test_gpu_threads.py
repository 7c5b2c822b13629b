"""Calls from more threads at once than the library has places for their counts, each
thread new, with the memory that the library caches given back in between.
"""
import threading

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def test_more_threads_than_places_for_counts():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2311_02029_amd as mt
    from paper_2311_02029_amd import _abi
    gen, reads, p = synth.workload_small(300)
    ga = gen.ascii()
    ix, dr = mt.Index(ga, p["k"], p["w"]), mt.to_device(reads)
    ref = oracle.Index(ga, p["k"], p["w"]).classify(reads, 3, 3, 0, 7)
    threads, wrong = 80, []
    start = threading.Barrier(threads)

    def call(i):
        try:
            stream = torch.cuda.Stream()
            start.wait()
            for mode in (i % 2, 1 - i % 2):
                r = ix.classify(dr, mode=mode, stream=stream)
                got = r.to_host()
                for f in ("cand_offsets", "genome", "diag", "hits", "approx", "unique", "multi"):
                    if not np.array_equal(got[f], ref[f]):
                        wrong.append((i, mode, f))
                if i % 8 == 0:
                    _abi.load().mt_trim()
        except Exception as e:  # noqa: BLE001
            wrong.append((i, repr(e)))

    for _ in range(3):
        ts = [threading.Thread(target=call, args=(i,)) for i in range(threads)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert not wrong, wrong[:5]
        _abi.load().mt_trim()
