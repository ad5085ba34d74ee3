"""Batches called on the null stream with use_graph: a thread's batches share
one side stream (each new one cost a batch's first pass 0.3 to 0.5 ms),
several threads have one each, and results equal the eager ones in every
order of use.  Whole numbers, and reconstructions from equal ones: equal.
"""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu


def _setup(seed, shapes=((65, 33, 65), (33, 33, 129))):
    from paper_2609_00205_amd import Batch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    b = Batch(shapes, M=1, L=1)
    xs = [torch.randn(s, device="cuda", generator=gen) for s in shapes]
    tols = [p.tolmap_from_boxes([(1, 1, 1, 9, 9, 9, 1e-4)], 1e-2) for p in b.plans]
    ref = b.decompose_quantize(xs, tols)
    return b, xs, tols, [r.clone() for r in ref], [o.clone() for o in b.dequantize_recompose(ref, tols)]


def _round(b, xs, tols, ref, back):
    codes = b.decompose_quantize(xs, tols, use_graph=True)
    outs = b.dequantize_recompose(codes, tols, use_graph=True)
    # read by the null stream right after
    return all(torch.equal(c, r) for c, r in zip(codes, ref)) and all(torch.equal(o, r) for o, r in zip(outs, back))


def test_batches_of_a_thread_share_a_side_stream():
    from paper_2609_00205_amd import api
    sets = [_setup(s) for s in range(3)]
    for k in range(9):
        assert _round(*sets[k % 3]), k
    assert api._side_stream() is api._side_stream()
    first = api._side_stream()
    assert _round(*_setup(7)) and api._side_stream() is first


def test_threads_have_their_own():
    from paper_2609_00205_amd import api
    bad, streams = [], []

    def work(k):
        try:
            s = _setup(20 + k)
            streams.append(api._side_stream().cuda_stream)
            if not all(_round(*s) for _ in range(6)):
                bad.append(k)
        except Exception as e:   # noqa: BLE001
            bad.append((k, repr(e)))

    th = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not bad
    assert len(set(streams)) == 3
