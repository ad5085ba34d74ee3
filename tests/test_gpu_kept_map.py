"""A map kept by a field's plan (bm_quant_prepare) and calls of the batch that
owns the plan: the batch writes its own maps' propagated tolerances and
scalar steps over the kept ones, so a later call of the plan under the kept
map builds them again.  The Python plan holds the kept tensor, whose address
is what the library knows it by.

Codes are whole numbers and the reconstructions come from equal codes and
widths: equal, no tolerance.
"""
import gc
import weakref

import pytest
import torch

pytestmark = pytest.mark.gpu


def _map(p, gen, lo):
    return 10.0 ** (torch.rand(p.block_grid, dtype=torch.float64, device="cuda", generator=gen) * 2 + lo)


@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("b,L,M", [(17, 2, 1), (9, 2, 0), (33, 2, 1), (17, 1, 2)])
def test_batch_under_another_map_drops_the_kept_one(b, L, M, use_graph):
    from paper_2609_00205_amd import Batch, Plan
    shape = (65, 65, 129)
    print("case", b, L, M, use_graph, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(shape, device="cuda", generator=gen)
    batch = Batch([shape, shape], block=b, L=L, M=M)
    p, fresh = batch.plans[0], Plan(shape, block=b, L=L, M=M)
    A, B = _map(p, gen, -3.0), _map(p, gen, -5.0)
    ref = fresh.decompose_quantize(x, A)
    back = fresh.dequantize_recompose(ref, A)
    other = batch.decompose_quantize([x, x], [B, B], use_graph=use_graph)
    for _ in range(3):                                   # (with use_graph: captured, then replayed)
        p.quant_prepare(A)
        batch.decompose_quantize([x, x], [B, B], codes=other, use_graph=use_graph)
        assert torch.equal(p.decompose_quantize(x, A), ref)
        p.quant_prepare(A)
        batch.dequantize_recompose(other, [B, B], use_graph=use_graph)
        assert torch.equal(p.dequantize_recompose(ref, A), back)
        assert torch.equal(p.quantize(p.decompose(x), A)[0], ref)
        # the kept map itself as the batch's: still kept, still right
        p.quant_prepare(A)
        assert torch.equal(batch.decompose_quantize([x, x], [A, B], use_graph=use_graph)[0], ref)
        assert torch.equal(p.decompose_quantize(x, A), ref)


def test_plan_holds_the_kept_tensor():
    from paper_2609_00205_amd import Plan
    p = Plan((33, 33, 33), block=17, L=1, M=1)
    t = p.tolmap_from_boxes([], 1e-3)
    w = weakref.ref(t)
    p.quant_prepare(t)
    del t
    gc.collect()
    assert w() is not None
    p.quant_prepare(None)
    gc.collect()
    assert w() is None
