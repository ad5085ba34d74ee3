"""Propagated tolerances (Eq. 2) on either side of the number of level-2
blocks that one workgroup propagates (512), one and several levels deep,
plain and nested, a plan's and a batch's: against the minimum over the
contributing blocks taken directly.

Delta is the block's tolerance times one constant of the level: ratios equal
to a rounding of the product, 4e-16.  Codes of the batch are whole numbers:
equal.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _next(t, nested):
    """The level-(s+1) map of a level-s map: the minimum over the blocks that share a node."""
    for a in range(3):
        n = t.shape[a]
        lo = torch.full_like(t.narrow(a, 0, 1), float("inf"))
        p = torch.cat([lo, t, lo], a)                    # p[k + 1] is block k
        if nested:
            t = torch.minimum(torch.minimum(p.narrow(a, 0, n), p.narrow(a, 1, n)), p.narrow(a, 2, n))
        else:                                            # block Z spans 2Z, 2Z+1 and touches 2Z-1, 2Z+2
            idx = torch.arange(0, n, 2, device=t.device)
            t = torch.stack([p.index_select(a, idx + k) for k in range(4)]).amin(0)
    return t


@pytest.mark.parametrize("dims,b,L,nested", [
    ((16, 16, 16), 9, 2, False), ((16, 16, 18), 9, 2, False),      # 512 and 576 blocks at level 2
    ((16, 16, 16), 9, 3, False), ((16, 16, 20), 9, 3, False),      # 512 and 640
    ((8, 8, 8), 17, 2, True), ((8, 8, 9), 17, 2, True),            # 512 and 576
    ((32, 32, 32), 9, 3, False),                                   # 4096
])
def test_levels_and_batch(dims, b, L, nested):
    from paper_2609_00205_amd import Batch, Plan
    print("case", dims, b, L, nested, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(21)
    shape = tuple(n * (b - 1) + 1 for n in dims)
    p = Plan(shape, dtype=torch.float64, block=b, L=L, M=1, nested=nested)
    assert p.block_grid == dims
    bt = 10.0 ** (torch.rand(dims, dtype=torch.float64, device="cuda", generator=gen) * 4 - 5)
    delta = p.dequantize(torch.ones(p.coeff_shape, dtype=torch.int32, device="cuda"), bt)
    t = bt
    for s in range(2, L + 1):
        t = _next(t, nested)
        # a detail of level s inside every block: an odd node of its grid
        o = [slice((1 << (s - 1)) + (0 if nested else 1 << s), None, (b - 1) << (0 if nested else s - 1))] * 3
        ratio = delta[o[0], o[1], o[2]] / t
        assert ratio.shape == t.shape
        assert bool(((ratio / ratio.reshape(-1)[0] - 1).abs() <= 4e-16).all()), s
    x = torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen)
    ref = p.quantize(p.decompose(x), bt)[0]
    assert torch.equal(p.decompose_quantize(x, bt), ref)
    if b == 9 or nested:
        batch = Batch([shape, shape], dtype=torch.float64, block=b, L=L, M=1, nested=nested)
        for c in batch.decompose_quantize([x, x], [bt, bt]):
            assert torch.equal(c, ref)
