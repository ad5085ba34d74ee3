"""The tail launch of the global levels (the last levels, whose grids fit one
workgroup, in one launch each way), and details written by the plane pass's
launch, against the launches they replace: a plan
created with BM_PLANE_PASS=0 runs every level by itself, from its own copy
of the input.  Coefficients, reconstructions and codes must be equal bit for
bit: a first tail level below and at level 1, padded and unpadded inputs,
axes that do not coarsen, one tail level and eight, grids on both sides of
the node limit, levels after fused and unfused block levels.
"""
import os

import numpy as np
import pytest
import torch

from paper_2609_00205_amd import synth

pytestmark = pytest.mark.gpu

CASES = [((65, 65, 65), 17, 0, 6), ((17, 17, 17), 17, 0, 4), ((17, 17, 19), 17, 0, 3), ((15, 16, 14), 17, 0, 3),
         ((3, 3, 3), 17, 0, 1), ((5, 9, 33), 17, 0, 3), ((2, 17, 40), 17, 0, 4), ((65, 1, 65), 17, 0, 6),
         ((2, 2, 95), 17, 0, 6), ((129, 129, 129), 17, 1, 4), ((41, 50, 61), 9, 1, 4), ((129, 65, 70), 33, 1, 3)]


def _ids(c):
    return "x".join(map(str, c[0])) + f"-b{c[1]}-L{c[2]}M{c[3]}"


def _plans(shape, b, L, M, dt):
    from paper_2609_00205_amd import Plan
    a = Plan(shape, dtype=dt, block=b, L=L, M=M)
    old = os.environ.get("BM_PLANE_PASS")
    os.environ["BM_PLANE_PASS"] = "0"
    try:
        z = Plan(shape, dtype=dt, block=b, L=L, M=M)
    finally:
        if old is None:
            del os.environ["BM_PLANE_PASS"]
        else:
            os.environ["BM_PLANE_PASS"] = old
    return a, z


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["float32", "float64"])
@pytest.mark.parametrize("case", CASES, ids=_ids)
def test_tail_equals_single_levels(case, dt):
    shape, b, L, M = case
    print("case", _ids(case), dt, flush=True)
    a, z = _plans(shape, b, L, M, dt)
    rng = np.random.default_rng(5)
    x = synth.gaussian_random_field(shape, 3.0, seed=72, dtype=np.float64) + 0.01 * rng.standard_normal(shape)
    x = torch.from_numpy(x).to(dt).cuda()
    x0 = x.clone()
    ca, cz = a.decompose(x), z.decompose(x)
    assert torch.equal(ca, cz), float((ca - cz).abs().max())
    c = ca + torch.from_numpy(0.01 * rng.standard_normal(tuple(ca.shape))).to(dt).cuda()
    ra, rz = a.recompose(c), z.recompose(c)
    assert torch.equal(ra, rz), float((ra - rz).abs().max())
    sc = float(x.abs().max())
    tol = a.tolmap_from_boxes([], 1e-3 * sc)
    qa, qz = a.decompose_quantize(x, tol), z.decompose_quantize(x, tol)
    assert torch.equal(qa, qz), int((qa != qz).sum())
    xa, xz = a.dequantize_recompose(qa, tol), z.dequantize_recompose(qa, tol)
    assert torch.equal(xa, xz), float((xa - xz).abs().max())
    assert torch.equal(x, x0)


@pytest.mark.parametrize("shape", [(17, 17, 17), (65, 33, 65)], ids=lambda s: "x".join(map(str, s)))
def test_in_place(shape):
    """Without block levels an unpadded input is read, and the result written,
    where it lies, unless it shares memory with the coefficients."""
    from paper_2609_00205_amd import Plan
    p = Plan(shape, block=17, L=0, M=2)
    x = torch.from_numpy(synth.gaussian_random_field(shape, 3.0, seed=73, dtype=np.float32)).cuda()
    c = p.decompose(x)
    y = x.clone()
    assert torch.equal(p.decompose(y, out=y), c)
    r = p.recompose(c)
    y = c.clone()
    assert torch.equal(p.recompose(y, out=y), r)
