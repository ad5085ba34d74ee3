"""The first level of the tail launch on either side of its size limit (27 KiB
of grid: 6912 nodes FP32, 3456 FP64), against a plan created with
BM_PLANE_PASS=0, which runs every level by itself.  The same operations in
the same order: equal bit for bit.
"""
import os

import numpy as np
import pytest
import torch

from paper_2609_00205_amd import synth

pytestmark = pytest.mark.gpu

F32, F64 = torch.float32, torch.float64


def _single(*args, **kw):
    from paper_2609_00205_amd import Plan
    old = os.environ.get("BM_PLANE_PASS")
    os.environ["BM_PLANE_PASS"] = "0"
    try:
        return Plan(*args, **kw)
    finally:
        if old is None:
            del os.environ["BM_PLANE_PASS"]
        else:
            os.environ["BM_PLANE_PASS"] = old


@pytest.mark.parametrize("shape,dt,L,M", [
    ((19, 19, 19), F32, 0, 2), ((17, 17, 23), F32, 0, 1), ((1, 83, 83), F32, 0, 3), ((15, 15, 15), F64, 0, 2),
    ((3, 33, 33), F64, 0, 2), ((17, 17, 25), F32, 0, 2), ((1, 89, 89), F32, 0, 2), ((3, 29, 93), F32, 0, 3), ((93, 1, 88), F32, 0, 1),
    ((17, 17, 33), F32, 0, 2), ((2, 64, 64), F32, 0, 3),
    ((13, 17, 17), F64, 0, 2), ((17, 17, 13), F64, 0, 3), ((1, 64, 64), F64, 0, 2), ((17, 17, 17), F64, 0, 3),
    ((65, 65, 65), F64, 1, 3),
], ids=str)
def test_either_side_of_the_limit(shape, dt, L, M):
    from paper_2609_00205_amd import Plan
    print("case", shape, dt, L, M, flush=True)
    kw = dict(dtype=dt, block=33 if L else 17, L=L, M=M)
    a, z = Plan(shape, **kw), _single(shape, **kw)
    x = torch.from_numpy(synth.gaussian_random_field(shape, 3.0, seed=74, dtype=np.float64)
                         + 0.01 * np.random.default_rng(6).standard_normal(shape)).to(dt).cuda()
    c = a.decompose(x)
    assert torch.equal(c, z.decompose(x))
    assert torch.equal(a.recompose(c), z.recompose(c))
    tol = a.tolmap_from_boxes([], 1e-3)
    q = a.decompose_quantize(x, tol)
    assert torch.equal(q, z.decompose_quantize(x, tol))
    assert torch.equal(a.dequantize_recompose(q, tol), z.dequantize_recompose(q, tol))


@pytest.mark.parametrize("shape,dt,M", [((515, 131, 129), F32, 1), ((1025, 145, 145), F32, 2), ((700, 97, 95), F64, 1)],
                         ids=str)
def test_details_of_many_planes(shape, dt, M):
    """Details written by the plane pass's launch on grids of more than 2^19 coarse cells."""
    from paper_2609_00205_amd import Plan
    print("case", shape, dt, M, flush=True)
    kw = dict(dtype=dt, block=17, L=0, M=M)
    a, z = Plan(shape, **kw), _single(shape, **kw)
    x = torch.randn(shape, dtype=dt, device="cuda", generator=torch.Generator(device="cuda").manual_seed(33))
    c = a.decompose(x)
    assert torch.equal(c, z.decompose(x))
    assert torch.equal(a.recompose(c), z.recompose(c))
    tol = a.tolmap_from_boxes([], 1e-2)
    q = a.decompose_quantize(x, tol)
    assert torch.equal(q, z.decompose_quantize(x, tol))
    assert torch.equal(a.dequantize_recompose(q, tol), z.dequantize_recompose(q, tol))
