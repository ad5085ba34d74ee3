"""Lanes of the block kernels: groups of two 17^3 (FP32) and six 9^3 blocks
with every kind of remainder, against the FP64 oracle; and the error flag of
the fused quantizer, which is formed apart from the codes, against the
unfused quantizer for a bad value at each kind of node (block corner, shared
face, even and odd columns and planes, the far faces).

Bar: 1e-6 (FP32) and 1e-13 (FP64) of max|x| per direction.
"""
import numpy as np
import pytest
import torch

from oracle import mgard
from paper_2609_00205_amd import synth

pytestmark = pytest.mark.gpu

TOL = {torch.float32: 1e-6, torch.float64: 1e-13}
SHAPES = [((9, 9, 9), 9), ((9, 9, 41), 9), ((9, 17, 49), 9), ((25, 17, 57), 9),     # 1, 5, 12, 42 blocks
          ((17, 17, 17), 17), ((17, 17, 33), 17), ((17, 49, 17), 17), ((33, 33, 49), 17)]   # 1, 2, 3, 12


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["float32", "float64"])
@pytest.mark.parametrize("M", [0, 1])
@pytest.mark.parametrize("shape,b", SHAPES, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_block_groups(shape, b, M, dt):
    from paper_2609_00205_amd import Plan
    print("case", shape, b, M, dt, flush=True)
    x = synth.gaussian_random_field(shape, 3.0, seed=5, dtype=np.float64)
    x = x.astype(np.float32 if dt == torch.float32 else np.float64)
    p = Plan(shape, dtype=dt, block=b, L=1, M=M)
    sc = float(np.abs(x).max())
    c = p.decompose(torch.from_numpy(x).cuda())
    ref = mgard.decompose(x.astype(np.float64), b, 1, M)
    assert float(np.abs(c.double().cpu().numpy() - ref).max()) <= TOL[dt] * sc
    back = mgard.recompose(c.double().cpu().numpy(), shape, b, 1, M)
    assert float(np.abs(p.recompose(c).double().cpu().numpy() - back).max()) <= TOL[dt] * sc


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["float32", "float64"])
@pytest.mark.parametrize("nested", [False, True], ids=["plain", "nested"])
@pytest.mark.parametrize("shape,b", [((20, 37, 70), 9), ((33, 33, 70), 9), ((40, 70, 33), 17), ((98, 33, 40), 17)],
                         ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_blocks_in_the_padding(shape, b, nested, dt):
    """Two block levels pad to whole level-2 blocks: level-1 blocks past the
    logical dims along one axis or several write nothing."""
    from paper_2609_00205_amd import Plan
    if nested and b == 9:
        pytest.skip("the nested pair starts with 17-node blocks")
    print("case", shape, b, nested, dt, flush=True)
    x = synth.gaussian_random_field(shape, 3.0, seed=6, dtype=np.float64)
    x = x.astype(np.float32 if dt == torch.float32 else np.float64)
    p = Plan(shape, dtype=dt, block=b, L=2, M=0, nested=nested)
    guard = torch.full((x.size + 64,), 7.0, dtype=dt, device="cuda")
    out = guard[:x.size].view(shape)
    c = p.decompose(torch.from_numpy(x).cuda())
    p.recompose(c, out=out)
    sc = float(np.abs(x).max())
    assert float(np.abs(out.double().cpu().numpy() - x).max()) <= 4 * TOL[dt] * sc   # (both directions, two levels)
    assert torch.all(guard[x.size:] == 7.0)


NODES = [(0, 0, 0), (16, 16, 16), (32, 32, 32), (2, 2, 2), (1, 2, 2), (2, 3, 4), (5, 7, 9), (31, 16, 5), (16, 3, 32),
         (32, 2, 2)]


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 3e9])
@pytest.mark.parametrize("M", [0, 1])
def test_error_flag(bad, M):
    from paper_2609_00205_amd import Plan
    p = Plan((33, 33, 33), block=17, L=1, M=M)
    tol = p.tolmap_from_boxes([], 1.0)
    for node in NODES:
        print("case", bad, M, node, flush=True)
        x = torch.zeros(33, 33, 33, device="cuda")
        x[node] = bad

        def run(f):
            try:
                f()
            except Exception as e:   # noqa: BLE001 (either raises the library's error or returns)
                return type(e).__name__
            return ""

        fused = run(lambda: p.decompose_quantize(x, tol))
        plain = run(lambda: p.quantize(p.decompose(x), tol))
        assert fused == plain and fused != "", (node, fused, plain)
