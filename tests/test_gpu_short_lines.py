"""Line passes on either side of the length (64 nodes) from which tiles of 32
lines and more take 512 lanes, against the FP64 oracle.

Bar: 1e-6 (FP32) and 1e-13 (FP64) of max|x| per direction.
"""
import numpy as np
import pytest
import torch

from oracle import mgard
from paper_2609_00205_amd import synth

pytestmark = pytest.mark.gpu

TOL = {torch.float32: 1e-6, torch.float64: 1e-13}


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["float32", "float64"])
@pytest.mark.parametrize("shape", [(3, 200, 210), (63, 190, 60), (65, 190, 60), (64, 20, 300), (190, 65, 40), (33, 257, 180)],
                         ids=lambda s: "x".join(map(str, s)))
def test_line_lengths(shape, dt):
    from paper_2609_00205_amd import Plan
    print("case", shape, dt, flush=True)
    x = synth.gaussian_random_field(shape, 3.0, seed=8, dtype=np.float64)
    x = x.astype(np.float32 if dt == torch.float32 else np.float64)
    p = Plan(shape, dtype=dt, L=0, M=1)
    sc = float(np.abs(x).max())
    c = p.decompose(torch.from_numpy(x).cuda())
    ref = mgard.decompose(x.astype(np.float64), 17, 0, 1)
    assert float(np.abs(c.double().cpu().numpy() - ref).max()) <= TOL[dt] * sc
    back = mgard.recompose(c.double().cpu().numpy(), shape, 17, 0, 1)
    assert float(np.abs(p.recompose(c).double().cpu().numpy() - back).max()) <= TOL[dt] * sc
