"""Tiles of the global levels' line passes, against the FP64 oracle: 512
lanes for tiles of 32 and more lines, 256 below, tiles dealt out to the eight
dies in runs of ceil(tiles / 8).

One global level without the plane pass on (n, 17, nx): the y pass has n
rows of (nx + 1) / 2 lines each, so tiles straddle rows and the last is
ragged; n >= 1024 keeps the tile as wide as the row allows (16, 32, 64
lines), (3, 17, 65) gives fewer tiles than dies.  Bar: 1e-6 (FP32) and 1e-13
(FP64) of max|x|.
"""
import os

import numpy as np
import pytest
import torch

from oracle import mgard
from paper_2609_00205_amd import synth

pytestmark = pytest.mark.gpu

TOL = {torch.float32: 1e-6, torch.float64: 1e-13}
SHAPES = [(1031, 17, 17), (1031, 17, 35), (1027, 17, 129), (3, 17, 65)]   # 9, 18, 65 and 33 lines a row


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["float32", "float64"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_line_tiles(shape, dt):
    from paper_2609_00205_amd import Plan
    print("case", shape, dt, flush=True)
    old = os.environ.get("BM_PLANE_PASS")
    os.environ["BM_PLANE_PASS"] = "0"
    try:
        plan = Plan(shape, dtype=dt, block=17, L=0, M=1)
    finally:
        if old is None:
            del os.environ["BM_PLANE_PASS"]
        else:
            os.environ["BM_PLANE_PASS"] = old
    x = synth.gaussian_random_field(shape, 3.0, seed=3, dtype=np.float64)
    x = x.astype(np.float32 if dt == torch.float32 else np.float64)
    ref = mgard.decompose(x.astype(np.float64), 17, 0, 1)
    c = plan.decompose(torch.from_numpy(x).cuda())
    sc = float(np.abs(x).max())
    assert float(np.abs(c.double().cpu().numpy() - ref).max()) <= TOL[dt] * sc
    r = plan.recompose(c)
    assert float(np.abs(r.cpu().numpy() - x).max()) <= 2 * TOL[dt] * sc   # (both directions)
