"""The search for the level lambda of the QoI widths (compacted shares,
brackets from concavity) against water-filling by sorting, at the ends of its
range: a budget that every cap fits, one that only the largest shares exceed,
one far below every share; grids whose last chunk of 64 shares is partial and
a grid with more chunks than wavefronts.

Tolerance: a sum of n <= 3e6 positive shares, formed as per-lane runs and
trees, is off by well under 1e-13 of itself, and the level moves by that much
times target / (n_above lambda), the inverse of the sum's slope there.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _level(a, target):
    """The root of sum min(a, level) = target by sorting; inf when every share fits."""
    a = np.sort(a)
    low = np.concatenate([[0.0], np.cumsum(a)])
    if low[-1] <= target:
        return np.inf, 0
    n_above = len(a) - np.arange(len(a) + 1)
    with np.errstate(divide="ignore"):
        lam = (target - low) / n_above
    k = int(np.nonzero(lam[:-1] <= a)[0][0])   # the first share above its own level
    return lam[k], n_above[k]


@pytest.mark.parametrize("shape,b,L,M,dt,frac", [
    ((33, 33, 33), 17, 1, 2, torch.float64, 2.0),        # every cap fits
    ((33, 33, 33), 17, 1, 2, torch.float64, 1.0 - 1e-6),
    ((33, 33, 33), 17, 1, 2, torch.float32, 0.5),
    ((20, 35, 50), 9, 2, 1, torch.float64, 1e-3),
    ((20, 35, 50), 17, 1, 0, torch.float64, 1e-12),      # far below every share
    ((129, 129, 160), 17, 1, 1, torch.float32, 0.3),     # several chunks per wavefront
])
def test_level_against_sorting(shape, b, L, M, dt, frac):
    from paper_2609_00205_amd import Plan
    print("case", shape, b, L, M, dt, frac, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    p = Plan(shape, dtype=dt, block=b, L=L, M=M)
    g = torch.randn(shape, dtype=dt, device="cuda", generator=gen) * 1e-3
    bt = p.tolmap_from_boxes([(0, 0, 0, 9, 9, 9, 1e-4)], 1e-2)
    cap, n0 = p.qoi_deltas(g, 1e30, bt)
    assert n0 == 0
    s = p.recompose_adjoint(g).double().abs().cpu().numpy().ravel()
    cap = cap.cpu().numpy().ravel()
    a = s * cap * 0.5
    tol_q = frac * a.sum() / (1.0 - p.eta)
    target = (1.0 - p.eta) * tol_q
    lam, n_above = _level(a, target)
    delta, nset = p.qoi_deltas(g, tol_q, bt)
    delta = delta.cpu().numpy().ravel()
    if n_above == 0:
        assert nset == 0 and np.array_equal(delta, cap)
        return
    rel = 1e-13 * target / (n_above * lam)
    near = np.abs(a - lam) <= 2 * rel * lam              # within the tolerance of the level itself
    assert abs(nset - int((a > lam).sum())) <= int(near.sum())
    ref = np.where(a > lam, 2.0 * lam / np.where(s > 0, s, 1.0), cap)
    assert np.all(np.abs(delta - ref)[~near] <= (rel + 4e-16) * ref[~near])
