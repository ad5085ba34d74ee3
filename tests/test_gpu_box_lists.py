"""Box lists that come with the launch (up to 32 boxes) and longer ones from
device memory give the same map: each list is padded with boxes that change
nothing (empty, or looser than the background) to either side of the limit;
several calls in a row with different lists do not mix."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [0, 1])
@pytest.mark.parametrize("n", [0, 1, 4, 31, 32])
def test_box_lists(n, L):
    from paper_2609_00205_amd import Plan
    print("case", n, L, flush=True)
    p = Plan((65, 50, 41), block=17, L=L, M=1)
    rng = np.random.default_rng(n)
    lists, maps = [], []
    for _ in range(3):
        lo = rng.integers(0, 40, size=(n, 3))
        hi = lo + rng.integers(1, 20, size=(n, 3))
        boxes = [(*map(int, a), *map(int, b), float(t)) for a, b, t in zip(lo, hi, rng.uniform(1e-4, 1.0, n))]
        lists.append(boxes)
        maps.append(p.tolmap_from_boxes(boxes, 0.5))
    for boxes, m in zip(lists, maps):
        for extra in (33 - n, 100):
            pad = [(3, 3, 3, 3, 9, 9, 1e-9), (0, 0, 0, 65, 50, 41, 0.75)] * extra
            assert torch.equal(p.tolmap_from_boxes(boxes + pad, 0.5), m)
