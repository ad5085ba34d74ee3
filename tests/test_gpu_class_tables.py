"""The block kernels' own Delta classes (from the blocks' tolerances, by lane
exchanges) against the class tables that the unfused quantizer builds, for a
map that differs from block to block; and the propagation by one workgroup
against the launch of many, on grids on either side of the limit.

Codes are whole numbers formed from the same coefficients: equal.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    ((17, 17, 17), 17, 1, 0, False, torch.float32),     # one block: every neighbour beyond the grid
    ((33, 17, 49), 17, 1, 0, False, torch.float64),     # odd block counts, coarsest values by block
    ((49, 65, 33), 17, 1, 1, False, torch.float32),     # pairs of blocks with one left over
    ((25, 41, 33), 9, 1, 2, False, torch.float32),      # three 9^3 blocks per workgroup, remainders
    ((40, 50, 61), 9, 2, 0, False, torch.float64),      # ragged, two levels
    ((65, 33, 49), 17, 2, 1, True, torch.float32),      # nested pair
    ((65, 33, 49), 17, 2, 0, True, torch.float64),
    ((70, 40, 100), 33, 1, 1, False, torch.float32),    # 33-node levels keep the tables
]


@pytest.mark.parametrize("shape,b,L,M,nested,dt", CASES)
def test_fused_codes_equal_unfused_codes(shape, b, L, M, nested, dt):
    from paper_2609_00205_amd import Batch, Plan
    print("case", shape, b, L, M, nested, dt, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(11)
    p = Plan(shape, dtype=dt, block=b, L=L, M=M, nested=nested)
    x = torch.randn(shape, dtype=dt, device="cuda", generator=gen)
    bt = 10.0 ** (torch.rand(p.block_grid, dtype=torch.float64, device="cuda", generator=gen) * 4 - 5)
    ref, _ = p.quantize(p.decompose(x), bt)
    codes = p.decompose_quantize(x, bt)
    assert torch.equal(codes, ref)
    assert torch.equal(p.dequantize_recompose(codes, bt), p.recompose(p.dequantize(codes, bt)))
    if nested or b == 33:
        return
    batch = Batch([shape, shape], dtype=dt, block=b, L=L, M=M)
    bc = batch.decompose_quantize([x, x], [bt, bt])
    assert torch.equal(bc[0], ref) and torch.equal(bc[1], ref)


@pytest.mark.parametrize("n", [257, 273])               # 16^3 and 17^3 blocks at level 2: one workgroup, many
def test_propagated_tolerances(n):
    from paper_2609_00205_amd import Plan
    gen = torch.Generator(device="cuda").manual_seed(12)
    p = Plan((n, n, n), dtype=torch.float64, block=9, L=2, M=0)
    nb = p.block_grid
    bt = 10.0 ** (torch.rand(nb, dtype=torch.float64, device="cuda", generator=gen) * 4 - 5)
    delta = p.dequantize(torch.ones(p.coeff_shape, dtype=torch.int32, device="cuda"), bt)
    t = bt.cpu().numpy()
    m = [v // 2 for v in nb]
    ref = np.full(m, np.inf)
    for z in range(m[0]):
        for y in range(m[1]):
            for x in range(m[2]):
                s = tuple(slice(max(0, 2 * c - 1), 2 * c + 3) for c in (z, y, x))
                ref[z, y, x] = t[s].min()
    # an inner detail of level 2 (an odd node of the grid of even nodes) of every block
    got = delta[10::16, 10::16, 10::16].cpu().numpy()
    ratio = got / ref
    assert np.all(np.abs(ratio / ratio.flat[0] - 1) <= 4e-16)   # tau * kappa: one rounding each
