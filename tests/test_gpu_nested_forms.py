"""The forms of the FP32 nested recomposition (one block a workgroup in groups
of 16 lanes or in rows, two blocks), on either side of where each is taken:
few blocks and 8192 and more, whole and cropped outputs, with and without a
global level above.

The fused dequantization equals recompose(dequantize) bit for bit, also where
the two take different forms; the round trip is within 8e-6 of max|x| (two
levels, both directions, 1e-6 each, doubled).
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [0, 1])
@pytest.mark.parametrize("shape", [
    (17, 17, 17), (40, 50, 61),           # few blocks, one alone and a row of odd length
    (321, 337, 321), (321, 321, 337),     # 8400: two blocks, or rows
    (305, 337, 321),                      # 7980
    (1, 1500, 1400), (3000, 5, 800),      # 8272 and 9400, most of them cropped
    (300, 320, 330),                      # 8379, cropped to 0.85
], ids=str)
def test_fused_equals_unfused(shape, M):
    from paper_2609_00205_amd import Plan
    gen = torch.Generator(device="cuda").manual_seed(31)
    p = Plan(shape, block=17, L=2, M=M, nested=True)
    print("case", shape, M, p.block_grid, flush=True)
    x = torch.randn(shape, device="cuda", generator=gen)
    c = p.decompose(x)
    guard = torch.full((x.numel() + 64,), 7.0, device="cuda")
    out = guard[:x.numel()].view(shape)
    p.recompose(c, out=out)
    assert float((out - x).abs().max()) <= 8e-6 * float(x.abs().max())
    bt = 10.0 ** (torch.rand(p.block_grid, dtype=torch.float64, device="cuda", generator=gen) * 3 - 4)
    codes = p.decompose_quantize(x, bt)
    ref = p.recompose(p.dequantize(codes, bt))
    p.dequantize_recompose(codes, bt, out=out)
    assert torch.equal(out, ref)
    assert bool((guard[x.numel():] == 7.0).all())


@pytest.mark.parametrize("shape,M", [((90, 70, 1), 1), ((40, 33, 17), 0), ((40, 33, 18), 0), ((17, 300, 9), 2)], ids=str)
def test_rows_of_one_block(shape, M):
    """The plain schedule where a row has one block and where it has two."""
    from paper_2609_00205_amd import Plan
    gen = torch.Generator(device="cuda").manual_seed(32)
    p = Plan(shape, block=17, L=1, M=M)
    print("case", shape, M, p.block_grid, flush=True)
    x = torch.randn(shape, device="cuda", generator=gen)
    guard = torch.full((x.numel() + 64,), 7.0, device="cuda")
    out = guard[:x.numel()].view(shape)
    p.recompose(p.decompose(x), out=out)
    assert float((out - x).abs().max()) <= 4e-6 * float(x.abs().max())
    bt = 10.0 ** (torch.rand(p.block_grid, dtype=torch.float64, device="cuda", generator=gen) * 3 - 4)
    codes = p.decompose_quantize(x, bt)
    p.dequantize_recompose(codes, bt, out=out)
    assert torch.equal(out, p.recompose(p.dequantize(codes, bt)))
    assert bool((guard[x.numel():] == 7.0).all())
