"""Transposes of block levels whose contributions take more than one slab
(128 MiB of scratch): <D x, y> = <x, D^T y> and <R c, g> = <c, R^T g> to
rounding.

Tolerance: as for the other dot-product checks, 1e-13 of |D x| |y| in FP64.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,b,L,M", [
    ((257, 257, 257), 33, 1, 1),     # two slabs of 33^3 blocks
    ((200, 257, 300), 9, 1, 1),      # two slabs of 9^3 blocks, every axis padded but one
    ((300, 150, 257), 17, 2, 0),     # two slabs at level 1, one at level 2
])
def test_dot_product_identity(shape, b, L, M):
    from paper_2609_00205_amd import Plan
    print("case", shape, b, L, M, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(7)
    p = Plan(shape, dtype=torch.float64, block=b, L=L, M=M)
    x = torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen)
    y = torch.randn(p.coeff_shape, dtype=torch.float64, device="cuda", generator=gen)
    for fwd, adj, u, v in ((p.decompose, p.decompose_adjoint, x, y), (p.recompose, p.recompose_adjoint, y, x)):
        fu, av = fwd(u), adj(v)
        gap = float((fu * v).sum() - (u * av).sum())
        assert abs(gap) <= 1e-13 * float(fu.norm() * v.norm())
        assert torch.equal(adj(v), av)      # a second call, on the kept scratch


def test_first_call_in_a_capture():
    """The scratch is allocated by the first call, also where that is captured."""
    from paper_2609_00205_amd import Plan
    p = Plan((65, 65, 65), dtype=torch.float64, block=17, L=1, M=1)
    y = torch.randn(p.coeff_shape, dtype=torch.float64, device="cuda")
    out = torch.empty(p.shape, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        p.decompose_adjoint(y, out=out)
    for k in range(3):
        y.copy_(torch.randn(p.coeff_shape, dtype=torch.float64, device="cuda"))
        graph.replay()
        assert torch.equal(out, p.decompose_adjoint(y)), k
