"""Transposes of block levels whose rows are so wide that the byte offset of a
block's last row passes 2^32 (the forward calls refuse such grids, the
transposes take them).

The input is zero but for windows of whole blocks at both ends of the rows; a
block level is local, so inside a window the gradient is that of a plan on
the window alone, of the same operations in the same order: equal.  Outside
it is zero.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

W = 12          # blocks of a window (the outermost two left zero)


def _skip_if_small(nbytes):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < nbytes:
        pytest.skip(f"needs {nbytes >> 30} GiB of device memory")


@pytest.mark.parametrize("b,dt,n", [(17, torch.float64, (1 << 25) + 1), (17, torch.float32, (1 << 26) + 1),
                                    (9, torch.float64, (1 << 26) + 1), (9, torch.float32, (1 << 27) + 1)])
@pytest.mark.parametrize("adj", ["decompose_adjoint", "recompose_adjoint"])
def test_rows_beyond_32_bit_offsets(b, dt, n, adj):
    from paper_2609_00205_amd import Plan
    print("case", b, dt, n, adj, flush=True)
    es = torch.finfo(dt).bits // 8
    assert (b - 1) * n * es >= 1 << 32
    _skip_if_small(int(1.5 * b * b * n * es) + (24 << 30))
    e = b - 1
    shape, full = (1, b, n), (b, b, n)
    p = Plan(shape, dtype=dt, block=b, L=1, M=0, pad_mode="zero")
    assert p.coeff_shape == full
    q = Plan((1, b, W * e + 1), dtype=dt, block=b, L=1, M=0, pad_mode="zero")
    src, win = (full, q.coeff_shape) if adj == "decompose_adjoint" else (shape, q.shape)
    gen = torch.Generator(device="cuda").manual_seed(9)
    x = torch.zeros(src, dtype=dt, device="cuda")
    parts, starts = [], [0, n - (W * e + 1)]             # (both on even blocks)
    assert starts[1] // e % 2 == 0
    for s in starts:
        w = torch.zeros(win, dtype=dt, device="cuda")
        w[..., e + 1: (W - 1) * e] = torch.randn(win[:-1] + ((W - 2) * e - 1,), dtype=dt, device="cuda",
                                                 generator=gen)
        x[..., s: s + W * e + 1] = w
        parts.append(getattr(q, adj)(w))
    out = getattr(p, adj)(x)
    del x
    for s, part in zip(starts, parts):
        got = out[..., s: s + W * e + 1]
        assert torch.equal(got, part)
        got.zero_()
    for z in range(out.shape[0]):
        assert not bool(out[z].any()), z
    assert bool(torch.stack([part.abs().max() for part in parts]).min() > 0)
    del out
    torch.cuda.empty_cache()
