"""The memory that container and stream calls keep between them (pool), the
histogram's 16-byte loads, and the code-length construction's key widths.

Everything here is whole numbers or bytes: results are equal, no tolerance.
"""
import threading

import numpy as np
import pytest
import torch

from paper_2609_00205_amd import synth


def test_code_lengths_of_counts_beyond_the_packed_key():
    # counts scaled by 2^30 merge in the same order (the wide keys are used
    # from 2^47 in all on)
    from paper_2609_00205_amd import api
    rng = np.random.default_rng(5)
    h = np.zeros(65536, np.uint64)
    s = rng.choice(65536, 3001, replace=False)
    h[s] = rng.integers(1, 1 << 16, s.size)
    h[s[:40]] = 7                                       # equal weights: ties go to the smaller symbol
    assert np.array_equal(api.huffman_code_lengths(h), api.huffman_code_lengths(h << np.uint64(30)))


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 3, 4, 5, 4095, 8192, 8197, 3 * 1024 * 1024 + 7])
def test_histogram_of_any_alignment(n):
    from paper_2609_00205_amd import api
    gen = torch.Generator(device="cuda").manual_seed(n)
    c = torch.randn(n + 3, device="cuda", generator=gen).mul_(3000).round_().to(torch.int32)
    edge = torch.tensor([-4096, -4097, 4095, 4096, 32767, 32768, -32767, -32768], dtype=torch.int32, device="cuda")
    c[: min(n, 8)] = edge[: min(n, 8)]                  # the LDS window's ends and the escape
    ref = bytes(api.huffman_encode(c[:n].clone()))
    assert torch.equal(api.huffman_decode(ref, n), c[:n])
    for k in (1, 2, 3):
        shifted = torch.empty(n + k, dtype=torch.int32, device="cuda")
        shifted[k:] = c[:n]
        assert bytes(api.huffman_encode(shifted[k:])) == ref


def _containers():
    from paper_2609_00205_amd import Plan
    out = []
    for i, shape in enumerate([(33, 33, 33), (65, 40, 50), (97, 65, 129)]):
        x = torch.from_numpy(synth.gaussian_random_field(shape, 3.0, seed=60 + i, dtype=np.float32)).cuda()
        p = Plan(shape, dtype=torch.float32, block=17, L=1, M=1)
        bt = p.tolmap_from_boxes([(1, 1, 1, 9, 9, 9, 1e-5)], 1e-3)
        out.append((p, x, bt, bytes(p.compress(x, bt))))
    return out


@pytest.mark.gpu
def test_calls_of_several_threads_and_streams_share_the_pool():
    from paper_2609_00205_amd import api
    cs = _containers()
    ref = [api.decompress(c[3]) for c in cs]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        try:
            st = torch.cuda.Stream()
            for r in range(8):
                p, x, bt, buf = cs[(k + r) % 3]
                with torch.cuda.stream(st):
                    if not torch.equal(api.decompress(buf), ref[(k + r) % 3]):
                        bad.append((k, r, "decompress"))
                    c = torch.full((5000 + 100 * k,), k, dtype=torch.int32, device="cuda")
                    st.synchronize()
                    if not torch.equal(api.huffman_decode(api.huffman_encode(c), c.numel()), c):
                        bad.append((k, r, "encode"))
                if r == 4:
                    api.release_memory()
        except Exception as e:   # noqa: BLE001
            bad.append((k, repr(e)))

    th = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not bad


@pytest.mark.gpu
def test_kept_memory_is_bounded_and_given_back():
    from paper_2609_00205_amd import api
    cs = _containers()
    api.release_memory()
    torch.cuda.synchronize()
    free0, total = torch.cuda.mem_get_info()
    for _ in range(5):
        for c in cs:
            api.decompress(c[3])
    torch.cuda.synchronize()
    assert free0 - torch.cuda.mem_get_info()[0] <= min(2 << 30, total)
    api.release_memory()
    torch.cuda.empty_cache()
    assert free0 - torch.cuda.mem_get_info()[0] <= 4 << 20   # (allocation granularity of the runtime)
