"""What the container calls keep between them does not grow with the number of
calls: the device memory held after a few rounds of containers is that held
after the second."""
import numpy as np
import pytest
import torch

from paper_2609_00205_amd import synth

pytestmark = pytest.mark.gpu


def test_held_memory_does_not_grow():
    from paper_2609_00205_amd import Plan, api
    bufs = []
    for i, shape in enumerate([(33, 33, 33), (65, 129, 100), (129, 129, 129)]):
        x = torch.from_numpy(synth.gaussian_random_field(shape, 3.0, seed=80 + i, dtype=np.float32)).cuda()
        p = Plan(shape, dtype=torch.float32, block=17, L=1, M=1)
        bufs.append(bytes(p.compress(x, p.tolmap_from_boxes([], 1e-3))))
        del p
    api.release_memory()
    torch.cuda.synchronize()
    used = []
    for _ in range(8):
        for b in bufs:
            api.decompress(b)
        torch.cuda.synchronize()
        used.append(torch.cuda.mem_get_info()[0])
    assert used[2:] == used[1:2] * 6, used
    api.release_memory()
    assert torch.cuda.mem_get_info()[0] > used[-1]
