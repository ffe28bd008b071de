"""The norm in one launch (up to 2,048 blocks): one workgroup and several, one counter of arrivals and several,
the last length of this form and the first of the other, again and again on the same counters, and captured."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2208_14228_amd import binding as B
    from paper_2208_14228_amd.job import ESTJob
    DEV = "cuda:0"

BLOCK = 4096


def _vector(n, seed):
    return np.random.default_rng([n, seed]).standard_normal(n, dtype=np.float32)


def _same(out, x):
    want = np.float32(oracle.tree_sumsq(x))
    got = out.cpu().numpy()
    assert got[0].view(np.uint32) == want.view(np.uint32)
    assert got[1].view(np.uint32) == np.sqrt(want).view(np.uint32)


# 4 blocks a workgroup; 64 workgroups share a counter, beyond there are 16 and one more
@pytest.mark.parametrize("blocks", [1, 4, 5, 255, 256, 257, 260, 261, 17 * 64, 2047, 2048, 2049])
@pytest.mark.parametrize("odd", [0, 1])
def test_again_and_again(blocks, odd):
    n = blocks * BLOCK - odd * 1235
    job = ESTJob(1, n, [(0, n)], 1)
    try:
        out = torch.full((2,), float("nan"), device=DEV)
        for k in range(4):
            x = _vector(n, k)
            vec = torch.from_numpy(x).to(DEV)
            torch.cuda.synchronize()
            B.check(B.es_grad_sq_norm(job.h, vec.data_ptr(), out.data_ptr()), "es_grad_sq_norm", job.h)
            job.sync()
            _same(out, x)
    finally:
        job.close()


def test_replays_of_a_captured_norm():
    n = 300 * BLOCK + 9
    job = ESTJob(1, n, [(0, n)], 1, use_streams="one")
    try:
        vec, out = torch.zeros(n, device=DEV), torch.zeros(2, device=DEV)
        norm = lambda: B.check(B.es_grad_sq_norm(job.h, vec.data_ptr(), out.data_ptr()), "es_grad_sq_norm", job.h)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=job.main):
            norm()
        for k in range(5):
            x = _vector(n, k)
            vec.copy_(torch.from_numpy(x))
            torch.cuda.synchronize()
            if k == 2:                          # an eager norm between the replays
                norm()
                job.sync()
            else:
                g.replay()
                torch.cuda.synchronize()
            _same(out, x)
    finally:
        job.close()
