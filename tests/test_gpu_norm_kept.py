"""The norm reads a long vector backwards, and its first 10,240 blocks without the streaming hint: lengths
where that line falls on the last block, the one before it and the one after it, and partial last blocks."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2208_14228_amd import binding as B
    from test_gpu_norm import gpu_norm

KEPT = 10240 * 4096


@pytest.mark.parametrize("n", [KEPT - 4096, KEPT - 1, KEPT, KEPT + 1, KEPT + 4096, KEPT + 2 * 4096 + 5])
def test_norm_kept_blocks(n):
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n, dtype=np.float32)
    got, want = gpu_norm(x), np.float32(oracle.tree_sumsq(x))
    assert got[0].view(np.uint32) == want.view(np.uint32)
    assert got[1].view(np.uint32) == np.sqrt(want).view(np.uint32)


@pytest.mark.parametrize("n", [1, 4096, 2048 * 4096 + 1, KEPT + 4096 + 5])
def test_norm_without_a_job(n):
    """es_grad_sq_norm_static streams all of the vector; the same bits."""
    x = np.random.default_rng(n).standard_normal(n, dtype=np.float32)
    vec, out = torch.from_numpy(x).to("cuda:0"), torch.full((2,), float("nan"), device="cuda:0")
    B.check(B.es_grad_sq_norm_static(vec.data_ptr(), n, out.data_ptr(), torch.cuda.current_stream().cuda_stream), "static")
    got, want = out.cpu().numpy(), gpu_norm(x)
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
    assert got[0].view(np.uint32) == np.float32(oracle.tree_sumsq(x)).view(np.uint32)
