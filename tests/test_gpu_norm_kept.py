"""The norm reads a long vector backwards, and its first 10,240 blocks without the streaming hint: lengths
where that line falls on the last block, the one before it and the one after it, and partial last blocks."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from test_gpu_norm import gpu_norm

KEPT = 10240 * 4096


@pytest.mark.parametrize("n", [KEPT - 4096, KEPT - 1, KEPT, KEPT + 1, KEPT + 4096, KEPT + 2 * 4096 + 5])
def test_norm_kept_blocks(n):
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n, dtype=np.float32)
    got, want = gpu_norm(x), np.float32(oracle.tree_sumsq(x))
    assert got[0].view(np.uint32) == want.view(np.uint32)
    assert got[1].view(np.uint32) == np.sqrt(want).view(np.uint32)
