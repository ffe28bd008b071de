"""The last stage of the fixed-tree norm where it changes from 8 loads ahead to 32: one vector of
8192 blocks (a whole round of 32 loads per lane), one block fewer, one more, and two rounds."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from test_gpu_norm import gpu_norm

ROUND = 32 * 256 * 4096


@pytest.mark.parametrize("n", [ROUND - 4096, ROUND - 4095, ROUND, ROUND + 1, 2 * ROUND + 300 * 4096 + 7])
def test_norm_partials_rounds(n):
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n, dtype=np.float32)
    got, want = gpu_norm(x), np.float32(oracle.tree_sumsq(x))
    assert got[0].view(np.uint32) == want.view(np.uint32)
    assert got[1].view(np.uint32) == np.sqrt(want).view(np.uint32)
