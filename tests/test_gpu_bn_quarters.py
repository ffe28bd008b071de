"""BatchNorm batch statistics whose channels end at, before and behind each quarter of a block of 4,096 terms (what lies
behind the end is neither added nor masked), bit for bit, in every form of the kernel."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from test_gpu_bn_clip import bits, gpu_bn

BLK = 4096


@pytest.mark.parametrize("blocks", [0, 1, 15, 16, 24, 25, 40, 257])
@pytest.mark.parametrize("images", [1, 3])
def test_channels_that_end_around_a_quarter(blocks, images):
    for end in (1, 1023, 1024, 1025, 2048, 2051, 3071, 3072, 3076, 4095):
        hw = (blocks * BLK + end + images - 1) // images
        rng = np.random.default_rng(hw)
        x = (rng.standard_normal((images, 3, hw)) * 3 - 7).astype(np.float32)
        x[-1, 1, -1] = -0.0
        want_m, want_v = oracle.bn_batch_stats(x)
        got_m, got_v = gpu_bn(x)
        assert np.array_equal(bits(got_m), bits(want_m)), ("mean", hw)
        assert np.array_equal(bits(got_v), bits(want_v)), ("var", hw)
