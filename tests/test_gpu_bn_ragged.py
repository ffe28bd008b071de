"""BatchNorm batch statistics of images that are no whole vectors, bit for bit: every place an image can end at inside a
vector, channels whose last vector is not full, both sides of the lines between single loads and vectors, and numbers of
channels that do not divide among eight compute dies."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from test_gpu_bn_clip import bits, gpu_bn


@pytest.mark.parametrize("hw,images", [
    (5, (1, 2, 3, 819, 820)), (6, (3, 682, 683)), (7, (5, 585, 586)), (9, (2, 455, 456)), (10, (409, 410)), (11, (4, 372, 373)),
    (13, (7, 315)), (25, (64, 333)), (35, (29, 118)), (49, (1, 32, 84, 700)), (121, (33, 67)), (127, (1, 3, 805)), (255, (9,)),
    (2558, (3, 41)), (2559, (2, 40)), (2561, (2, 40)), (2562, (3, 41))])
def test_every_end_of_a_ragged_image(hw, images):
    for n in images:
        for c in (1, 3, 9, 37):
            rng = np.random.default_rng(hw * 1000 + n + c)
            x = (rng.standard_normal((n, c, hw)) * 2 + rng.standard_normal((1, c, 1)) * 5).astype(np.float32)
            want_m, want_v = oracle.bn_batch_stats(x)
            for shift in (0, 1):
                got_m, got_v = gpu_bn(x, shift)
                assert np.array_equal(bits(got_m), bits(want_m)), ("mean", n, c, shift)
                assert np.array_equal(bits(got_v), bits(want_v)), ("var", n, c, shift)


@pytest.mark.parametrize("blocks,c", [(9, 48), (10, 48), (10, 49), (14, 48), (14, 49), (15, 64), (15, 65), (25, 64)])
def test_images_of_one_vector_in_one_launch_and_in_three(blocks, c):
    rng = np.random.default_rng(blocks + c)
    for n in (1024 * blocks, 1024 * blocks - 7):
        x = (rng.standard_normal((n, c, 4), dtype=np.float32) * 3 + 1).astype(np.float32)
        want_m, want_v = oracle.bn_batch_stats(x)
        got_m, got_v = gpu_bn(x)
        assert np.array_equal(bits(got_m), bits(want_m)) and np.array_equal(bits(got_v), bits(want_v)), n
