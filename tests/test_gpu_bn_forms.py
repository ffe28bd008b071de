"""BatchNorm batch statistics at the edges of the kernel's forms, bit for bit: channels of one
block, of up to 16 (registers), up to 25 (registers and LDS), up to 256 (three launches) and more
(four), in every memory form (whole vectors, long and short ragged images, images below four
positions), and byte offsets beyond 32 bits."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2208_14228_amd import binding as B
    from test_gpu_bn_clip import bits, gpu_bn
    DEV = "cuda:0"

BLK = 4096
# terms per channel just at, below and above each form's limit, as (images, positions)
SHAPES = [
    (1, BLK), (1, BLK - 1), (1, BLK + 1), (4, 1024), (4, 1025), (5, 1023), (1, 16 * BLK), (1, 16 * BLK + 4),
    (13, 5041), (64, 1024 + 1), (1, 25 * BLK), (1, 25 * BLK + 4), (25, BLK - 1), (3, 25 * BLK // 3 + 1),
    (1, 32 * BLK), (1, 32 * BLK + 1), (7, 9 * BLK + 3), (100, 3 * BLK + 2), (1, 256 * BLK), (1, 256 * BLK + 1),
    (255, 1), (4097, 1), (1400, 3), (70_001, 2), (40_000, 5), (30_000, 7), (1, 1), (2, 4), (1, 6),
    (3, 255), (3, 256), (3, 257), (17, 258),
    # both sides of the line between short and long images, in every form
    (32, 127), (31, 129), (400, 127), (400, 129), (700, 127), (700, 129), (1100, 127), (1100, 131), (8500, 127), (8500, 129),
    # few channels of tiny images, around where they are spread over several workgroups
    (7 * BLK, 1), (7 * BLK + 1, 1), (8 * BLK, 1), (16 * BLK + 5, 1), (25 * BLK, 1), (12_289, 3), (21_850, 3), (9 * BLK // 4, 4),
    (7_400, 5), (13_106, 5), (20_479, 5), (6_144, 8), (6_145, 8), (3_641, 15), (6_826, 15), (5_000, 16), (26 * BLK - 9, 1),
]


@pytest.mark.parametrize("Bn,HW", SHAPES)
def test_every_form_at_its_edges(Bn, HW):
    for C in (1, 5):                       # 5: a last workgroup with idle waves in the one-block form
        rng = np.random.default_rng(Bn * 131 + HW + C)
        x = (rng.standard_normal((Bn, C, HW)) * 3 + rng.standard_normal((1, C, 1)) * 10).astype(np.float32)
        want_m, want_v = oracle.bn_batch_stats(x)
        for shift in (0, 3):
            got_m, got_v = gpu_bn(x, shift)
            assert np.array_equal(bits(got_m), bits(want_m)), ("mean", C, shift)
            assert np.array_equal(bits(got_v), bits(want_v)), ("var", C, shift)


@pytest.mark.parametrize("Bn,C,HW", [(7_373, 128, 5), (7_373, 129, 5), (9_300, 48, 4), (9_300, 49, 4),
                                      (15_000, 64, 4), (15_000, 65, 4), (4_800, 64, 12), (4_800, 65, 12)])
def test_both_sides_of_the_channel_lines_for_tiny_images(Bn, C, HW):
    rng = np.random.default_rng(C)
    x = (rng.standard_normal((Bn, C, HW), dtype=np.float32) * 3 + 1).astype(np.float32)
    want_m, want_v = oracle.bn_batch_stats(x)
    got_m, got_v = gpu_bn(x)
    assert np.array_equal(bits(got_m), bits(want_m)) and np.array_equal(bits(got_v), bits(want_v))


@pytest.mark.parametrize("HW", [49, 196, 4 * BLK + 3, 20 * BLK, 40 * BLK + 1])
def test_infinities_and_nan_stay_in_their_channel(HW):
    rng = np.random.default_rng(HW)
    x = rng.standard_normal((2, 6, HW)).astype(np.float32)
    x[1, 1, HW - 1] = np.inf
    x[0, 3, 0] = np.nan
    x[0, 4, :] = -0.0
    x[1, 4, :] = -0.0
    want_m, want_v = oracle.bn_batch_stats(x)
    got_m, got_v = gpu_bn(x)
    for got, want in ((got_m, want_m), (got_v, want_v)):
        assert np.array_equal(np.isnan(got), np.isnan(want))
        fine = ~np.isnan(want)
        assert np.array_equal(bits(got)[fine], bits(want)[fine])
    assert np.isfinite(got_m[[0, 2, 4, 5]]).all() and np.isinf(got_m[1]) and np.isnan(got_m[3])


@pytest.mark.parametrize("Bn,C,HW", [
    (2, 140_000 // 4, 15_361), (2, 9_000, 60_000), (1, 1_100, 1_000_001),
    # short ragged images and images below four positions: up to 16 blocks, up to 25, up to 256, more
    (600, 40_000, 49), (1_700, 13_000, 49), (3_000, 7_400, 49), (25_000, 900, 49),
    (20_000, 20_000, 3), (30_000, 12_000, 3), (50_000, 7_200, 3), (400_000, 900, 3),
    # short ragged images read in single loads
    (9_000, 17_100, 7), (14_000, 11_000, 7), (40_000, 3_900, 7), (200_000, 780, 7), (50_000, 4_400, 5), (250_000, 880, 5),
    # long images and whole vectors in the forms not reached above
    (100, 12_000, 901), (1_200, 1_000, 901), (100, 12_000, 900), (1_200, 1_000, 900)])
def test_offsets_beyond_32_bits(Bn, C, HW):
    """x of more than 4 GiB: the same bits as its channels a slice at a time (32-bit offsets).  A channel of
    one block cannot get there: 65,535 of them are 1.07 GB."""
    assert 4 * Bn * C * HW > 1 << 32
    g = torch.Generator(device=DEV)
    g.manual_seed(HW)
    x = torch.empty((Bn, C, HW), device=DEV).normal_(0.5, 2.0, generator=g)

    def stats(t):
        c = t.shape[1]
        out = torch.full((2, c), float("nan"), device=DEV)
        n = B.es_bn_workspace_floats(*t.shape)
        ws = torch.full((n,), float("nan"), device=DEV)
        torch.cuda.synchronize()
        print(f"[gpu-case] es_bn_batch_stats {tuple(t.shape)}", flush=True)
        assert B.es_bn_batch_stats(t.data_ptr(), *t.shape, out[0].data_ptr(), out[1].data_ptr(), ws.data_ptr(), n) == B.ES_OK
        torch.cuda.synchronize()
        return out.view(torch.int32)

    whole = stats(x)
    for lo in (0, C // 2, C - 300):
        assert torch.equal(whole[:, lo:lo + 300], stats(x[:, lo:lo + 300].contiguous())), lo
