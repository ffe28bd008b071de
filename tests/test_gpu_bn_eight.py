"""BatchNorm batch statistics where workgroups of eight waves share a channel, bit for bit: both sides of the line to those of
four, more than sixteen blocks to a workgroup (their sums are two rows of lanes), and workgroups that do not wait."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2208_14228_amd import binding as B
    from test_gpu_bn_shared import Case

BLK = 4096


@pytest.mark.parametrize("shape", [(26, 57, BLK), (26, 58, BLK), (33, 45, 4096), (33, 46, 4097), (50, 30, BLK), (50, 31, BLK),
                                   (1, 23, 64 * BLK), (1, 24, 64 * BLK - 8), (129, 11, BLK + 4), (17, 5, 15 * BLK + 1)])
def test_both_sides_of_the_line(shape):
    c = Case(*shape)
    for k in range(2):
        c.run()
        c.check(k)


@pytest.mark.parametrize("polls", [0, 1])
@pytest.mark.parametrize("shape", [(50, 30, BLK), (64, 23, BLK), (1, 1, 1000 * BLK + 5), (99, 14, BLK + 1)])
def test_workgroups_that_do_not_wait(shape, polls):
    f = B.lib()._ZN2es27launch_bn_batch_stats_pollsEP12ihipStream_tPKfjjjPfS4_S4_j
    p, u = ctypes.c_void_p, ctypes.c_uint32
    f.argtypes, f.restype = [p, p, u, u, u, p, p, p, u], ctypes.c_int
    c = Case(*shape)
    for k in range(2):
        a = c.args()
        print(f"[gpu-case] bn shared {shape} polls {polls}", flush=True)
        assert f(0, a[0], *shape, *a[4:7], polls) == 0
        c.check(k)
