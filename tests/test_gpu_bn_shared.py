"""BatchNorm batch statistics where several workgroups share a channel and wait for each other's sums,
bit for bit: both sides of every number of workgroups, whole vectors and ragged images, one round of
workgroups and several, a workspace that holds anything, launches in flight on three streams, workgroups
that do not wait (every look at the others' sums the last), and captured launches replayed, with other
values in x and with eager calls on the same workspace in between."""
import ctypes

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2208_14228_amd import binding as B
    from test_gpu_bn_clip import bits
    DEV = "cuda:0"

BLK = 4096


class Case:
    def __init__(self, images, channels, positions, seed=0):
        rng = np.random.default_rng(seed * 7919 + images * 131 + channels * 17 + positions)
        self.shape = (images, channels, positions)
        self.x = torch.empty(self.shape, device=DEV)
        self.fill(rng)
        self.out = torch.empty((2, channels), device=DEV)
        self.n = B.es_bn_workspace_floats(*self.shape)
        self.ws = torch.full((self.n + 5,), float("nan"), device=DEV)   # at an address that is no multiple of 8
        self.ws[:] = torch.from_numpy(rng.integers(0, 1 << 32, self.n + 5, dtype=np.uint32).view(np.float32)).to(DEV)
        self.guard = self.ws.view(torch.int32).clone()

    def fill(self, rng):
        h = (rng.standard_normal(self.shape, dtype=np.float32) * 3 + rng.standard_normal((1, self.shape[1], 1)) * 5).astype(np.float32)
        self.want = oracle.bn_batch_stats(h)
        self.x.copy_(torch.from_numpy(h))
        torch.cuda.synchronize()

    def args(self):
        return (self.x.data_ptr(), *self.shape, self.out[0].data_ptr(), self.out[1].data_ptr(), self.ws[1:].data_ptr(), self.n)

    def run(self, stream=None):
        print(f"[gpu-case] es_bn_batch_stats {self.shape}", flush=True)
        assert B.es_bn_batch_stats(*self.args(), stream.cuda_stream if stream else 0) == B.ES_OK

    def check(self, what=""):
        torch.cuda.synchronize()
        got = self.out.cpu().numpy()
        assert np.array_equal(bits(got[0]), bits(self.want[0])), ("mean", self.shape, what)
        assert np.array_equal(bits(got[1]), bits(self.want[1])), ("var", self.shape, what)
        now = self.ws.view(torch.int32)
        assert bool((now[0] == self.guard[0]).all()) and bool((now[1 + self.n:] == self.guard[1 + self.n:]).all())
        self.out.fill_(3.0)


# terms of a channel at and just above the blocks where the number of workgroups (2 to 64) or the form changes
EDGES = [26 * BLK - 3000, 32 * BLK, 32 * BLK + 4, 64 * BLK, 65 * BLK - 8, 128 * BLK + 400, 255 * BLK, 256 * BLK + 12,
         512 * BLK + 4, 1024 * BLK, 1024 * BLK + 4]


@pytest.mark.parametrize("terms", EDGES)
def test_both_sides_of_every_number_of_workgroups(terms):
    for shape in ((1, 1, terms), (2, 3, terms // 2), (3, 2, terms // 3 + 1)):
        c = Case(*shape)
        for k in range(2):                      # the second finds the sums of the first in the workspace
            c.run()
            c.check(k)


@pytest.mark.parametrize("shape", [(13, 64, 2 * BLK), (27, 70, BLK + 1), (8, 300, 14400), (26, 160, 4225), (500, 40, 225 * 4), (250, 40, 901)])
def test_many_channels(shape):
    c = Case(*shape)
    c.run()
    c.check()


# up to 1,500 blocks workgroups of eight waves, beyond of four; ragged long images are the second of each pair
@pytest.mark.parametrize("whole,ragged", [(40, 30), (60, 50)])
def test_launches_in_flight_together(whole, ragged):
    cases = ([Case(26, whole + k, 4096 + 4 * k, seed=k) for k in range(3)]
             + [Case(33, ragged + k, 4097, seed=k) for k in range(3)])
    streams = [torch.cuda.Stream(DEV) for _ in range(3)]
    for _ in range(3):
        for k, c in enumerate(cases):
            c.run(streams[k % 3])
        for c in cases:
            c.check()


@pytest.mark.parametrize("polls", [0, 1])
@pytest.mark.parametrize("shape", [(26, 5, BLK), (1, 3, 33 * BLK + 4), (100, 4, 5041), (3, 2, 300 * BLK + 1), (27, 300, 4096)])
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


# little work (another form where it is captured) and more (workgroups of eight waves, beyond 1,500 blocks of four), on both
# sides of the lines between them, and much
@pytest.mark.parametrize("shape", [(26, 4, BLK), (26, 38, BLK), (26, 39, BLK), (130, 9, BLK + 1), (130, 10, BLK + 1), (26, 57, BLK),
                                   (26, 58, BLK), (130, 11, BLK + 1), (130, 12, BLK + 1), (32, 64, 12544)])
def test_captured_launches_replayed(shape):
    c = Case(*shape)
    s = torch.cuda.Stream(DEV)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        c.run(s)
    rng = np.random.default_rng(5)
    for k in range(4):
        if k:
            c.fill(rng)
        g.replay()
        c.check(k)
        c.run()
        c.check((k, "eager"))
