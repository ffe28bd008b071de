"""Masks of more than one workgroup, drawn and advanced in one launch: one counter of arrivals and
several, one workgroup per share of the mask and several shares each, two states of one job in turn on
the same counters, and a captured draw replayed: between eager ones, after a regrouping, after its job's
end, and beside the draws of another state; bit for bit with the state left behind."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2208_14228_amd import binding as B
    from paper_2208_14228_amd.job import ESTJob
    DEV = "cuda:0"

GROUP = 4096                                    # bytes a workgroup draws at a time
ONE_COUNTER, RESIDENT = 64 * GROUP, 2048 * GROUP


def _set(job, seg, seed, off):
    st = np.array([seed, off], dtype=np.uint64)
    job.live_of(0)[seg].copy_(torch.from_numpy(st.view(np.uint8)))
    torch.cuda.synchronize()
    return st


def _state(job, seg):
    return job.live_of(0)[seg].cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("n", [ONE_COUNTER, ONE_COUNTER + 1, 65 * GROUP + 3, 79 * GROUP, 80 * GROUP + 17, RESIDENT,
                               RESIDENT + 1, RESIDENT + GROUP + 5])
def test_two_states_in_turn(n):
    job = ESTJob(1, 4, [(0, 4)], 1, [16, 40, 16])
    try:
        segs = (0, 2)
        st = {s: _set(job, s, 0x9E3779B97F4A7C15 * (s + 1) & (1 << 63) - 1, (1 << 32) - n // 8 + s) for s in segs}
        masks = {s: torch.full((n + 16,), 7, dtype=torch.uint8, device=DEV) for s in segs}
        for _ in range(2):
            for s in segs:
                job.dropout_mask(0, s, masks[s][:n], 0.3)
        job.sync()
        for s in segs:
            oracle.dropout_mask(st[s], n, 0.3)
            want = oracle.dropout_mask(st[s], n, 0.3)
            assert np.array_equal(masks[s][:n].cpu().numpy(), want), s
            assert bool((masks[s][n:] == 7).all()) and np.array_equal(_state(job, s), st[s]), s
    finally:
        job.close()


def test_replays_of_a_captured_draw():
    n = 70 * GROUP + 9
    job = ESTJob(1, 4, [(0, 4)], 1, [16], use_streams="one")
    try:
        st = _set(job, 0, 12345, 77)
        mask = torch.zeros(n, dtype=torch.uint8, device=DEV)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=job.main):
            job.dropout_mask(0, 0, mask, 0.5)
        for k in range(4):
            if k == 2:                          # an eager draw between the replays
                job.dropout_mask(0, 0, mask, 0.5)
                job.sync()
            else:
                g.replay()
                torch.cuda.synchronize()
            assert np.array_equal(mask.cpu().numpy(), oracle.dropout_mask(st, n, 0.5)), k
            assert np.array_equal(_state(job, 0), st), k
    finally:
        job.close()


def _captured(job, mask, p):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=job.main):
        job.dropout_mask(0, 0, mask, p)
    return g


@pytest.mark.parametrize("n", [16 * 1024 + 1, 70 * GROUP + 9, RESIDENT + GROUP + 5])
def test_a_captured_draw_outlives_the_grouping_and_the_job(n):
    """What is recorded uses the live state and the mask alone, so memory that the library gives back is left alone."""
    live = torch.zeros(32, dtype=torch.uint8, device=DEV)[:16]
    job = ESTJob(2, 4, [(0, 4)], 1, [16], use_streams="one", live_alloc=lambda nb: live)
    mask = torch.zeros(n, dtype=torch.uint8, device=DEV)
    st = _set(job, 0, 987654321, (1 << 32) - 3)
    g = _captured(job, mask, 0.25)
    others = []
    for k in range(4):
        if k == 1:
            job.set_grouping([0, 0], [1, 0])
        if k == 3:
            job.close()
        # whatever has been given back is now someone else's: 512 bytes are torch's smallest block
        others += [torch.full((nb,), 0x5A, dtype=torch.uint8, device=DEV) for nb in [512] * 8 + [4096] * 8]
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(mask.cpu().numpy(), oracle.dropout_mask(st, n, 0.25)), k
        assert np.array_equal(live.cpu().numpy().view(np.uint64), st), k
        assert all(bool((t == 0x5A).all()) for t in others), k
        if k < 3:                               # and an eager draw of the job as it is now
            job.dropout_mask(0, 0, mask, 0.25)
            job.sync()
            assert np.array_equal(mask.cpu().numpy(), oracle.dropout_mask(st, n, 0.25)), k


def test_captured_and_eager_draws_side_by_side():
    """Two states bound one after the other: the first's draws replayed on a stream of their own while the second's
    are enqueued."""
    n = 3000 * GROUP + 1
    lives = [torch.zeros(16, dtype=torch.uint8, device=DEV) for _ in range(2)]
    job = ESTJob(1, 4, [(0, 4)], 1, [16], use_streams="one", live_alloc=lambda nb: lives[0])
    try:
        masks = [torch.zeros(n, dtype=torch.uint8, device=DEV) for _ in range(2)]
        st = [np.array([seed, 5], dtype=np.uint64) for seed in (11, 22)]
        for live, s in zip(lives, st):
            live.copy_(torch.from_numpy(s.view(np.uint8)))
        torch.cuda.synchronize()
        g = _captured(job, masks[0], 0.5)
        B.check(B.es_bind_live_state(job.h, 0, [lives[1].data_ptr()]), "es_bind_live_state", job.h)
        own = torch.cuda.Stream(DEV)
        for _ in range(6):
            with torch.cuda.stream(own):
                g.replay()
            job.dropout_mask(0, 0, masks[1], 0.5)
        torch.cuda.synchronize()
        for live, mask, s in zip(lives, masks, st):
            for _ in range(5):
                oracle.dropout_mask(s, n, 0.5)
            assert np.array_equal(mask.cpu().numpy(), oracle.dropout_mask(s, n, 0.5))
            assert np.array_equal(live.cpu().numpy().view(np.uint64), s)
    finally:
        job.close()
