"""The wave-tile form of the reduce (the default below 5 M parameters and up to 64 ranks, 8 M below 8) at the edges
of its rule and of its tiles: against the oracle's ring where that is small enough, and everywhere
against the tiled kernels an explicit launch-shape option selects, bit for bit."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2208_14228_amd import binding as B
    from paper_2208_14228_amd.job import ESTJob
    DEV = "cuda:0"

LR, MU = 0.1, 0.9


def make(N, lens, A, seed, special=False):
    """A job whose slots hold seeded gradients (written in place), and its rows on the host."""
    buckets, off = [], 0
    for n in lens:
        buckets.append((off, n))
        off += n
    job = ESTJob(N, off, buckets, A, use_streams="one")
    base = B.es_grad_slot(job.h, 0, 0)
    block = job.memory.blocks[base].view(torch.float32)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    rows = []
    for e in range(N):
        a = (B.es_grad_slot(job.h, e, 0) - base) // 4
        row = block[a:a + off]
        row.normal_(0.0, 1.0, generator=g)
        row.mul_(torch.exp2(torch.randint(-8, 8, (off,), device=DEV, generator=g).float()))
        if special:
            row[::7] = -0.0
            row[1::11] = 1e-41 * (e + 1)
            row[3::13] = float("inf")
            row[5::17] = float("-inf") if e % 2 else float("inf")
            row[6::19] = float("nan")
        rows.append(row)
    p0 = torch.empty(off, device=DEV).normal_(0.0, 1.0, generator=g)
    v0 = torch.empty(off, device=DEV).normal_(0.0, 1.0, generator=g)
    torch.cuda.synchronize()
    return job, rows, p0, v0, buckets


def step(job, p0, v0, how):
    job.p.copy_(p0); job.v.copy_(v0); job.avg.fill_(3.0)
    torch.cuda.synchronize()
    print(f"[gpu-case] wave reduce N={job.N} P={job.P} {how}", flush=True)
    B.check(B.es_accumulate_many(job.h, list(range(job.N)), [B.es_grad_slot(job.h, e, 0) for e in range(job.N)]),
            "es_accumulate_many", job.h)
    if how == "reduce":
        job.ring_order_reduce()
    else:
        job.reduce_sgd_step(LR, MU, store_avg=how == "fused+avg")
    job.sync()
    return [t.clone().view(torch.int32) for t in (job.avg, job.p, job.v)]


def same(a, b):
    """Equal bits; a NaN equals any NaN."""
    for x, y in zip(a, b):
        nan = torch.isnan(x.view(torch.float32)) & torch.isnan(y.view(torch.float32))
        if not bool(((x == y) | nan).all()):
            return False
    return True


def check(N, lens, A, seed, special=False, with_oracle=False):
    job, rows, p0, v0, buckets = make(N, lens, A, seed, special)
    try:
        got = {}
        for nt in (0, 1):
            job.set_option("nontemporal_pv", nt)
            for how in ("reduce", "fused", "fused+avg"):
                got[nt, how] = step(job, p0, v0, how)
        assert (B.es_get_option(job.h, "reduce_wave_width")[1] != 0) == (
            N <= 64 and job.P < (8_000_000 if N < 8 else 5_000_000))
        job.set_option("reduce_unroll", 2)                     # an explicit shape: the tiled kernels
        assert B.es_get_option(job.h, "reduce_wave_width")[1] == 0
        for (nt, how), w in got.items():
            assert same(w, step(job, p0, v0, how)), (N, A, nt, how)
        if with_oracle:
            host = [r.cpu().numpy() for r in rows]
            want = np.concatenate([oracle.ring_order_reduce(np.stack([h[o:o + n] for h in host]), A)
                                   for o, n in buckets if n])
            pw, vw = p0.cpu().numpy().copy(), v0.cpu().numpy().copy()
            oracle.sgd_momentum(pw, vw, want, LR, MU)
            for nt in (0, 1):
                avg, p, v = (t.cpu().numpy().view(np.uint32) for t in got[nt, "fused+avg"])
                assert np.array_equal(avg, want.view(np.uint32)), (N, A, nt)
                assert np.array_equal(p, pw.view(np.uint32)) and np.array_equal(v, vw.view(np.uint32)), (N, A, nt)
                assert torch.equal(got[nt, "reduce"][0], got[nt, "fused+avg"][0])
    finally:
        job.close()


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 23, 24, 31, 32, 33, 48, 63, 64, 65])
def test_ragged_layouts_against_the_ring(N):
    """Empty, tiny and odd buckets, chunks of every remainder, at chunk alignments 1 and 4."""
    for A in (1, 4):
        check(N, [3 * 4096 + 37, 0, 3, 1, 1001, 4 * N + 1, 2, 20_000 + N, 257 * N, 63, 64 * N + 1], A, N, with_oracle=True)


@pytest.mark.parametrize("N", [1, 2, 8, 17, 64])
def test_infinities_nan_and_denormals(N):
    check(N, [5000, 3, 40_001], 1, 100 + N, special=True)


@pytest.mark.parametrize("N,P", [
    (8, (128 << 10) - 1), (8, 128 << 10), (64, (128 << 10) + 1), (40, 131_073), (8, 299_999), (64, 300_000), (7, 300_001),
    (23, 400_003), (24, 400_003), (7, 1_499_999), (7, 1_500_000), (8, 1_500_001), (1, 1_500_003), (33, 1_000_000), (32, 999_999),
    (3, 7_999_999), (3, 8_000_000), (64, 1_200_005), (65, 100_003),
    (8, 4_999_999), (12, 5_000_000), (8, 8_000_001), (10, 8_100_019), (11, 8_000_001), (24, 2_000_003), (8, 64_000_000), (9, 63_999_999)])
def test_both_sides_of_every_line_of_the_rule(N, P):
    for A in (1, 4):
        check(N, [P // 3 + 1, P - 2 * (P // 3) - 2, P // 3 + 1], A, P + N)


def test_options_choose_the_shape_and_keep_their_values():
    job, rows, p0, v0, _ = make(9, [70_001], 1, 5)
    try:
        want = step(job, p0, v0, "fused+avg")
        assert B.es_set_option(job.h, "reduce_unroll", 3) == B.ES_EINVAL        # refused: nothing changes
        assert B.es_set_option(job.h, "reduce_tile_elems", 100) == B.ES_EINVAL
        n = B.es_query(job.h)[1]["n_reduce_tiles"]
        assert n >= 70_001 // 64
        job.set_option("reduce_lds_pad_kib", -1)
        job.set_option("nontemporal", 1)
        assert B.es_query(job.h)[1]["n_reduce_tiles"] == n
        for name, value in (("nontemporal", 0), ("reduce_rank_batch", 4), ("reduce_lds_pad_kib", 0),
                            ("reduce_tile_elems", 1024), ("reduce_big_unroll", 8)):
            job.set_option(name, value)
            assert B.es_get_option(job.h, name) == (B.ES_OK, value)
            assert same(want, step(job, p0, v0, "fused+avg")), name
            assert B.es_query(job.h)[1]["n_reduce_tiles"] < n
    finally:
        job.close()
