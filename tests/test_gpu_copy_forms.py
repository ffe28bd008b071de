"""Staging copies on both sides of the line between the short form (two waves per workgroup, plain
loads) and the long one (one wave, streaming loads): every entry point, sources aligned with the slot
and not, bytes outside the bucket untouched."""
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2208_14228_amd import binding as B
    from paper_2208_14228_amd.job import ESTJob
    DEV = "cuda:0"

LINE = 3 << 20


@pytest.mark.parametrize("total", [1, 5, 511, 512, 513, 4099, LINE - 1, LINE, LINE + 1])
@pytest.mark.parametrize("shift", [0, 1, 7])
def test_copies_around_the_line(total, shift):
    lens = [total // 3, total - total // 3] if total > 2 else [total]
    buckets, off = [], 0
    for n in lens:
        buckets.append((off, n))
        off += n
    N = 4
    job = ESTJob(N, total, buckets, 1, [16], use_streams="one")
    try:
        g = torch.Generator(device=DEV)
        g.manual_seed(total + shift)
        src = [torch.empty(total + 16, device=DEV).normal_(0, 1, generator=g) for _ in range(N)]
        flat = [s[shift:shift + total] for s in src]
        ptr = [[f.data_ptr() + 4 * o for o, _ in buckets] for f in flat]
        base = B.es_grad_slot(job.h, 0, 0)
        arena = job.memory.blocks[base].view(torch.float32)
        arena.fill_(-7.0)
        for e in range(N):
            job.ctx_save(e)
        job.sync()
        torch.cuda.synchronize()
        ids = list(range(len(buckets)))
        print(f"[gpu-case] staging total={total} shift={shift}", flush=True)
        for b in ids:
            B.check(B.es_accumulate(job.h, 0, b, ptr[0][b]), "es_accumulate", job.h)
        B.check(B.es_accumulate_batch(job.h, 1, ids, ptr[1]), "es_accumulate_batch", job.h)
        B.check(B.es_est_boundary(job.h, 2, None, ids, ptr[2]), "es_est_boundary", job.h)
        B.check(B.es_accumulate_many(job.h, [3], [flat[3].data_ptr()]), "es_accumulate_many", job.h)
        job.sync()
        for e in range(N):
            a = (B.es_grad_slot(job.h, e, 0) - base) // 4
            assert torch.equal(arena[a:a + total].view(torch.int32), flat[e].view(torch.int32)), e
            end = (B.es_grad_slot(job.h, e + 1, 0) - base) // 4 if e + 1 < N else arena.numel()
            assert bool((arena[a + total:end] == -7.0).all()), e
    finally:
        job.close()
