"""The work a training job has libes do, as cases that can be timed and compared.

Kinds of case (the ``kind`` of a case), each through the public entry points:

  step     one whole global step on one worker: every EST's state is switched in, its dropout mask
           is drawn (if it has one), its flat gradient is staged and its state saved by
           es_est_boundary, then es_reduce_sgd_step
  hooks    the same step as a framework's gradient hooks drive it: one es_accumulate per bucket as
           it becomes ready, staging on a stream of its own, the averaged gradient stored as well
  update   the zero-copy step: backward passes wrote into the slots, so the ESTs are marked as
           present and es_reduce_sgd_step is all that is left
  clip     the zero-copy step with clipping: es_ring_order_reduce, es_grad_sq_norm, es_clip_sgd_step
  mask     one dropout mask from an EST's live RNG state
  bn       BatchNorm batch statistics of one layer
  switch   the small-state path alone: every EST draws a small mask and hands over to the next

Layouts are given as numbers: "resnet50", "bert-base" and "gpt2-medium" are the lengths of the DDP
buckets (25 MiB, reversed tensor order) of those tensor lists; "flat" is one bucket; "ragged" cuts
the vector into buckets of about ``cap`` elements whose lengths are odd and even in turn.

Every result is defined bit for bit (the order of every sum is fixed), so the tolerance is "exact";
``exact`` gives the same values from plain torch in 64 bits.
"""
import math

import numpy as np
import torch

from paper_2208_14228_amd import binding as B
from paper_2208_14228_amd.job import ESTJob

DEV = "cuda:0"
LR, MU = 0.1, 0.9
MAX_NORM, EPS = 0.5, 1e-6
GRAD_SIGMA = 1e-2 / math.sqrt(512.0)

LAYOUTS = {
    "resnet50": [7564264, 6563840, 7091712, 4337216],
    "bert-base": [7087872] * 12 + [24427776],
    "gpt2-medium": [8395776, 8397824, 8398848] * 12 + [52513792],
}
# channels of ResNet-50's 53 BatchNorm layers, as running mean and running variance each
BN_CHANNELS = ([64, 64, 64, 256, 256] + [64, 64, 256] * 2 + [128, 128, 512, 512] + [128, 128, 512] * 3
               + [256, 256, 1024, 1024] + [256, 256, 1024] * 5 + [512, 512, 2048, 2048] + [512, 512, 2048] * 2)


def listed():
    return [
        # the smallest step: N(0, 1e-2) gradients of a 1 M vector, four ESTs; launches and latency
        {"name": "step-1m-4", "kind": "step", "layout": "flat", "n": 4, "p": 1 << 20, "cap": 0, "align": 4,
         "bn": 0, "mask": 0},
        # a convolutional model with 8 ESTs, driven by gradient hooks, staging beside the compute
        {"name": "hooks-resnet50-8", "kind": "hooks", "layout": "resnet50", "n": 8, "p": 25557032, "cap": 0,
         "align": 4},
        # the same model with BatchNorm and RNG state switched at every one of 32 EST boundaries
        {"name": "step-resnet50-bn-32", "kind": "step", "layout": "resnet50", "n": 32, "p": 25557032, "cap": 0,
         "align": 4, "bn": 53, "mask": 0},
        # a language model with Dropout: every EST draws a 32x128x768 mask from its own RNG state
        {"name": "step-bert-mask-16", "kind": "step", "layout": "bert-base", "n": 16, "p": 109482240, "cap": 0,
         "align": 4, "bn": 0, "mask": 32 * 128 * 768},
        # the largest: 48 ESTs of a 355 M parameter model, gradients produced in the slots (68 GB read)
        {"name": "update-gpt2m-48", "kind": "update", "layout": "gpt2-medium", "n": 48, "p": 354823168, "cap": 0,
         "align": 4, "avg": 0},
        # a language model trained with gradient clipping
        {"name": "clip-bert-16", "kind": "clip", "layout": "bert-base", "n": 16, "p": 109482240, "cap": 0,
         "align": 4},
        # a small model (a few M parameters, odd bucket lengths, unaligned chunks) on many ESTs
        {"name": "update-ragged-4m-16", "kind": "update", "layout": "ragged", "n": 16, "p": 4000037, "cap": 1000003,
         "align": 1, "avg": 0},
        # the shortest vectors with the most ESTs
        {"name": "update-ragged-200k-64", "kind": "update", "layout": "ragged", "n": 64, "p": 200003, "cap": 66667,
         "align": 1, "avg": 1},
        # BatchNorm statistics of the first layer of a convolutional model, batch 32 ...
        {"name": "bn-32x64x112x112", "kind": "bn", "images": 32, "channels": 64, "positions": 112 * 112},
        # ... and of its last one: many channels, few and odd positions
        {"name": "bn-32x2048x7x7", "kind": "bn", "images": 32, "channels": 2048, "positions": 49},
        # a dropout mask over attention probabilities, 16x12x512x512
        {"name": "mask-50m", "kind": "mask", "n": 16 * 12 * 512 * 512, "drop": 0.1},
        # EST switches alone: RNG state and the 106 BatchNorm tensors of eight ESTs
        {"name": "switch-bn-8", "kind": "switch", "n": 8, "bn": 53, "mask": 1003},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["update"] * 4 + ["step"] * 3 + ["hooks", "clip", "bn", "bn", "mask", "switch"])
    if kind == "bn":
        images, side = _log(rng, 1, 256), rng.randint(1, 120)
        positions = side * side if rng.random() < 0.7 else rng.randint(1, 14400)
        channels = max(1, min(_log(rng, 3, 2048), 25_000_000 // (images * positions)))
        return {"kind": kind, "images": images, "channels": channels, "positions": positions}
    if kind == "mask":
        return {"kind": kind, "n": _log(rng, 1000, 150_000_000), "drop": rng.choice([0.1, 0.2, 0.5])}
    if kind == "switch":
        return {"kind": kind, "n": rng.randint(2, 16), "bn": rng.randint(0, 53), "mask": _log(rng, 100, 100_000)}
    n = _log(rng, 1, 64) if kind in ("update", "clip") else _log(rng, 2, 32)
    most = {"update": 5_000_000_000, "clip": 1_700_000_000, "step": 900_000_000, "hooks": 900_000_000}[kind]
    p = min(_log(rng, 20_000, 200_000_000), most // n)
    c = {"kind": kind, "layout": rng.choice(["flat", "ragged"]), "n": n, "p": p,
         "cap": rng.choice([p // 3 + 1, 6553600]), "align": rng.choice([1, 4])}
    if kind == "step":
        c["bn"] = rng.choice([0, 0, rng.randint(1, 53)])
        c["mask"] = rng.choice([0, _log(rng, 1000, 4_000_000)])
    if kind == "update":
        c["avg"] = rng.choice([0, 1])
    return c


# ---- inputs: a pure function of (case, seed), made on the GPU ------------------------------

def _lens(case):
    if case["layout"] == "flat":
        return [case["p"]]
    if case["layout"] in LAYOUTS:
        return list(LAYOUTS[case["layout"]])
    out, left, k = [], case["p"], 0
    while left:
        out.append(min(left, case["cap"] + (1237 * k) % 1024))
        left -= out[-1]
        k += 1
    return out


def _buckets(case):
    out, off = [], 0
    for n in _lens(case):
        out.append((off, n))
        off += n
    assert off == case["p"]
    return out


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1_000_003 + stream) & 0x7FFFFFFFFFFFFFFF)
    return g


def _normal(out, seed, stream, sigma):
    return out.normal_(0.0, sigma, generator=_gen(seed, stream))


def _grad(case, seed, e, out=None):
    out = torch.empty(case["p"], device=DEV) if out is None else out
    return _normal(out, seed, e, 1e-2 if case["layout"] == "flat" else GRAD_SIGMA)


def _param(case, seed):
    return _normal(torch.empty(case["p"], device=DEV), seed, 5000, 0.05)


def _momentum(case, seed):
    return _normal(torch.empty(case["p"], device=DEV), seed, 5001, 2 * GRAD_SIGMA)


def _philox_state(seed, e):
    return (0x9E3779B97F4A7C15 * (seed * 64 + e + 1)) & 0x7FFFFFFFFFFFFFFF, (e << 33) + seed % 97


def _segs(case):
    return [16] + [4 * c for c in BN_CHANNELS[:case["bn"]] for _ in (0, 1)]


class _Live:
    """The live tensors of one worker, cut out of one block at the 512-byte steps of torch's allocator."""

    def __init__(self, segs):
        self.at, off = [], 0
        for nb in segs:
            self.at.append((off, nb))
            off += -(-nb // 512) * 512
        self.block = torch.zeros(max(off, 512), dtype=torch.uint8, device=DEV)
        self.k = 0

    def __call__(self, nb):
        off, have = self.at[self.k]
        assert nb == have
        self.k += 1
        return self.block[off:off + nb]


def _fill_context(live, seed, e):
    """EST e's RNG state and running statistics, into the live tensors."""
    off, _ = live.at[0]
    live.block[off:off + 16].copy_(torch.from_numpy(np.array(_philox_state(seed, e), dtype=np.uint64).view(np.uint8)))
    for j, (off, nb) in enumerate(live.at[1:]):
        x = torch.empty(nb // 4, device=DEV)
        _normal(x, seed, 100_000 + 1000 * e + j, 1.0)
        live.block[off:off + nb].copy_(x.view(torch.uint8))


class State:
    pass


def prepare(case, seed):
    s, kind = State(), case["kind"]
    s.case, s.kind = case, kind
    if kind == "bn":
        shape = (case["images"], case["channels"], case["positions"])
        s.x = _bn_input(case, seed)
        s.mean = torch.zeros(case["channels"], device=DEV)
        s.var = torch.zeros(case["channels"], device=DEV)
        s.nws = B.es_bn_workspace_floats(*shape)
        s.ws = torch.zeros(s.nws, device=DEV)
        s.args = (s.x.data_ptr(), *shape, s.mean.data_ptr(), s.var.data_ptr(), s.ws.data_ptr(), s.nws,
                  torch.cuda.current_stream().cuda_stream)
        return s
    if kind in ("mask", "switch"):
        n, segs, p, buckets, align = (1, [16], 4, [(0, 4)], 4) if kind == "mask" else (case["n"], _segs(case), 4, [(0, 4)], 4)
    else:
        n, p, buckets, align = case["n"], case["p"], _buckets(case), case["align"]
        segs = _segs(case) if kind == "step" and (case["bn"] or case["mask"]) else []
    s.n, s.ids = n, list(range(len(buckets)))
    s.live = _Live(segs) if segs else None
    s.job = job = ESTJob(n, p, buckets, align, segs, use_streams="two" if kind == "hooks" else "one", live_alloc=s.live)
    s.h = job.h
    if segs:
        for e in range(n):
            _fill_context(s.live, seed, e)
            torch.cuda.synchronize()
            job.ctx_save(e)
            job.sync()
    if kind == "mask":
        job.ctx_restore(0)
        s.masks = [torch.zeros(case["n"], dtype=torch.uint8, device=DEV)]
    elif kind == "switch" or (kind == "step" and case["mask"]):
        s.masks = [torch.zeros(case["mask"], dtype=torch.uint8, device=DEV) for _ in range(n)]
    if kind == "switch":
        job.ctx_restore(0)
    if kind in ("mask", "switch"):
        torch.cuda.synchronize()
        return s
    job.p.copy_(_param(case, seed))
    job.v.copy_(_momentum(case, seed))
    if kind in ("step", "hooks"):
        s.grads = [_grad(case, seed, e) for e in range(n)]
        ptrs = [[g.data_ptr() + 4 * off for off, _ in buckets] for g in s.grads]
        s.ptrs = ptrs
        s.batch = [B.Marshalled(s.ids, q) for q in ptrs]
    else:
        base = B.es_grad_slot(s.h, 0, 0)
        slots = job.memory.blocks[base].view(torch.float32)
        s.ests, s.slots = list(range(n)), [B.es_grad_slot(s.h, e, 0) for e in range(n)]
        for e in range(n):
            a = (s.slots[e] - base) // 4
            _grad(case, seed, e, slots[a:a + p])
        s.norm2 = torch.zeros(2, device=DEV)
    torch.cuda.synchronize()
    return s


def _bn_input(case, seed):
    x = torch.empty(case["images"], case["channels"], case["positions"], device=DEV)
    _normal(x, seed, 1, 1.5)
    off = torch.empty(case["channels"], device=DEV)
    _normal(off, seed, 2, 1.0)
    return x.add_(off[None, :, None])


# ---- one pass ------------------------------------------------------------------------------

def run(s):
    case, kind = s.case, s.kind
    if kind == "bn":
        B.check(B.es_bn_batch_stats(*s.args), "es_bn_batch_stats")
        return {"mean": s.mean, "var": s.var}
    job, h, n = s.job, s.h, s.n
    if kind == "mask":
        B.check(B.es_dropout_mask(h, 0, 0, s.masks[0].data_ptr(), case["n"], case["drop"]), "es_dropout_mask", h)
        return {"mask": s.masks[0], "live": s.live.block}
    if kind == "switch":
        for e in range(n):
            job.dropout_mask(e, 0, s.masks[e], 0.1)
            job.ctx_switch(e, (e + 1) % n)
        return {"masks": s.masks, "live": s.live.block}
    if kind == "step":
        if s.live:
            job.ctx_restore(0)
        for e in range(n):
            if case["mask"]:
                job.dropout_mask(e, 0, s.masks[e], 0.1)
            B.check(B.es_est_boundary_m(h, e, e + 1 if e + 1 < n else B.ES_NO_EST, s.batch[e]), "es_est_boundary", h)
        job.reduce_sgd_step(LR, MU, store_avg=False)
        out = {"p": job.p, "v": job.v}
        if s.live:
            out["live"] = s.live.block
        if case["mask"]:
            out["masks"] = s.masks
        return out
    if kind == "hooks":
        for e in range(n):
            for b, q in zip(s.ids, s.ptrs[e]):
                B.check(B.es_accumulate(h, e, b, q), "es_accumulate", h)
        job.reduce_sgd_step(LR, MU, store_avg=True)
        return {"p": job.p, "v": job.v, "avg": job.avg}
    B.check(B.es_accumulate_many(h, s.ests, s.slots), "es_accumulate_many", h)
    if kind == "update":
        job.reduce_sgd_step(LR, MU, store_avg=bool(case["avg"]))
        return {"p": job.p, "v": job.v, "avg": job.avg} if case["avg"] else {"p": job.p, "v": job.v}
    job.ring_order_reduce()
    B.check(B.es_grad_sq_norm(h, job.avg.data_ptr(), s.norm2.data_ptr()), "es_grad_sq_norm", h)
    B.check(B.es_clip_sgd_step(h, job.p.data_ptr(), job.v.data_ptr(), job.avg.data_ptr(), s.norm2.data_ptr(),
                               MAX_NORM, EPS, LR, MU), "es_clip_sgd_step", h)
    return {"p": job.p, "v": job.v, "avg": job.avg, "norm2": s.norm2}


# ---- what a pass cannot do without ---------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "bn":
        m = case["images"] * case["channels"] * case["positions"]
        return {"bytes": 4 * m + 8 * case["channels"], "flops": 4 * m}
    if kind == "mask":
        # ten rounds of two 32x32->64 products and four exclusive ors per four bytes
        return {"bytes": case["n"], "flops": 60 * (case["n"] // 4)}
    ctx = sum(_segs(case)) if kind in ("switch", "step") else 0
    if kind == "switch":
        # save and restore: each EST's state is read and written once in each direction
        return {"bytes": case["n"] * (4 * ctx + case["mask"]), "flops": 60 * case["n"] * (case["mask"] // 4)}
    n, p = case["n"], case["p"]
    flops = (n + 4) * p
    if kind == "update":
        return {"bytes": 4 * p * (n + 4 + case["avg"]), "flops": flops}
    if kind == "clip":
        # the norm needs the whole average before the first parameter can change
        return {"bytes": 4 * p * (n + 1 + 1 + 5), "flops": flops + 3 * p}
    if kind == "hooks":
        return {"bytes": 4 * p * (3 * n + 5), "flops": flops}
    if not (case["bn"] or case["mask"]):
        ctx = 0
    # staging is a copy (the caller reuses its gradient buffers), and the reduce reads the copies
    return {"bytes": 4 * p * (3 * n + 4) + n * (4 * ctx + case["mask"]), "flops": flops + 60 * n * (case["mask"] // 4)}


def tolerance(case):
    """Bit for bit: the library fixes the order of every sum, and determinism is what it is for."""
    return "exact"


# ---- the same values in 64 bits, from plain torch ------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind in ("mask", "switch"):
        return None                     # bytes and copies only: compared as they are
    if kind == "bn":
        x = _bn_input(case, seed).double()
        mean = x.mean(dim=(0, 2))
        return {"mean": mean, "var": x.sub_(mean[None, :, None]).square_().mean(dim=(0, 2))}
    lr, mu = float(np.float32(LR)), float(np.float32(MU))
    g = torch.zeros(case["p"], dtype=torch.float64, device=DEV)
    row = torch.empty(case["p"], device=DEV)
    for e in range(case["n"]):
        g += _grad(case, seed, e, row)
    g /= case["n"]
    p, v = _param(case, seed).double(), _momentum(case, seed).double()
    out = {"avg": g.clone()} if kind in ("hooks", "clip") or case.get("avg") else {}
    if kind == "clip":
        sq = g.square().sum()
        out["norm2"] = torch.stack([sq, sq.sqrt()])
        coef = (float(np.float32(MAX_NORM)) / (sq.sqrt() + float(np.float32(EPS)))).clamp(max=1.0)
        g = g * coef
    v = v * mu + g
    return {**out, "p": p - lr * v, "v": v}
