"""Staging behind main without an event where main is idle: the rule on the CPU; on the GPU what the first staging call of a
handle asks of a main that works or is idle, for several writers of the gradient and every staging entry point, and many steps
of which the rule remembers the ones before."""
import ctypes
import os
import subprocess

import pytest
import torch

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

if torch.cuda.is_available():
    from paper_2208_14228_amd import binding as B
    from paper_2208_14228_amd.job import ESTJob
    DEV = "cuda:0"

    class Probe(ctypes.Structure):
        _fields_ = [("idle", ctypes.c_void_p), ("done", ctypes.c_void_p)]

    ASK = ctypes.CFUNCTYPE(ctypes.c_bool, ctypes.c_void_p)


@pytest.fixture
def answers():
    """What the library asks the runtime about main from here on, with the answers: [("idle" or "done", answer)]."""
    probe = Probe.in_dll(B.lib(), "_ZN2es12stream_probeE")
    kept = probe.idle, probe.done
    log = []

    def listen(name, address):
        ask = ASK(address)

        def asked(of):
            log.append((name, ask(of)))
            return log[-1][1]
        return ASK(asked)

    ears = [listen("idle", kept[0]), listen("done", kept[1])]
    probe.idle, probe.done = (ctypes.cast(f, ctypes.c_void_p).value for f in ears)
    yield log
    probe.idle, probe.done = kept


def keep_busy(slow):
    """Some milliseconds of work on the current stream."""
    for _ in range(20):
        slow.add_(1.0)


def test_the_rule(tmp_path):
    exe = str(tmp_path / "host_probe")
    pkg = os.path.join(ROOT, "paper_2208_14228_amd", "csrc")
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"),
                           "-I", pkg, "-I", "/opt/rocm/include", os.path.join(HERE, "c_abi", "host_probe.cpp"),
                           os.path.join(pkg, "es_api.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and "passed" in out.stdout, out.stdout + out.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("streams", ["two", "three"])
def test_staged_gradients_are_those_of_the_last_write(streams):
    """Many steps on one handle: gradients written by a kernel on main, by a copy on main, by another stream that main waits for,
    and long before, each right in front of the staging calls and each behind work that takes a while.  Which of the calls ask
    is the rule's to say here."""
    P, N = 1 << 20, 4
    job = ESTJob(N, P, [(0, P // 4)] + [(P // 4 + k, 1) for k in range(3)] + [(P // 4 + 3, P - P // 4 - 3)], 4, use_streams=streams)
    g = torch.zeros(P, device=DEV)
    slow = torch.zeros(1 << 27, device=DEV)
    other = torch.cuda.Stream(DEV)
    values = torch.arange(64, dtype=torch.float32, device=DEV).repeat_interleave(P).view(64, P)
    for step in range(12):
        want = []
        for e in range(N):
            v = float((step * N + e) % 64)
            want.append(v)
            how = (step + e) % 4
            busy = (step // 4) % 2 == 0
            if how == 2:                                    # another stream that main waits for
                other.wait_stream(job.stage)                # (the buffer is written again: behind the last copies)
                with torch.cuda.stream(other):
                    if busy:
                        slow.add_(1.0)
                    g.fill_(v)
                job.main.wait_stream(other)
            else:
                job.main.wait_stream(job.stage)
                with torch.cuda.stream(job.main):
                    if busy:
                        slow.add_(1.0)
                    if how == 1:
                        g.copy_(values[int(v)])
                    else:
                        g.fill_(v)
                if how == 3:
                    torch.cuda.synchronize()                # main is idle
            for b, (off, _) in enumerate(job.buckets):
                B.check(B.es_accumulate(job.h, e, b, g.data_ptr() + 4 * off), "es_accumulate", job.h)
        job.ring_order_reduce()
        job.sync()
        torch.cuda.synchronize()
        slots = [job.memory.blocks[B.es_grad_slot(job.h, 0, 0)].view(torch.float32)]
        base = B.es_grad_slot(job.h, 0, 0)
        for e in range(N):
            a = (B.es_grad_slot(job.h, e, 0) - base) // 4
            assert bool((slots[0][a:a + P] == want[e]).all()), (step, e)
    job.close()


def enter(job, entry, g):
    """All of EST 0's gradient by the named entry point."""
    if entry == "many":
        return B.es_accumulate_many(job.h, [0], [g.data_ptr()])
    if entry == "one":
        return B.es_accumulate(job.h, 0, 0, g.data_ptr())
    f = {"batch": B.es_accumulate_batch, "boundary": lambda h, e, b, d: B.es_est_boundary(h, e, B.ES_NO_EST, b, d)}[entry]
    return f(job.h, 0, [0], [g.data_ptr()])


@pytest.mark.gpu
@pytest.mark.parametrize("busy", [True, False])
@pytest.mark.parametrize("writer,entry", [("kernel", e) for e in ("one", "batch", "many", "boundary")]
                         + [(w, "one") for w in ("copy", "host copy", "another stream", "graph")])
def test_first_staging_call_asks_main(writer, entry, busy, answers):
    """A new handle has learned nothing and asks main itself: an event where it works, none where it is idle (which the
    runtime may deny where a stream's last work was a copy from the host, a graph or a wait for another stream), and the staged
    values are the last ones written, whoever writes them."""
    P = 1 << 20
    job = ESTJob(1, P, [(0, P)], 4, use_streams="two")
    g = torch.full((P,), -1.0, device=DEV)
    new = torch.arange(P, dtype=torch.float32, device=DEV)
    pinned = torch.empty(P, pin_memory=True)
    pinned.copy_(new)
    slow = torch.zeros(1 << 27, device=DEV)
    other = torch.cuda.Stream(DEV)
    graph = torch.cuda.CUDAGraph()
    if writer == "graph":
        with torch.cuda.graph(graph, stream=job.main):
            g.copy_(new).mul_(1.0)
    g.fill_(-1.0)
    torch.cuda.synchronize()
    with torch.cuda.stream(other if writer == "another stream" else job.main):
        if busy:
            keep_busy(slow)
        if writer == "graph":
            graph.replay()
        elif writer == "host copy":
            g.copy_(pinned, non_blocking=True)
        elif writer == "kernel":
            torch.add(new, 0.0, out=g)
        else:
            g.copy_(new)
    job.main.wait_stream(other)
    if not busy:
        torch.cuda.synchronize()
    print(f"[gpu-case] first staging call: {writer}, {entry}, busy {busy}", flush=True)
    B.check(enter(job, entry, g), "staging", job.h)
    print(answers, flush=True)
    assert answers == [("idle", False)] or (not busy and answers == [("idle", True)])
    assert busy or answers[0][1] or writer not in ("kernel", "copy")
    job.ring_order_reduce()
    job.sync()
    torch.cuda.synchronize()
    slot = job.memory.blocks[B.es_grad_slot(job.h, 0, 0)].view(torch.float32)[:P]
    assert torch.equal(slot, new) and torch.equal(job.avg, new)
    job.close()


@pytest.mark.gpu
def test_an_error_of_somebody_else_stays(answers):
    """Main and the event on it are asked while they work, which is answered with a status that is no error: an error that
    another library has left in this thread is still there afterwards."""
    hip = ctypes.CDLL([line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line][0])
    P = 1 << 16
    job = ESTJob(6, P, [(0, P)], 4, use_streams="two")
    g = torch.ones(P, device=DEV)
    slow = torch.zeros(1 << 27, device=DEV)
    for e in range(6):                                  # loads the kernels
        B.check(B.es_accumulate(job.h, e, 0, g.data_ptr()), "es_accumulate", job.h)
    job.ring_order_reduce()
    B.check(B.es_set_streams(job.h, *(s.cuda_stream for s in (job.main, job.ctx, job.stage))), "es_set_streams", job.h)
    torch.cuda.synchronize()
    answers.clear()
    with torch.cuda.stream(job.main):
        keep_busy(slow)
    left = hip.hipSetDevice(9999)
    status = [B.es_accumulate(job.h, e, 0, g.data_ptr()) for e in range(6)]
    still = hip.hipGetLastError()
    assert status == [B.ES_OK] * 6 and left != 0
    assert answers == [("idle", False), ("done", False), ("done", False)]
    assert still == left
    job.ring_order_reduce()
    job.sync()
    torch.cuda.synchronize()
    assert bool((job.avg == 1.0).all())
    job.close()
