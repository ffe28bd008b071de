"""Staging behind main without an event where main is idle: the rule on the CPU, and on the GPU every way in which main can
have work left when a copy is asked for."""
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
    """Gradients written by a kernel on main, by a copy on main, by another stream that main waits for, and long before, each
    right in front of the staging call and each behind work that takes a while."""
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
