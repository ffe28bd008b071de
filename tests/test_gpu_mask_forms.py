"""Dropout masks where the kernel's forms change, bit for bit with the state they leave: the longest
mask of one workgroup and one byte more, whole and part workgroups and lanes, counters whose low word
carries inside a wave, at its first and last counter and just outside it, thresholds 0, 1, 2^32 - 1
and 2^32 (nothing kept), aligned and unaligned masks."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2208_14228_amd.job import ESTJob
    DEV = "cuda:0"

SHORT = 16 * 1024
NS = [1, 15, 16, 17, 1023, 1024, 1025, 2 * SHORT, 2 * SHORT + 1, SHORT - 1, SHORT, SHORT + 1, SHORT + 16,
      4096 * 16 + 5, 300_007]
# a wave's counters are 256 in a row, the first one a multiple of 256 past the offset
OFFS = [0, (1 << 32) - 256, (1 << 32) - 255, (1 << 32) - 300, (5 << 32) - 1, (1 << 64) - 100]


@pytest.mark.parametrize("p", [0.0, 0.1, 2.0 ** -32, 1.0 - 2.0 ** -32, 1.0])
def test_mask_forms(p):
    for n in NS:
        job = ESTJob(1, 4, [(0, 4)], 1, [16])
        try:
            for off in OFFS:
                for shift in (0, 3):
                    st = np.array([0x0123456789ABCDEF * 3, off], dtype=np.uint64)
                    job.live_of(0)[0].copy_(torch.from_numpy(st.view(np.uint8)))
                    buf = torch.full((n + 40,), 7, dtype=torch.uint8, device=DEV)
                    torch.cuda.synchronize()
                    mask = buf[shift:shift + n]
                    want = []
                    for _ in range(2):          # the second draws from the state the first has left
                        job.dropout_mask(0, 0, mask, p)
                        job.sync()
                        want = oracle.dropout_mask(st, n, p)
                        assert np.array_equal(mask.cpu().numpy(), want), (n, off, shift)
                    assert np.array_equal(job.live_of(0)[0].cpu().numpy().view(np.uint64), st), (n, off, shift)
                    assert bool((buf[:shift] == 7).all()) and bool((buf[shift + n:] == 7).all()), (n, off, shift)
        finally:
            job.close()
