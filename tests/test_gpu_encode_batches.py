"""Stroke encoding of large batches: on both sides of the size above which the sample offsets have
a launch of their own, the result is that of the same samples encoded a thousand at a time, and
the time grows with the batch, not with its square."""
import time

import numpy as np
import pytest
import torch

from tests.gpu_harness import log

pytestmark = pytest.mark.gpu


def _strokes(N, batch, seed):
    """One stroke of three points a sample."""
    pts = np.random.default_rng(seed).integers(0, N, size=(batch, 3, 2))

    def dev(a):
        return torch.tensor(np.ascontiguousarray(a), dtype=torch.int32).cuda()

    def part(lo, hi):
        return dev(pts[lo:hi].reshape(-1, 2)), dev(np.arange(0, 3 * (hi - lo) + 1, 3)), dev(np.arange(hi - lo))

    return part


@pytest.mark.parametrize("batch", [24576, 24577, 40000])
def test_offsets_of_large_batches(batch):
    from paper_1409_6070_amd.sscn import StrokeEncoder
    N, step = 12, 1000
    log(f"[encode] batch {batch}")
    part = _strokes(N, batch, 5)
    whole = StrokeEncoder(N, batch, batch * 40, "f32")
    c, f = whole.encode(*part(0, batch), batch)
    small = StrokeEncoder(N, step, step * 40, "f32")
    want_c, want_f = [], []
    for lo in range(0, batch, step):
        hi = min(batch, lo + step)
        pc, pf = small.encode(*part(lo, hi), hi - lo)
        want_c.append(pc + torch.tensor([lo, 0, 0], dtype=torch.int32, device="cuda"))
        want_f.append(pf.clone())
    assert torch.equal(c, torch.cat(want_c))
    assert torch.equal(f, torch.cat(want_f))


def test_time_grows_with_the_batch():
    """Eight times the samples: 6 to 7 times the time when every part is linear (the fixed part of a
    call is small), 20 and more with the offsets summed by every sample's workgroup."""
    from paper_1409_6070_amd.sscn import StrokeEncoder
    N, best = 12, {}
    for batch in (32768, 262144):
        p = _strokes(N, batch, 6)(0, batch)
        enc = StrokeEncoder(N, batch, batch * 40, "f32")
        t = []
        for _ in range(12):
            t0 = time.perf_counter()
            enc.encode(*p, batch)  # waits for the device
            t.append(time.perf_counter() - t0)
        best[batch] = min(t)
        log(f"[encode] batch {batch}: {min(t) * 1e6:.0f} us")
    assert best[262144] < 12 * best[32768], best
