"""Snapshots of batches past what the device holds at once, whose classes are launched
several times per snapshot interval."""
import numpy as np
import pytest

from paper_1706_07413_amd import adscl
from test_gpu_parity import FIELDS

pytestmark = pytest.mark.gpu

# grids, steps before, steps with snapshots, interval, threshold: a class alone whose last
# launch wraps round to instances that are through (300 instances on 256 compute units); a
# start off a multiple of the interval; both, for several classes; intervals that leave one
# launch each; instances at different steps, since some have collapsed
CASES = [([4097] * 300, 0, 256, 64, 0.0), ([2049] * 600, 50, 512, 256, 0.0),
         ([2049] * 520 + [4097] * 70 + [65], 7, 150, 48, 0.0), ([1025] * 900 + [2049] * 300 + [513], 50, 128, 33, 0.0),
         ([4097] * 300, 0, 60, 20, 0.0), ([2049] * 600, 30, 400, 100, 0.5)]


@pytest.mark.parametrize("Ns,before,steps,every,thr", CASES)
def test_every_snapshot_of_a_sliced_batch_is_written(Ns, before, steps, every, thr):
    """Every slot due, and no other, holds bit for bit the state of the instance alone."""
    Ns = np.array(Ns, np.int32)
    n = len(Ns)
    eps = np.linspace(0.5, 2.0 if thr == 0.0 else 30.0, n)
    sig = np.full(n, 0.2)
    slots = (before + steps) // every + 1
    print("sliced snapshots", n, before, steps, every, flush=True)

    def run(sel):
        b = adscl.Batch(Ns[sel], a_collapse=thr)
        b.init_gaussian(eps[sel], sig[sel])
        if before:
            b.step(before, 1e9)
        snaps = np.full((slots, 5, b.total), np.nan)
        b.step(steps, 1e9, every, snaps)
        st, off = b.status(), b.off
        b.close()
        return st, off, snaps

    st, off, snaps = run(slice(0, n))
    assert np.all((st["steps"] == before + steps) | (st["state"] == adscl.COLLAPSED))
    if thr == 0.0:
        assert np.all(st["state"] == adscl.RUNNING)
    else:
        assert np.any(st["state"] == adscl.COLLAPSED) and np.any(st["state"] == adscl.RUNNING)
    for b in range(n):
        for s in range(slots):
            # from the step at which the call finds the instance (it may have stopped before)
            due = min(before, st["steps"][b]) <= s * every <= st["steps"][b]
            got = snaps[s, :, off[b]:off[b] + Ns[b]]
            assert np.all(np.isnan(got) != due), (b, int(Ns[b]), s)
    for b in sorted({0, 79, 80, 255, 256, n // 2, n - 2, n - 1}):
        st1, _, alone = run(slice(b, b + 1))
        assert st1["steps"][0] == st["steps"][b]
        for s in range(slots):
            for f, name in enumerate(FIELDS):
                assert np.array_equal(snaps[s, f, off[b]:off[b] + Ns[b]], alone[s, f], equal_nan=True), (b, s, name)
