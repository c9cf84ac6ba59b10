"""Kernel timing of eager ticks: every launch is bracketed on the stream it runs
on, also where a tick runs in two chains (windows on both sides of m = 64)."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _tick_times(shapes, modes):
    import paper_1612_07875_amd as dmd
    rng = np.random.default_rng(5)
    streams = [dmd.Stream(n, m, r) for n, m, r in shapes]
    data = [torch.from_numpy(rng.standard_normal((m + 1, n)).astype(np.float32)).cuda() for n, m, _ in shapes]
    batch = dmd.Batch(max_streams=len(shapes))
    for s, x in zip(streams, data):
        for f in x:
            s.push(f)
        batch.attach(s)
    out = [torch.zeros((r, n), dtype=torch.complex64, device="cuda").T for n, _, r in shapes]
    torch.cuda.synchronize()
    dmd.profile_enable(True)
    dmd.profile_reset()
    batch.tick(streams, [x[0] for x in data], [o if w else None for o, w in zip(out, modes)])
    torch.cuda.synchronize()
    dmd.profile_enable(False)
    got = {k: dmd.profile_read("batch_" + k) for k in ("gram", "solve", "project")}
    dmd.profile_reset()
    batch.close()
    return got


def test_both_chains_are_timed():
    wide, narrow = (20000, 120, 32), (20000, 16, 6)
    for shapes, modes, launches in (([wide, narrow], [1, 1], (1, 2, 2)), ([wide, narrow], [0, 1], (1, 2, 1)),
                                    ([wide, narrow], [1, 0], (1, 2, 2)), ([wide, wide], [1, 1], (1, 1, 1)),
                                    ([narrow, narrow], [1, 1], (1, 1, 1))):
        got = _tick_times(shapes, modes)
        assert tuple(got[k][0] for k in ("gram", "solve", "project")) == launches, (shapes, modes, got)
        assert all(ms > 0 for _, ms in got.values()), got
