"""Ticks of windows on both sides of the size where a tick forks into two chains
(m = 64 | 65), and of one side alone: every member's results equal its own
pushes' bit for bit, eagerly and replayed as graphs, with eager work and
synchronizations between the ticks."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPES = [(3000, 16, 6), (40000, 65, 20), (5003, 64, 24), (20000, 128, 32), (1025, 8, 3), (6000, 130, 16)]


@pytest.mark.parametrize("graphs", [0, 4])
def test_chains_equal_alone(graphs):
    import paper_1612_07875_amd as dmd
    rng = np.random.default_rng(12)
    ticks = 140
    data = [torch.from_numpy(rng.standard_normal((8, n)).astype(np.float32)).cuda() for n, _, _ in SHAPES]
    frame = lambda i, t: data[i][t % 8] * (1.0 + 0.01 * ((7 * t) % 11)) + data[i][(3 * t + 1) % 8]
    alone = [dmd.Stream(n, m, r) for n, m, r in SHAPES]
    members = [dmd.Stream(n, m, r) for n, m, r in SHAPES]
    batch = dmd.Batch(max_streams=len(SHAPES), graphs=graphs)
    for s in members:
        batch.attach(s)
    both = list(range(len(SHAPES)))
    subsets = [both, [0, 2, 4], both[::-1], [1, 3, 5], both, [0, 3], both]
    for t in range(ticks):
        which = both if t < 132 else subsets[t - 132] if t - 132 < len(subsets) else both
        xs = [frame(i, t) for i in which]
        want = t >= 130
        out = [torch.full((SHAPES[i][2], SHAPES[i][0]), -1.0, dtype=torch.complex64, device="cuda").T
               for i in which] if want else None
        batch.tick([members[i] for i in which], xs, out)
        for k, i in enumerate(which):
            alone[i].push(xs[k])
        if not want:
            continue
        for k, i in enumerate(which):
            a, b = alone[i].eigs(), members[i].eigs()
            assert a[2] == b[2]  # (the data has fewer directions than some r)
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), (t, i)
            phi = alone[i].modes(torch.full_like(out[k], -1.0))
            assert torch.equal(phi, out[k]), (t, i)
        torch.cuda.synchronize()


def test_shared_event_orders_streams():
    """A tick records one event for its members: their later work on other
    streams, and other batches' ticks, still follow it, also after the batch
    is gone."""
    import paper_1612_07875_amd as dmd
    rng = np.random.default_rng(13)
    shapes = [(300000, 16, 6), (200000, 66, 20), (100000, 32, 12)]
    data = [torch.from_numpy(rng.standard_normal((80, n)).astype(np.float32)).cuda() for n, _, _ in shapes]
    streams = [torch.cuda.Stream() for _ in range(3)]
    alone = [dmd.Stream(n, m, r) for n, m, r in shapes]
    members = [dmd.Stream(n, m, r) for n, m, r in shapes]
    torch.cuda.synchronize()
    batch = None
    for t in range(80):
        if t % 16 == 0:
            if batch is not None:
                batch.close()
            batch = dmd.Batch(max_streams=3)
            for s in members:
                batch.attach(s)
        which = [0, 1, 2] if t % 3 else [t % 2, 2]
        batch.tick([members[i] for i in which], [data[i][t] for i in which], stream=streams[t % 3])
        for i in set(range(3)) - set(which):  # the others by pushes of their own, on another stream
            members[i].push(data[i][t], stream=streams[(t + 1) % 3])
        for i in range(3):
            alone[i].push(data[i][t])
    batch.close()
    for i in range(3):
        phi = members[i].modes(stream=streams[i])
        a, b = alone[i].eigs(), members[i].eigs()
        want = alone[i].modes()
        torch.cuda.synchronize()
        assert a[2] == b[2] == 0 and np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
        assert torch.equal(phi, want)
