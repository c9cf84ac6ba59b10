"""A tick reads every member's frame before it writes any member's modes: one
member follows the modes that another wrote, in place, in the tick before
(windows on both sides of the line where a tick runs in two chains, and on one
side), eagerly and replayed as graphs."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graphs", [0, 4])
@pytest.mark.parametrize("m_src,m_dst", [(66, 8), (8, 66), (16, 8), (66, 70)])
def test_frames_in_modes_buffers(m_src, m_dst, graphs):
    import paper_1612_07875_amd as dmd
    n, r = 300000, 4
    rng = np.random.default_rng(m_src + m_dst)
    data = [torch.from_numpy(rng.standard_normal(n).astype(np.float32)).cuda() for _ in range(5)]
    src = [dmd.Stream(n, m_src, r) for _ in range(2)]
    dst = [dmd.Stream(2 * n, m_dst, r) for _ in range(2)]
    batch = dmd.Batch(max_streams=2, graphs=graphs)
    batch.attach(src[0])
    batch.attach(dst[0])
    out = torch.zeros((r, n), dtype=torch.complex64, device="cuda").T
    out2 = torch.zeros((r, 2 * n), dtype=torch.complex64, device="cuda").T
    frame = torch.view_as_real(out.T[0]).reshape(-1)  # the first mode, interleaved, in place
    assert frame.data_ptr() == out.data_ptr()
    for t in range(m_src + m_dst + 8):
        x = sum(np.float32(np.cos(0.37 * t * (k + 1) + k)) * data[k] for k in range(5))
        before = frame.clone()
        batch.tick([src[0], dst[0]], [x, frame], [out, out2])
        src[1].push(x)
        dst[1].push(before)
        if t <= m_src:
            out.copy_(torch.view_as_complex(torch.stack([x, 0.5 * x + data[t % 5]], 1))[:, None].expand(n, r))
    torch.cuda.synchronize()
    for pair, o in ((src, out), (dst, out2)):
        a, b = pair[0].eigs(), pair[1].eigs()
        assert a[2] == b[2] and np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
        if pair is dst:
            assert torch.equal(pair[1].modes(torch.zeros_like(o.T).T)[:, :a[0].size], o[:, :a[0].size])
