"""Windows on both sides of the length (8 columns) up to which the vectors'
kernel finds the eigenvalues itself: against LAPACK on the library's own Gram,
and alone, in blocks, in ticks and in a build-up start alike, bit for bit."""

import numpy as np
import pytest
import torch

from test_gpu_trid import check

pytestmark = pytest.mark.gpu


def _frames(m, n, count):
    rng = np.random.default_rng([8, m])
    return torch.from_numpy((rng.standard_normal((count, n)) * np.linspace(1.0, 3.0, n)).astype(np.float32)).cuda()


@pytest.mark.parametrize("m", [5, 7, 8, 9])
def test_short_windows(m):
    import paper_1612_07875_amd as dmd
    n, r = 200, min(m, 6)
    X = _frames(m, n, m + 9)
    with dmd.Stream(n, m, r, dtype="f64") as s:
        for x in X[:m + 1].double():
            s.push(x)
        check(s, s.gram(), m, r)
    with dmd.Stream(n, m, r, dtype="c64_csr") as s:
        idx = torch.arange(n, dtype=torch.int32, device="cuda")
        for t in range(m + 1):
            s.push_csr(idx, torch.complex(X[t], X[t + 4].flip(0)))
        check(s, s.gram(), m, r)
    alone, member, other = dmd.Stream(n, m, r), dmd.Stream(n, m, r), dmd.Stream(n, 33, 6)
    batch = dmd.Batch(max_streams=2)
    batch.attach(member)
    batch.attach(other)
    for x in X:
        alone.push(x)
        batch.tick([member, other], [x, x])
    a, b = alone.eigs(), member.eigs()
    assert a[2] == b[2] == 0 and np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    block, single = dmd.Stream(n, m, r, max_block=4), dmd.Stream(n, m, r, max_block=4)
    block.push_block(X[:4])
    block.push_block(X[4:8])
    block.push_block(X[m:m + 4])
    for x in [*X[:8], *X[m:m + 4]]:
        single.push_block(x[None])
    a, b = block.eigs(), single.eigs()
    assert a[2] == b[2] and np.allclose(a[1], b[1], rtol=1e-6) and a[0].size == b[0].size
    with dmd.Stream(n, m, r, dtype="f64", buildup=True) as s:  # partial windows of the same class
        for k, x in enumerate(X[:m + 1].double()):
            s.push(x)
            if k >= 2:
                sigma = s.svd()[0]
                ev = np.linalg.eigvalsh(s.gram()[:k, :k])[::-1]
                assert np.abs(sigma[:k] ** 2 - ev).max() <= 8 * (m + 8) * 2.0 ** -52 * ev[0]
