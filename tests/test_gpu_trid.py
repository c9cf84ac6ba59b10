"""The tridiagonal solve at the edges of its size classes: every window length
where the thread grid, the number of register blocks, the kernels or the padding
change, against LAPACK on the library's own Gram."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def check(s, G, m, r):
    """Residuals and values of the solve of the (m+1)-column Gram G (FP64).

    A backward stable reduction perturbs X^*X by at most a small multiple of
    m eps ||X^*X||: 8 m eps bounds eigenvalues and residuals.  The multisection
    adds eps (absolute, T scaled to a Gershgorin radius of at most 2 ||T||).
    Vectors of eigenvalues a gap g apart are orthogonal to within that
    perturbation over g.
    """
    sigma, V, rc = s.svd()
    At, W, _ = s.atilde()
    assert rc == 0 and V.shape == (m, min(r, m))
    k = V.shape[1]
    X2, xty = G[:m, :m], G[:m, 1:m + 1]
    ev = np.sort(np.abs(np.linalg.eigvalsh(X2)))[::-1]
    tol = 8 * (m + 8) * EPS * ev[0]
    assert np.abs(sigma ** 2 - ev).max() <= tol
    assert np.linalg.norm(X2 @ V - V * sigma[:k] ** 2, axis=0).max() <= tol
    gap = np.abs(ev[:k, None] - ev[None, :])
    gap[np.arange(k), np.arange(k)] = np.inf
    assert np.abs(V.conj().T @ V - np.eye(k)).max() <= 1e-13 + 2 * tol / gap.min()
    want = (V.conj().T @ xty @ V) / np.outer(sigma[:k], sigma[:k])
    assert np.abs(At - want).max() <= 64 * m * EPS * ev[0] / sigma[k - 1] ** 2
    R = At @ W - W * s.eigs()[0]
    assert np.abs(R).max() <= 1e-10 * max(1.0, np.abs(At).max())


@pytest.mark.parametrize("m", [2, 3, 15, 16, 17, 32, 33, 49, 64, 65, 95, 96, 97, 128, 129, 192, 193, 241, 256])
def test_real_windows(m):
    import paper_1612_07875_amd as dmd
    r = min(m, 32)
    rng = np.random.default_rng([5, m])
    n = 3 * m + 40
    X = torch.from_numpy(rng.standard_normal((m + 1, n)) * np.linspace(1.0, 3.0, n)).cuda()
    with dmd.Stream(n, m, r, dtype="f64", auto_solve=False) as s:
        for t in range(m + 1):
            s.push(X[t])
        s.solve()
        check(s, s.gram(), m, r)
    with dmd.Stream(n, m, r, dtype="f64") as s:  # the finalize fused with the reduction
        for t in range(m + 1):
            s.push(X[t])
        check(s, s.gram(), m, r)


@pytest.mark.parametrize("m", [2, 3, 16, 17, 32, 33, 64, 65, 127, 128, 129])
def test_hermitian_windows(m):
    import paper_1612_07875_amd as dmd
    r = min(m, 32)
    rng = np.random.default_rng([6, m])
    n = 3 * m + 40
    with dmd.Stream(n, m, r, dtype="c64_csr") as s:
        idx = torch.arange(n, dtype=torch.int32, device="cuda")
        for t in range(m + 1):
            v = (rng.standard_normal(n) + 1j * rng.standard_normal(n)) * np.linspace(1.0, 3.0, n)
            s.push_csr(idx, torch.from_numpy(v.astype(np.complex64)).cuda())
        check(s, s.gram(), m, r)


@pytest.mark.parametrize("scale", [1e-60, 1e60])
def test_extreme_scales(scale):
    """The reduction scales the Gram (squares of the data) by a power of two."""
    import paper_1612_07875_amd as dmd
    m, r, n = 24, 8, 300
    rng = np.random.default_rng(7)
    X = rng.standard_normal((m + 1, n))
    out = []
    for f in (1.0, scale):
        with dmd.Stream(n, m, r, dtype="f64") as s:
            for t in range(m + 1):
                s.push(torch.from_numpy(X[t] * f).cuda())
            lam, sigma, rc = s.eigs()
            assert rc == 0
            out.append((lam, sigma / f))
    assert np.abs(out[0][1] / out[1][1] - 1).max() < 1e-12
    assert np.abs(out[0][0] - out[1][0]).max() < 1e-9
