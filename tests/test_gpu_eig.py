"""The nonsymmetric solve at the edges of its runs of eight and four and at the
full 32 x 32: eigenpairs, amplitudes and modes against A~, V and sigma as the
library returns them."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def check(s, k):
    """Residuals of the eigenpairs and of the amplitudes.

    The Schur form is backward stable: 64 k eps ||A~|| bounds the residual of a
    unit eigenvector.  The amplitudes solve Y x = Z^* alpha by back
    substitution, so W Lambda b misses alpha by at most a small multiple of
    k eps sum |lambda_q b_q| (unit columns of W); the member of a conjugate
    pair that is set to its partner's conjugate moves by its conditioning,
    which cond(W) bounds.
    """
    lam, _, rc = s.eigs()
    At, W, _ = s.atilde()
    sigma, V, _ = s.svd()
    b = s.amplitudes()[0]
    assert rc == 0 and len(lam) == k and W.shape == (k, k)
    nrm = np.linalg.norm(At)
    assert np.abs(np.linalg.norm(W, axis=0) - 1).max() <= 64 * EPS
    assert np.linalg.norm(At @ W - W * lam, axis=0).max() <= 64 * (k + 4) * EPS * nrm
    top = np.abs(W) >= np.abs(W).max(axis=0) * (1 - 64 * EPS)  # (ties to rounding: either may be the real one)
    assert (top & (np.abs(W.imag) <= 64 * EPS) & (W.real > 0)).any(axis=0).all()
    assert (np.diff(np.abs(lam)) <= 4 * EPS * np.abs(lam[0])).all()
    alpha = sigma[:k] * V[0].conj()
    tol = 64 * (k + 4) * EPS * np.linalg.cond(W) * (np.linalg.norm(alpha) + np.abs(lam * b).sum())
    assert np.linalg.norm(W @ (lam * b) - alpha) <= tol
    return lam, W, sigma, V


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 10, 16, 17, 24, 25, 26, 31, 32])
def test_real(k):
    import paper_1612_07875_amd as dmd
    m, n = 40, 200
    X = np.random.default_rng([8, k]).standard_normal((m + 1, n)) * np.linspace(1.0, 3.0, n)
    with dmd.Stream(n, m, k, dtype="f64") as s:
        for t in range(m + 1):
            s.push(torch.from_numpy(X[t]).cuda())
        lam, W, sigma, V = check(s, k)
        cplx = lam[lam.imag != 0]
        assert np.isin(cplx.conj(), cplx).all()  # exact pairs
        C = (V[:, :k] / sigma[:k]) @ W
        phi = s.modes().cpu().numpy()  # (an n x m product: 64 m eps of its largest terms)
        tol = 64 * m * np.finfo(phi.dtype).eps * (np.abs(X[1:]).T @ np.abs(C)).max()
        assert np.abs(phi - X[1:].T @ C).max() <= tol


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 10, 16, 17, 24, 25, 26, 31, 32])
def test_complex(k):
    import paper_1612_07875_amd as dmd
    m, n = 40, 200
    rng = np.random.default_rng([9, k])
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    with dmd.Stream(n, m, k, dtype="c64_csr") as s:
        for t in range(m + 1):
            v = (rng.standard_normal(n) + 1j * rng.standard_normal(n)) * np.linspace(1.0, 3.0, n)
            s.push_csr(idx, torch.from_numpy(v.astype(np.complex64)).cuda())
        check(s, k)


@pytest.mark.parametrize("pairs", [1, 3, 16])
def test_rotations(pairs):
    """Undamped rotations: A~ is near-orthogonal and no 2 x 2 block splits into reals."""
    import paper_1612_07875_amd as dmd
    k = 2 * pairs
    m, n = 2 * k + 1, 4 * k
    Q = np.linalg.qr(np.random.default_rng(10).standard_normal((n, k)))[0]
    w = 0.3 + 2.5 * np.arange(pairs) / pairs
    t = np.arange(m + 1)[:, None]
    X = np.concatenate([np.cos(w * t), np.sin(w * t)], axis=1) @ Q.T
    with dmd.Stream(n, m, k, dtype="f64") as s:
        for x in X:
            s.push(torch.from_numpy(np.ascontiguousarray(x)).cuda())
        lam = check(s, k)[0]
    want = np.exp(1j * np.concatenate([w, -w]))
    assert max(np.abs(lam - v).min() for v in want) <= 1e-9
