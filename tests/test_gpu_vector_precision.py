"""Eigenvectors of graded windows (singular values over three decades), where a
loss of one or two bits shows.

The eigenvalues of the tridiagonal T are resolved to d(l) = 8 eps l + 2^-59 l_1
(Sturm counts in FP64 down to the bracket, against the same counts in extended
precision).  A vector for an eigenvalue off by d, taken where it is largest, has
at most sqrt(m) d / gap of another one, and the back-transformation leaves
2 m eps: |v_i^* v_j| <= sqrt(m) (d(l_i) + d(l_j)) / |l_i - l_j| + 2 m eps.
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


def _patterns(rng, m, r, low):
    t = np.arange(m + 1)
    w = r // 2
    cols = []
    for j in range(w):
        f, a, ph = np.pi * (j + 0.5) / w, low ** (j / (w - 1)), rng.uniform(0, 6)
        cols += [a * np.cos(f * t + ph), a * np.sin(f * t + ph)]
    return np.stack(cols, 1)


def _check_orthogonal(V, sigma, m):
    k = V.shape[1]
    lam = sigma[:k] ** 2
    VL = V.astype(np.clongdouble)
    off = np.abs((VL.conj().T @ VL - np.eye(k)).astype(np.complex128))
    d = 8 * EPS * lam + 2.0 ** -59 * lam[0]
    gap = np.abs(lam[:, None] - lam[None, :]) + np.diag(np.full(k, np.inf))
    bound = np.sqrt(m) * (d[:, None] + d[None, :]) / gap + 2 * m * EPS
    assert (off <= bound).all(), (off / bound).max()


@pytest.mark.parametrize("m,r", [(24, 10), (32, 10), (64, 20), (120, 16), (160, 16), (250, 16)])
def test_vectors_of_graded_windows(m, r):
    import paper_1612_07875_amd as dmd
    for seed in range(8):
        rng = np.random.default_rng([seed, m, r])
        X = _patterns(rng, m, r, 3e-3) @ rng.standard_normal((r, 2000)) + 1e-6 * rng.standard_normal((m + 1, 2000))
        with dmd.Stream(2000, m, r, dtype="f64") as s:
            s.load_window(torch.from_numpy(X).cuda())
            s.solve()
            sigma, V, status = s.svd()
        assert status == 0 and V.shape[1] == r
        _check_orthogonal(V, sigma, m)


@pytest.mark.parametrize("m,r", [(24, 10), (64, 20), (120, 16)])
def test_vectors_of_graded_hermitian_windows(m, r):
    import paper_1612_07875_amd as dmd
    n, nnz = 4096, 600
    for seed in range(4):
        rng = np.random.default_rng([seed, m, r, 1])
        C = _patterns(rng, m, r, 1e-2) * np.exp(0.3j * np.arange(m + 1))[:, None]
        X = C @ (rng.standard_normal((r, nnz)) + 1j * rng.standard_normal((r, nnz)))
        idx = torch.from_numpy(np.sort(rng.choice(n, nnz, replace=False)).astype(np.int32)).cuda()
        with dmd.Stream(n, m, r, dtype="c64_csr", max_nnz=nnz) as s:
            for x in X.astype(np.complex64):
                s.push_csr(idx, torch.from_numpy(x).cuda())
            sigma, V, status = s.svd()
        assert status == 0 and V.shape[1] == r
        _check_orthogonal(V, sigma, m)
