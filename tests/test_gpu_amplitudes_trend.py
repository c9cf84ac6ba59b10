"""Mode amplitudes where A~ is nearly defective (a linear trend: a Jordan block of
eigenvalue 1) or has an eigenvalue of zero: b = (W Lambda)^-1 alpha_1 has to hold
for the W and lambda that the library gives out, whatever the size of b.

A backward stable solve leaves |alpha_1 - W Lambda b| of a few k eps |W Lambda| |b|
(16 k eps here: elimination with partial pivoting, growth of 16); b that pass
the library's own check leave 64 eps |alpha_1|.
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


def _windows(rng, m, n):
    t = np.arange(m + 1)[:, None]
    a, b, c = rng.standard_normal((3, 1, n))
    yield "linear trend", t * a + b
    yield "trend and waves", t * a + b + np.cos(0.7 * t) * c + np.sin(0.7 * t) * a[:, ::-1]
    yield "quadratic trend", (t / m) ** 2 * a + t / m * b + c
    yield "pairs of equal frames", rng.standard_normal((m // 2 + 1, n))[np.arange(m + 1) // 2]
    yield "last frame zero", np.vstack([rng.standard_normal((m, n)), np.zeros((1, n))])
    yield "waves", np.cos(0.7 * t) * a + np.sin(0.7 * t) * b + 0.9 ** t * c


@pytest.mark.parametrize("m,r", [(2, 2), (5, 5), (9, 9), (16, 8), (33, 20), (64, 32), (120, 15), (200, 12)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_amplitudes(dtype, m, r):
    import paper_1612_07875_amd as dmd
    rng = np.random.default_rng([m, r])
    n = 300
    for name, X in _windows(rng, m, n):
        with dmd.Stream(n, m, r, dtype=dtype) as s:
            for x in torch.from_numpy(X.astype(np.float64 if dtype == "f64" else np.float32)).cuda():
                s.push(x)
            lam = s.eigs()[0]
            sigma, V, _ = s.svd()
            _, W, _ = s.atilde()
            b, _, _ = s.amplitudes()
        k = lam.size
        assert np.isfinite(b).all(), name
        A = (W * lam).astype(np.clongdouble)
        alpha = sigma[:k] * V[0]
        res = np.linalg.norm((A @ b.astype(np.clongdouble) - alpha).astype(complex))
        if np.abs(lam).min() < 1e-12:  # (an eigenvalue of zero: its mode cannot be fitted)
            continue
        bound = 64 * EPS * np.linalg.norm(alpha) + 16 * k * EPS * np.linalg.norm(A.astype(complex)) * np.linalg.norm(b)
        assert res <= bound, (name, res / bound)


@pytest.mark.parametrize("m,r", [(12, 4), (40, 8), (130, 6)])
def test_hermitian(m, r):
    import paper_1612_07875_amd as dmd
    rng = np.random.default_rng([m, r, 1])
    n = 200
    t = np.arange(m + 1)[:, None]
    a, b = rng.standard_normal((2, 1, n)) + 1j * rng.standard_normal((2, 1, n))
    idx = torch.arange(n, dtype=torch.int32, device="cuda")
    for X in (t * a + b, np.exp(0.4j * t) * (t * a + b), np.exp(0.4j * t) * a + np.exp(-1.1j * t) * b):
        with dmd.Stream(n, m, r, dtype="c64_csr", max_nnz=n) as s:
            for x in X.astype(np.complex64):
                s.push_csr(idx, torch.from_numpy(x).cuda())
            lam = s.eigs()[0]
            sigma, V, _ = s.svd()
            _, W, _ = s.atilde()
            amp, _, _ = s.amplitudes()
        k = lam.size
        A = (W * lam).astype(np.clongdouble)
        alpha = sigma[:k] * V[0].conj()
        res = np.linalg.norm((A @ amp.astype(np.clongdouble) - alpha).astype(complex))
        bound = 64 * EPS * np.linalg.norm(alpha) + 16 * k * EPS * np.linalg.norm(A.astype(complex)) * np.linalg.norm(amp)
        assert res <= bound, res / bound
