"""Eigenvalues of A~ against extended precision: a double-shift QR iteration with
reflectors that are orthogonal to their rounding is as exact as LAPACK's on the
same matrix; sqrt(2) of its error is allowed in the geometric mean.
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _eigenvalues(A):
    """Eigenvalues in extended precision (LAPACK's, corrected twice to first order), and LAPACK's."""
    lam, W = np.linalg.eig(A)
    Al, Wl, Wi = A.astype(np.clongdouble), W.astype(np.clongdouble), np.linalg.inv(W).astype(np.clongdouble)
    for _ in range(2):
        Wi = Wi + (np.eye(len(lam)) - Wi @ Wl) @ Wi
        M = Wi @ Al @ Wl
        d = np.diag(M)
        D = d[None, :] - d[:, None] + np.eye(len(d))
        E = (M - np.diag(d)) / D
        Wl, Wi = Wl + Wl @ E, Wi - E @ Wi
    return np.diag(Wi @ Al @ Wl), lam


@pytest.mark.parametrize("m,r", [(16, 5), (32, 10), (64, 20), (64, 32)])
def test_eigenvalues_as_exact_as_lapack(m, r):
    import paper_1612_07875_amd as dmd
    ours, lapack = [], []
    t = np.arange(m + 1)
    for seed in range(40):
        rng = np.random.default_rng([seed, m, r, 2])
        cols = [np.ones(m + 1)] if r % 2 else []
        w = r // 2
        for j in range(w):
            f, ph = np.pi * (j + 1) / (w + 1), rng.uniform(0, 6)
            a = 10.0 ** (-j / w) * np.exp(-0.002 * j * t)
            cols += [a * np.cos(f * t + ph), a * np.sin(f * t + ph)]
        X = np.stack(cols, 1) @ rng.standard_normal((r, 2000)) + 1e-3 * rng.standard_normal((m + 1, 2000))
        with dmd.Stream(2000, m, r, dtype="f64") as s:
            s.load_window(torch.from_numpy(X).cuda())
            s.solve()
            A, _, status = s.atilde()
            lam = s.eigs()[0]
        assert status == 0 and lam.size == r
        exact, theirs = _eigenvalues(A)
        near = lambda x: np.linalg.norm((x - exact[np.argmin(np.abs(exact[:, None] - x[None, :]), axis=0)]).astype(complex))
        ours.append(near(lam))
        lapack.append(near(theirs))
    ratio = np.exp(np.mean(np.log(ours) - np.log(lapack)))
    print(f"m={m} r={r}: error {ratio:.2f} of LAPACK's")
    assert ratio <= np.sqrt(2)
