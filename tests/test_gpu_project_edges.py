"""Single-window projections at their edges: ragged rows, windows that end
inside a group of k-steps, every number of column tiles, and outputs that allow
only narrow stores, against X' (V Sigma^-1 W) and X (V Sigma^-1) in FP64 from the
library's own V, sigma and W.

Bound per entry: (m + 8) u (|X'| |C|), u the unit roundoff of the coefficients
and sums (m products and additions, and the coefficients' own rounding).
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,precision,u", [("f32", "default", 2.0 ** -23), ("f64", "default", 2.0 ** -52),
                                               ("f32", "fp64", 2.0 ** -52)])
@pytest.mark.parametrize("n,m,r", [(1, 2, 1), (63, 5, 3), (64, 16, 8), (65, 17, 9), (257, 33, 16), (300, 40, 17),
                                   (511, 64, 24), (1000, 90, 25), (4097, 130, 32)])
def test_projection(dtype, precision, u, n, m, r):
    import paper_1612_07875_amd as dmd
    rng = np.random.default_rng([n, m, r])
    X = rng.standard_normal((m + 1, n))
    if dtype == "f32":
        X = X.astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    with dmd.Stream(n, m, r, dtype=dtype, precision=precision, rcond=1e-6) as s:
        for t in range(m + 1):
            s.push(Xd[t])
        sigma, V, _ = s.svd()
        _, W, _ = s.atilde()
        k = V.shape[1]
        C = (V / sigma[:k]) @ W
        P = V / sigma[:k]
        X64 = X.astype(np.float64)
        ref, pref = X64[1:].T @ C, X64[:m].T @ P
        bound = (m + 8) * u * (np.abs(X64[1:].T) @ np.abs(C)) + 1e-300
        pbound = (m + 8) * u * (np.abs(X64[:m].T) @ np.abs(P)) + 1e-300
        # aligned, an odd leading dimension, and a start 8 bytes past alignment
        for ld, off in ((n + (n & 1), 0), (n + 1 - (n & 1), 0), (n + 2 + (n & 1), 1)):
            buf = torch.full((r * ld + off + 1,), 7.0, dtype=s.mode_dtype, device="cuda")
            out = buf[off:off + r * ld].view(r, ld)[:, :n].T
            got = s.modes(out).cpu().numpy()
            assert (np.abs(got[:, :k] - ref) <= bound).all()
            pad = buf[off:off + r * ld].view(r, ld)[:, n:]
            assert (pad == 7).all() and buf[-1] == 7  # nothing written past the rows
            pbuf = torch.full((r * ld + off + 1,), 7.0, dtype=s.pod_dtype, device="cuda")
            pout = pbuf[off:off + r * ld].view(r, ld)[:, :n].T
            pgot = s.pod(pout).cpu().numpy()
            assert (np.abs(pgot[:, :k] - pref) <= pbound).all()
            assert (pbuf[off:off + r * ld].view(r, ld)[:, n:] == 7).all() and pbuf[-1] == 7
