"""Single-window projections on both sides of each line between their forms:
window length, column tiles and rows, and FP64 modes on both sides of the size
where they are stored plainly, against X' (V Sigma^-1 W) and X (V Sigma^-1) in
FP64 from the library's own V, sigma and W.

Bound per entry: (m + 8) u (|X'| |C|), u the unit roundoff of the coefficients
and sums (m products and additions, and the coefficients' own rounding).
"""

import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [("f32", 131072, 48, 20), ("f32", 131073, 48, 20), ("f32", 131072, 49, 6), ("f32", 5000, 48, 24),
         ("f32", 5000, 32, 25), ("f32", 131073, 40, 8), ("f32", 131073, 41, 8), ("f32", 140001, 12, 12),
         ("f32", 140001, 13, 12), ("f32", 140001, 12, 3), ("f64", 1000, 32, 8), ("f64", 1000, 33, 8),
         ("f64", 1000, 32, 9), ("f64", 200001, 128, 8), ("f64", 200000, 128, 8), ("f64", 200001, 129, 8),
         ("f64", 524289, 32, 16), ("f64", 524288, 32, 16), ("f64", 524289, 33, 16)]


@pytest.mark.parametrize("dtype,n,m,r", CASES)
def test_forms(dtype, n, m, r):
    import paper_1612_07875_amd as dmd
    g = torch.Generator(device="cuda")
    g.manual_seed(n + m + r)
    u = 2.0 ** -23 if dtype == "f32" else 2.0 ** -52
    X = torch.randn((m + 1, n), generator=g, device="cuda", dtype=torch.float64 if dtype == "f64" else torch.float32)
    with dmd.Stream(n, m, r, dtype=dtype) as s:
        s.load_window(X)
        s.solve()
        sigma, V, _ = s.svd()
        _, W, _ = s.atilde()
        assert V.shape[1] == r
        P = torch.from_numpy(V / sigma[:r]).cuda()
        C = P.to(torch.complex128) @ torch.from_numpy(W).cuda()
        X64 = X.double()
        def within(out, got, Xw, coef):
            for part in ("real", "imag") if out.is_complex() else ("real",):
                c = getattr(coef, part).contiguous()
                err = (getattr(got, part).double() - c.T.contiguous() @ Xw).abs()
                assert (err <= (m + 8) * u * (coef.abs().T.contiguous() @ Xw.abs()) + 1e-300).all()
        for ld in (n + n % 2, n + 1 - n % 2):
            for fn, dt, Xw, coef in ((s.modes, s.mode_dtype, X64[1:], C), (s.pod, s.pod_dtype, X64[:m], P)):
                buf = torch.full((r, ld), 7.0, dtype=dt, device="cuda")
                fn(buf[:, :n].T)
                within(buf, buf[:, :n], Xw, coef)
                assert (buf[:, n:] == 7).all()
