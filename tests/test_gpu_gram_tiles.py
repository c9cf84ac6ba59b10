"""The whole-window Gram where its tiling changes: 16-column blocks, the groups
of tiles (one to 112 columns, three to 208, six beyond in FP64; by the row
ranges in FP32 and split BF16), ragged rows and windows shorter than a stage.

Tolerances as for the whole Gram elsewhere: |dG_ij| <= tol sqrt(G_ii G_jj), 1e-12
for FP64 products, 2e-5 for FP32, 2e-4 for split BF16.
"""

import pytest
import torch

pytestmark = pytest.mark.gpu

KS = [1, 2, 15, 16, 17, 31, 33, 65, 80, 96, 112, 113, 128, 129, 160, 177, 208, 209, 224, 240, 256, 257]


@pytest.mark.parametrize("dtype,precision,tol", [("f64", "default", 1e-12), ("f32", "fp64", 1e-12),
                                                 ("f32", "default", 2e-5), ("f32", "bf16x3", 2e-4)])
@pytest.mark.parametrize("n", [1, 31, 64, 65, 1000, 8197, 70001])
def test_block_edges(dtype, precision, tol, n):
    import paper_1612_07875_amd as dmd
    dt = torch.float64 if dtype == "f64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(n)
    ld = -(-n // 4) * 4
    full = torch.randn((257, ld), generator=g, device="cuda", dtype=torch.float64).to(dt) + 0.5
    full[:, n:] = float("nan")  # never read
    for k in KS:
        X = full[:k, :n]
        G = dmd.window_gram(X, precision=precision)
        again = dmd.window_gram(X, precision=precision, noalloc=True)
        assert torch.equal(G, again)
        ref = X.double() @ X.double().T
        d = ref.diagonal().clamp_min(1e-300).sqrt()
        assert torch.equal(G, G.T)
        err = ((G - ref).abs() / (d[:, None] * d[None, :])).max().item()
        assert err <= tol, (k, err)
