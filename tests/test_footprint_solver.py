"""Only the Jacobi solver keeps all eigenvectors of a window, m x m values per
window in flight; no stream of the tridiagonal solver allocates them."""

import pytest

import paper_1612_07875_amd as dmd


@pytest.mark.parametrize("m,block", [(16, 1), (100, 1), (100, 8), (250, 32)])
def test_eigenvector_storage(m, block):
    size = {s: dmd.footprint(5000, m, 8, max_block=block, eig_solver=s) for s in ("default", "tridiag", "jacobi")}
    assert size["default"] == size["tridiag"]
    assert size["jacobi"] - size["tridiag"] == 8 * m * m * block
