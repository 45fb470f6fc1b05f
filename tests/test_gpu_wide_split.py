"""Batched sweeps that give a row several lane groups (few rows, long rows):
every column of a batched solve against the same column's oracle solve, for
widths with one, some and all lanes of a group live and rows from one entry to
full length (parts of a row without entries included).  Counts within one of
the oracle's, solutions at equal counts to 1e-9 (the solve parity bound)."""
import numpy as np
import pytest

from paper_2606_09001_amd import matrices as M
from gpu_util import dev, host, pair
from test_gpu_two_sweep import _arrow

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [2, 5, 32, 64])
@pytest.mark.parametrize("case", ["arrow", "cube", "systems"])
def test_split_rows(case, width):
    from paper_2606_09001_amd.solver import AmgHierarchy
    import oracle
    if case == "arrow":
        rp, ci, v = _arrow(900)
        kw = dict(max_coarse=8)
    else:
        rp, ci, v = M.diffusion(np.exp(M.grf(13, 3, seed=3)))
        kw = dict(max_coarse=30)
    n = len(rp) - 1
    B = M.rhs_normal(n, 4, width)
    scale = 1.0 + 0.1 * np.arange(width) if case == "systems" else None
    vals = v[:, None] * scale[None, :] if case == "systems" else v
    H = AmgHierarchy(dev(rp), dev(ci), dev(vals), **kw)
    X, info = H.solve(dev(B), 1e-10)
    X, it = host(X), H.columns(width)["iters"]
    assert info["status"] == 0
    for c in sorted({0, width // 2, width - 1}):
        O = oracle.OracleHierarchy(rp, ci, v * scale[c] if case == "systems" else v, **kw)
        xo, io = O.pcg(np.ascontiguousarray(B[:, c]), tol=1e-10)
        assert abs(it[c] - io["iters"]) <= 1
        if it[c] == io["iters"]:
            assert np.linalg.norm(X[:, c] - xo) <= 1e-9 * np.linalg.norm(xo)
