"""Plain CG (precondition = 0): <r, z> = ||r||^2 carried by the update, folded
(few partials) and with finalize kernels, against the FP64 oracle's
unpreconditioned CG; the flexible beta, a tolerance of 0, a zero right-hand
side and a restart-free limit.  Counts within 1 + 1 %, fixed-count iterates to
1e-9 (the parity rules of unpreconditioned solves)."""
import numpy as np
import pytest

from paper_2606_09001_amd import matrices as M
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 257, 4097, 600_001], ids=str)
@pytest.mark.parametrize("flexible", [0, 1])
def test_plain_cg_vs_oracle(n, flexible):
    import oracle
    from paper_2606_09001_amd.solver import AmgHierarchy
    rp, ci, v = M.tridiagonal(n, 2.5)
    b = M.rhs_normal(n, 3)
    O = oracle.OracleHierarchy(rp, ci, v, max_levels=1) if n <= 2000 else None
    H = AmgHierarchy(dev(rp), dev(ci), dev(v), precondition=0, flexible=flexible)
    x, info = H.solve(dev(b), 1e-10)
    assert info["status"] == 0 and info["restarts"] == 0
    assert oracle.rel_residual(rp, ci, v, b, host(x)) <= 1e-10
    if O is not None:
        xo, io = O.pcg(b, tol=1e-10, precondition=False)
        assert abs(info["iters"] - io["iters"]) <= 1 + 0.01 * io["iters"]
        k = max(1, min(io["iters"] - 1, 20))
        Hk = AmgHierarchy(dev(rp), dev(ci), dev(v), precondition=0, flexible=flexible, maxiter=k)
        xk, ik = Hk.solve(dev(b), 0.0)
        xok, iok = O.pcg(b, tol=0.0, maxiter=k, precondition=False)
        assert ik["iters"] == iok["iters"]
        assert np.linalg.norm(host(xk) - xok) <= 1e-9 * np.linalg.norm(xok)
    z, iz = H.solve(dev(np.zeros(n)), 1e-10)
    assert iz["iters"] == 0 and not host(z).any()
    x2, _ = H.solve(dev(b), 1e-10)
    assert np.array_equal(host(x).view(np.int64), host(x2).view(np.int64))
