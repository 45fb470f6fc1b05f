"""The one-workgroup solve's coarse product over the sizes where its split
changes: 1-D Poisson systems whose coarsest levels hold 1 unknown (one pair of
rows, eight column blocks), 128 and 129 (eight and seven blocks), 168 and 170
(the whole inverse in registers; columns beyond them read every cycle) and 256
unknowns (the largest).  Against the FP64 oracle: the iterate after one and
five iterations.  Each cycle's sums differ from the oracle's in order only:
with condition numbers up to 940^2 / 2.5 = 3.5e5 and a few hundred rounding
errors of 1.1e-16 per component, 1e-9 leaves a factor of ten or more."""
import numpy as np
import pytest

from paper_2606_09001_amd import matrices as M
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nc", [(3, 1), (467, 128), (470, 129), (623, 168), (629, 170), (940, 256)])
def test_coarse_product_split(n, nc):
    import oracle
    from paper_2606_09001_amd.solver import AmgHierarchy
    rp, ci, v = M.poisson(n, 1)
    b = M.rhs_normal(n, nc)
    kw = {"max_coarse": 2} if n == 3 else {}
    O = oracle.OracleHierarchy(rp, ci, v, **kw)
    assert O.level_sizes(1)["n"] == nc
    print(f"[case] one-workgroup coarse product n={n} n_c={nc}", flush=True)
    for k in (1, 5) if n > 3 else (1,):
        H = AmgHierarchy(dev(rp), dev(ci), dev(v), maxiter=k, **kw)
        assert H.stats()["single_workgroup"] == 1
        x, info = H.solve(dev(b), 0.0)
        xo, _ = O.pcg(b, tol=0.0, maxiter=k)
        assert info["iters"] == k
        assert np.linalg.norm(host(x) - xo) <= 1e-9 * np.linalg.norm(xo)
