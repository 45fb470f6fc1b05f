"""Values that are not symmetric on a handle made for symmetric ones (CG's
default, also the preconditioner of another solver): the cycle uses A as it is
stored, as the oracle's does, whichever sweeps a level takes; and value
refreshes between symmetric and nonsymmetric values leave nothing behind.

FP64 tolerance: regrouped sums of at most a few hundred rounded terms per row,
1e-12 (the bound of the other V-cycle tests)."""
import numpy as np
import pytest

from paper_2606_09001_amd import matrices as M
from gpu_util import dev, host, pair

pytestmark = pytest.mark.gpu


def _wind(N, d, speed):
    return M.convection_diffusion(N, d, M.recirculating_wind(N, d, speed))


def _row_scaled(N, d, by):
    rp, ci, v = M.poisson(N, d)
    i = len(rp) // 2
    v = v.copy()
    v[rp[i]:rp[i + 1]] *= 1.0 + by
    return rp, ci, v


def _one_sided(N):
    """Entries (i, i + 1) of every third row dropped: a structurally nonsymmetric pattern."""
    rp, ci, v = M.poisson(N, 2)
    rows = np.repeat(np.arange(len(rp) - 1), np.diff(rp))
    keep = ~((ci == rows + 1) & (rows % 3 == 0))
    n = len(rp) - 1
    rp2 = np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=n))]).astype(np.int32)
    return rp2, ci[keep], v[keep]


CASES = {
    "wind_2d_60": (lambda: _wind(60, 2, 15.0), {}),
    "wind_2d_deep": (lambda: _wind(45, 2, 30.0), dict(max_coarse=12)),
    "wind_3d_54": (lambda: _wind(54, 3, 20.0), {}),
    "one_row_1e-6": (lambda: _row_scaled(50, 2, 1e-6), {}),
    "one_sided_40": (lambda: _one_sided(40), dict(max_coarse=60)),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_cycle_uses_the_stored_values(case):
    make, kw = CASES[case]
    rp, ci, v = make()
    b = M.rhs_normal(len(rp) - 1, 5)
    H, O = pair(rp, ci, v, fused_small=0, **kw)
    zo = O.vcycle(b)
    z = host(H.apply_vcycle(dev(b)))
    assert np.linalg.norm(z - zo) <= 1e-12 * np.linalg.norm(zo)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("N,d", [(60, 2), (54, 3)])
def test_refreshes_leave_nothing_behind(N, d, prec):
    from paper_2606_09001_amd.solver import AmgHierarchy
    rp, ci, v = M.poisson(N, d)
    w = _wind(N, d, 15.0)[2]
    b = dev(M.rhs_normal(len(rp) - 1, 3))
    rpd, cid = dev(rp), dev(ci)
    H = AmgHierarchy(rpd, cid, dev(v), vcycle_prec=prec)
    print(f"[case] {N}^{d} {prec}", flush=True)
    for values in (w, v, w * 1.5, v * 0.5, v):
        H.update_values(dev(values))
        got = host(H.apply_vcycle(b))
        F = AmgHierarchy(rpd, cid, dev(values), vcycle_prec=prec, max_levels=19)   # (not the cached one)
        assert np.array_equal(got.view(np.int64), host(F.apply_vcycle(b)).view(np.int64))
        F.close()
    x, info = H.solve(b, 1e-8)
    assert info["status"] == 0
