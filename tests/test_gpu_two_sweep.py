"""The two-sweep V-cycle levels and the folded CG scalars at the sizes where
their forms change: levels left out because of their padding, levels around
the dense limit of 512 rows, deep hierarchies folded into one dense matrix,
level 0 with and without folded reductions, FP32 transfers, and nonsymmetric
values (structurally symmetric, and not).

FP64 tolerance: the products are regrouped sums of at most a few hundred
rounded terms per row, so a cycle agrees with the oracle's to 1e-12 (the bound
of the other V-cycle tests).  FP32 cycle with FP32 transfers: a few hundred
FP32 roundings of relative size 6e-8 over up to five levels stay below 1e-5."""
import numpy as np
import pytest

from paper_2606_09001_amd import matrices as M
from gpu_util import dev, host, pair

pytestmark = pytest.mark.gpu


def _arrow(n):
    """First row and column full, diagonally dominant, symmetric."""
    rp, ci, v = [0], [], []
    for i in range(n):
        if i == 0:
            ci += list(range(n))
            v += [float(n)] + [-0.5] * (n - 1)
        else:
            cols = sorted({0, max(i - 1, 1), i, min(i + 1, n - 1)})
            ci += cols
            v += [3.0 if c == i else -0.5 for c in cols]
        rp.append(len(ci))
    return np.array(rp, np.int32), np.array(ci, np.int32), np.array(v)


CASES = {
    "arrow_900": (lambda: _arrow(900), dict(max_coarse=8)),
    "deep_75": (lambda: M.poisson(75, 2), dict(max_coarse=3)),
    "n529": (lambda: M.diffusion(np.exp(M.grf(23, 2, seed=1))), dict(max_coarse=16)),
    "n484": (lambda: M.diffusion(np.exp(M.grf(22, 2, seed=1))), dict(max_coarse=16)),
    "cube_13": (lambda: M.diffusion(np.exp(M.grf(13, 3, seed=2))), dict(max_coarse=40)),
    "tridiag_5001": (lambda: M.tridiagonal(5001, 2.5), dict(max_coarse=20)),
    "folded_45": (lambda: M.poisson(45, 3), {}),
    "unfolded_54": (lambda: M.poisson(54, 3), {}),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_two_sweep_cycle_and_solve(case):
    make, kw = CASES[case]
    rp, ci, v = make()
    b = M.rhs_normal(len(rp) - 1, 5)
    H, O = pair(rp, ci, v, fused_small=0, **kw)
    zo = O.vcycle(b)
    z = host(H.apply_vcycle(dev(b)))
    assert np.linalg.norm(z - zo) <= 1e-12 * np.linalg.norm(zo)
    x, info = H.solve(dev(b), 1e-10)
    xo, io = O.pcg(b, tol=1e-10)
    assert info["status"] == 0 and abs(info["iters"] - io["iters"]) <= 1
    if info["iters"] == io["iters"]:
        assert np.linalg.norm(host(x) - xo) <= 1e-9 * np.linalg.norm(xo)
    H.update_values(dev(v * 1.25))          # refreshed values reach every form
    z2 = host(H.apply_vcycle(dev(b)))
    assert np.linalg.norm(z2 * 1.25 - zo) <= 1e-12 * np.linalg.norm(zo)


@pytest.mark.parametrize("case", ["n529", "cube_13", "deep_75"])
def test_two_sweep_cycle_fp32(case):
    make, kw = CASES[case]
    rp, ci, v = make()
    b = M.rhs_normal(len(rp) - 1, 6)
    H, O = pair(rp, ci, v, vcycle_prec="fp32", transfer_bf16=0, **kw)
    zo = O.vcycle(b)
    z = host(H.apply_vcycle(dev(b)))
    assert np.linalg.norm(z - zo) <= 1e-5 * np.linalg.norm(zo)


@pytest.mark.parametrize("drop", [0.0, 0.2], ids=["symmetric_pattern", "nonsymmetric_pattern"])
def test_two_sweep_cycle_nonsymmetric(drop):
    rp, ci, v = M.convection_diffusion(30, 2, (40.0, 20.0))
    if drop:
        rp, ci, v = M.drop_entries(rp, ci, v, drop, 4)
    b = M.rhs_normal(len(rp) - 1, 7)
    H, O = pair(rp, ci, v, symmetric=False, solver="bicgstab", max_coarse=12)
    zo = O.vcycle(b)
    z = host(H.apply_vcycle(dev(b)))
    assert np.linalg.norm(z - zo) <= 1e-12 * np.linalg.norm(zo)


def test_two_sweep_cycle_nonsymmetric_without_product_map():
    # six random neighbours per row: a product map of R (A P) would exceed 16
    # pairs per entry of A, so D's values come from the search through P's rows
    n, rng = 1500, np.random.default_rng(11)
    i, j = rng.integers(0, n, 3 * n), rng.integers(0, n, 3 * n)
    D = np.zeros((n, n))
    D[i, j] = -rng.uniform(0.2, 1.0, 3 * n)
    D[j, i] = -rng.uniform(0.2, 1.0, 3 * n)
    np.fill_diagonal(D, 0.0)
    np.fill_diagonal(D, 1.0 + np.abs(D).sum(axis=1))
    rows, cols = np.nonzero(D)
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    ci, v = cols.astype(np.int32), D[rows, cols]
    b = M.rhs_normal(n, 8)
    H, O = pair(rp, ci, v, symmetric=False, solver="bicgstab", max_coarse=12)
    L = O.level(0)
    P = np.zeros((n, O.level_sizes(0)["nagg"]))
    P[np.repeat(np.arange(n), np.diff(L["P_rp"])), L["P_ci"]] = 1.0
    ap_rows = ((D != 0).astype(float) @ P != 0).sum(axis=1)
    assert P.sum(axis=1) @ ap_rows > 16 * len(v)
    zo = O.vcycle(b)
    z = host(H.apply_vcycle(dev(b)))
    assert np.linalg.norm(z - zo) <= 1e-12 * np.linalg.norm(zo)
