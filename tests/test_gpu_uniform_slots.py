"""Operators whose slots hold one value each (constant coefficients): the
sweeps that read a value per slot give the bits of the sweeps that read one
per entry, across value refreshes in both directions, and the explicit-value
form is taken as soon as one entry differs."""
import numpy as np
import pytest

from paper_2606_09001_amd import matrices as M
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", ["poisson3d_17", "poisson2d_65", "tridiag_1000"])
def test_uniform_slots(case, prec):
    from paper_2606_09001_amd.solver import AmgHierarchy
    rp, ci, v = {"poisson3d_17": lambda: M.poisson(17, 3), "poisson2d_65": lambda: M.poisson(65, 2),
                 "tridiag_1000": lambda: M.tridiagonal(1000, 2.5)}[case]()
    n = len(rp) - 1
    b = dev(M.rhs_normal(n, 2))
    kw = dict(vcycle_prec=prec, max_coarse=40)
    U = AmgHierarchy(dev(rp), dev(ci), dev(v), **kw)
    assert U.stats()["form_a"][0] == 3
    uni = U.kernel_bytes("spmv_dot")
    zu, xu = host(U.apply_vcycle(b)), host(U.solve(b, 1e-9)[0])
    # one entry changed: values per entry; changed back: one per slot again
    w = v.copy()
    w[rp[n // 2]:rp[n // 2 + 1]] *= 1.0 + 1e-12
    U.update_values(dev(w))
    assert U.kernel_bytes("spmv_dot") > uni + 7 * len(v)
    zw = host(U.apply_vcycle(b))
    V = AmgHierarchy(dev(rp), dev(ci), dev(w), **kw)
    assert np.array_equal(zw.view(np.int64), host(V.apply_vcycle(b)).view(np.int64))
    assert np.linalg.norm(zw - zu) <= (1e-9 if prec == "fp64" else 1e-4) * np.linalg.norm(zu)
    U.update_values(dev(v))
    assert U.kernel_bytes("spmv_dot") == uni
    assert np.array_equal(host(U.apply_vcycle(b)).view(np.int64), zu.view(np.int64))
    assert np.array_equal(host(U.solve(b, 1e-9)[0]).view(np.int64), xu.view(np.int64))
