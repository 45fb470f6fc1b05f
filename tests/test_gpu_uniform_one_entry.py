"""Constant-coefficient operators with exactly one entry (and its mirror)
changed, in the first slice, in the middle and in the last, partly filled one:
the sweeps read a value per entry again, and the cycle follows the oracle's on
the changed matrix (1e-12, the bound of the other V-cycle tests)."""
import numpy as np
import pytest

from paper_2606_09001_amd import matrices as M
from gpu_util import dev, host, pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["first", "middle", "last"])
@pytest.mark.parametrize("N,d", [(66, 2), (55, 3)])
def test_one_entry_changed(N, d, where):
    rp, ci, v = M.poisson(N, d)
    n = len(rp) - 1
    assert n % 64 not in (0, 1)                 # the last slice has some rows, not all
    i = {"first": 1, "middle": n // 2, "last": n - 2}[where]
    w = v.copy()
    k = rp[i] + int(np.flatnonzero(ci[rp[i]:rp[i + 1]] == i + 1)[0])
    m = rp[i + 1] + int(np.flatnonzero(ci[rp[i + 1]:rp[i + 2]] == i)[0])
    w[k] = w[m] = np.nextafter(-1.0, 0.0)
    assert np.count_nonzero(w != v) == 2
    H, _ = pair(rp, ci, v)
    uniform = H.kernel_bytes("spmv_dot")
    H.update_values(dev(w))
    assert H.kernel_bytes("spmv_dot") > uniform + 7 * len(v)
    b = M.rhs_normal(n, 4)
    F, O = pair(rp, ci, w, max_levels=19)       # (not the cached one)
    z = host(H.apply_vcycle(dev(b)))
    assert np.array_equal(z.view(np.int64), host(F.apply_vcycle(dev(b))).view(np.int64))
    zo = O.vcycle(b)
    assert np.linalg.norm(z - zo) <= 1e-12 * np.linalg.norm(zo)
    H.update_values(dev(v))
    assert H.kernel_bytes("spmv_dot") == uniform
