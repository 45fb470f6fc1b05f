"""amg_apply_vcycle with z = r (the same buffer): the result of the call with
two buffers, bit for bit, on every form level 0 can take (two-sweep, four-sweep,
one dense level of several workgroups, several sweeps, no preconditioner)."""
import numpy as np
import pytest
import torch

from paper_2606_09001_amd import _lib
from paper_2606_09001_amd import matrices as M
from gpu_util import dev, host

pytestmark = pytest.mark.gpu

CASES = {
    "two_sweep_150": (lambda: M.poisson(150, 2), {}),
    "two_sweep_21": (lambda: M.diffusion(np.exp(M.grf(21, 3, seed=2))), dict(max_coarse=30)),
    "four_sweep_60": (lambda: M.poisson(60, 3), {}),
    "sweeps_2_2": (lambda: M.poisson(60, 2), dict(nu_pre=2, nu_post=2)),
    "one_level_900": (lambda: M.poisson(30, 2), dict(max_coarse=1000)),
    "identity": (lambda: M.poisson(40, 2), dict(precondition=0)),
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_in_place_equals_two_buffers(case, prec):
    from paper_2606_09001_amd.solver import AmgHierarchy
    make, kw = CASES[case]
    rp, ci, v = make()
    n = len(rp) - 1
    print(f"[case] {case} {prec} n={n}", flush=True)
    H = AmgHierarchy(dev(rp), dev(ci), dev(v), vcycle_prec=prec, **kw)
    r = dev(M.rhs_normal(n, 8))
    z = host(H.apply_vcycle(r))
    for _ in range(3):
        y = r.clone()
        st = _lib.load().amg_apply_vcycle(H.handle, y.data_ptr(), y.data_ptr(),
                                          torch.cuda.current_stream().cuda_stream)
        assert st == _lib.AMG_OK
        assert np.array_equal(host(y).view(np.int64), z.view(np.int64))
    assert np.array_equal(host(r), M.rhs_normal(n, 8))
    H.close()
