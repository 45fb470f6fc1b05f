"""Device memory of small handles: their arena (slabs of 2 MB and up) and the
workspaces of their own sizes, nothing sized for larger hierarchies.  A handle
of 1,024 unknowns keeps well under 6 MB; the memory comes back with the handles."""
import numpy as np
import pytest
import torch

from paper_2606_09001_amd import matrices as M
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [{}, dict(nu_pre=2, nu_post=2), dict(symmetric=False, solver="bicgstab"),
                                dict(vcycle_prec="fp32")], ids=["cg", "sweeps", "nonsym", "fp32"])
def test_small_handles(kw):
    from paper_2606_09001_amd import solver
    cap, count, limit = 8, 24, 6 << 20
    solver.finalize()
    solver.set_cache_capacity(0)
    try:
        rp, ci, v = M.poisson(32, 2)
        n = len(rp) - 1
        b = dev(M.rhs_normal(n, 1))
        rpd, cid = dev(rp), dev(ci)
        vals = [dev(v * (1.0 + 0.01 * i)) for i in range(count + 1)]
        first = solver.AmgHierarchy(rpd, cid, vals[0], **kw)
        first.solve(b, 1e-8)
        torch.cuda.synchronize()
        free0 = torch.cuda.mem_get_info()[0]
        hs = [solver.AmgHierarchy(rpd, cid, vals[i + 1], **kw) for i in range(count)]
        torch.cuda.synchronize()
        used = (free0 - torch.cuda.mem_get_info()[0]) / count
        print(f"[case] {kw}: {used / 2**20:.2f} MB per handle", flush=True)
        assert used <= limit
        x0 = host(first.solve(b, 1e-8)[0])
        x1 = host(hs[0].solve(b, 1e-8)[0])
        assert np.allclose(x1 * 1.01, x0, rtol=1e-6, atol=1e-9 * np.abs(x0).max())
        for h in hs:
            h.close()
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] >= free0 - (4 << 20)
        first.close()
    finally:
        solver.set_cache_capacity(cap)
