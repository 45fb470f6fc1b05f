"""Captured iterations replayed into another output buffer than the one they
were captured with: every solve writes its own x and leaves earlier ones
alone, for the single-column, batched and BiCGSTAB solves."""
import numpy as np
import pytest
import torch

from paper_2606_09001_amd import matrices as M
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["pcg", "batched", "bicgstab"])
def test_replay_into_new_buffers(form):
    from paper_2606_09001_amd.solver import AmgHierarchy
    if form == "bicgstab":
        rp, ci, v = M.convection_diffusion(40, 2, M.recirculating_wind(40, 2, 100.0))
        kw = dict(symmetric=False, solver="bicgstab")
    else:
        rp, ci, v = M.diffusion(np.exp(M.grf(40, 2, seed=9)))
        kw = {}
    n = len(rp) - 1
    H = AmgHierarchy(dev(rp), dev(ci), dev(v), **kw)
    E = AmgHierarchy(dev(rp), dev(ci), dev(v), use_graphs=0, **kw)
    rhs = [M.rhs_normal(n, s) if form != "batched" else M.rhs_normal(n, s, 3) for s in (1, 2, 3)]
    xs = [torch.full_like(dev(b), float("nan")) for b in rhs]
    for b, x in zip(rhs, xs):
        H.solve(dev(b), 1e-9, out=x)
    for b, x in zip(rhs, xs):
        ref, _ = E.solve(dev(b), 1e-9)
        assert np.array_equal(host(x).view(np.int64), host(ref).view(np.int64))
