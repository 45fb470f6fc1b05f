"""What the autotuner of the batched sweeps records: matrices whose sweeps take
the split kernel (few long rows), which has no form or stream count to choose,
are not timed, except the level-0 matrix for the sweeps with sums, under a key
of its own; the others are recorded as before."""
import os
import re
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import sys
sys.path[:0] = ["tests", "."]
import numpy as np
from paper_2606_09001_amd import matrices as M
from paper_2606_09001_amd.solver import AmgHierarchy
from gpu_util import dev, host
from test_gpu_two_sweep import _arrow
for name, (rp, ci, v), kw in (("cube", M.diffusion(np.exp(M.grf(26, 3, seed=3))), dict(max_coarse=30)),
                              ("dense_rows", M.poisson(12, 3), {})):
    n = len(rp) - 1
    if name == "dense_rows":      # every row couples to its 40 neighbours in index
        import scipy.sparse as sp
        A = sp.diags([60.0] + [-1.0] * 40, [0] + [s * k for k in range(1, 21) for s in (1, -1)], shape=(n, n)).tocsr()
        A.sort_indices()
        rp, ci, v = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    print("[case]", name, n, len(ci), flush=True)
    B = dev(M.rhs_normal(n, 4, 32))
    H = AmgHierarchy(dev(rp), dev(ci), dev(v), autotune=1, **kw)
    X, info = H.solve(B, 1e-10)
    assert info["status"] == 0
    P = AmgHierarchy(dev(rp), dev(ci), dev(v), **kw)
    Y, _ = P.solve(B, 1e-10)
    assert np.linalg.norm(host(X) - host(Y)) <= 1e-8 * np.linalg.norm(host(Y))
"""


def _parts(n, nnz, groups):
    parts = 1
    while parts < groups and n * parts < 1024 * groups and nnz >= 16 * parts * n:
        parts *= 2
    return parts


def test_recorded_choices(tmp_path):
    cache = tmp_path / "tune.txt"
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, env=dict(os.environ, AMG_TUNE_CACHE=str(cache)),
                       capture_output=True, text=True, timeout=100)
    print(r.stdout)
    assert r.returncode == 0, r.stderr
    seen = set()
    for line in cache.read_text().splitlines():
        m = re.match(r"wide([APR]):n(\d+):nnz(\d+):W32:\S*?br\d+(:red)? ", line)
        if not m:
            continue
        split = _parts(int(m[2]), int(m[3]), 256 // 16) > 1       # 16 lanes of two FP64 columns
        assert split == bool(m[4]), line
        assert not split or m[1] == "A", line
        seen.add((m[1], split))
    assert ("A", True) in seen and ("A", False) in seen and ("P", False) in seen
