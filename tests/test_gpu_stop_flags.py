"""Solves that end inside a queue of iterations (the product, the update, a
BiCGSTAB half or full step finds the end, and everything queued behind it
returns) against solves that are read back after every iteration: the same
iterations, so the same counts and the same bits of x.  Level 0 in every sweep
form, reductions folded by their consumers and totalled beforehand."""
import numpy as np
import pytest

from paper_2606_09001_amd import matrices as M
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def _arrow(n, far):
    """First row and column hold every far-th unknown; diagonally dominant, symmetric."""
    rp, ci, v = [0], [], []
    first = list(range(0, n, far))
    for i in range(n):
        cols = sorted({0, max(i - 1, 0), i, min(i + 1, n - 1)} if i % far == 0 else
                      {max(i - 1, 0), i, min(i + 1, n - 1)}) if i else sorted({0, 1, *first})
        ci += cols
        v += [float(len(cols)) + 1.0 if c == i else -0.5 for c in cols]
        rp.append(len(ci))
    return np.array(rp, np.int32), np.array(ci, np.int32), np.array(v)


def _shuffled(N):
    """2D Poisson under a permutation of the unknowns: no common offsets."""
    import scipy.sparse as sp
    rp, ci, v = M.poisson(N, 2)
    n = len(rp) - 1
    p = np.random.default_rng(4).permutation(n)
    A = sp.csr_matrix((v, ci, rp), shape=(n, n))[p][:, p].tocsr()
    A.sort_indices()
    return A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data


MATRICES = {
    # level-0 form: 0 lanes per row, 1 CSR-stream, 2 sliced, 3 offsets
    "vec_4001": (lambda: _arrow(4001, 1), 0),
    "stream_3000": (lambda: _arrow(3000, 2), 1),
    "sliced_70": (lambda: _shuffled(70), 2),
    "offsets_61": (lambda: M.poisson(61, 2), 3),
    "totals_90": (lambda: M.poisson(90, 3), 3),
}


@pytest.mark.parametrize("solver", ["pcg", "bicgstab"])
@pytest.mark.parametrize("case", sorted(MATRICES))
def test_end_inside_a_queue(case, solver):
    from paper_2606_09001_amd.solver import AmgHierarchy
    make, form = MATRICES[case]
    rp, ci, v = make()
    n = len(rp) - 1
    b = dev(M.rhs_normal(n, 6))
    print(f"[case] {case} {solver} n={n}", flush=True)
    out = []
    for every in (1, 5, 64):
        for pre in (1, 0):
            H = AmgHierarchy(dev(rp), dev(ci), dev(v), solver=solver, check_every=every, fused_small=0,
                             precondition=pre, maxiter=3000)
            assert H.stats()["form_a"][0] == form
            x, info = H.solve(b, 1e-9)
            assert info["status"] == 0
            out.append((pre, info["iters"], host(x).view(np.int64)))
            H.close()
    for pre in (1, 0):
        runs = [(i, x) for p, i, x in out if p == pre]
        for i, x in runs[1:]:
            assert i == runs[0][0]
            assert np.array_equal(x, runs[0][1])
