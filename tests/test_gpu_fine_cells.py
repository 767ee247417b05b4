"""The fine smoother's fused phase on cells of every size class (1 to 8 rows, 9 to 16, 17 to 32, more) against the oracle:
scattered points of strongly varying density, each coupled to its nearest neighbours, so that cells hold dense blocks.
Both sides do the same operations but for the order of a row's subtractions, so a sweep's error is a few roundings of
rows of at most 40 entries of comparable size: within 1e-11 of the largest value in FP64 and 1e-4 in FP32."""
import numpy as np
import pytest
import scipy.sparse as sp
from scipy.spatial import cKDTree

import oracle
from paper_1209_5421_amd import meshgen as mg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def scattered(n, power, seed, neighbours=12):
    rng = np.random.default_rng(seed)
    pts = np.column_stack([rng.random(n) ** power, rng.random(n)])
    _, near = cKDTree(pts).query(pts, neighbours + 1)
    i = np.repeat(np.arange(n), neighbours)
    A = sp.csr_matrix((-(0.5 + rng.random(n * neighbours)), (i, near[:, 1:].ravel())), shape=(n, n))
    A = A.minimum(A.T)
    A = (A + sp.diags(1.0 - np.asarray(A.sum(axis=1)).ravel())).tocsr()
    A.sort_indices()
    return mg.Problem("scattered", pts, A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data,
                      rng.standard_normal(n), (0.0, 1.0, 0.0, 1.0), {})


# cells of 1 to 8 rows with some of 9 to 16; up to 32; beyond 32; the smallest multi-level systems
@pytest.mark.parametrize("n,power,classes", [(3000, 1.0, (8, 16)), (6000, 2.0, (8, 16, 32)), (6000, 4.0, (8, 16, 32, 64)),
                                             (700, 1.5, (8,))])
@pytest.mark.parametrize("smoother", [0, 1])
def test_cells_of_every_size(n, power, classes, smoother):
    from paper_1209_5421_amd import amg
    prob = scattered(n, power, seed=n)
    print(f"[fine cells] n={n} power={power} smoother={smoother}", flush=True)
    g = amg.Hierarchy.from_problem(prob, device="cuda:0", smoother=smoother)
    o = oracle.setup_problem(prob)
    o.set_block_smoother(bool(smoother))
    side = int(round(np.sqrt(g.level_info(1)["n"])))
    cell = np.minimum((prob.coords * side).astype(int), side - 1)
    sizes = np.bincount(cell[:, 1] * side + cell[:, 0])
    for c in classes:
        assert np.any((sizes > (c // 2 if c > 8 else 0)) & (sizes <= c)), (c, sizes.max())
    rng = np.random.default_rng(3)
    x, f = rng.standard_normal(n), rng.standard_normal(n)
    for fwd in (True, False):
        want = o.smooth(0, f, x, fwd)
        for prec, tol in ((0, 1e-11), (1, 1e-4)):
            got = g.smooth(0, T(f), T(x), fwd, precision=prec).cpu().numpy()
            np.testing.assert_allclose(got, want, rtol=0, atol=tol * np.abs(want).max(), err_msg=f"{fwd} {prec}")
    r = rng.standard_normal(n)
    z = o.apply_precond(r)
    assert np.linalg.norm(g.apply_precond(T(r)).cpu().numpy() - z) <= 1e-10 * np.linalg.norm(z)
    g.close()
