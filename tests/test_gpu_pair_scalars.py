"""The second inner step's scalars from sums of products of p0 and p1 (engine on) against those from A d (engine off) where
B^ is a poor preconditioner: point smoothing and square aggregates on a diffusion of ratio 10^-2 and 10^-4. The form
subtracts (p1, q0)^2 / (p0, q0) from (p1, A p1), of which at least 4 / k is left for a condition number k of B^ A, so its
rounding grows by k / 4 at most over the tolerances of the isotropic meshes (1e-11 and 1e-4, test_gpu_tiles). k from the
outer iterations N to 1e-8, N = sqrt(k) / 2 ln(2e8): about 50 for 10^-2 and 2,500 for 10^-4."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1209_5421_amd import meshgen as mg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def anisotropic(m, ratio):
    n = m - 1
    one, lap = sp.identity(n), sp.diags([-np.ones(n - 1), 2 * np.ones(n), -np.ones(n - 1)], [-1, 0, 1])
    A = (sp.kron(one, lap) + ratio * sp.kron(lap, one)).tocsr()
    A.sort_indices()
    g = (np.arange(n) + 1) / m
    X, Y = np.meshgrid(g, g)
    return mg.Problem("anisotropic", np.stack([X.ravel(), Y.ravel()], 1), A.indptr.astype(np.int64),
                      A.indices.astype(np.int32), A.data, np.random.default_rng(1).standard_normal(n * n),
                      (0.0, 1.0, 0.0, 1.0), {})


# 4,225 unknowns: the engine alone; 16,641: tiles above it
@pytest.mark.parametrize("m", [66, 130])
@pytest.mark.parametrize("ratio,k", [(1e-2, 50.0), (1e-4, 2500.0)])
@pytest.mark.parametrize("precision", [0, 1])
def test_poor_preconditioner(m, ratio, k, precision):
    from paper_1209_5421_amd import amg
    p = anisotropic(m, ratio)
    ga = amg.Hierarchy.from_problem(p, engine=1, precision=precision)
    gb = amg.Hierarchy.from_problem(p, engine=0, precision=precision)
    r = torch.as_tensor(np.random.default_rng(5).standard_normal(p.n), device="cuda")
    za, zb = ga.apply_precond(r, precision=precision), gb.apply_precond(r, precision=precision)
    tol = (1e-11 if precision == 0 else 1e-4) * k / 4
    assert torch.linalg.norm(za - zb) <= tol * torch.linalg.norm(zb)
    b = torch.as_tensor(p.b, device="cuda")
    xa, ia = ga.solve(b)
    xb, ib = gb.solve(b)
    print(f"[pair] m={m} ratio={ratio} precision={precision}: {ia['iters']} and {ib['iters']} iterations", flush=True)
    assert ia["status"] == 0 and ib["status"] == 0
    # two residuals of 1e-8, and the condition number of A
    assert torch.linalg.norm(xa - xb) <= 2e-8 * 2.0 / (1.0 - np.cos(np.pi / m)) * torch.linalg.norm(xb)
    ga.close()
    gb.close()
