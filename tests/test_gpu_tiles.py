"""Tiled tree levels with A u and its inner products formed in the post-smoothing tile, against one launch per color
phase (engine off), over the tile sizes and cycle options: the same preconditioner to rounding (other reduction trees,
and beta and alpha1 of the second inner step from sums of products of p1 and p0 instead of their combination)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1209_5421_amd import amg
from paper_1209_5421_amd import meshgen as mg

pytestmark = pytest.mark.gpu

# uniform lattices couple no cell beyond its neighbours at about one unknown per cell, so every level is tiled: n just
# above 4^k gives level k; 513^2 has a level of 262,144 cells (squares of 16 x 16 super-cells), the others levels of
# 16,384 and 65,536 cells (squares of 8 x 8). The disk has empty cells.
_cache = {}


def _problem(name):
    if name not in _cache:
        _cache[name] = mg.disk_problem(200) if name == "disk200" else mg.uniform_problem(int(name[7:]) - 1)
    return _cache[name]


@pytest.mark.parametrize("name,sweeps,inner", [("uniform131", 1, 2), ("uniform259", 1, 2), ("uniform515", 1, 2),
                                               ("disk200", 1, 2), ("uniform259", 2, 2), ("uniform259", 1, 1)])
@pytest.mark.parametrize("precision", [0, 1])
def test_tiled_levels_with_products(name, sweeps, inner, precision):
    prob = _problem(name)
    ga = amg.Hierarchy.from_problem(prob, sweeps=sweeps, inner_iters=inner, engine=1)
    gb = amg.Hierarchy.from_problem(prob, sweeps=sweeps, inner_iters=inner, engine=0)
    r = torch.as_tensor(np.random.default_rng(7).standard_normal(prob.n), device="cuda")
    za = ga.apply_precond(r, precision=precision)
    zb = gb.apply_precond(r, precision=precision)
    tol = 1e-11 if precision == 0 else 1e-4
    assert torch.linalg.norm(za - zb) <= tol * torch.linalg.norm(zb)
    assert torch.equal(za, ga.apply_precond(r, precision=precision))  # fixed summation order
    ga.set_precision(precision)
    gb.set_precision(precision)
    b = torch.as_tensor(prob.b, device="cuda")
    xa, ia = ga.solve(b)
    xb, ib = gb.solve(b)
    assert ia["status"] == 0 and abs(ia["iters"] - ib["iters"]) <= 1
    assert torch.linalg.norm(xa - xb) <= 1e-6 * torch.linalg.norm(xb)
    ga.close()
    gb.close()


def test_tiled_levels_against_the_oracle():
    prob = _problem("uniform131")
    g = amg.Hierarchy.from_problem(prob)
    r = np.random.default_rng(8).standard_normal(prob.n)
    z = g.apply_precond(torch.as_tensor(r, device="cuda"), precision=0).cpu().numpy()
    o = oracle.setup_problem(prob)
    z_o = o.apply_precond(r)
    assert np.linalg.norm(z - z_o) <= 1e-10 * np.linalg.norm(z_o)
    o.close()
    g.close()
