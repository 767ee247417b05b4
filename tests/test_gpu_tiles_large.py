"""Tiles on a level of more than 256 workgroups, whose partial sums a launch of their own adds up (k_finish): a uniform
lattice just above 4^10 unknowns, coupled to no cell beyond its neighbours, against one launch per color phase (engine off).
Tolerances as in test_gpu_tiles: the same preconditioner up to the order of its sums."""
import time

import numpy as np
import pytest

from paper_1209_5421_amd import meshgen as mg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

_cache = {}


def problem():
    if "p" not in _cache:
        _cache["p"] = mg.uniform_problem(1026)
    return _cache["p"]


@pytest.mark.parametrize("inner", [2, 1])
@pytest.mark.parametrize("precision", [0, 1])
def test_partial_sums_of_1024_tiles(inner, precision):
    from paper_1209_5421_amd import amg
    p = problem()
    print(f"[tiles large] n={p.n} inner={inner} precision={precision} {time.strftime('%X')}", flush=True)
    ga = amg.Hierarchy.from_problem(p, inner_iters=inner, engine=1)
    gb = amg.Hierarchy.from_problem(p, inner_iters=inner, engine=0)
    top = ga.level_info(1)
    assert top["n"] == 4 ** 10 and top["ovf_nnz"] == 0  # 262,144 super-cells: 1,024 squares of 16 x 16
    r = torch.as_tensor(np.random.default_rng(7).standard_normal(p.n), device="cuda")
    za, zb = ga.apply_precond(r, precision=precision), gb.apply_precond(r, precision=precision)
    assert torch.linalg.norm(za - zb) <= (1e-11 if precision == 0 else 1e-4) * torch.linalg.norm(zb)
    assert torch.equal(za, ga.apply_precond(r, precision=precision))
    ga.set_precision(precision)
    gb.set_precision(precision)
    b = torch.as_tensor(p.b, device="cuda")
    xa, ia = ga.solve(b)
    xb, ib = gb.solve(b)
    assert ia["status"] == 0 and abs(ia["iters"] - ib["iters"]) <= 1
    assert torch.linalg.norm(xa - xb) <= 1e-6 * torch.linalg.norm(xb)
    ga.close()
    gb.close()
