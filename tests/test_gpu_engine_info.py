"""What amg_engine_info reports is what runs: the octree's persistent workgroup on the systems it is meant for, with the
top level and the couplings beyond one cell that each of its instances needs, and none with the engine off or a cycle
outside its shape; its launches are timed. The instance of a 512-cell top level with couplings of any reach is compared
with one launch per step and the oracle (the same preconditioner up to the order of its sums)."""
import numpy as np
import pytest

import oracle
from paper_1209_5421_amd import meshgen as mg
from tests import helpers as H

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

_cache = {}


def prob(m):
    if m not in _cache:
        _cache[m] = mg.cube_problem(m)
    return _cache[m]


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


# m, the engine's top level k, couplings beyond one cell on that level. 9: 900 unknowns, L = 3; 12: 2,028, L = 3;
# 17: 5,508, L = 4; 24: 15,000, L = 4; 34: 41,650 and 45: 95,220, L = 5
@pytest.mark.parametrize("m,k,ovf", [(9, 3, False), (12, 3, False), (17, 4, True), (24, 4, False), (34, 4, False),
                                     (45, 4, False)])
def test_octree_engine_is_selected(m, k, ovf):
    from paper_1209_5421_amd import amg
    p = prob(m)
    h = amg.Hierarchy.from_problem(p)
    off = amg.Hierarchy.from_problem(p, engine=0)
    two = amg.Hierarchy.from_problem(p, sweeps=2)
    b = T(p.b)
    for precision, kind in ((0, "engine64"), (1, "engine32")):
        info = h.engine_info(precision)
        top = h.level_info(info["top_level"])
        assert top["k"] == k and (top["ovf_nnz"] > 0) == ovf, (info, top)
        assert h.level_info(info["lds_level"])["k"] == 3 and info["steps"] == {3: 38, 4: 112}[k]
        assert 0 < info["lds_bytes"] <= 160 * 1024
        assert off.engine_info(precision)["top_level"] == -1 and two.engine_info(precision)["top_level"] == -1
        for g, runs in ((h, True), (off, False), (two, False)):
            g.set_precision(precision)
            g.timing_enable(kind)
            _, i = g.solve(b)
            t = g.timing_read()
            g.timing_enable(None)
            # B~ of the top level runs once per iteration at the finest tree level, twice for each level above it
            assert t["launches"] == (i["iters"] * 2 ** (info["top_level"] - 1) if runs else 0)
            assert (t["bytes_per_launch"] > 0) == runs
    for g in (h, off, two):
        g.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_octree_engine_on_a_top_level_of_512_cells_with_far_couplings(precision):
    from paper_1209_5421_amd import amg
    p = H.longrange_problem_3d(n=2000, extra=150)
    ga = amg.Hierarchy.from_problem(p, engine=1)
    gb = amg.Hierarchy.from_problem(p, engine=0)
    top = ga.level_info(ga.engine_info(precision)["top_level"])
    assert top["k"] == 3 and top["ovf_nnz"] > 0
    r = T(np.random.default_rng(5).standard_normal(p.n))
    za, zb = ga.apply_precond(r, precision=precision), gb.apply_precond(r, precision=precision)
    assert torch.linalg.norm(za - zb) <= (1e-11 if precision == 0 else 1e-4) * torch.linalg.norm(zb)
    assert torch.equal(za, ga.apply_precond(r, precision=precision))
    if precision == 0:
        o = oracle.setup_problem(p)
        z_o = o.apply_precond(r.cpu().numpy())
        assert np.linalg.norm(za.cpu().numpy() - z_o) <= 1e-10 * np.linalg.norm(z_o)
        o.close()
    ga.set_precision(precision)
    gb.set_precision(precision)
    xa, ia = ga.solve(T(p.b))
    xb, ib = gb.solve(T(p.b))
    assert ia["status"] == 0 and abs(ia["iters"] - ib["iters"]) <= 1
    assert torch.linalg.norm(xa - xb) <= 1e-6 * torch.linalg.norm(xb)
    ga.close()
    gb.close()


# squares of 8 and of 16 super-cells: 4^7, 4^8 and 4^9 cells, none coupled beyond its neighbours
@pytest.mark.parametrize("side,cells", [(131, 16384), (259, 65536), (515, 262144)])
def test_uniform_levels_are_tiled(side, cells):
    from paper_1209_5421_amd import amg
    h = amg.Hierarchy.from_problem(mg.uniform_problem(side - 1))
    top = h.level_info(1)
    assert top["n"] == cells and top["ovf_nnz"] == 0  # at least 256 super-cells, no couplings beyond one cell
    for precision in (0, 1):
        assert h.engine_info(precision)["top_level"] >= 2  # the finest tree level lies above the engine
    h.close()
