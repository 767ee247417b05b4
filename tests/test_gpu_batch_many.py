"""Batches of more systems than a launch takes by value (64) and by address (256): every system's solution, iterations and
status equal amg_solve's bit for bit, of two depths and both precisions, by either entry point."""
import numpy as np
import pytest

from paper_1209_5421_amd import meshgen as mg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


# 2,601 and 9,604 unknowns, in step in both precisions (depths 5 and 6; not every lattice is, with couplings beyond one cell
# on the engine's levels)
@pytest.mark.parametrize("count,noalloc", [(65, False), (65, True), (256, False), (256, True), (300, False)])
def test_many_systems_equal_amg_solve(count, noalloc):
    from paper_1209_5421_amd import amg
    probs = [mg.jittered_problem(s, rhs_seed=s, fast=True) for s in (53, 100)]
    hs, bs, ref = [], [], []
    print(f"[batch many] {count} noalloc {noalloc}", flush=True)
    for i in range(count):
        p = probs[i % 3 == 2]
        hs.append(amg.Hierarchy.from_problem(p, precision=1 if i % 5 else 0))
        bs.append(T(p.b) * (1.0 + i))
    xs = [torch.full_like(b, float("nan")) for b in bs]
    code, infos = amg.solve_batch(hs, bs, xs, [1e-8] * count, noalloc=noalloc)
    assert code == 0
    for i, (h, b, x, info) in enumerate(zip(hs, bs, xs, infos)):
        y, one = h.solve(b)
        assert info["iters"] == one["iters"] and info["relres"] == one["relres"] and torch.equal(x, y), i
        h.close()


# every count up to 64, so that each kernel meets its own limit of calls by value and the counts on either side of it
@pytest.mark.parametrize("precision", [0, 1])
def test_every_count_equals_amg_solve(precision):
    from paper_1209_5421_amd import amg
    print(f"[batch counts] precision {precision}", flush=True)
    p = mg.jittered_problem(53, rhs_seed=53, fast=True)
    hs = [amg.Hierarchy.from_problem(p, precision=precision) for _ in range(64)]
    bs = [T(p.b) * (1.0 + i) for i in range(64)]
    ref = [h.solve(b)[0] for h, b in zip(hs, bs)]
    for count in range(1, 65):
        xs = [torch.full_like(b, float("nan")) for b in bs[:count]]
        code, _ = amg.solve_batch(hs[:count], bs[:count], xs, [1e-8] * count)
        assert code == 0 and all(torch.equal(x, y) for x, y in zip(xs, ref)), count
    for h in hs:
        h.close()
