"""amg_solve_batch's systems that run in step (more than 2,500 unknowns, specialised engine): every system's solution,
iterations and status equal amg_solve's bit for bit, whatever depth, precision, right-hand side or iteration limit its
neighbours have, and in batches of more systems than one launch takes."""
import numpy as np
import pytest

from paper_1209_5421_amd import meshgen as mg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

_cache = {}


def prob(side):
    if side not in _cache:
        _cache[side] = mg.jittered_problem(side, rhs_seed=500 + side, fast=True)
    return _cache[side]


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def run(spec, noalloc):
    """spec: (side, precision, zero right-hand side, max_iters) per system."""
    from paper_1209_5421_amd import amg
    print(f"[batch in step] {len(spec)} systems, first {spec[0]}, noalloc {noalloc}", flush=True)
    hs = [amg.Hierarchy.from_problem(prob(s), device="cuda:0", precision=p, max_iters=m) for s, p, _, m in spec]
    bs = [T(np.zeros(prob(s).n) if z else prob(s).b) for s, _, z, _ in spec]
    xs = [torch.full_like(b, float("nan")) for b in bs]
    _, infos = amg.solve_batch(hs, bs, xs, [1e-8] * len(hs), noalloc=noalloc)
    torch.cuda.synchronize()
    for h, b, x, i, (side, _, zero, limit) in zip(hs, bs, xs, infos, spec):
        ref = torch.full_like(b, float("nan"))
        _, one = h.solve(b, x=ref, check=False)
        torch.cuda.synchronize()
        assert i["status"] == one["status"] and i["iters"] == one["iters"] and i["restarts"] == one["restarts"], (side, i, one)
        assert i["relres"] == one["relres"], (side, i, one)
        assert torch.equal(x, ref), side
        assert (one["status"] == 0) == (limit > 3)
        if zero:
            assert not x.any()
    for h in hs:
        h.close()


# 2,601 unknowns (the limit is 2,500), two depths, both precisions, a zero right-hand side, a limit of
# three iterations, the largest size
MIXED = [(53, 0, False, 1000), (53, 1, False, 1000), (100, 1, False, 1000), (100, 1, True, 1000), (258, 1, False, 3),
         (258, 0, False, 1000), (258, 1, False, 1000), (180, 0, False, 3), (180, 1, False, 1000)]


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("spec", [MIXED, MIXED[::-1], [(53, 1, False, 1000)], [(54, 1, False, 1000)] * 67],
                         ids=["mixed", "reversed", "one", "many"])
def test_in_step_equals_amg_solve(spec, noalloc):
    run(spec, noalloc)
