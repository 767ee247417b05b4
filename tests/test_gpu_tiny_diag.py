"""Systems whose diagonals lie below the smallest normal number of the preconditioner's precision, where 1 / d overflows:
a system scaled by a power of two takes the iterations of the unscaled one and has its solution, scaled, in both
smoothers, both engines and in a batch; values updates in and out of that range equal a setup from scratch.

The right-hand side is scaled so that solution and residuals are normal numbers. In FP32 the matrix itself is rounded to
subnormal numbers (16 bits are left at the smallest scale here), a perturbation of the preconditioner only: one iteration
more or less at most. Both solutions stop at a residual of 1e-8."""
import numpy as np
import pytest

from paper_1209_5421_amd import meshgen as mg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

_cache = {}


def prob(name):
    if name not in _cache:
        make = {"jittered": lambda s: mg.jittered_problem(s, fast=True), "uniform": mg.uniform_problem,
                "cube": mg.cube_problem}
        kind = name.rstrip("0123456789")
        _cache[name] = make[kind](int(name[len(kind):]))
    return _cache[name]


def scaled(p, e, eb):
    return mg.Problem(**{**p.__dict__, "val": np.ldexp(p.val, e), "b": np.ldexp(p.b, eb)})


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


# 2^e of the matrix and of the right-hand side. (In FP64 the coarsest level's inverse has to stay finite as well: the
# cube's smallest diagonal is 0.06, the squares' 4.)
SCALES = {1: [(-130, -60), (-134, -60)], 0: [(-1026, -300)]}
CUBE64 = [(-1021, -300)]


# 3,969 unknowns (the engine's top is the finest tree level); 65,536 (levels above the engine); the octree
@pytest.mark.parametrize("name", ["jittered65", "jittered258", "uniform130", "cube12"])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("smoother", [0, 1])
def test_scaled_system(name, precision, smoother):
    from paper_1209_5421_amd import amg
    p = prob(name)
    g = amg.Hierarchy.from_problem(p, precision=precision, smoother=smoother)
    x1, i1 = g.solve(T(p.b))
    for e, eb in CUBE64 if name == "cube12" and precision == 0 else SCALES[precision]:
        q = scaled(p, e, eb)
        print(f"[tiny] {name} precision={precision} smoother={smoother} 2^{e}", flush=True)
        h = amg.Hierarchy.from_problem(q, precision=precision, smoother=smoother)
        x, i = h.solve(T(q.b), check=False)
        assert i["status"] == 0 and abs(i["iters"] - i1["iters"]) <= 1, (i, i1)
        want = x1 * 2.0 ** (eb - e)
        assert torch.linalg.norm((x - want) * 2.0 ** (e - eb)) <= 1e-6 * torch.linalg.norm(x1)
        # in and out of the range by values updates: what a setup from scratch gives, bit for bit
        t = lambda a, dt: torch.as_tensor(a, dtype=dt, device="cuda:0")
        pattern = t(p.row_ptr, torch.int64), t(p.col, torch.int32)
        h.update_values(*pattern, T(p.val))
        y, j = h.solve(T(p.b))
        assert torch.equal(y, x1) and j["iters"] == i1["iters"]
        h.update_values(*pattern, T(q.val))
        y, j = h.solve(T(q.b))
        assert torch.equal(y, x) and j["iters"] == i["iters"]
        h.close()
    g.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("noalloc", [False, True])
def test_batch_of_scaled_and_unscaled_systems(precision, noalloc):
    from paper_1209_5421_amd import amg
    e, eb = SCALES[precision][0]
    ps = [prob("jittered65"), scaled(prob("jittered65"), e, eb), scaled(prob("jittered258"), e, eb), prob("jittered258")]
    hs = [amg.Hierarchy.from_problem(p, precision=precision) for p in ps]
    bs = [T(p.b) for p in ps]
    xs = [torch.full_like(b, float("nan")) for b in bs]
    code, infos = amg.solve_batch(hs, bs, xs, [1e-8] * len(hs), noalloc=noalloc)
    assert code == 0
    for h, b, x, i in zip(hs, bs, xs, infos):
        y, j = h.solve(b)
        assert i["iters"] == j["iters"] and torch.equal(x, y)
        h.close()
