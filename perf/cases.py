"""Timed cases: the work a program hands to the solver, through the public entry points.

A program keeps its system on the GPU and either solves it again and again on one hierarchy ("solve"), meets it for the
first time ("new": setup, solve, release), gives a resident hierarchy new coefficients each time step ("step": device
assembly, values update, solve), or hands over several systems at once ("batch"). The systems are those of the
generators: jittered P1 lattices of the unit square (plain, or with a 16 x 16 checkerboard of coefficients over six
decades), a lattice graded towards a corner, and the heat step on the unit cube. Sizes run from the small systems of the
tests to the meshes of the benchmark; the smoother and the precision are options a caller sets, and every solve stops at
the benchmark's 1e-8.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1209_5421_amd import amg, meshgen

TOL = 1e-8
KAPPA_TILES = 16
DEVICE = "cuda:0"


def _case(name, kind, mesh, side, precision, smoother, count=1):
    c = dict(kind=kind, mesh=mesh, side=side, precision=precision, smoother=smoother, count=count)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest system of the tests and the smoke check (3,969 unknowns) on the library's defaults: latency
        _case("solve_4k_fp64", "solve", "jittered", 65, 0, 0),
        # a new mesh of the serving stream's smallest size (10,201 unknowns): setup counts as much as the solve
        _case("new_10k_fp32", "new", "jittered", 103, 1, 0),
        # the middle of the serving stream (99,856 unknowns) on a cached hierarchy
        _case("solve_100k_fp32", "solve", "jittered", 318, 1, 0),
        # an odd size (301,401 unknowns) in plain FP64, the library's default form
        _case("solve_301k_fp64", "solve", "jittered", 551, 0, 0),
        # the benchmark's system (1,044,484 unknowns), further right-hand sides on a resident hierarchy
        _case("solve_1m_fp32", "solve", "jittered", 1024, 1, 1),
        # the benchmark's step: setup and solve of a system met for the first time
        _case("new_1m_fp32", "new", "jittered", 1024, 1, 1),
        # the benchmark's coefficient checkerboard (1,999,396 unknowns)
        _case("solve_2m_checker_fp32", "solve", "checker", 1416, 1, 1),
        # a mesh graded towards a corner (498,436 unknowns): cells of very uneven size, couplings of long reach
        _case("solve_498k_graded_fp32", "solve", "graded", 708, 1, 1),
        # a time step with new coefficients (260,100 unknowns): assembly, values update, solve
        _case("step_260k_fp32", "step", "jittered", 512, 1, 1),
        # a serving batch of eight small systems (about 10,000 to 65,000 unknowns), the default smoother
        _case("batch_8_fp32", "batch", "jittered", 254, 1, 0, count=8),
        # the octree variant at the size of its tests (8,820 unknowns) on the defaults
        _case("solve_8k_cube_fp64", "solve", "cube", 20, 0, 0),
        # the benchmark's cube heat step (1,020,100 unknowns)
        _case("solve_1m_cube_fp32", "solve", "cube", 100, 1, 1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "new", "step", "batch"])
    precision = 1 if rng.random() < 0.7 else 0
    smoother = rng.randrange(2)
    if kind == "batch":  # the default smoother, sizes up to the whole-solve limit
        return _case(None, kind, "jittered", rng.randint(102, 256), precision, 0, count=rng.randint(2, 12))
    mesh = rng.choice(["jittered", "jittered", "checker", "graded", "cube"]) if kind == "solve" else "jittered"
    side = {"jittered": lambda: _log_int(rng, 65, 1400), "checker": lambda: _log_int(rng, 130, 1100),
            "graded": lambda: _log_int(rng, 65, 600), "cube": lambda: _log_int(rng, 12, 90)}[mesh]()
    return _case(None, kind, mesh, side, precision, smoother)


# ---- inputs ----

def _graded_points(side, seed):
    """A jittered lattice pulled towards (0, 0): a point at max-norm distance t from the corner moves along its ray to
    distance r(t) with dr/dt ~ (r + 0.01)^0.75, the spacing of the generators' graded mesh."""
    p = torch.as_tensor(meshgen.jittered_points(side, seed, 0.2), device=DEVICE)
    e = 0.01 ** 0.25
    t = p.amax(1)
    s = 1.01 ** 0.25 - e
    r = (e + s * t) ** 4 - 0.01
    return p * torch.where(t > 0, r / t.clamp_min(1e-300), torch.zeros_like(t))[:, None].clamp(max=1.0)


def _square_system(mesh, side, seed):
    pts = _graded_points(side, seed) if mesh == "graded" else \
        torch.as_tensor(meshgen.jittered_points(side, seed), device=DEVICE)
    return meshgen.lattice_p1_assemble(side, pts, meshgen.lattice_diagonals(side, pts),
                                       KAPPA_TILES if mesh == "checker" else 0, kappa_seed=seed)


def _cube_system(m, seed):
    """The heat step of the generators (dt = h, jittered (m+1)^3 lattice, six tetrahedra per cube, inlet face x = 0
    eliminated), assembled cube by cube on the GPU in a fixed order."""
    h, w = 1.0 / m, m + 1
    g = np.arange(w, dtype=np.float64) * h
    z, y, x = np.meshgrid(g, g, g, indexing="ij")
    pts = np.stack([x, y, z], -1)
    d = np.random.default_rng(seed).uniform(-0.15 * h, 0.15 * h, size=pts.shape)
    d[(pts <= 0.0) | (pts >= 1.0)] = 0.0
    P = torch.as_tensor(pts + d, device=DEVICE)
    off = [(c & 1, (c >> 1) & 1, c >> 2) for c in range(8)]
    corner = [P[oz:oz + m, oy:oy + m, ox:ox + m] for ox, oy, oz in off]
    S = torch.zeros((w, w, w, 27), dtype=torch.float64, device=DEVICE)
    has = torch.zeros((w, w, w, 27), dtype=torch.bool, device=DEVICE)
    for a in range(3):
        for b in range(3):
            if a == b:
                continue
            tet = (0, 1 << a, (1 << a) | (1 << b), 7)
            e = [corner[tet[i]] - corner[0] for i in (1, 2, 3)]
            n = [torch.linalg.cross(e[1], e[2]), torch.linalg.cross(e[2], e[0]), torch.linalg.cross(e[0], e[1])]
            det = (e[0] * n[0]).sum(-1)
            vol = det.abs() / 6.0
            grad = [v / det[..., None] for v in n]
            grad = [-(grad[0] + grad[1] + grad[2])] + grad
            for i in range(4):
                for j in range(4):
                    v = vol * (grad[i] * grad[j]).sum(-1)
                    if i == j:
                        v = v + vol / 4.0 / h
                    (ox, oy, oz), (qx, qy, qz) = off[tet[i]], off[tet[j]]
                    slot = (qz - oz + 1) * 9 + (qy - oy + 1) * 3 + (qx - ox + 1)
                    S[oz:oz + m, oy:oy + m, ox:ox + m, slot] += v
                    has[oz:oz + m, oy:oy + m, ox:ox + m, slot] = True
    ar = lambda k: torch.arange(k, device=DEVICE)
    dz, dy, dx = torch.meshgrid(ar(3) - 1, ar(3) - 1, ar(3) - 1, indexing="ij")
    Z, Y, X = torch.meshgrid(ar(w), ar(w), ar(w), indexing="ij")
    nx = X[..., None] + dx.reshape(-1)
    col = ((Z[..., None] + dz.reshape(-1)) * w + Y[..., None] + dy.reshape(-1)) * m + nx - 1
    keep = (has & (nx >= 1))[:, :, 1:]
    rp = torch.zeros(w * w * m + 1, dtype=torch.int64, device=DEVICE)
    rp[1:] = torch.cumsum(keep.reshape(-1, 27).sum(1), 0)
    return (P[:, :, 1:].reshape(-1, 3).contiguous(), rp, col[:, :, 1:][keep].to(torch.int32).contiguous(),
            S[:, :, 1:][keep].contiguous())


def _system(case, seed):
    if case["mesh"] == "cube":
        return _cube_system(case["side"], seed)
    return _square_system(case["mesh"], case["side"], seed)


def _rhs(n, seed):
    return torch.as_tensor(meshgen.rhs(n, seed + 1_000_000), device=DEVICE)


def _mesh_arrays(side, seed):
    """Points, triangles and unknown numbers of a jittered lattice mesh, on the GPU."""
    pts = torch.as_tensor(meshgen.jittered_points(side, seed), device=DEVICE)
    m = side - 1
    ac = meshgen.lattice_diagonals(side, pts).reshape(-1)[:, None]
    a = (torch.arange(m, device=DEVICE)[:, None] * side + torch.arange(m, device=DEVICE)[None, :]).reshape(-1)
    b, c, d = a + 1, a + side + 1, a + side
    t1 = torch.where(ac, torch.stack([a, b, c], 1), torch.stack([a, b, d], 1))
    t2 = torch.where(ac, torch.stack([a, c, d], 1), torch.stack([b, c, d], 1))
    tris = torch.cat([t1, t2]).to(torch.int32).contiguous()
    dof = torch.full((side, side), -1, dtype=torch.int32, device=DEVICE)
    n = side - 2
    dof[1:-1, 1:-1] = torch.arange(n * n, dtype=torch.int32, device=DEVICE).reshape(n, n)
    return pts, tris, dof.reshape(-1).contiguous()


def _kappa(pts, tris, seed):
    """A smooth coefficient per triangle, 1 + sin(2 pi (x + s)) sin(2 pi y) / 2 at its centroid."""
    s = (seed % 64) / 64.0
    c = (pts[tris[:, 0].long()] + pts[tris[:, 1].long()] + pts[tris[:, 2].long()]) / 3.0
    return 1.0 + 0.5 * torch.sin(2 * math.pi * (c[:, 0] + s)) * torch.sin(2 * math.pi * c[:, 1])


def _batch_sides(case):
    """The sides of a batch's systems: from 102 (10,000 unknowns) up to the case's side, evenly in the logarithm."""
    k = case["count"]
    lo, hi = math.log(102), math.log(case["side"])
    return [int(round(math.exp(lo + (hi - lo) * i / max(1, k - 1)))) for i in range(k)]


def _hierarchy(case, system):
    coords, rp, col, val = system
    return amg.Hierarchy(coords, rp, col, val, box=meshgen.UNIT_CUBE if coords.shape[1] == 3 else meshgen.UNIT_BOX,
                         precision=case["precision"], smoother=case["smoother"])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        hs, bs = [], []
        for i, side in enumerate(_batch_sides(case)):
            system = _square_system("jittered", side, seed + 1000 * i)
            hs.append(_hierarchy(case, system))
            bs.append(_rhs(len(system[0]), seed + 1000 * i))
        return dict(case=case, h=hs, b=bs, x=[torch.empty_like(b) for b in bs])
    if kind == "step":
        pts, tris, dof = _mesh_arrays(case["side"], seed)
        mesh = amg.P1Mesh(pts, tris, dof, (case["side"] - 2) ** 2)
        rp, col = mesh.pattern()
        val = mesh.assemble()
        h = _hierarchy(case, (pts.reshape(case["side"], -1, 2)[1:-1, 1:-1].reshape(-1, 2).contiguous(), rp, col, val))
        b = _rhs(mesh.ndof, seed)
        return dict(case=case, mesh=mesh, h=h, rp=rp, col=col, val=val, kappa=_kappa(pts, tris, seed), b=b,
                    x=torch.empty_like(b))
    system = _system(case, seed)
    b = _rhs(len(system[0]), seed)
    s = dict(case=case, system=system, b=b, x=torch.empty_like(b))
    if kind == "solve":
        s["h"] = _hierarchy(case, system)
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind == "batch":
        code, infos = amg.solve_batch(s["h"], s["b"], s["x"], [TOL] * len(s["h"]))
        if code != amg.OK:
            raise RuntimeError(f"amg_solve_batch: {code}")
        return dict(x=s["x"], iters=[i["iters"] for i in infos])
    if kind == "step":
        s["mesh"].assemble(s["kappa"], out=s["val"])
        s["h"].update_values(s["rp"], s["col"], s["val"])
        x, info = s["h"].solve(s["b"], tol=TOL, x=s["x"])
        return dict(val=s["val"], x=x, iters=info["iters"])
    if kind == "new":
        h = _hierarchy(s["case"], s["system"])
        x, info = h.solve(s["b"], tol=TOL, x=s["x"])
        h.close()
        return dict(x=x, iters=info["iters"])
    x, info = s["h"].solve(s["b"], tol=TOL, x=s["x"])
    return dict(x=x, iters=info["iters"])


# ---- what a pass cannot do without ----

def work(case):
    """Bytes and operations of one pass, from the method alone: the system read and the solution written once, and for
    about 14 outer iterations (11 on the cube, 55 on the checkerboard, 45 on the graded mesh) the matrix and vectors of
    the outer product in 64 bits, three passes of the preconditioner over the matrix in its precision, the vectors of
    the outer iteration, and the tree levels (each level's cells visited 2^depth times, about 1,000 bytes a finest cell
    in 32 bits)."""
    sides = _batch_sides(case) if case["kind"] == "batch" else [case["side"]]
    cube = case["mesh"] == "cube"
    its = 11 if cube else {"jittered": 14, "checker": 55, "graded": 45}[case["mesh"]]
    word = 4 if case["precision"] else 8
    total, flops = 0.0, 0.0
    for side in sides:
        n = (side + 1) ** 2 * side if cube else (side - 2) ** 2
        nnz = (15 if cube else 7) * n
        tree = 0.5 * n * 250 * word
        per = 12 * nnz + 24 * n + 108 * n + 3 * ((4 + word) * nnz + 3 * word * n) + tree
        total += its * per + 12 * nnz + 16 * n
        flops += its * (8 * nnz + 20 * n + 0.5 * n * 8 * 20)
        if case["kind"] == "new":
            total += 40 * nnz + 60 * n
        elif case["kind"] == "step":
            total += 60 * nnz + 200 * n
    return dict(bytes=total, flops=flops)


# ---- the same in 64 bits ----

def _cg(rp, col, val, b, tol=1e-13, max_iters=60000):
    """Jacobi-preconditioned conjugate gradients in 64 bits on padded rows, or None if they do not end in time."""
    n = len(b)
    cnt = rp[1:] - rp[:-1]
    w = int(cnt.max())
    row = torch.repeat_interleave(torch.arange(n, device=b.device), cnt)
    at = (torch.arange(len(col), device=b.device) - rp[:-1][row]) * n + row
    C = torch.arange(n, device=b.device).repeat(w)
    C[at] = col.long()
    V = torch.zeros(w * n, dtype=torch.float64, device=b.device)
    V[at] = val
    C, V = C.reshape(w, n), V.reshape(w, n)
    mul = lambda v: (V * v[C]).sum(0)
    diag = torch.zeros(n, dtype=torch.float64, device=b.device)
    on = col.long() == row
    diag[row[on]] = val[on]
    x = torch.zeros_like(b)
    r = b.clone()
    norm = float(b.norm())
    for start in range(6):  # restarts from the true residual
        z = r / diag
        p, rz = z.clone(), torch.dot(r, z)
        for it in range(max_iters):
            q = mul(p)
            a = rz / torch.dot(p, q)
            x += a * p
            r -= a * q
            if it % 100 == 99 and float(r.norm()) <= tol * norm:
                break
            z = r / diag
            new = torch.dot(r, z)
            p = z + (new / rz) * p
            rz = new
        r = b - mul(x)
        if float(r.norm()) <= 20 * tol * norm:
            break
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        xs = []
        for i, side in enumerate(_batch_sides(case)):
            coords, rp, col, val = _square_system("jittered", side, seed + 1000 * i)
            xs.append(_cg(rp, col, val, _rhs(len(coords), seed + 1000 * i)))
        return dict(x=xs, iters=None)
    if kind == "step":
        side = case["side"]
        pts, tris, dof = _mesh_arrays(side, seed)
        kappa = _kappa(pts, tris, seed)
        n = (side - 2) ** 2
        P = [pts[tris[:, k].long()] for k in range(3)]
        E = [P[2] - P[1], P[0] - P[2], P[1] - P[0]]
        area2 = (E[2][:, 0] * -E[1][:, 1] + E[2][:, 1] * E[1][:, 0]).abs()
        D = [dof[tris[:, k].long()].long() for k in range(3)]
        key, v = [], []
        for a in range(3):
            for b in range(3):
                keep = (D[a] >= 0) & (D[b] >= 0)
                key.append((D[a] * n + D[b])[keep])
                v.append((kappa * (E[a] * E[b]).sum(1) / (2.0 * area2))[keep])
        key, pos = torch.unique(torch.cat(key), return_inverse=True)
        val = torch.zeros(len(key), dtype=torch.float64, device=DEVICE).index_add_(0, pos, torch.cat(v))
        rp = torch.zeros(n + 1, dtype=torch.int64, device=DEVICE)
        rp[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
        return dict(val=val, x=_cg(rp, key % n, val, _rhs(n, seed)), iters=None)
    coords, rp, col, val = _system(case, seed)
    return dict(x=_cg(rp, col, val, _rhs(len(coords), seed)), iters=None)
