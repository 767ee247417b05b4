"""The fine smoother's fused phase against the oracle where its windows take other forms than test_gpu_fine_cells': more
than 256 windows in a color (four wavefronts, a thread per cell), and windows that end with empty cells (lane groups
without a cell). The windows are counted here by setup's rule: a color's cells in storage order, a new window at every 512th
cell, at a cell whose first row lies in another band of 225 rows than the previous cell's, and around cells of more than
256 rows. Tolerances as there: the same operations up to the order of a row's subtractions, so a few roundings of rows of
at most 40 entries."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_fine_cells import T, scattered

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BAND, CELLS, BIG = 225, 512, 256


def spread(v):
    v = v.astype(np.uint32)
    for s, m in ((8, 0x00FF00FF), (4, 0x0F0F0F0F), (2, 0x33333333), (1, 0x55555555)):
        v = (v | (v << np.uint32(s))) & np.uint32(m)
    return v


def windows(coords, side):
    """(windows of each color, windows that end with an empty cell, sizes of the cells)"""
    t = np.minimum((coords * side).astype(int), side - 1)
    m = spread(t[:, 0]) | (spread(t[:, 1]) << np.uint32(1))
    n4 = side * side // 4
    q = (m & 3).astype(np.int64) * n4 + (m >> 2)
    sizes = np.bincount(q, minlength=4 * n4)
    first = np.concatenate([[0], np.cumsum(sizes)])
    counts, empty_end = [], 0
    for c in range(4):
        s = sizes[c * n4:(c + 1) * n4]
        f = first[c * n4:(c + 1) * n4] - first[c * n4]
        mark = np.zeros(n4, bool)
        mark[::CELLS] = True
        big = s > BIG
        mark[1:] |= big[1:] | big[:-1] | (f[1:] // BAND != f[:-1] // BAND)
        counts.append(int(mark.sum()))
        last = np.append(np.flatnonzero(mark)[1:], n4) - 1
        empty_end += int((s[last] == 0).sum())
    return counts, empty_end, sizes


# 262,200 unknowns, density rising towards x = 0; 5,000 unknowns of which most cells hold none
@pytest.mark.parametrize("n,power,many", [(262200, 1.7, True), (5000, 6.0, False)])
@pytest.mark.parametrize("smoother", [0, 1])
def test_windows_of_other_forms(n, power, many, smoother):
    from paper_1209_5421_amd import amg
    p = scattered(n, power, seed=n)
    print(f"[fine windows] n={n} power={power} smoother={smoother}", flush=True)
    g = amg.Hierarchy.from_problem(p, device="cuda:0", smoother=smoother)
    o = oracle.setup_problem(p)
    o.set_block_smoother(bool(smoother))
    counts, empty_end, sizes = windows(p.coords, int(round(np.sqrt(g.level_info(1)["n"]))))
    assert (min(counts) > 256) == many, counts
    assert empty_end > 0
    for lo, hi in ((1, 8), (9, 16), (17, 32)):
        assert np.any((sizes >= lo) & (sizes <= hi)), (lo, hi)
    rng = np.random.default_rng(3)
    x, f = rng.standard_normal(n), rng.standard_normal(n)
    for fwd in (True, False):
        want = o.smooth(0, f, x, fwd)
        for prec, tol in ((0, 1e-11), (1, 1e-4)):
            got = g.smooth(0, T(f), T(x), fwd, precision=prec).cpu().numpy()
            np.testing.assert_allclose(got, want, rtol=0, atol=tol * np.abs(want).max(), err_msg=f"{fwd} {prec}")
    g.close()
    o.close()
