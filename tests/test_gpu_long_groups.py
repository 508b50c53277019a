"""Row groups of very many rows: few columns met over and over, so that a group's
columns fit long after its rows are many.  Boundaries and lists against the
greedy rule, products of integers (exact), and a set-up that stays linear."""
import time

import numpy as np
import pytest
import scipy.sparse as sp

from device_blocks import Blocks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def stretch(m, first, count, seed):
    """m rows of 6 runs of 4 columns among the `count` columns from `first` on."""
    rng = np.random.default_rng([seed, first])
    b = np.sort(np.argpartition(rng.random((m, count // 8)), 6, axis=1)[:, :6], axis=1)
    return (first + 8 * b[:, :, None] + np.arange(4)).reshape(m, 24)


def system(stretches, seed=0):
    col = np.concatenate([stretch(m, f, c, seed) for m, f, c in stretches])
    rp = np.arange(len(col) + 1, dtype=np.int64) * 24
    val = np.random.default_rng(seed + 1).integers(1, 9, size=col.size).astype(float)
    return rp, col.reshape(-1).astype(np.int32), val


def greedy(rp, col, n, cap):
    seen, size, gp, lists = np.zeros(n, bool), 0, [0], []
    for i in range(len(rp) - 1):
        c = col[rp[i]:rp[i + 1]]
        new = len(c) - int(seen[c].sum())
        if size + new > cap and i > gp[-1]:
            lists.append(np.nonzero(seen)[0])
            gp.append(i)
            seen[:], size, new = False, 0, len(c)
        seen[c] = True
        size += new
    return np.array(gp + [len(rp) - 1], np.int32), lists + [np.nonzero(seen)[0]]


# a grid within the group size; one group although the grid is larger; long
# groups, then short ones, then long ones again, with a last column alone
@pytest.mark.parametrize("grid,stretches", [
    ((10, 10, 10), [(60000, 0, 1000)]),
    ((11, 10, 10), [(60000, 40, 1000)]),
    ((50, 20, 10), [(20000, 0, 800), (20000, 2000, 1000), (300, 0, 10000), (25000, 7000, 1016), (1, 9992, 8 * 7)]),
])
def test_groups(monkeypatch, grid, stretches):
    from paper_2604_11920_amd import Solver, lsqr
    n = grid[0] * grid[1] * grid[2]
    stretches = [(m, min(f, n - c), c) for m, f, c in stretches]
    rp, col, val = system(stretches)
    gp, lists = greedy(rp, col, n, 1024)
    blocks = Blocks()
    monkeypatch.setattr(lsqr, "torch_allocator", blocks)
    G = sp.csr_matrix((val, col, rp), shape=(len(rp) - 1, n))
    rng = np.random.default_rng(3)
    x, y = rng.integers(-4, 5, n).astype(float), rng.integers(-4, 5, len(rp) - 1 + 2 * n).astype(float)
    y[len(rp) - 1:] = 0.0
    with Solver(rp, col, val, *grid, 0.0, 0.0, row_format="groups") as sol:
        st = sol.kernel_stats()
        assert (st["row_format"], st["groups"]) == (4, len(gp) - 1)
        assert st["staged_cols"] == sum(len(v) for v in lists)
        assert blocks.holds(gp) and blocks.holds(np.concatenate(lists).astype(np.int32))
        yy = sol.apply(torch.from_numpy(x).cuda()).cpu().numpy()
        xx = sol.apply_t(torch.from_numpy(y).cuda()).cpu().numpy()
        assert np.array_equal(yy[:len(rp) - 1], G @ x) and np.array_equal(xx, G.T @ y[:len(rp) - 1])
        assert blocks.intact()


def test_linear_in_the_rows():
    """400,000 rows in one group on a grid of more columns than a group holds: a
    walk over all later rows from every row is 2e11 runs; the whole set-up is
    allowed what 1e9 of them take."""
    from paper_2604_11920_amd import Solver
    rp, col, val = system([(400000, 40, 1000)])
    arrays = [torch.from_numpy(a).cuda() for a in (rp, col, val)]
    best = np.inf
    for _ in range(3):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        with Solver(*arrays, 11, 10, 10, 0.1, 0.5, row_format="groups") as sol:
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
            assert sol.kernel_stats()["groups"] == 1
    assert best < 1.0, best
