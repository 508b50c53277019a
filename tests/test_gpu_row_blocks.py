"""Block products where rows share their lateral nodes (row blocks on the matrix
cores): integer data, so that every sum is exact in FP32 and the results equal
the FP64 products, at the edges of the tiles: depths around multiples of 4 and
16, rows a path around 16 and 20, paths of few rows, every tile width; and
infinities, which must reach exactly the rows and columns with an entry there.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def path_system(nz, rows, npath, seed, nx=9, ny=7):
    """Paths of `rows` rows (0: 1 to 24) over their own random nodes; a row skips a
    node now and then and reaches from the first to the last third of the depths of
    the others (windows that differ more hold too few values per stored one)."""
    rng = np.random.default_rng([nz, rows, seed])
    ptr, col = [0], []
    for _ in range(npath):
        nodes = np.sort(rng.choice(nx * ny, rng.integers(1, 14), replace=False))
        for _ in range(rows or rng.integers(1, 25)):
            for k in nodes:
                if rng.random() < 0.08:
                    continue
                a = rng.integers(0, max(1, nz // 3))
                b = rng.integers(max(a + 1, 2 * nz // 3 + 1), nz + 1)
                col.extend(range(k * nz + a, k * nz + b))
            ptr.append(len(col))
    col = np.array(col, dtype=np.int32)
    val = rng.integers(1, 6, size=len(col)).astype(np.float64)
    m = len(ptr) - 1
    return synth.RandomSystem(m=m, n=nx * ny * nz, nx=nx, ny=ny, nz=nz, row_ptr=np.array(ptr, dtype=np.int64),
                              col=col, val=val, dt=np.zeros(m), damp=0.25, smooth=0.5)


@pytest.mark.parametrize("nz,rows", [(1, 6), (4, 16), (5, 17), (12, 20), (13, 21), (16, 15), (17, 19),
                                     (20, 20), (21, 16), (32, 20), (32, 8), (33, 12), (9, 0)])
def test_products_exact(nz, rows):
    from paper_2604_11920_amd import Solver
    s = path_system(nz, rows, 40, 0)
    op = oracle.Operator.from_system(s)
    rng = np.random.default_rng(nz)
    with Solver.from_system(s) as sol:
        for R in (1, 2, 4, 8, 16, 32):
            X = rng.integers(-4, 5, size=(s.n, R)).astype(np.float32)
            Y = rng.integers(-4, 5, size=(op.mbar, R)).astype(np.float32)
            yg = sol.apply_block(torch.from_numpy(X).cuda()).cpu().numpy()
            xg = sol.apply_t_block(torch.from_numpy(Y).cuda()).cpu().numpy()
            for r in range(R):
                assert np.array_equal(yg[:, r].astype(np.float64), op.apply(X[:, r].astype(np.float64))), (R, r)
                assert np.array_equal(xg[:, r].astype(np.float64), op.apply_t(Y[:, r].astype(np.float64))), (R, r)


@pytest.mark.parametrize("R", [2, 32])
def test_infinities_stay_in_their_entries(R):
    from paper_2604_11920_amd import Solver
    s = path_system(13, 18, 40, 1)
    dense = np.zeros((s.m, s.n))
    for i in range(s.m):
        p = slice(s.row_ptr[i], s.row_ptr[i + 1])
        dense[i, s.col[p]] = s.val[p]
    j, i = int(s.col[len(s.col) // 2]), s.m // 2
    X = np.ones((s.n, R), dtype=np.float32)
    X[j, 1] = np.inf
    Y = np.zeros((s.m + 2 * s.n, R), dtype=np.float32)
    Y[:s.m] = 1.0
    Y[i, 0] = -np.inf
    with Solver.from_system(s) as sol:
        yg = sol.apply_block(torch.from_numpy(X).cuda()).cpu().numpy()[:s.m]
        xg = sol.apply_t_block(torch.from_numpy(Y).cuda()).cpu().numpy()
    want = np.repeat(dense.sum(1)[:, None], R, 1)
    want[dense[:, j] != 0, 1] = np.inf
    assert np.array_equal(yg, want)
    want = np.repeat(dense.sum(0)[:, None], R, 1)
    want[dense[i] != 0, 0] = -np.inf
    assert np.array_equal(xg, want)
