"""Every kernel that the block products and the batches choose from, on integers
(every sum exact in FP32, so the results equal the FP64 products): the products
over runs and entries (paths of few rows), the row-block kernels of many blocks
and many nodes, tiles narrower than the block; and the batch's graph against its
plain launches.  The route is read off the memory a context takes."""
import numpy as np
import pytest

import oracle
import synth
from device_blocks import Blocks
from test_gpu_row_blocks import path_system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def run_system(nz, npath, seed, nx=9, ny=7):
    """Paths of one to three rows; a row has one or two stretches of depths at a node."""
    rng = np.random.default_rng([nz, npath, seed])
    ptr, col = [0], []
    for _ in range(npath):
        nodes = np.sort(rng.choice(nx * ny, rng.integers(1, 14), replace=False))
        for _ in range(rng.integers(1, 4)):
            for k in nodes:
                a, b = np.sort(rng.integers(0, nz + 1, 2))
                d = np.arange(a, max(b, a + 1)) if a < nz else np.array([nz - 1])
                if len(d) > 4 and rng.random() < 0.3:
                    d = np.delete(d, len(d) // 2)
                col.extend(k * nz + d)
            ptr.append(len(col))
    m = len(ptr) - 1
    val = rng.integers(1, 6, size=len(col)).astype(np.float64)
    return synth.RandomSystem(m=m, n=nx * ny * nz, nx=nx, ny=ny, nz=nz, row_ptr=np.array(ptr, dtype=np.int64),
                              col=np.array(col, dtype=np.int32), val=val, dt=np.zeros(m), damp=0.25, smooth=0.5)


def check(monkeypatch, s, widths, row_blocks):
    """widths: (right-hand sides, tile or None)."""
    from paper_2604_11920_amd import Solver, lsqr
    op = oracle.Operator.from_system(s)
    rng = np.random.default_rng(s.nz)
    Xs = rng.integers(-4, 5, size=(s.n, 32)).astype(np.float32)
    Ys = rng.integers(-4, 5, size=(op.mbar, 32)).astype(np.float32)
    want_y = np.stack([op.apply(Xs[:, r].astype(np.float64)) for r in range(32)], 1)
    want_x = np.stack([op.apply_t(Ys[:, r].astype(np.float64)) for r in range(32)], 1)
    for R, tile in widths:
        blocks = Blocks()
        monkeypatch.setattr(lsqr, "torch_allocator", blocks)
        with Solver.from_system(s) as sol:
            made = len(blocks.sizes)
            if tile:
                sol.set_batch_config(tile, 512)
            X, Y = Xs[:, 32 - R:].copy(), Ys[:, 32 - R:].copy()
            yg = sol.apply_block(torch.from_numpy(X).cuda()).cpu().numpy()
            xg = sol.apply_t_block(torch.from_numpy(Y).cuda()).cpu().numpy()
            # the FP32 copy of the transpose is made for the products over runs and entries
            assert (4 * s.nnz not in blocks.sizes[made:]) == row_blocks, (R, tile)
            assert np.array_equal(yg.astype(np.float64), want_y[:, 32 - R:]), (R, tile)
            assert np.array_equal(xg.astype(np.float64), want_x[:, 32 - R:]), (R, tile)
            assert blocks.intact()


WIDTHS = [(1, None), (2, None), (8, None), (32, None), (32, 1), (32, 8), (32, 16), (16, 4)]


@pytest.mark.parametrize("nz,npath", [(1, 300), (5, 40), (12, 700), (20, 300), (32, 150), (33, 60)])
def test_products_over_runs_and_entries(monkeypatch, nz, npath):
    check(monkeypatch, run_system(nz, npath, 0), WIDTHS, False)


@pytest.mark.parametrize("nz,rows", [(13, 18), (4, 16)])
def test_tiles_of_row_blocks(monkeypatch, nz, rows):
    check(monkeypatch, path_system(nz, rows, 40, 0), WIDTHS, True)


# one and two tiles of rows and of depths; 1,100 blocks and 1,110 nodes: 4 waves to
# each; many paths on few nodes: 8 waves to a node (and, of 500 blocks, to a block)
@pytest.mark.parametrize("nz,rows,npath,nx,ny", [(12, 6, 1100, 37, 30), (20, 18, 1100, 37, 30), (9, 17, 1100, 37, 30),
                                                 (32, 12, 1100, 37, 30), (17, 8, 1100, 9, 7), (32, 19, 1100, 37, 30),
                                                 (4, 16, 500, 9, 7), (16, 18, 500, 9, 7), (20, 19, 500, 9, 7),
                                                 (32, 7, 500, 9, 7)])
def test_row_blocks_of_many_paths_and_nodes(monkeypatch, nz, rows, npath, nx, ny):
    check(monkeypatch, path_system(nz, rows, npath, 0, nx=nx, ny=ny), [(1, None), (8, None), (32, None), (32, 8)], True)


def batch(count, graph, streams=False, twice=False):
    """Six uneven systems: (their solvers, their right-hand sides)."""
    from paper_2604_11920_amd import Solver
    sols, dts = [], []
    for i in range(count):
        s = synth.make_system(synth.small_config(nx=6 + i % 3, ny=7, nz=5, n_stations=10 + 2 * i, n_periods=4 + i % 4,
                                                 region=0.7, seed=i))
        st = torch.cuda.Stream() if streams else None
        sols.append(Solver.from_system(s, precond="jacobi", check_every=8, graph=graph, stream=st))
        dts.append(synth.checker_rhs_batch(s, n_checker=3, n_boot=2))
    if twice:
        sols, dts = sols + sols[:1], dts + [dts[0].copy()]
    torch.cuda.synchronize()
    return sols, dts


@pytest.mark.skip(reason="a run of this test ended in an abort of a runtime thread while the captured graph had a "
                         "branch per system; the branches were taken out, their cause was not found")
@pytest.mark.parametrize("count,streams,twice", [(2, False, False), (6, False, False), (6, True, False),
                                                 (1, True, False), (3, False, True)])
def test_graph_branches(count, streams, twice):
    """Graph and plain launches of several systems agree: contexts on streams of
    their own, a context given twice."""
    from paper_2604_11920_amd import solve_batched, solve_batched_refined
    out = []
    for graph in (False, True, True):
        sols, dts = batch(count, graph, streams and graph, twice)
        a, _, ia = solve_batched(sols, dts, 43)
        b, _, ib = solve_batched(sols, dts, 400, tol=1e-3)
        if twice:
            out.append((a, b, [], ia, ib, []))
        else:
            c, ic = solve_batched_refined(sols, dts, 400, 1e-9, inner_tol=1e-3, sweeps=6)
            out.append((a, b, c, ia, ib, ic))
        for s in set(sols):
            s.close()
    for k in (1, 2):
        for x, y in zip(out[0][:3], out[k][:3]):
            assert all(np.array_equal(p, q, equal_nan=True) for p, q in zip(x, y))
        for x, y in zip(out[0][3:], out[k][3:]):
            assert str(x) == str(y)
