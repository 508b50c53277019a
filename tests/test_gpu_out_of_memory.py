"""An allocator that refuses: the call reports LSQR_E_OOM, and the context goes on
working when there is memory again."""
import numpy as np
import pytest

import synth
from device_blocks import Blocks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def make(monkeypatch, s, blocks, **kw):
    from paper_2604_11920_amd import Solver, lsqr
    monkeypatch.setattr(lsqr, "torch_allocator", blocks)
    return Solver.from_system(s, **kw)


def shared_paths(seed):
    """Paths of 12 rows over the same nodes: row blocks."""
    rng = np.random.default_rng(seed)
    nx, ny, nz = 6, 5, 4
    ptr, col = [0], []
    for _ in range(15):
        nodes = np.sort(rng.choice(nx * ny, 7, replace=False))
        for _ in range(12):
            col.extend(np.add.outer(nodes * nz, np.arange(nz)).reshape(-1))
            ptr.append(len(col))
    m = len(ptr) - 1
    return synth.RandomSystem(m=m, n=nx * ny * nz, nx=nx, ny=ny, nz=nz, row_ptr=np.array(ptr, dtype=np.int64),
                              col=np.array(col, dtype=np.int32), val=rng.integers(1, 6, len(col)).astype(float),
                              dt=rng.standard_normal(m), damp=0.25, smooth=0.5)


def test_solves(monkeypatch):
    """A solve of more iterations needs more state rows, a batch of more
    right-hand sides new buffers: refused once, then served."""
    from paper_2604_11920_amd import lsqr
    s = shared_paths(5)
    dt = np.random.default_rng(6).standard_normal((s.m, 4))
    blocks = Blocks()
    with make(monkeypatch, s, blocks) as sol:
        want, want5 = sol.solve(s.dt, 700)[0], sol.solve(s.dt, 5)[0]
        batch = lsqr.solve_batched_refined([sol], [dt], 700, 1e-8)[0][0]
    blocks = Blocks()
    with make(monkeypatch, s, blocks) as sol:
        sol.solve(s.dt, 5)
        sol.apply_block(torch.zeros(s.n, 2, device="cuda"))
        blocks.fail_at, blocks.fail_on = blocks.count, True
        for f in (lambda: sol.solve(s.dt, 700), lambda: lsqr.solve_batched_refined([sol], [dt], 700, 1e-8)):
            with pytest.raises(lsqr.LsqrError) as e:
                f()
            assert e.value.status == lsqr.LSQR_E_OOM
        blocks.fail_at = None
        assert np.array_equal(sol.solve(s.dt, 5)[0], want5)
        assert np.array_equal(sol.solve(s.dt, 700)[0], want)
        assert np.array_equal(lsqr.solve_batched_refined([sol], [dt], 700, 1e-8)[0][0], batch)
        assert blocks.intact()


def test_widths_in_turn_hold_no_more_memory(monkeypatch):
    from paper_2604_11920_amd import lsqr
    s = shared_paths(7)
    blocks = Blocks()
    with make(monkeypatch, s, blocks) as sol:
        def round_trip():
            for R in (2, 32):
                sol.apply_block(torch.zeros(s.n, R, device="cuda"))
            return sum(n for _, n in blocks.live.values())
        first = round_trip()
        assert [round_trip() for _ in range(3)] == [first] * 3
