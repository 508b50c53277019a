"""An allocator that refuses: every entry point reports LSQR_E_OOM (or does
without the memory), whichever of its allocations it is, gives back what it had,
and the context goes on working when there is memory again."""
import ctypes

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


CASES = [dict(precision="fp64", precond="jacobi"), dict(precision="fp32"), dict(precision="bf16", method="lsqr"),
         dict(precision="bf16", col_format="runs"), dict(precision="fp64", row_format="groups", method="lsmr"),
         dict(precision="fp32", col_format="csc", row_format="csr")]


@pytest.mark.parametrize("kw", CASES)
def test_create(monkeypatch, kw):
    from paper_2604_11920_amd import lsqr
    s = synth.random_system(60, 5, 4, 6, row_len=(0, 30), seed=1)
    whole = Blocks()
    with make(monkeypatch, s, whole, **kw):
        pass
    assert whole.count > 15
    for i in range(whole.count):
        for on in (False, True):
            blocks = Blocks(fail_at=i, fail_on=on)
            with pytest.raises(lsqr.LsqrError) as e:
                make(monkeypatch, s, blocks, **kw)
            assert e.value.status == lsqr.LSQR_E_OOM, (i, str(e.value))
            assert not blocks.live and blocks.damaged == 0


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


def last_error_allocator(blocks):
    """The refusals come from hipMalloc, which leaves its error behind."""
    def factory(device, stream):
        from paper_2604_11920_amd import lsqr
        hip = ctypes.CDLL("libamdhip64.so")
        inner, free = blocks(device, stream)

        def alloc(nbytes, user):
            p = inner(nbytes, None)
            if not p:
                q = ctypes.c_void_p()
                assert hip.hipMalloc(ctypes.byref(q), ctypes.c_size_t(1 << 50)) != 0
            return p

        return lsqr._ALLOC_FN(alloc), free
    return factory


@pytest.mark.parametrize("hip_error", [False, True])
def test_block_products(monkeypatch, hip_error):
    """The planning of the row blocks does without them; the rest is refused.
    Afterwards both products are right, with the memory and on the other layouts
    (integers: every sum is exact)."""
    from paper_2604_11920_amd import lsqr
    s = shared_paths(3)
    rng = np.random.default_rng(4)
    X = rng.integers(-4, 5, size=(s.n, 8)).astype(np.float32)
    Y = rng.integers(-4, 5, size=(s.m, 8)).astype(np.float32)
    G = s.dense()
    Xg, Yg = torch.from_numpy(X).cuda(), torch.zeros(s.m + 2 * s.n, 8, device="cuda")
    Yg[:s.m] = torch.from_numpy(Y).cuda()

    def check(sol):
        y = sol.apply_block(Xg).cpu().numpy()
        x = sol.apply_t_block(Yg).cpu().numpy()
        assert np.array_equal(y[:s.m], G @ X) and np.array_equal(x, G.T @ Y)

    blocks = Blocks()
    with make(monkeypatch, s, blocks) as sol:
        first = blocks.count
        check(sol)
        last = blocks.count
    other = refused = 0
    for i in range(first, last):
        blocks = Blocks(fail_at=i)
        factory = last_error_allocator(blocks) if hip_error else blocks
        with make(monkeypatch, s, factory) as sol:
            try:
                check(sol)
                other += 1
            except lsqr.LsqrError as e:
                assert e.status == lsqr.LSQR_E_OOM, (i, str(e))
                refused += 1
            check(sol)
            assert blocks.intact()
        assert not blocks.live and blocks.intact()
    assert other > 10 and refused > 10


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
