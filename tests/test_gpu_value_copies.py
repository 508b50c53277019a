"""The FP32 copies of G's values serve the batched products over entries and the
FP32 inner solves of a stalled refinement, whichever asks first: the solve after
block products equals the solve of a fresh context bit for bit, and nothing is
written past a buffer's end."""
import numpy as np
import pytest

import synth
from device_blocks import Blocks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# one period a path (no row blocks); the second grid has no node runs, and its
# longer rows the plain CSR kernels
@pytest.mark.parametrize("nx,ny,nz,row_len", [(9, 8, 6, (1, 30)), (6, 5, 66, (100, 300)), (24, 20, 12, (390, 800))])
def test_block_products_then_fp32_inner_solves(monkeypatch, nx, ny, nz, row_len):
    from paper_2604_11920_amd import Solver, lsqr
    s = synth.random_system(301, nx, ny, nz, row_len=row_len, seed=nz)
    kw = dict(precision="bf16", precond="jacobi", refine_sweeps=3, refine_stall_ratio=1e-300)
    z = torch.randn(s.n, 4, device="cuda")
    y = torch.randn(s.m + 2 * s.n, 4, device="cuda")
    out = []
    for first in (False, True):
        blocks = Blocks()
        monkeypatch.setattr(lsqr, "torch_allocator", blocks)
        with Solver.from_system(s, **kw) as sol:
            if first:
                sol.apply_block(z)
                sol.apply_t_block(y)
            dm, _, info = sol.solve(s.dt, 200, tol=1e-14)
            assert info["inner_fp32"] == 1
            out.append((dm, sol.apply_block(z).cpu(), sol.apply_t_block(y).cpu()))
            assert blocks.intact()
        assert blocks.intact()
    (a, ya, xa), (b, yb, xb) = out
    assert np.array_equal(a, b) and torch.equal(ya, yb) and torch.equal(xa, xb)


def test_first_call_under_capture():
    """A capture only records the conversion: an eager call before the first replay
    makes the copies itself."""
    from paper_2604_11920_amd import Solver
    s = synth.random_system(301, 9, 8, 6, row_len=(1, 30), seed=2, integer=True)
    G = s.dense()
    rng = np.random.default_rng(1)
    Xs = [rng.integers(-4, 5, size=(s.n, 4)).astype(np.float32) for _ in range(4)]
    st = torch.cuda.Stream()
    x = torch.from_numpy(Xs[0]).cuda()
    y, eager = (torch.zeros(s.m + 2 * s.n, 4, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    sol = Solver.from_system(s, stream=st)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        sol.apply_block(x, y)
    sol.apply_block(x, eager)
    torch.cuda.synchronize()
    assert np.array_equal(eager.cpu().numpy()[:s.m], G @ Xs[0])
    for X in Xs:
        x.copy_(torch.from_numpy(X))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy()[:s.m], G @ X)
    sol.close()
