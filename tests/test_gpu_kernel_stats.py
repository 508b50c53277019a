"""The bytes lsqr_kernel_stats counts for one launch, against the arrays that the
launch reads and writes: with the update in the forward launch (small grids, 16-bit
columns) and without it, and the part offsets of 4 and of 16 waves a node."""
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def expected(s, sol, sv, sx, fused, lsmr, sigma, waves):
    m, n, nnz, mb = s.m, s.n, s.nnz, s.m + 2 * s.n
    fwd = nnz * sv + 8 * (m + 1) + n * sx + 2 * mb * sx + (4 * m + m * sx if sigma else 0)
    if fused:
        fwd += 2 * nnz + 8 * n + sx * n + 32 * n + (16 * n if lsmr else 0)
    else:
        fwd += 4 * nnz
    runs = 0
    for i in range(m):
        c = s.col[s.row_ptr[i]:s.row_ptr[i + 1]]
        if len(c):
            runs += 1 + int(((c[1:] != c[:-1] + 1) | (c[1:] % s.nz == 0)).sum())
    nn = n // s.nz
    adj = nnz * sv + 6 * runs + 8 * (nn + 1) + 8 * waves * nn + 4 * nn + mb * sx + n * (8 + 2 * sx)
    return fwd, adj


@pytest.mark.parametrize("precision,sv,sx", [("fp64", 8, 8), ("fp32", 4, 4), ("bf16", 2, 4)])
@pytest.mark.parametrize("method", ["lsqr", "lsmr"])
@pytest.mark.parametrize("m,nx,ny,nz,waves", [(300, 6, 5, 4, 4), (900, 2, 1, 9, 16)])
def test_bytes(precision, sv, sx, method, m, nx, ny, nz, waves):
    from paper_2604_11920_amd import Solver
    s = synth.random_system(m, nx, ny, nz, row_len=(1, 12), seed=m)
    for rf in ("auto", "csr"):
        with Solver.from_system(s, precision=precision, method=method, row_format=rf) as sol:
            st = sol.kernel_stats()
            fwd, adj = expected(s, sol, sv, sx, rf == "auto", method == "lsmr", precision == "bf16", waves)
            assert st["row_format"] == 1 and (st["fwd_bytes"], st["adj_bytes"]) == (fwd, adj)


@pytest.mark.parametrize("nx,ny,per,waves", [(8, 8, 390, 4), (8, 8, 410, 16), (16, 16, 500, 4), (16, 16, 525, 16),
                                             (27, 27, 700, 4), (27, 27, 1470, 16), (28, 29, 4000, 4)])
def test_waves_of_a_node(nx, ny, per, waves):
    """16 waves share a node's runs where there are enough of them: `per` rows of
    two depths at every node, on either side of the rule."""
    import numpy as np
    from paper_2604_11920_amd import Solver
    nn, nz = nx * ny, 3
    n, m = nn * nz, nn * per
    col = (np.repeat(np.arange(nn), per)[:, None] * nz + [0, 1]).reshape(-1).astype(np.int32)
    rp = 2 * np.arange(m + 1, dtype=np.int64)
    with Solver(rp, col, np.ones(2 * m), nx, ny, nz, 0.1, 0.5) as sol:
        got = sol.kernel_stats()["adj_bytes"]
        q = sol.apply_t(torch.cat([torch.ones(m, dtype=torch.float64), torch.zeros(2 * n, dtype=torch.float64)]).cuda())
    adj = 16 * m + 6 * m + 8 * (nn + 1) + 8 * waves * nn + 4 * nn + 8 * (m + 2 * n) + 24 * n
    assert got == adj
    assert np.array_equal(q.cpu().numpy().reshape(nn, nz), np.tile([per, per, 0.0], (nn, 1)))
