"""The formats planned on the device, against the structure they describe:
the transpose bitwise against SciPy's CSC, the row groups' boundaries and
column lists against the greedy rule, the padded lengths against their
definition, and products of integer values (every sum exact) in every format
and value type, on ragged structures: empty rows and nodes, several runs of a
row in one node, runs up to a node's last depth, single entries, long rows.
"""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def ragged(m, nx, ny, nz, seed, longest=None):
    """Random rows made of stretches of columns; integer values."""
    rng = np.random.default_rng(seed)
    n = nx * ny * nz
    rows = []
    for i in range(m):
        kind = rng.integers(0, 6)
        if kind == 0:
            cols = np.zeros(0, dtype=np.int64)
        elif kind == 1:
            cols = rng.choice(n, size=min(n, int(rng.integers(1, 90))), replace=False)
        else:
            base = rng.integers(0, n, size=int(rng.integers(1, 12)))
            cols = np.concatenate([np.arange(b, min(n, b + int(rng.integers(1, 2 * nz + 3)))) for b in base])
        if i == m // 2 and longest:
            cols = rng.choice(n, size=longest, replace=False)
        rows.append(np.unique(cols))
    rows[-1] = np.unique(np.append(rows[-1], n - 1))
    rp = np.zeros(m + 1, dtype=np.int64)
    rp[1:] = np.cumsum([len(r) for r in rows])
    col = np.concatenate(rows).astype(np.int32)
    val = rng.integers(1, 9, size=len(col)) * rng.choice([-1.0, 1.0], size=len(col))
    return rp, col, val


def greedy_groups(rp, col, cap):
    """Boundaries and total list length: a row joins while the union fits."""
    sizes, cur, first = [], set(), True
    for i in range(len(rp) - 1):
        row = col[rp[i]:rp[i + 1]].tolist()
        new = cur.union(row)
        if len(new) > cap and not first:
            sizes.append(len(cur))
            new, first = set(row), False
        cur, first = new, False
    return len(sizes) + 1, sum(sizes) + len(cur)


def padded_zeros(rp, col, nz, W):
    tot = 0
    for i in range(len(rp) - 1):
        r = col[rp[i]:rp[i + 1]].astype(np.int64)
        if not len(r):
            continue
        st = np.nonzero(np.r_[True, (np.diff(r) != 1) | (r[1:] % nz == 0)])[0]
        ln = np.diff(np.r_[st, len(r)])
        pre = (r[st] % nz) & (W - 1)
        tot += int(((ln + pre + W - 1) // W * W - ln).sum())
    return tot


def laplacian(x, nx, ny, nz):
    u = x.reshape(ny, nx, nz)
    y = np.zeros_like(u)
    for ax in range(3):
        d = np.diff(u, axis=ax)
        lo, hi = [slice(None)] * 3, [slice(None)] * 3
        lo[ax], hi[ax] = slice(0, u.shape[ax] - 1), slice(1, None)
        y[tuple(lo)] += d
        y[tuple(hi)] -= d
    return y.reshape(-1)


@pytest.mark.parametrize("m,nx,ny,nz,longest", [
    (1, 3, 2, 5, None), (70, 5, 4, 1, None), (300, 7, 5, 20, None), (257, 4, 6, 31, 700),
    (200, 6, 5, 33, 990), (130, 5, 3, 64, 960), (60, 3, 3, 65, None),
    (400, 20, 12, 20, None),
    (90, 117, 112, 20, 3000), (40, 130, 101, 20, 2500)])
@pytest.mark.parametrize("device", [False, True])
def test_formats_of_ragged_structures(m, nx, ny, nz, longest, device):
    """nz = 65 has no node runs; the last two grids lie on either side of the
    columns a device-planned group can index (262,144)."""
    from paper_2604_11920_amd import Solver
    n = nx * ny * nz
    rp, col, val = ragged(m, nx, ny, nz, seed=m + nz, longest=longest)
    G = sp.csr_matrix((val, col, rp), shape=(m, n))
    arrays = (rp, col, val)
    if device:
        arrays = tuple(torch.from_numpy(a).cuda() for a in arrays)
    rng = np.random.default_rng(5)
    x, y = rng.integers(-4, 5, size=n).astype(float), rng.integers(-4, 5, size=m + 2 * n).astype(float)
    ref_y = np.concatenate([G @ x, 2.0 * laplacian(x, nx, ny, nz), 3.0 * x])
    ref_q = G.T @ y[:m] + 2.0 * laplacian(y[m:m + n], nx, ny, nz) + 3.0 * y[m + n:]
    ng, ncols = greedy_groups(rp, col, max(1024, -(-int(np.diff(rp).max()) // 1024) * 1024))
    cols = ("pairs", "runs", "csc") if nz <= 64 else ("csc",)
    for prec, W in (("fp64", 2), ("fp32", 4), ("bf16", 8)):
        for cf in cols:
            for rf in ("groups", "csr"):
                with Solver(*arrays, nx, ny, nz, 3.0, 2.0, precision=prec, row_format=rf, col_format=cf) as sol:
                    st = sol.kernel_stats()
                    if rf == "groups":
                        assert (st["groups"], st["staged_cols"]) == (ng, ncols)
                    if cf == "pairs":
                        assert st["padded_values"] == padded_zeros(rp, col, nz, W)
                    dt = torch.float64 if prec == "fp64" else torch.float32
                    yy = sol.apply_stored(torch.from_numpy(x).to("cuda", dt)).cpu().numpy()
                    t = torch.from_numpy(y).to("cuda", dt)
                    tg = None
                    if prec == "bf16":
                        tg = (t[:m] * torch.from_numpy(sol.quantised()[0]).cuda()).contiguous()
                    qq = sol.apply_t_stored(t, tg).cpu().numpy()
                    assert np.array_equal(yy, ref_y.astype(yy.dtype)), (prec, cf, rf)
                    assert np.array_equal(qq, ref_q.astype(qq.dtype)), (prec, cf, rf)
                    if prec == "fp64":
                        cp, ri, cv = sol.transpose()
                        C = G.tocsc()
                        C.sort_indices()
                        assert np.array_equal(cp, C.indptr) and np.array_equal(ri, C.indices)
                        assert np.array_equal(cv, C.data)


def test_device_csr_refusals():
    """A malformed device CSR is refused with its own status, rows whose bounds
    lie outside the arrays included (they are not read)."""
    from paper_2604_11920_amd import Solver
    from paper_2604_11920_amd.lsqr import LSQR_E_BAD_CSR, LSQR_E_NONFINITE, LsqrError
    rp, col, val = ragged(50, 4, 4, 6, seed=1)
    k = int(np.argmax(np.diff(rp)))

    def bad(change):
        a = [rp.copy(), col.copy(), val.copy()]
        change(*a)
        with pytest.raises(LsqrError) as e:
            Solver(*[torch.from_numpy(v).cuda() for v in a], 4, 4, 6, 1.0, 1.0)
        return e.value.status

    def set_at(arr, i, v):
        arr[i] = v

    assert bad(lambda r, c, v: set_at(r, 20, r[19] - 1 if r[19] else -1)) == LSQR_E_BAD_CSR
    assert bad(lambda r, c, v: set_at(r, 20, len(col) + 10 ** 6)) == LSQR_E_BAD_CSR
    assert bad(lambda r, c, v: set_at(r, 20, -5)) == LSQR_E_BAD_CSR
    assert bad(lambda r, c, v: set_at(r, 0, 1)) == LSQR_E_BAD_CSR
    assert bad(lambda r, c, v: set_at(c, rp[k], -1)) == LSQR_E_BAD_CSR
    assert bad(lambda r, c, v: set_at(c, rp[k + 1] - 1, 96)) == LSQR_E_BAD_CSR
    assert bad(lambda r, c, v: set_at(c, rp[k] + 1, c[rp[k]])) == LSQR_E_BAD_CSR
    assert bad(lambda r, c, v: set_at(v, rp[k], np.inf)) == LSQR_E_NONFINITE
