"""The fused step of small systems (update and forward product in one launch)
against the separate launches (row_format="csr" keeps them): early iterates
and histories at the repository's bar for them (1e-10, 8 iterations), stops by
tolerance at the same iteration, breakdowns, zero data; at the edges of its
range: one unknown, one row, the most unknowns it takes and one lateral node
more, rows of 1 to 300 entries, fewer and more rows than workgroups hold.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def pair(s, **kw):
    from paper_2604_11920_amd import Solver
    return Solver.from_system(s, **kw), Solver.from_system(s, row_format="csr", **kw)


@pytest.mark.parametrize("m,nx,ny,nz,row_len", [
    (1, 1, 1, 1, (1, 1)), (1, 4, 3, 5, (3, 9)), (40, 1, 1, 7, (0, 7)), (700, 5, 4, 3, (0, 60)),
    (9000, 12, 8, 6, (1, 5)), (3000, 32, 16, 12, (20, 200)), (900, 13, 7, 67, (40, 300)),
    (500, 35, 16, 11, (100, 300))])
@pytest.mark.parametrize("method,precond", [("lsqr", "none"), ("lsqr", "jacobi"), ("lsmr", "jacobi")])
def test_fused_iterations_match_the_separate_launches(m, nx, ny, nz, row_len, method, precond):
    """32 x 16 x 12 = 6,144 unknowns are the most that are fused; 35 x 16 x 11
    and 13 x 7 x 67 keep the separate launches or have no node runs."""
    s = synth.random_system(m, nx, ny, nz, row_len=row_len, seed=m + nz)
    a, b = pair(s, method=method, precond=precond)
    with a, b:
        for K in (0, 1, 2, 3, 8):
            xa, ha, ia = a.solve(s.dt, K)
            xb, hb, ib = b.solve(s.dt, K)
            assert (ia["istop"], ia["iters"]) == (ib["istop"], ib["iters"])
            if ia["istop"] != 2:                       # exhausted Krylov space: rounding noise
                continue
            assert np.linalg.norm(xa - xb) <= 1e-10 * max(np.linalg.norm(xb), 1e-300)
            k = ia["iters"] + 1
            scale = np.abs(hb[0])
            assert np.all(np.abs(ha[:k] - hb[:k]) <= 1e-10 * scale)
            assert np.isnan(ha[k:]).all()
        x0 = np.random.default_rng(1).standard_normal(s.n)
        xa, _, _ = a.solve(s.dt, 4, x0=x0)
        xb, _, _ = b.solve(s.dt, 4, x0=x0)
        assert np.linalg.norm(xa - xb) <= 1e-10 * np.linalg.norm(xb)


@pytest.mark.parametrize("check_every", [2, 8, 32])
@pytest.mark.parametrize("graph", [True, False])
def test_fused_stops(check_every, graph):
    """Tolerances met at each of the first 8 iterations (inside a block of
    iterations and at its end), where eta agrees to 1e-10: the stop falls on
    the same iteration; then the limit, a repeat and zero data."""
    s = synth.make_system(synth.small_config())
    a, b = pair(s, precond="jacobi", check_every=check_every, graph=graph)
    with a, b:
        eta = b.solve(s.dt, 8)[1][:, 2]
        for k in range(1, 9):
            tol = eta[k] * (1 + 1e-6)
            first = next(i for i in range(1, 9) if eta[i] <= tol)
            xa, ha, ia = a.solve(s.dt, 500, tol=tol)
            xb, hb, ib = b.solve(s.dt, 500, tol=tol)
            assert (ia["istop"], ia["iters"]) == (ib["istop"], ib["iters"]) == (1, first)
            assert np.linalg.norm(xa - xb) <= 1e-10 * np.linalg.norm(xb)
            assert abs(ia["eta"] - eta[first]) <= 1e-9 * eta[first] and ha[first, 2] == ia["eta"]
            assert abs(ia["eta_final_fp64"] - ia["eta"]) <= 1e-9 * ia["eta"]
            assert not np.isnan(ha[:first + 1]).any() and np.isnan(ha[first + 1:]).all()
        xa, _, ia = a.solve(s.dt, 7, tol=1e-14)
        xb, _, ib = b.solve(s.dt, 7, tol=1e-14)
        assert (ia["istop"], ia["iters"]) == (ib["istop"], ib["iters"]) == (2, 7)
        assert np.linalg.norm(xa - xb) <= 1e-10 * np.linalg.norm(xb)
        again, _, _ = a.solve(s.dt, 7, tol=1e-14)
        assert np.array_equal(xa, again)
        z, _, iz = a.solve(np.zeros(s.m), 7)
        assert iz["istop"] == 0 and iz["iters"] == 0 and not z.any()


def test_fused_breakdown():
    """One unknown: the Krylov space is exhausted after one iteration."""
    s = synth.random_system(6, 1, 1, 1, row_len=(1, 1), seed=3, integer=True)
    a, b = pair(s, method="lsqr")
    with a, b:
        xa, _, ia = a.solve(s.dt, 20)
        xb, _, ib = b.solve(s.dt, 20)
    ref = np.linalg.lstsq(np.vstack([s.dense(), [[0.0]], [[s.damp]]]), np.r_[s.dt, 0.0, 0.0], rcond=None)[0]
    assert np.allclose(xa, ref, rtol=1e-12) and np.allclose(xb, ref, rtol=1e-12)


@pytest.mark.parametrize("precision", ["fp32", "bf16", "fp16"])
def test_fused_reduced_precision(precision):
    s = synth.make_system(synth.small_config(seed=4))
    a, b = pair(s, precond="jacobi", precision=precision, refine_sweeps=20)
    with a, b:
        if precision == "fp32":
            xa, xb = a.solve(s.dt, 6)[0], b.solve(s.dt, 6)[0]
            assert np.linalg.norm(xa - xb) <= 1e-4 * np.linalg.norm(xb)   # the FP32 bar of early iterates
        else:
            xa, _, ia = a.solve(s.dt, 2000, tol=1e-12)
            xb, _, ib = b.solve(s.dt, 2000, tol=1e-12)
            assert ia["istop"] == ib["istop"] == 1
            assert np.linalg.norm(xa - xb) <= 1e-9 * np.linalg.norm(xb)
