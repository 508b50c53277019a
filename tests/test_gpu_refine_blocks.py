"""The FP64 residual blocks of the refined batch, at widths with and without
padding: the eta and |rbar| reported for the returned solution equal those of
the FP64 operator applied to it (both sides round at 1e-16 of |A| |rbar|, some
hundred entries a row: 1e-12 of |Abar^T bbar| and |bbar| is two digits above)."""
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


@pytest.mark.parametrize("nrhs", [1, 2, 3, 5, 17, 32])
def test_reported_residuals(nrhs):
    from paper_2604_11920_amd import Solver, solve_batched_refined
    systems = [synth.make_system(synth.small_config(nx=9, ny=7, nz=5, n_stations=12, n_periods=6, region=0.8, seed=1)),
               synth.make_system(synth.small_config(nx=6, ny=8, nz=3, n_stations=9, n_periods=5, region=0.7, seed=2))]
    rng = np.random.default_rng(nrhs)
    dts = [rng.standard_normal((s.m, nrhs)) for s in systems]
    sols = [Solver.from_system(s, precond="jacobi") for s in systems]
    try:
        dms, infos = solve_batched_refined(sols, dts, 500, 1e-11, inner_tol=1e-3, sweeps=2)
    finally:
        for so in sols:
            so.close()
    for s, dt, dm, info in zip(systems, dts, dms, infos):
        op = oracle.Operator.from_system(s)
        x = dm.cpu().numpy() if torch.is_tensor(dm) else dm
        for r in range(nrhs):
            b = np.concatenate([dt[:, r], np.zeros(2 * s.n)])
            res = b - op.apply(x[:, r])
            ar = np.linalg.norm(op.apply_t(b))
            assert abs(info[r]["eta"] - np.linalg.norm(op.apply_t(res)) / ar) <= 1e-12
            assert abs(info[r]["phibar"] - np.linalg.norm(res)) <= 1e-12 * np.linalg.norm(b)
