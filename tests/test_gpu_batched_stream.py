"""A refined batch on a context's own, non-blocking stream, launched without a
graph: what the sweeps report (iterations, stop reasons) is read back after the
stream has finished, and equals a run on the default stream."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("iters,check_every", [(41, 32), (7, 32), (300, 8)])
def test_own_stream(iters, check_every):
    from paper_2604_11920_amd import Solver, solve_batched_refined
    s = synth.make_system(synth.small_config(nx=12, ny=10, nz=6, n_stations=24, n_periods=6, region=1.0, seed=3))
    dt = synth.checker_rhs_batch(s, n_checker=3, n_boot=2)
    out = []
    for stream in (None, torch.cuda.Stream()):
        with Solver.from_system(s, precond="jacobi", graph=False, check_every=check_every, stream=stream) as sol:
            out.append(solve_batched_refined([sol], [dt], iters, 1e-9, inner_tol=1e-3, sweeps=6))
    (a, ia), (b, ib) = out
    assert np.array_equal(a[0], b[0]) and str(ia) == str(ib)
