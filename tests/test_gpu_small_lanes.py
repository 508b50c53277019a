"""The fused step at every number of lanes a row can take and on either side of
the rule for its sizes: iterates against the separate launches (row_format="csr"
keeps them) at the bars of early iterates, and which of the two runs, read off
the counted bytes."""
import numpy as np
import pytest

import synth
from test_gpu_small_step import pair

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def fused(a, b):
    return a.kernel_stats()["fwd_bytes"] != b.kernel_stats()["fwd_bytes"]


# average rows of 4 to 300 entries; 6,144 unknowns are the most that are fused,
# 1,537 and more need entries for it
@pytest.mark.parametrize("m,nx,ny,nz,row_len,f64,f32,f16", [
    (500, 12, 10, 8, (1, 7), 1, 1, 1), (400, 12, 10, 8, (8, 16), 1, 1, 1), (400, 16, 12, 8, (15, 25), 1, 1, 1),
    (300, 12, 10, 8, (35, 60), 1, 1, 1), (300, 16, 12, 8, (60, 120), 1, 1, 1), (300, 12, 10, 8, (130, 170), 1, 1, 1),
    (250, 16, 12, 8, (220, 380), 1, 1, 1),
    (1700, 29, 53, 1, (80, 90), 0, 0, 0), (2000, 29, 53, 1, (75, 85), 1, 0, 0), (4000, 29, 53, 1, (75, 85), 1, 1, 0),
    (9700, 29, 53, 1, (75, 85), 1, 1, 1), (6000, 32, 16, 12, (60, 150), 1, 0, 0), (16000, 32, 16, 12, (180, 230), 1, 1, 1)])
def test_lanes_and_sizes(m, nx, ny, nz, row_len, f64, f32, f16):
    s = synth.random_system(m, nx, ny, nz, row_len=row_len, seed=m + nz)
    for precision, want in (("fp64", f64), ("fp32", f32), ("bf16", f16), ("fp16", f16)):
        a, b = pair(s, precision=precision, precond="jacobi", refine_sweeps=20)
        with a, b:
            assert fused(a, b) == bool(want), precision
            if precision in ("fp64", "fp32"):
                bar = 1e-10 if precision == "fp64" else 1e-4
                for K in (1, 5):
                    xa, xb = a.solve(s.dt, K)[0], b.solve(s.dt, K)[0]
                    assert np.linalg.norm(xa - xb) <= bar * np.linalg.norm(xb), (precision, K)
            else:
                xa, _, ia = a.solve(s.dt, 2000, tol=1e-11)
                xb, _, ib = b.solve(s.dt, 2000, tol=1e-11)
                assert ia["istop"] == ib["istop"] == 1
                # either is within eta cond(Abar)^2 of the solution: singular values from
                # damp = 0.1 to about 45
                assert np.linalg.norm(xa - xb) <= 1e-5 * np.linalg.norm(xb), precision
