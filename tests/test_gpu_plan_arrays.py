"""The arrays planned on the device against those of the host builders
(csrc/runs_host.h, themselves checked exhaustively on the CPU), element by
element: node runs in both orders, value offsets of every layout, node order, row
groups with their column lists and slots, on ragged structures."""
import numpy as np
import pytest

from device_blocks import Blocks
from test_gpu_plan import ragged
from test_host_runs import driver, run_builders  # noqa: F401  (driver: fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m,nx,ny,nz,longest", [
    (1, 3, 2, 5, None), (70, 5, 4, 1, None), (300, 7, 5, 20, None), (257, 4, 6, 31, 700), (200, 6, 5, 33, 990),
    (130, 5, 3, 64, 960), (400, 20, 12, 20, None), (2500, 16, 9, 12, 1100), (90, 117, 112, 20, 3000)])
@pytest.mark.parametrize("precision,W", [("fp64", 2), ("fp32", 4), ("bf16", 8)])
def test_device_arrays(monkeypatch, driver, tmp_path, m, nx, ny, nz, longest, precision, W):  # noqa: F811
    from paper_2604_11920_amd import Solver, lsqr
    n, nn = nx * ny * nz, nx * ny
    rp, col, val = ragged(m, nx, ny, nz, seed=m + nz, longest=longest)
    cap = max(1024, -(-int(np.diff(rp).max()) // 1024) * 1024)
    o = run_builders(driver, tmp_path, rp, col, n, nz, cap)
    assert o["nodes_ok"] and o["groups_ok"] and o[f"pairs_ok{W}"]
    blocks = Blocks()
    monkeypatch.setattr(lsqr, "torch_allocator", blocks)
    with Solver(rp, col, val, nx, ny, nz, 3.0, 2.0, precision=precision, row_format="groups"):
        for k in ("nrp", "row", "desc", "order", "gp", "gcp", "gcol"):
            assert blocks.holds(o[k]), k
        assert blocks.holds(np.r_[o["slot"], np.zeros(8, np.uint16)])
        if nz <= 32:
            assert blocks.holds(o["rrp"]) and blocks.holds(o["rrid"])
        # 16 parts of a node's runs here, 4 there: every fourth offset
        parts = blocks.of_size(8 * (16 * nn + 1), np.int64)
        for k in ("nvq", "nvqp2", f"nvqp{W}"):
            assert any(np.array_equal(p[::4], o[k]) and np.all(np.diff(p) >= 0) for p in parts), k
        assert blocks.intact()
