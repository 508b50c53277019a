"""Polylines of many points are checked on the device, of few on the host: the
same inputs are refused with the same message on either side of the line, the
first fault in the order of the points deciding; and the split of many paths
equals the splits of its parts."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def paths(count, npts=50, h=0.25, nx=40, ny=30):
    rng = np.random.default_rng(count)
    a = rng.uniform(0.0, 0.9, (count, 2)) * [(nx - 1) * h, (ny - 1) * h]
    d = rng.uniform(-0.2, 0.2, (count, 2)) * h
    t = np.arange(npts)[None, :, None]
    pts = np.clip(a[:, None, :] + d[:, None, :] * t, 0.0, [(nx - 1) * h, (ny - 1) * h]).reshape(-1, 2)
    return dict(pt_ptr=np.arange(count + 1, dtype=np.int64) * npts, px=pts[:, 0].copy(), py=pts[:, 1].copy(),
                plen=np.full(count * npts, 3.0), h=h, nx=nx, ny=ny, km_per_deg=111.0)


FAULTS = [([("px", 1007, np.nan)], "non-finite point"),
          ([("plen", 1010, -1.0), ("py", 2222, np.inf)], "non-finite point"),
          ([("plen", 1010, -1.0), ("px", 2020, 1e3)], "piece lengths"),
          ([("plen", 3010, np.nan), ("px", 2020, 1e3)], "spans a whole cell"),
          ([("plen", 2019, np.nan), ("px", 2020, 1e3)], "piece lengths"),
          ([("px", 99, 1e3)], "spans a whole cell")]


@pytest.mark.parametrize("count", [80, 1400])
@pytest.mark.parametrize("faults,message", FAULTS)
def test_refusals(count, faults, message):
    from paper_2604_11920_amd import LsqrError
    from paper_2604_11920_amd.lsqr import split_polylines
    p = paths(count)
    for k, i, v in faults:
        p[k][i] = v
    with pytest.raises(LsqrError, match=message):
        split_polylines(p)


def test_length_of_a_path_end_is_not_read():
    from paper_2604_11920_amd.lsqr import split_polylines
    p = paths(1400)
    want = split_polylines(p)
    p["plen"][49::50] = np.nan
    got = split_polylines(p)
    assert np.array_equal(got[0], want[0]) and torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])


def test_parts(monkeypatch):
    from paper_2604_11920_amd import lsqr
    p = paths(1400)
    ptr, k, length = lsqr.split_polylines(p)
    half = dict(p, pt_ptr=p["pt_ptr"][:701])
    hp, hk, hl = lsqr.split_polylines(half)
    assert np.array_equal(hp, ptr[:701]) and torch.equal(hk, k[:hp[-1]]) and torch.equal(hl, length[:hp[-1]])
    monkeypatch.setattr(lsqr, "_SPLIT_ONE_CALL", 0)
    p2, k2, l2 = lsqr.split_polylines(p)
    assert np.array_equal(p2, ptr) and torch.equal(k2, k) and torch.equal(l2, length)
