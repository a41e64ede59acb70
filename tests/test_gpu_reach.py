"""Fits that list the points within reach of each node tile (Gaussian): the
listing's rounds and segments, points on no tile's list, and inputs that are
not finite, which reach every node as when all points are summed.

The bounds are those of the precision's other tests: tests/test_gpu_fit_lp.py
for 16 bit (max 2e-3, rms 1e-4 on the well-conditioned nodes), 1e-5 for
float64."""
import sys

import numpy as np
import pytest

from tests.parity import compare

pytestmark = pytest.mark.gpu

BOUND = {"bf16": (2e-3, 1e-4, 1e-2), "fp16": (2e-3, 1e-4, 1e-2)}


def note(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def gpu_fit(torch, pts, vals, grid, **kw):
    from paper_1408_0677_amd import api
    P = torch.from_numpy(np.ascontiguousarray(pts, np.float32)).cuda()
    V = torch.from_numpy(np.ascontiguousarray(vals, np.float32)).cuda()
    f, d = api.fit(P, V, grid, **kw)
    torch.cuda.synchronize()
    return f.cpu().numpy().reshape(V.shape[1], -1), d.cpu().numpy().ravel()


def check(prec, F, deg, of, od, dm, vals):
    max_err, rms_err, dmin = BOUND[prec]
    st = compare(F, deg, of, od, dm, vals, dmin_pass=dmin)
    note(str({k: v for k, v in st.items() if k != "per_field_max_pass"}))
    assert st["nan_ok"] and st["max_err_pass"] <= max_err and st["rms_err_pass"] <= rms_err, st
    assert st["degree_mismatch"] <= max(2, 0.03 * st["nodes"]), st
    return st


# (n, h): either side of a test round and of the list's capacity with every
# point in reach, rounds with few in reach, more points than one segment's
# offsets span
SIZES = [(64, 0.3), (1535, 0.2), (1536, 0.2), (1537, 0.2), (4096, 0.15), (4097, 0.15),
         (6001, 0.5), (9000, 0.004), (70001, 0.01)]


@pytest.mark.parametrize("n,h", SIZES)
@pytest.mark.parametrize("prec,d", [("fp16", 5), ("bf16", 5), ("bf16", 33)])
def test_listing_rounds_and_segments(torch_dev, oracle, prec, d, n, h):
    from paper_1408_0677_amd import workloads as wl
    note(f"case listing {prec} n={n} d={d} h={h}")
    rng = np.random.default_rng(n + d)
    pts = wl.uniform_points(rng, n).astype(np.float32)
    vals = wl.smooth_fields(rng, pts, d).astype(np.float32)
    # a window of the square, fine enough against h for every form; h = 0.004
    # leaves most tiles a handful of points
    dx = min(h / 20.0, 0.01)
    grid = {"x0": 0.31, "y0": 0.42, "dx": dx, "dy": dx, "width": 37, "height": 19}
    F, deg = gpu_fit(torch_dev, pts, vals, grid, basis="linear", h=h, precision=prec)
    of, od, dm = oracle.fit_grid(pts, vals, grid, basis="linear", h=h)
    check(prec, F, deg, of.reshape(d, -1), od.ravel(), dm.ravel(), vals)


@pytest.mark.parametrize("prec,d", [("fp16", 3), ("bf16", 3), ("bf16", 40)])
def test_not_finite(torch_dev, prec, d):
    """What a point beyond every tile's reach does when all points are summed
    (0 x NaN): a NaN attribute makes that field NaN everywhere and leaves the
    others; a point at infinity makes the first moments NaN, which leaves
    every node the constant basis and a NaN value."""
    from paper_1408_0677_amd import workloads as wl
    note(f"case not finite {prec} d={d}")
    rng = np.random.default_rng(3)
    pts = wl.uniform_points(rng, 800).astype(np.float32)
    vals = wl.smooth_fields(rng, pts, d).astype(np.float32)
    grid = {"x0": 0.2, "y0": 0.2, "dx": 0.004, "dy": 0.004, "width": 40, "height": 24}
    kw = dict(basis="linear", h=0.08, precision=prec)
    far = np.vstack([pts, [[50.0, 50.0]]]).astype(np.float32)
    F0, d0 = gpu_fit(torch_dev, far, np.vstack([vals, vals[:1]]), grid, **kw)
    bad = np.vstack([vals, vals[:1]])
    bad[-1, 1] = np.nan
    F1, d1 = gpu_fit(torch_dev, far, bad, grid, **kw)
    others = [k for k in range(d) if k != 1]
    assert np.isnan(F1[1]).all() and np.isfinite(F1[others]).all()
    assert np.array_equal(F1[others], F0[others]) and np.array_equal(d0, d1)
    inf = far.copy()
    inf[-1] = [np.inf, 0.0]
    F2, d2 = gpu_fit(torch_dev, inf, np.vstack([vals, vals[:1]]), grid, **kw)
    assert (d2 == 0).all() and np.isnan(F2).all()
