"""Float64 Gaussian fits where what lies beyond the usual reach decides:
weight floors small enough that far points determine a node, and attributes
whose sizes differ by more than the weights."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


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


# the cluster right of the grid and left of it, above and below (each half of a
# tile starts its factors at one end), tiles of 4 rows and of 16
@pytest.mark.parametrize("side", ["right", "left", "above", "below"])
@pytest.mark.parametrize("width,height", [(23, 23), (23, 4200)])
@pytest.mark.parametrize("basis,d", [("constant", 3), ("linear", 5)])
def test_tiny_weight_floor(torch_dev, oracle, basis, d, width, height, side):
    """Nodes 17 h to 29 h from a cluster of points, on tiles of 8 h, with a
    weight floor of 1e-300: determined up to 26.3 h.  The factors of a half tile
    whose first node is 28 h away underflow there and not at its last node."""
    print(f"case tiny floor {basis} {side} {width} x {height}", flush=True)
    rng = np.random.default_rng(3)
    h = 0.01
    dx = 8.0 / 15.0 * h
    if side in ("above", "below"):
        width, height = height, width
    pts = (0.02 * h * rng.random((500, 2))).astype(np.float32)
    vals = rng.random((500, d)).astype(np.float32)
    grid = {"x0": -3 * dx, "y0": -3 * dx, "dx": dx, "dy": dx, "width": width, "height": height}
    if side == "right":
        grid["x0"] = -29.0 * h
    elif side == "left":
        grid["x0"] = 17.0 * h
    elif side == "above":
        grid["y0"] = -29.0 * h
    else:
        grid["y0"] = 17.0 * h
    kw = dict(basis=basis, h=h, weight_floor=1e-300)
    F, deg = gpu_fit(torch_dev, pts, vals, grid, **kw)
    of, od, dm = oracle.fit_grid(pts, vals, grid, **kw)
    of, od = of.reshape(d, -1), od.ravel()
    assert (od != 255).any() and (od == 255).any()
    # (the ladder's degrees above 0 are rounding noise: the cluster is a point
    # from there)
    assert np.array_equal(deg == 255, od == 255)
    both = (deg == 0) & (od == 0)
    if basis == "constant":
        assert both.sum() == (od == 0).sum()
    if both.any():
        assert np.abs(F - of)[:, both].max() <= 1e-5


# values that every tile looks through itself, and by one launch for all tiles
@pytest.mark.parametrize("n", [700, 1500, 12000])
@pytest.mark.parametrize("basis,d", [("constant", 1), ("constant", 7), ("linear", 2),
                                     ("linear", 5), ("quadratic", 3), ("quadratic", 14)])
@pytest.mark.parametrize("size", [1e30, 1e12])
def test_markers_among_the_values(torch_dev, oracle, basis, d, n, size):
    """A few points hold 1e30 (or 1e12) in one attribute, as a marker of a
    missing value would: at 8 h (6 h) from a node they still add e^-64 1e30 =
    160 (e^-36 1e12 = 2e-4) to fields near 1.  Bound: 1e-5 of the field at the
    node (the oracle's float64 sums; the results are float32), on nodes whose
    smallest pivot is at least 1e-3."""
    print(f"case markers {basis} d={d} n={n} size={size}", flush=True)
    rng = np.random.default_rng(n + d)
    h = 0.02
    pts = rng.random((n, 2)).astype(np.float32)
    vals = (1.0 + rng.random((n, d))).astype(np.float32)
    mark = rng.integers(0, n, 3)
    vals[mark, d // 2] = size
    if d > 2:   # an attribute in other units, one that is 0, one at float32's ends
        vals[:, 0] *= 1e-20
        vals[:, -1] = 0.0
    grid = {"x0": 0.2, "y0": 0.2, "dx": 0.012, "dy": 0.012, "width": 50, "height": 40}
    kw = dict(basis=basis, h=h)
    F, deg = gpu_fit(torch_dev, pts, vals, grid, **kw)
    of, od, dm = oracle.fit_grid(pts, vals, grid, **kw)
    of, od, dm = of.reshape(d, -1), od.ravel(), dm.ravel()
    ok = (deg == od) & (od != 255) & (dm >= 1e-3)
    assert ok.sum() > 100 and (deg != od).mean() <= 0.01
    err = np.abs(F - of)[:, ok]
    assert (err <= 1e-5 * np.abs(of[:, ok])).all(), (err / np.abs(of[:, ok])).max()


@pytest.mark.parametrize("n,d", [(60, 255), (200, 255), (3000, 83)])
def test_exponential_attributes(torch_dev, oracle, n, d):
    """Attributes that grow by up to e^80 over the square, the constant basis
    (all weights and products positive, so that the error is relative)."""
    print(f"case exponential n={n} d={d}", flush=True)
    rng = np.random.default_rng(d)
    pts = rng.random((n, 2)).astype(np.float32)
    rate = np.linspace(0.0, 80.0, d)
    vals = np.exp(rate[None, :] * (pts[:, :1] - 0.5)).astype(np.float32)
    grid = {"x0": 0.1, "y0": 0.1, "dx": 0.02, "dy": 0.02, "width": 40, "height": 37}
    kw = dict(basis="constant", h=0.05)
    F, deg = gpu_fit(torch_dev, pts, vals, grid, **kw)
    of, od, _ = oracle.fit_grid(pts, vals, grid, **kw)
    of, od = of.reshape(d, -1), od.ravel()
    assert np.array_equal(deg, od)
    ok = od == 0
    assert (np.abs(F - of)[:, ok] <= 1e-6 * np.abs(of[:, ok])).all()
