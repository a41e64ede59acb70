"""A missing value (NaN) among the attributes of a 16-bit fit: with the compact
support it stays with the tiles that list its point, with the Gaussian, whose
sums meet every point, it reaches every node of its field.

Beyond the NaN's tiles the fit is compared with that of the same points with
another of the attribute's values in its place, which leaves the attribute's
range and so every other bit as it was, and with the oracle at the 16-bit
bounds of tests/test_gpu_fit_lp.py."""
import numpy as np
import pytest

from tests.parity import compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# (n, d): ranges reduced by the staging blocks, and by their own kernel
@pytest.mark.parametrize("n,d", [(3000, 3), (45000, 50)])
@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("weight", ["wendland", "gaussian"])
def test_missing_value(torch_dev, oracle, weight, prec, n, d):
    from paper_1408_0677_amd import api, workloads as wl
    torch = torch_dev
    print(f"case missing value {weight} {prec} n={n} d={d}", flush=True)
    rng = np.random.default_rng(n)
    pts = wl.uniform_points(rng, n).astype(np.float32)
    vals = wl.smooth_fields(rng, pts, d).astype(np.float32)
    h = float(np.sqrt(60.0 / (np.pi * n)))
    W, H = 160, 120
    dx = 0.1 * h
    grid = {"x0": 0.5 - 80 * dx, "y0": 0.5 - 60 * dx, "dx": dx, "dy": dx, "width": W, "height": H}
    # the point nearest to the grid's first node, and a value of another point
    # that is neither end of the range
    p = int(np.argmin((pts[:, 0] - grid["x0"]) ** 2 + (pts[:, 1] - grid["y0"]) ** 2))
    vals[p, 1] = np.sort(vals[:, 1])[n // 2]
    bad = vals.copy()
    bad[p, 1] = np.nan
    P = torch.from_numpy(pts).cuda()
    kw = dict(basis="linear", weight=weight, h=h, precision=prec)
    F0, d0 = api.fit(P, torch.from_numpy(vals).cuda(), grid, **kw)
    F1, d1 = api.fit(P, torch.from_numpy(bad).cuda(), grid, **kw)
    F0, F1 = F0.cpu().numpy(), F1.cpu().numpy()
    assert np.array_equal(d0.cpu().numpy(), d1.cpu().numpy())
    others = [k for k in range(d) if k != 1]
    assert np.array_equal(F0[others].view(np.uint32), F1[others].view(np.uint32))
    if weight == "gaussian":
        assert np.isnan(F1[1]).all()
        return
    # tiles of 16 x 16 nodes whose every node is farther than h from the point
    # in x or y do not list it
    x = grid["x0"] + dx * np.arange(W)
    y = grid["y0"] + dx * np.arange(H)
    far_c = np.add.reduceat(np.abs(x - pts[p, 0]) <= h, np.arange(0, W, 16)) == 0
    far_r = np.add.reduceat(np.abs(y - pts[p, 1]) <= h, np.arange(0, H, 16)) == 0
    far = np.repeat(far_r, 16)[:H, None] | np.repeat(far_c, 16)[None, :W]
    near = np.hypot(x[None, :] - pts[p, 0], y[:, None] - pts[p, 1]) < h
    assert near.any() and far.mean() > 0.5 and not (near & far).any()
    assert np.isnan(F1[1][near]).all()
    assert np.array_equal(F1[1][far].view(np.uint32), F0[1][far].view(np.uint32))
    pix = np.flatnonzero(far.ravel())[::37]
    of, od, dm = oracle.fit_grid(pts, vals, grid, basis="linear", weight="wendland", h=h,
                                 pixels=pix)
    st = compare(F1.reshape(d, -1)[:, pix], d1.cpu().numpy().ravel()[pix], of, od, dm, vals,
                 dmin_pass=1e-2)
    assert st["nan_ok"] and st["max_err_pass"] <= 2e-3 and st["rms_err_pass"] <= 1e-4, st
