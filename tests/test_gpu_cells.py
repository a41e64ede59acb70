"""Cell list and tile order at the edges of their one-workgroup forms: scans
of up to 16,384 values, up to 4,096 supertiles, staging blocks that reduce up
to 2,048 partial ranges themselves; Wendland fits on sampled nodes against the
oracle, at the 16-bit bounds of tests/test_gpu_fit_lp.py (max 2e-3, rms 1e-4 on
the nodes with a smallest pivot of at least 1e-2)."""
import math

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


# (n, d, width, height): one sort block; a ragged grid of few supertiles; more
# than 16,384 histogram entries (n > 131,072); more than 16,384 tiles; more
# partial ranges than the staging blocks reduce (131 x 17); 65 x 64 supertiles
@pytest.mark.parametrize("n,d,width,height", [(700, 3, 97, 61), (2049, 2, 300, 190),
                                              (131073, 2, 500, 333), (140001, 17, 300, 200),
                                              (60000, 1, 2100, 2050), (40000, 1, 4113, 4096)])
@pytest.mark.parametrize("prec", ["bf16", "fp16"])
def test_wendland(torch_dev, oracle, prec, n, d, width, height):
    from paper_1408_0677_amd import api, workloads as wl
    torch = torch_dev
    print(f"case cells {prec} n={n} d={d} {width} x {height}", flush=True)
    rng = np.random.default_rng(n)
    pts = wl.uniform_points(rng, n).astype(np.float32)
    vals = wl.smooth_fields(rng, pts, d).astype(np.float32)
    h = math.sqrt(60.0 / (math.pi * n))
    # the grid covers the square unless that would be too coarse against h
    dx = min(1.0 / max(width, height), 0.2 * h)
    grid = {"x0": 0.1, "y0": 0.1, "dx": 0.8 * dx, "dy": 0.8 * dx, "width": width,
            "height": height}
    F, deg = api.fit(torch.from_numpy(pts).cuda(), torch.from_numpy(vals).cuda(), grid,
                     basis="linear", weight="wendland", h=h, precision=prec)
    P = width * height
    pix = np.unique(np.concatenate([rng.integers(0, P, 500), np.arange(P - 40, P)]))
    idx = torch.from_numpy(pix).cuda()
    of, od, dm = oracle.fit_grid(pts, vals, grid, basis="linear", weight="wendland", h=h,
                                 pixels=pix)
    st = compare(F.reshape(d, -1)[:, idx].cpu().numpy(), deg.reshape(-1)[idx].cpu().numpy(), of,
                 od, dm, vals, dmin_pass=1e-2)
    print({k: v for k, v in st.items() if k != "per_field_max_pass"}, flush=True)
    assert st["pass_set"] > 0.9 * st["nodes"] and st["nan_ok"], st
    assert st["max_err_pass"] <= 2e-3 and st["rms_err_pass"] <= 1e-4, st
    assert st["degree_mismatch"] <= max(2, 0.03 * st["nodes"]), st
