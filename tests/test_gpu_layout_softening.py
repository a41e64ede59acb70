"""Layout iterations with a softening at the bottom of float64's range, where
the repulsion of a node from itself, C / (0 + eta) times 0, must stay 0; against
the oracle's sampled-node step at the bounds of tests/test_gpu_layout.py (1e-6
of the canvas), in both kernels."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("n", [300, 16400])
@pytest.mark.parametrize("scale,eta", [(1.0, 1e-290), (1.0, 1e-310), (1.0, 5e-324),
                                       (1e20, 1e-295), (1e40, 1e-308)])
def test_tiny_softening(torch_dev, oracle, n, scale, eta):
    from paper_1408_0677_amd import api, workloads as wl
    torch = torch_dev
    print(f"case layout softening n={n} C x {scale} eta={eta}", flush=True)
    pts, mesh, prm = wl.layout_workload(n)
    p32 = pts.astype(np.float32)
    prm = dict(prm, C=prm["C"] * scale, eta=eta)
    m = {k: torch.from_numpy(np.ascontiguousarray(v.reshape(-1))).cuda() for k, v in mesh.items()
         if k != "triangles"}
    pos = torch.from_numpy(p32).cuda()
    api.layout(pos, m, iterations=1, **prm)
    nodes = np.arange(0, n, max(1, n // 200))
    ref = oracle.layout_step_nodes(p32.astype(np.float64), mesh, prm["C"], prm["D"], prm["eta"],
                                   prm["t0"], nodes)
    got = pos.cpu().numpy()
    assert np.isfinite(got).all() and np.isfinite(ref).all()
    err = np.abs(got[nodes] - ref).max() / 600.0
    assert err <= 1e-6, err
