"""Layout sizes at the edges of the small-mesh kernel: fewer nodes than a
wave, one to four nodes per workgroup, a last workgroup that is not full, and
the last size of that kernel beside the first of the other; one iteration
against the oracle's sampled-node step, at the bounds of
tests/test_gpu_layout.py (positions are float32 at the boundary: 1e-6 of the
canvas)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("n", [3, 4, 63, 64, 65, 255, 257, 300, 767, 1023, 1025, 2245, 2306, 4001,
                               16383, 16384])
def test_one_iteration(torch_dev, oracle, n):
    from paper_1408_0677_amd import api, workloads as wl
    torch = torch_dev
    pts, mesh, prm = wl.layout_workload(n)
    p32 = pts.astype(np.float32)
    print(f"case layout group n={n}", flush=True)
    m = {k: torch.from_numpy(np.ascontiguousarray(v.reshape(-1))).cuda() for k, v in mesh.items()
         if k != "triangles"}
    pos = torch.from_numpy(p32).cuda()
    api.layout(pos, m, iterations=1, **prm)
    nodes = np.unique(np.concatenate([np.arange(min(n, 200)), np.arange(max(0, n - 200), n)]))
    ref = oracle.layout_step_nodes(p32.astype(np.float64), mesh, prm["C"], prm["D"], prm["eta"],
                                   prm["t0"], nodes)
    err = np.abs(pos.cpu().numpy()[nodes] - ref).max() / 600.0
    assert err <= 1e-6, err
