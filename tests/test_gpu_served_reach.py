"""Served batches of bfloat16 fits whose tiles are summed a second time without
the adaptive reach (a call of its own in the batch kernel) among tiles that are
not: each request computes the bits that it computes alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("basis,d", [("linear", 1), ("linear", 12), ("quadratic", 2),
                                     ("quadratic", 5)])
def test_tiles_summed_again_in_a_batch(basis, d):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1408_0677_amd import api
    print(f"case summed again in a batch {basis} d={d}", flush=True)
    h = 1.0 / 64
    dx = h / 8
    rng = np.random.default_rng(d)
    # nodes on a point and on their tile's anchor, whose neighbours are 6 h away
    # and more, see past the reach; nodes among many points do not
    c = 8 + 48 * np.arange(3)
    lone = np.stack(np.meshgrid(c, c), -1).reshape(-1, 2) * dx
    many = rng.random((2000, 2)) * 112 * dx
    grid = {"x0": 0.0, "y0": 0.0, "dx": dx, "dy": dx, "width": 112, "height": 112}
    kw = dict(basis=basis, h=h, precision="bf16")
    srv = api.Server(slots=1, hbm_budget=1 << 30, slot_scratch=64 << 20)
    subs = []
    for pts in (lone, many, np.concatenate([lone[:4], many[many[:, 0] > 56 * dx]])):
        P = torch.from_numpy(pts.astype(np.float32)).cuda()
        V = torch.from_numpy(rng.random((len(pts), d)).astype(np.float32)).cuda()
        out = torch.empty((d, 112, 112), device="cuda")
        deg = torch.empty((112, 112), dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        subs.append((srv.submit(srv.put_points(P, V), grid, out, deg, **kw), P, V, out, deg))
    for t, *_ in subs:
        assert srv.wait(t)["status"] == 0
    srv.close()
    for _, P, V, out, deg in subs:
        F, D = api.fit(P, V, grid, **kw)
        torch.cuda.synchronize()
        assert torch.equal(F.view(torch.int32), out.view(torch.int32))
        assert torch.equal(D, deg)
