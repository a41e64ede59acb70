"""Float64 fits store planes of any width at any float address: four columns a
store where every row of the fields (and of the slopes) is 16-byte aligned, one
elsewhere, the same values, nothing around them."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("width", [1, 4, 17, 20, 64])
@pytest.mark.parametrize("basis,d", [("linear", 13), ("linear", 35), ("quadratic", 14)])
@pytest.mark.parametrize("slopes", [False, True])
def test_stores(torch_dev, slopes, basis, d, width):
    from paper_1408_0677_amd import _lib, api
    torch = torch_dev
    print(f"case f64 stores {basis} d={d} width={width} slopes={slopes}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(width)
    P = torch.rand(400, 2, generator=g, device="cuda")
    V = torch.rand(400, d, generator=g, device="cuda")
    height, lib, ctx = 21, _lib.load(), api.Context()
    gs = api.grid_struct({"x0": 0.1, "y0": 0.1, "dx": 0.006, "dy": 0.006, "width": width,
                          "height": height})
    wt = _lib.MlsWeight(0, 0.15, 1.0)
    count = d * height * width
    got = []
    for off_f, off_g in ((0, 0), (1, 0), (0, 1), (3, 2), (4, 8)):
        F = torch.full((count + 16,), 7.0, device="cuda")
        G = torch.full((2 * count + 16,), 7.0, device="cuda")
        args = [ctx.handle, P.data_ptr(), V.data_ptr(), 400, d, api.BASIS[basis],
                ctypes.byref(wt), ctypes.byref(gs), 0, None, F.data_ptr() + 4 * off_f]
        args = [ctypes.c_void_p(a) if i in (1, 2, 10) else a for i, a in enumerate(args)]
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        if slopes:
            st = lib.mls_fit_grad(*args, ctypes.c_void_p(G.data_ptr() + 4 * off_g), None, stream)
        else:
            st = lib.mls_fit(*args, None, stream)
        assert st == 0
        bufs = ((F, off_f, count), (G, off_g, 2 * count if slopes else 0))
        for buf, off, k in bufs:
            assert bool((buf[:off] == 7.0).all()) and bool((buf[off + k:] == 7.0).all())
        got.append([buf[off:off + k].view(torch.int32).clone() for buf, off, k in bufs])
        assert bool(got[-1][0].view(torch.float32).isfinite().all())
    for f, s in got[1:]:
        assert torch.equal(f, got[0][0]) and torch.equal(s, got[0][1])
