"""Performance cases: the calls that a user of this framework makes, over
their range of sizes, precisions and options.

Each listed case is one pass through the public entry points of
``paper_1408_0677_amd.api`` on inputs resident on the GPU.  Inputs are drawn
on the GPU from the seed: scattered points in the unit square and smooth
attributes (sums of plane waves plus 1% noise), the shapes of the
generators in ``paper_1408_0677_amd.workloads``.  ``exact`` evaluates the same
definitions in float64 with plain torch.
"""
from __future__ import annotations

import math

import torch

from paper_1408_0677_amd import api, workloads

DEV = "cuda:0"


def _fit(name, n, d, width, height, basis, weight, h, precision, points, **more):
    return dict(name=name, kind="fit", n=n, d=d, width=width, height=height, basis=basis,
                weight=weight, h=h, precision=precision, points=points, **more)


def listed():
    return [
        # the smallest call: a CPU-scale point set on a thumbnail grid
        _fit("fit_f64_small", 200, 4, 128, 128, "linear", "gaussian", 0.05, "f64", "uniform"),
        # one interactive redraw of the headline workload: 13 attributes of
        # 5,000 projected points at screen resolution, plain precision
        _fit("fit_f64_screen", 5000, 13, 1024, 1024, "linear", "gaussian", 0.03, "f64",
             "mixture"),
        # the paper's own timing shape: inverse-distance weight, two
        # attributes, 600 x 600 canvas
        _fit("fit_invpow_600", 2245, 2, 600, 600, "linear", "invpow", 0.05, "f64", "uniform",
             alpha=1.0),
        # slopes for the adaptive line mapping: quadratic basis, a window of
        # odd size
        _fit("grad_f64_quadratic", 3001, 5, 517, 389, "quadratic", "gaussian", 0.065, "f64",
             "uniform", grads=True),
        # many attributes at high resolution in bfloat16 (two-pass form)
        _fit("fit_bf16_64attr", 50000, 64, 2048, 2048, "quadratic", "gaussian", 0.015, "bf16",
             "uniform"),
        # one request of the served mix as a direct call, ragged sizes
        _fit("fit_fp16_request", 7351, 19, 701, 643, "quadratic", "gaussian", 0.0416, "fp16",
             "uniform"),
        # a million points with compact support, many small clusters
        _fit("fit_wendland_1m", 1000000, 16, 4096, 4096, "quadratic", "wendland", 0.01, "bf16",
             "clusters"),
        # a mid-size compact-support fit in float16
        _fit("fit_wendland_20k", 20011, 5, 777, 513, "linear", "wendland", 0.05, "fp16",
             "clusters"),
        # contour lines of every field of one screen (segments and ids)
        dict(name="contour_screen", kind="contour", d=13, width=1024, height=1024, n_iso=10),
        # colour bands and adaptive lines of the same fields
        dict(name="maps_screen", kind="maps", d=13, width=1024, height=1024, n_iso=10,
             n_levels=3),
        # one animation frame's iterations of the planar layout at the timing
        # table's largest mesh
        dict(name="layout_2245", kind="layout", n=2245, iterations=20),
        # a burst of requests at the server
        dict(name="serve_burst", kind="serve", count=8, n=6000, d=12, side=512,
             precision="fp16"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["f64", "f64", "invpow", "grad", "lp", "lp", "wendland", "wendland",
                       "contour", "maps", "layout", "serve"])
    width, height = int(_log(rng, 128, 1024)), int(_log(rng, 128, 1024))
    if kind in ("f64", "grad"):
        n, d = int(_log(rng, 200, 5000)), rng.randint(1, 13)
        basis = rng.choice(["constant", "linear", "linear", "quadratic"])
        # mean number of points within h of a node
        near = rng.uniform(10, 40) if basis != "quadratic" else rng.uniform(20, 40)
        c = _fit("", n, d, width, height, basis, "gaussian", math.sqrt(near / (math.pi * n)),
                 "f64", rng.choice(["uniform", "mixture"]))
        if kind == "grad":
            c.update(grads=True, points="uniform")
    elif kind == "invpow":
        basis = rng.choice(["constant", "linear", "rigid"])
        c = _fit("", int(_log(rng, 306, 2245)), 2, width, height, basis, "invpow", 0.05, "f64",
                 "uniform", alpha=rng.choice([1.0, 1.0, 1.5, 2.0]))
    elif kind == "lp":
        n, d = int(_log(rng, 500, 20000)), rng.randint(4, 40)
        basis = rng.choice(["linear", "quadratic"])
        near = 20.0 if basis == "linear" else 40.0
        c = _fit("", n, d, max(width, 256), max(height, 256), basis, "gaussian",
                 math.sqrt(near / (math.pi * n)), rng.choice(["bf16", "fp16"]), "uniform")
    elif kind == "wendland":
        n, d = int(_log(rng, 10000, 500000)), rng.randint(2, 16)
        h = math.sqrt(300.0 / (math.pi * n))
        # fine enough against h for the 16-bit paths (16 nodes within 2.5 h)
        width = max(2 * width, int(7.0 / h))
        c = _fit("", n, d, width, 2 * height, rng.choice(["linear", "quadratic"]), "wendland",
                 h, rng.choice(["bf16", "fp16"]), "clusters")
    elif kind == "contour":
        c = dict(kind="contour", d=rng.randint(1, 13), width=2 * width, height=2 * height,
                 n_iso=rng.randint(4, 12))
    elif kind == "maps":
        c = dict(kind="maps", d=rng.randint(1, 16), width=2 * width, height=2 * height,
                 n_iso=rng.randint(4, 16), n_levels=rng.randint(2, 4))
    elif kind == "layout":
        c = dict(kind="layout", n=int(_log(rng, 306, 4000)), iterations=rng.randint(8, 20))
    else:
        c = dict(kind="serve", count=rng.randint(4, 12), n=int(_log(rng, 1000, 15000)),
                 d=rng.randint(4, 24), side=int(_log(rng, 256, 800)),
                 precision=rng.choice(["fp16", "fp16", "bf16"]))
    c.pop("name", None)
    return c


# ---- inputs ----

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float64)


def _points(g, n, how):
    """(n, 2) float32 points in the unit square."""
    if how == "uniform":
        return _rand(g, n, 2).float()
    if how == "mixture":   # eight wide components and a quarter spread evenly
        k, lo, hi, s_lo, s_hi, bg = 8, 0.15, 0.85, 0.03, 0.1, 0.25
    else:                  # uniform background and 32 tight clusters
        k, lo, hi, s_lo, s_hi, bg = 32, 0.05, 0.95, 0.002, 0.02, 0.2
    centre = lo + (hi - lo) * _rand(g, k, 2)
    sigma = s_lo + (s_hi - s_lo) * _rand(g, k)
    comp = torch.randint(k, (n,), generator=g, device=DEV)
    pts = centre[comp] + sigma[comp, None] * _randn(g, n, 2)
    for _ in range(8):     # outside the square: again from the same component
        bad = ((pts < 0) | (pts > 1)).any(1, keepdim=True)
        pts = torch.where(bad, centre[comp] + sigma[comp, None] * _randn(g, n, 2), pts)
    pts = torch.where(_rand(g, n, 1) < bg, _rand(g, n, 2), pts.clamp(0, 1))
    return pts.float()


def _waves(g, x, y, d):
    """d sums of 8 plane waves (wave vectors in [-3, 3]^2) at (x, y)."""
    out = torch.zeros((d,) + x.shape, device=DEV, dtype=torch.float64)
    for j in range(d):
        k = torch.randint(-3, 4, (8, 2), generator=g, device=DEV).double()
        k[:, 0] += (k.abs().sum(1) == 0).double()
        a, ph = _randn(g, 8) / k.norm(dim=1), 2 * math.pi * _rand(g, 8)
        for q in range(8):
            out[j] += a[q] * torch.sin(2 * math.pi * (k[q, 0] * x + k[q, 1] * y) + ph[q])
    return out


def _values(g, pts, d):
    """(n, d) float32 attributes: smooth fields and 1% noise."""
    f = _waves(g, pts[:, 0].double(), pts[:, 1].double(), d)
    f += 0.01 * (f.amax(1) - f.amin(1))[:, None] * _randn(g, *f.shape)
    return f.t().contiguous().float()


def _grid(width, height):
    # pixel centres of a canvas whose longer side has unit length
    s = 1.0 / max(width, height)
    return {"x0": 0.5 * s, "y0": 0.5 * s, "dx": s, "dy": s, "width": width, "height": height}


def _fields(g, c):
    """Smooth fields on the grid (float32 (d, H, W)), their slopes and range."""
    gr = _grid(c["width"], c["height"])
    x = (gr["x0"] + gr["dx"] * torch.arange(c["width"], device=DEV, dtype=torch.float64))
    y = (gr["y0"] + gr["dy"] * torch.arange(c["height"], device=DEV, dtype=torch.float64))
    X, Y = x.expand(c["height"], -1), y[:, None].expand(-1, c["width"])
    f = _waves(g, X, Y, c["d"])
    lo, hi = f.amin((1, 2)), f.amax((1, 2))
    return gr, f.float().contiguous(), lo, hi


def _serve_requests(case):
    """Sizes of a burst: requests from half to one and a half times the case's."""
    reqs = []
    for q in range(case["count"]):
        t = 0.5 + q / max(1, case["count"] - 1)
        basis = "linear" if q % 2 else "quadratic"
        n = int(case["n"] * t) + q
        near = 20.0 if basis == "linear" else 40.0
        reqs.append(dict(n=n, d=max(1, int(case["d"] * (1.5 - 0.5 * t))), basis=basis,
                         width=int(case["side"] * (1.25 - 0.5 * t)) + q, weight="gaussian",
                         height=int(case["side"] * (0.75 + 0.5 * t)),
                         h=math.sqrt(near / (math.pi * n)), precision=case["precision"],
                         points="uniform"))
    return reqs


def _contour_capacity(case):
    return 8 * case["d"] * case["n_iso"] * (case["width"] + case["height"])


def _layout_mesh(case, seed):
    pts, mesh, prm = workloads.layout_workload(case["n"], seed=seed % 1000003)
    return pts, mesh, prm


def prepare(case, seed):
    g, kind = _gen(seed), case["kind"]
    s = {"case": case}
    if kind == "fit":
        s["grid"] = _grid(case["width"], case["height"])
        s["points"] = _points(g, case["n"], case["points"])
        s["values"] = _values(g, s["points"], case["d"])
    elif kind == "contour":
        s["grid"], s["fields"], lo, hi = _fields(g, case)
        k = torch.arange(1, case["n_iso"] + 1, device=DEV) / (case["n_iso"] + 1)
        s["iso"] = (lo[:, None] + k * (hi - lo)[:, None]).float().contiguous()
        # room for the lines of every field, kept from redraw to redraw
        cap = _contour_capacity(case)
        s["segments"] = torch.zeros(cap, 4, device=DEV)
        s["ids"] = torch.zeros(cap, 3, dtype=torch.int32, device=DEV)
        s["count"] = torch.zeros(1, dtype=torch.int64, device=DEV)
    elif kind == "maps":
        s["grid"], s["fields"], lo, hi = _fields(g, case)
        f, gr = s["fields"], s["grid"]
        gy, gx = torch.gradient(f, dim=(1, 2)) if min(f.shape[1:]) > 1 else (f, f)
        s["grads"] = torch.stack([gx / gr["dx"], gy / gr["dy"]], 1).contiguous()
        k = torch.arange(1, case["n_iso"] + 1, device=DEV) / (case["n_iso"] + 1)
        s["iso"] = (lo[:, None] + k * (hi - lo)[:, None]).float().contiguous()
        s["levels"] = torch.stack([lo, (hi - lo) / (case["n_iso"] + 1)], 1).float().contiguous()
        s["colormap"] = torch.randint(1 << 31, (case["d"], case["n_iso"] + 1), generator=g,
                                      device=DEV).int()
    elif kind == "layout":
        pts, mesh, s["params"] = _layout_mesh(case, seed)
        s["start"] = torch.from_numpy(pts).float().to(DEV)
        s["pos"] = torch.empty_like(s["start"])
        s["mesh"] = {k: torch.from_numpy(v.reshape(-1)).to(DEV) for k, v in mesh.items()
                     if k != "triangles"}
    else:
        reqs = _serve_requests(case)
        scratch = sum(api.fit_scratch_bytes(r["n"], r["d"], _grid(r["width"], r["height"]),
                                            r["precision"]) for r in reqs) + (1 << 20)
        s["server"] = api.Server(0, (1 << 30) + 6 * scratch, 4, scratch)
        s["requests"] = []
        for r in reqs:
            p = _points(g, r["n"], "uniform")
            pid = s["server"].put_points(p, _values(g, p, r["d"]))
            gr = _grid(r["width"], r["height"])
            out = torch.empty((r["d"], r["height"], r["width"]), device=DEV)
            deg = torch.empty((r["height"], r["width"]), dtype=torch.uint8, device=DEV)
            s["requests"].append((pid, gr, out, deg, r))
    return s


# ---- one pass ----

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "fit":
        call = api.fit_grad if c.get("grads") else api.fit
        return call(s["points"], s["values"], s["grid"], basis=c["basis"], weight=c["weight"],
                    h=c["h"], alpha=c.get("alpha", 1.0), precision=c["precision"])
    if kind == "contour":
        api.contour_static(s["fields"], s["grid"], s["iso"], s["segments"], s["count"],
                           ids=s["ids"])
        return s["segments"], s["ids"], s["count"]
    if kind == "maps":
        bands, rgba = api.map_bands(s["fields"], s["grid"], s["iso"], colormap=s["colormap"])
        lines = api.map_adaptive(s["fields"], s["grads"], s["grid"], s["levels"],
                                 n_levels=c["n_levels"])
        return bands, rgba, lines
    if kind == "layout":
        s["pos"].copy_(s["start"])
        return api.layout(s["pos"], s["mesh"], iterations=c["iterations"], **s["params"])
    tickets = [s["server"].submit(pid, gr, out, deg, basis=r["basis"], h=r["h"],
                                  precision=r["precision"])
               for pid, gr, out, deg, r in s["requests"]]
    for t in tickets:
        res = s["server"].wait(t)
        if res["status"] != 0:
            raise RuntimeError(res["detail"])
    return [(out, deg) for _, _, out, deg, _ in s["requests"]]


# ---- what a pass cannot do without ----

def _fit_work(c):
    nodes = c["width"] * c["height"]
    m = {"constant": 1, "linear": 3, "quadratic": 6, "rigid": 3}[c["basis"]]
    nmom = {1: 1, 3: 6, 6: 15}[m]
    # points whose weight a node can tell from zero in float64 (Gaussian) or
    # that lie in the support (Wendland), at the mean density; every point
    # for the inverse-distance weight
    reach = {"gaussian": 6.0, "wendland": 1.0, "invpow": math.inf}[c["weight"]]
    near = min(c["n"], math.pi * (reach * c["h"]) ** 2 * c["n"])
    planes = c["d"] * (3 if c.get("grads") else 1)
    return {"bytes": 4.0 * c["n"] * (2 + c["d"]) + nodes * (4.0 * planes + 1),
            "flops": 2.0 * nodes * near * (nmom + c["d"])}


def work(case):
    kind = case["kind"]
    if kind == "fit":
        return _fit_work(case)
    if kind == "contour":
        # one read of the fields, and 28 bytes for each segment: a field's
        # level crosses about as many cells as two grid sides hold
        segs = 2 * case["d"] * case["n_iso"] * (case["width"] + case["height"])
        return {"bytes": 4.0 * case["d"] * case["width"] * case["height"] + 28.0 * segs,
                "flops": 0.0}
    if kind == "maps":
        return {"bytes": 25.0 * case["d"] * case["width"] * case["height"], "flops": 0.0}
    if kind == "layout":
        return {"bytes": 80.0 * case["n"] * case["iterations"],
                "flops": 15.0 * case["n"] * (case["n"] - 1) * case["iterations"]}
    w = [_fit_work(r) for r in _serve_requests(case)]
    return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}


# ---- the same definitions in float64 ----

_BASIS_EXP = [(0, 0), (1, 0), (0, 1), (2, 0), (1, 1), (0, 2)]


def _ladder(M, floor_w=1e-6, tau=1e-8):
    """Degree ladder on node-frame moment matrices (P, m, m): the rows
    A[:, j] = M'^-1 e_j of the accepted degree for j = 0, 1, 2 (zero past the
    accepted terms) and whether the node is determined."""
    P, m = M.shape[0], M.shape[1]
    out = torch.zeros(P, 3, m, device=DEV, dtype=torch.float64)
    done = ~(M[:, 0, 0] >= floor_w)
    known = ~done
    for mk in [k for k in (6, 3, 1) if k <= m]:
        D = torch.diagonal(M[:, :mk, :mk], dim1=1, dim2=2)
        ok = (D > 0).all(1)
        sc = 1.0 / torch.sqrt(torch.where(D > 0, D, torch.ones_like(D)))
        A = sc[:, :, None] * M[:, :mk, :mk] * sc[:, None, :]
        L = [[None] * mk for _ in range(mk)]
        for j in range(mk):
            p = A[:, j, j]
            for q in range(j):
                p = p - L[j][q] ** 2
            ok = ok & (p >= tau)
            L[j][j] = torch.sqrt(torch.where(p >= tau, p, torch.ones_like(p)))
            for r in range(j + 1, mk):
                v = A[:, r, j]
                for q in range(j):
                    v = v - L[r][q] * L[j][q]
                L[r][j] = v / L[j][j]
        take = ok & ~done
        for e in range(min(3, mk)):
            z = []
            for r in range(mk):
                v = sc[:, r] if r == e else torch.zeros_like(sc[:, 0])
                for q in range(r):
                    v = v - L[r][q] * z[q]
                z.append(v / L[r][r])
            w = [None] * mk
            for r in reversed(range(mk)):
                v = z[r]
                for q in range(r + 1, mk):
                    v = v - L[q][r] * w[q]
                w[r] = v / L[r][r]
            for r in range(mk):
                out[:, e, r] = torch.where(take, sc[:, r] * w[r], out[:, e, r])
        done = done | ok
    return out, known & done


def _rigid(M, R, h):
    """Eq. 9-10 from the linear node-frame moments (P, 3, 3) and products."""
    w0 = M[:, 0, 0]
    P, Q = h * M[:, 0, 1:3] / w0[:, None], R[:, 0, :] / w0[:, None]
    c = h * R[:, 1:3, :] - w0[:, None, None] * P[:, :, None] * Q[:, None, :]
    mu, nu = c[:, 0, 0] + c[:, 1, 1], c[:, 1, 0] - c[:, 0, 1]
    rho = torch.sqrt(mu * mu + nu * nu)
    f = torch.stack([-P[:, 0] * mu - P[:, 1] * nu, P[:, 0] * nu - P[:, 1] * mu], 1)
    return Q + torch.where((rho > 0)[:, None], f / rho.clamp_min(1e-300)[:, None], 0.0)


def _exact_fit(c, grid, points, values):
    """Fields and slopes by the definition, in blocks of nodes with each
    block's own coordinate frame."""
    W, H, h, d = c["width"], c["height"], c["h"], c["d"]
    X, Y, V = points[:, 0].double(), points[:, 1].double(), values.double()
    m = {"constant": 1, "linear": 3, "quadratic": 6, "rigid": 3}[c["basis"]]
    exps = _BASIS_EXP[:m]
    # beyond 12 h a Gaussian weighs less than 1e-62
    reach = {"gaussian": 12.0 * h, "wendland": h, "invpow": math.inf}[c["weight"]]
    out = torch.full((d, H, W), math.nan, device=DEV, dtype=torch.float64)
    grads = torch.full((d, 2, H, W), math.nan, device=DEV, dtype=torch.float64)
    strip, side = 512, 64
    for s0 in range(0, H, strip):
        s1 = min(H, s0 + strip)
        M = torch.zeros(s1 - s0, W, m, m, device=DEV, dtype=torch.float64)
        R = torch.zeros(s1 - s0, W, m, d, device=DEV, dtype=torch.float64)
        E = torch.zeros(2, s1 - s0, W, device=DEV, dtype=torch.float64)
        for r0 in range(s0, s1, side):
            for c0 in range(0, W, side):
                r1, c1 = min(s1, r0 + side), min(W, c0 + side)
                gx = grid["x0"] + grid["dx"] * torch.arange(c0, c1, device=DEV).double()
                gy = grid["y0"] + grid["dy"] * torch.arange(r0, r1, device=DEV).double()
                near = ((X >= gx[0] - reach) & (X <= gx[-1] + reach) &
                        (Y >= gy[0] - reach) & (Y <= gy[-1] + reach)).nonzero()[:, 0]
                cx, cy = gx.mean(), gy.mean()
                ux, uy, f = (X[near] - cx) / h, (Y[near] - cy) / h, V[near]
                ex = ((gx - cx) / h).expand(r1 - r0, -1)
                ey = ((gy - cy) / h)[:, None].expand(-1, c1 - c0)
                E[0, r0 - s0:r1 - s0, c0:c1] = ex
                E[1, r0 - s0:r1 - s0, c0:c1] = ey
                r2 = (ux - ex.reshape(-1, 1)) ** 2 + (uy - ey.reshape(-1, 1)) ** 2
                if c["weight"] == "gaussian":
                    w = torch.exp(-r2)
                elif c["weight"] == "wendland":
                    t = torch.sqrt(r2)
                    w = (1 - t).clamp_min(0) ** 4 * (4 * t + 1)
                else:
                    w = r2 ** (-c.get("alpha", 1.0))
                b = torch.stack([ux ** i * uy ** j for i, j in exps], 1)
                feats = torch.cat([(b[:, :, None] * b[:, None, :]).reshape(-1, m * m),
                                   (b[:, :, None] * f[:, None, :]).reshape(-1, m * d)], 1)
                G = (w @ feats).reshape(r1 - r0, c1 - c0, -1)
                M[r0 - s0:r1 - s0, c0:c1] = G[..., :m * m].reshape(r1 - r0, c1 - c0, m, m)
                R[r0 - s0:r1 - s0, c0:c1] = G[..., m * m:].reshape(r1 - r0, c1 - c0, m, d)
        # to the node's own frame: b(u - e) = T b(u)
        M, R, (ex, ey) = M.reshape(-1, m, m), R.reshape(-1, m, d), E.reshape(2, -1)
        T = torch.zeros(M.shape[0], m, m, device=DEV, dtype=torch.float64)
        T[:, 0, 0] = 1
        if m >= 3:
            T[:, 1, 0], T[:, 1, 1], T[:, 2, 0], T[:, 2, 2] = -ex, 1, -ey, 1
        if m >= 6:
            T[:, 3, 0], T[:, 3, 1], T[:, 3, 3] = ex * ex, -2 * ex, 1
            T[:, 4, 0], T[:, 4, 1], T[:, 4, 2], T[:, 4, 4] = ex * ey, -ey, -ex, 1
            T[:, 5, 0], T[:, 5, 2], T[:, 5, 5] = ey * ey, -2 * ey, 1
        M = sum(T[:, :, q, None] * M[:, q, None, :] for q in range(m))
        M = sum(M[:, :, q, None] * T[:, None, :, q] for q in range(m))
        shape = (d, s1 - s0, W)
        if c["basis"] == "rigid":
            R = sum(T[:, :, q, None] * R[:, q, None, :] for q in range(m))
            out[:, s0:s1] = _rigid(M, R, h).t().reshape(shape)
            continue
        A, known = _ladder(M)
        for e in range(3 if c.get("grads") else 1):
            # (M'^-1 e_e)^T T R, the node's row taken to the block's frame first
            y = sum(A[:, e, q, None] * T[:, q, :] for q in range(m))
            v = sum(y[:, q, None] * R[:, q, :] for q in range(m))
            v = torch.where(known[:, None], v, math.nan).t().reshape(shape)
            if e == 0:
                out[:, s0:s1] = v
            else:
                grads[:, e - 1, s0:s1] = v / h
    return out, grads


def _exact_contour(s):
    """Marching squares on the float32 fields, positions in float64."""
    f, gr = s["fields"], s["grid"]
    D, H, W = f.shape
    # segments per case as (from, to) edges, the above side on the left;
    # cases 5 and 10 join the above corners when the centre is above
    one = [[], [(0, 3)], [(1, 0)], [(1, 3)], [(2, 1)], [], [(2, 0)], [(2, 3)], [(3, 2)],
           [(0, 2)], [], [(1, 2)], [(3, 1)], [(0, 1)], [(3, 0)], []]
    joined = {5: [(0, 1), (2, 3)], 10: [(3, 0), (1, 2)]}
    split = {5: [(0, 3), (2, 1)], 10: [(1, 0), (3, 2)]}
    table = torch.full((32, 2, 2), -1, dtype=torch.long)
    for k in range(16):
        for j, two in enumerate((split, joined)):
            for q, e in enumerate(two.get(k, one[k])):
                table[k + 16 * j, q] = torch.tensor(e)
    table = table.to(DEV)
    segs = []
    for d in range(D):
        v = torch.stack([f[d, :-1, :-1], f[d, :-1, 1:], f[d, 1:, 1:], f[d, 1:, :-1]], 0)
        v = v.reshape(4, -1)
        for iso in s["iso"][d]:
            above = v >= iso
            case = (above.long() * torch.tensor([1, 2, 4, 8], device=DEV)[:, None]).sum(0)
            centre = ((v[0] + v[1]) + (v[2] + v[3])) * 0.25 >= iso
            cells = ((case > 0) & (case < 15)).nonzero()[:, 0]
            edges = table[case[cells] + 16 * centre[cells].long()]        # (c, 2, 2)
            live = edges[:, :, 0] >= 0
            cell = cells[:, None].expand(-1, 2)[live]
            edges = edges[live]                                           # (s, 2)
            i, j = (cell // (W - 1)).double(), (cell % (W - 1)).double()
            ends = []
            for q in range(2):
                e = edges[:, q]
                a = torch.tensor([0, 1, 3, 0], device=DEV)[e]
                b = torch.tensor([1, 2, 2, 3], device=DEV)[e]
                va, vb = v[a, cell].double(), v[b, cell].double()
                t = (iso.double() - va) / (vb - va)
                x = torch.where(e % 2 == 0, j + t, j + (e == 1).double())
                y = torch.where(e % 2 == 1, i + t, i + (e == 2).double())
                ends += [gr["x0"] + x * gr["dx"], gr["y0"] + y * gr["dy"]]
            segs.append(torch.stack(ends, 1))
    segs = torch.cat(segs)
    out = torch.zeros(s["segments"].shape, device=DEV, dtype=torch.float64)
    out[:segs.shape[0]] = segs
    return out


def _exact_lines(s, n_levels, halfwidth=1.0, lo=4.0, hi=12.0):
    f, g, gr = s["fields"].double(), s["grads"].double(), s["grid"]
    origin, spacing = (s["levels"][:, k].double()[:, None, None] for k in (0, 1))
    r = torch.sqrt((g[:, 0] * gr["dx"]) ** 2 + (g[:, 1] * gr["dy"]) ** 2)
    best = torch.zeros_like(f)
    for j in range(n_levels):
        step = spacing / 2 ** j
        sp = step / r
        t = (f - origin) / step
        op = torch.ones_like(f) if j == 0 else ((sp - lo) / (hi - lo)).clamp(0, 1)
        best = torch.maximum(best, op * (1 - (t - torch.round(t)).abs() * sp /
                                         halfwidth).clamp_min(0))
    return torch.where(r > 0, best, 0.0)


def _exact_layout(pts, mesh, prm, iterations):
    """Eq. 1-3 with the temperature and the limiting lines, all nodes at once."""
    n = pts.shape[0]
    x = torch.from_numpy(pts).float().double().to(DEV)
    C, D, eta, t = prm["C"], prm["D"], prm["eta"], prm["t0"]
    deg = torch.from_numpy(mesh["adj_start"]).long().diff()
    av = torch.repeat_interleave(torch.arange(n), deg).to(DEV)
    au = torch.from_numpy(mesh["adj"]).long().to(DEV)
    tri = torch.from_numpy(mesh["fan_start"]).long().diff()
    fv = torch.repeat_interleave(torch.arange(n), tri).to(DEV)
    fan = torch.from_numpy(mesh["fan"]).long().reshape(-1, 2).to(DEV)

    def offset(c, a, b):   # from the foot on the line (a, b) to c
        e = b - a
        return c - (a + (((c - a) * e).sum(1) / (e * e).sum(1))[:, None] * e)

    for _ in range(iterations):
        F = torch.zeros_like(x)
        for r0 in range(0, n, 1024):
            V = x[r0:r0 + 1024, None, :] - x[None, :, :]
            F[r0:r0 + 1024] = (C * V / ((V * V).sum(2) ** 1.5 + eta)[:, :, None]).sum(1)
        V = x[av] - x[au]
        L = V.norm(dim=1)
        F.index_add_(0, av, -(L * torch.log((L + eta) / D))[:, None] * V)
        c, a, b = x[fv], x[fan[:, 0]], x[fan[:, 1]]
        R = -offset(c, a, b)
        F.index_add_(0, fv, -C * R / ((R * R).sum(1) + eta)[:, None])
        fl = F.norm(dim=1, keepdim=True)
        F = torch.where(fl > t, F * (t / fl), F)
        scale = torch.ones(n, device=DEV, dtype=torch.float64)
        for o in (-0.5 * offset(c, a, b), 0.5 * offset(a, b, c), 0.5 * offset(b, c, a)):
            rl = o.norm(dim=1)
            proj = (F[fv] * o).sum(1) / rl
            lim = torch.where(proj > 0, (rl - eta).clamp_min(0) / proj, 1.0)
            scale.scatter_reduce_(0, fv, lim, "amin")
        x = x + scale[:, None] * F
        t *= prm["lam"]
    return x


def exact(case, seed):
    g, kind = _gen(seed), case["kind"]
    if kind == "layout":
        pts, mesh, prm = _layout_mesh(case, seed)
        return _exact_layout(pts, mesh, prm, case["iterations"])
    if kind == "serve":
        out = []
        for r in _serve_requests(case):
            p = _points(g, r["n"], "uniform")
            f, _ = _exact_fit(r, _grid(r["width"], r["height"]), p, _values(g, p, r["d"]))
            out.append((f, None))
        return out
    s = prepare(case, seed)
    if kind == "fit":
        f, gr = _exact_fit(case, s["grid"], s["points"], s["values"])
        return (f, gr, None) if case.get("grads") else (f, None)
    if kind == "contour":
        return _exact_contour(s), None, None
    return None, None, _exact_lines(s, case["n_levels"])
