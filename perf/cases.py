"""Performance cases of the framework: the calls its users make, with inputs
and a 64-bit definition of each result.

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  what a program holds before the call (on the GPU)
  run(state)           one pass through the public entry points; its outputs
  work(case)           bytes and operations the pass cannot do without
  exact(case, seed)    the outputs in 64 bits by plain torch (no code of this
                       package), or None where that would take too long

Volumes are ellipsoids on a faint noise floor (attenuations per mm),
projections for timing are uniform in [0, 1) (the paper's timing input), the
solvers' data are the ellipsoids' line integrals plus 1 % noise.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2110_09841_amd as _pkg  # noqa: F401
from paper_2110_09841_amd import autograd, cvp, solvers, unet

DEV = "cuda"
EXACT_LIMIT = 1.0e9          # voxel-view updates that exact() takes on


# ------------------------------------------------------------------ the cases

def _op(name, dims, vox, det, pitch, sid, sdd, views, arc, **kw):
    vox = (vox,) * 3 if np.isscalar(vox) else vox
    c = dict(name=name, kind="operators", n1=dims[0], n2=dims[1], n3=dims[2], a1=vox[0], a2=vox[1], a3=vox[2],
             cols=det[0], rows=det[1], pitch=pitch, sid=sid, sdd=sdd, views=views, arc=arc, variant="relaxed", ec=True,
             scaling="solid_angle", cached=False, matrices=False, autograd=False)
    c.update(kw)
    return c


def listed():
    return [
        # the benchmark's C-arm short scan: A x and A^T b, record table kept, as an iterative solver applies them
        _op("carm_512", (512, 512, 512), 0.25, (616, 480), 0.616, 749.0, 1198.0, 248, 200.0, cached=True),
        # the 12 degree cone workload as a differentiable layer: forward and backward with the default options
        _op("cone_256_autograd", (256, 256, 256), 0.5, (512, 384), 0.388, 600.0, 900.0, 360, 360.0, variant="exact",
            autograd=True),
        # the paper's "Pfeiffer" speed benchmark (pixels small against the voxels), the relaxed form
        _op("pfeiffer_256", (256, 256, 256), 0.5, (1280, 960), 0.25, 750.0, 1000.0, 100, 198.0),
        # the smallest workload of the tests and the benchmark, default options: few blocks, launches count
        _op("small_64", (64, 64, 64), 1.0, (96, 96), 1.6, 750.0, 1200.0, 32, 360.0, variant="exact"),
        # a general trajectory (one camera matrix per view), ragged sizes, the flat-panel scaling without the
        # elevation correction
        _op("matrices_ragged", (107, 93, 131), (0.9, 1.0, 0.8), (181, 163), 1.1, 560.0, 910.0, 75, 360.0,
            matrices=True, ec=False, scaling="cos"),
        # the separable-footprint projector that the paper compares with
        _op("tt_128", (128, 128, 128), 1.0, (256, 256), 1.0, 750.0, 1200.0, 90, 360.0, variant="tt", ec=False,
            scaling="cos"),
        # the two CGLS iterates that feed the learned warm start, on its workload
        dict(_op("cgls_128", (128, 128, 128), 1.0, (256, 256), 1.0, 750.0, 1200.0, 180, 360.0), kind="cgls", iters=2),
        # one OS-SART sweep: many launches over few views each
        dict(_op("ossart_80", (80, 80, 72), 1.0, (128, 112), 1.6, 750.0, 1200.0, 96, 360.0), kind="ossart",
             subsets=12),
        # uneven problems in one persistent launch per direction
        dict(name="batch_6", kind="batch", problems=6, edge_min=64, edge_max=128, views_min=40, views_max=120,
             draw_seed=41, cached=True),
        # the warm-start network: inference at its workload's size
        dict(name="unet_forward_128", kind="unet_forward", d=128, h=128, w=128),
        # and one gradient evaluation (forward, loss, backward) on a ragged volume
        dict(name="unet_gradients", kind="unet_gradients", d=64, h=72, w=88),
        # one 3x3x3 convolution layer by itself: forward, backward-data, backward-weight, bias gradient
        dict(name="conv_64_32", kind="conv", d=48, h=50, w=66, ci=64, co=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["operators"] * 6 + ["cgls", "ossart", "batch", "unet_forward", "unet_gradients", "conv"])
    if kind in ("operators", "cgls", "ossart"):
        edge = _log(rng, 40, 224 if kind == "operators" else 112)
        dims = tuple(max(16, int(edge * rng.uniform(0.7, 1.2))) for _ in range(3))
        vox = rng.uniform(0.4, 1.2)
        vox = tuple(vox * rng.uniform(0.85, 1.15) for _ in range(3))
        pitch = rng.choice([0.55, 0.8, 1.0, 1.25, 1.6]) * 1.6 * vox[0]       # about that many voxels per pixel
        width = 1.7 * max(dims[0] * vox[0], dims[1] * vox[1]) * math.sqrt(2.0)
        cols = max(24, int(width / pitch * rng.uniform(0.85, 1.1)))
        rows = max(20, int(1.75 * dims[2] * vox[2] / pitch * rng.uniform(0.8, 1.1)))
        views = _log(rng, 16, 240)
        if kind != "operators":
            views = min(views, 120)
        c = _op(None, dims, vox, (cols, rows), pitch, 750.0, 1200.0, views, rng.choice([200.0, 360.0]),
                variant=rng.choice(["exact", "relaxed", "relaxed"]), ec=rng.random() < 0.8,
                cached=rng.random() < 0.5)
        del c["name"]
        c["kind"] = kind
        if kind == "operators":
            c["matrices"] = rng.random() < 0.25
            c["autograd"] = rng.random() < 0.3
            c["scaling"] = rng.choice(["solid_angle", "solid_angle", "cos"])
            if rng.random() < 0.15:
                c.update(variant="tt", ec=False, scaling="cos", cached=False)
        elif kind == "cgls":
            c["iters"] = rng.randint(1, 3)
        else:
            c["subsets"] = rng.randint(3, max(4, views // 5))
        return c
    if kind == "batch":
        lo = rng.choice([48, 64])
        return dict(kind="batch", problems=rng.randint(2, 8), edge_min=lo, edge_max=rng.randint(lo + 8, 140),
                    views_min=20, views_max=rng.randint(40, 110), draw_seed=rng.randrange(1 << 20),
                    cached=rng.random() < 0.5)
    if kind == "conv":
        ci, co = rng.choice([(16, 16), (16, 32), (32, 16), (32, 32), (32, 64), (64, 32), (64, 64)])
        e = _log(rng, 16, 96)
        return dict(kind="conv", d=max(4, int(e * rng.uniform(0.6, 1.1))), h=max(4, int(e * rng.uniform(0.6, 1.1))),
                    w=max(4, int(e * rng.uniform(0.6, 1.3))), ci=ci, co=co)
    e = _log(rng, 5, 32 if kind == "unet_forward" else 24)
    return dict(kind=kind, **{k: 4 * max(2, int(e * rng.uniform(0.7, 1.15))) for k in ("d", "h", "w")})


# --------------------------------------------------------- geometry and inputs

def _batch_members(case):
    """The uneven problems of a batch: edge, voxel, detector, views and arc
    drawn per problem, the pitch such that the volume fits the detector."""
    r = np.random.Generator(np.random.PCG64(case["draw_seed"]))
    out = []
    for _ in range(case["problems"]):
        edge = int(r.integers(case["edge_min"], case["edge_max"] + 1))
        vox = float(r.uniform(0.5, 1.0))
        cols, rows = [(128, 96), (160, 120), (192, 144), (256, 192)][int(r.integers(0, 4))]
        views = int(r.integers(case["views_min"], case["views_max"] + 1))
        arc = float(r.choice([360.0, 200.0]))
        out.append(_op(None, (edge,) * 3, vox, (cols, rows), 1.05 * 1.6 * edge * vox * math.sqrt(2.0) / cols, 750.0,
                       1200.0, views, arc))
    return out


def _frames(c):
    """Per view: source s, horizontal axes e1 and d, f/b1, f/b2, principal
    point.  A camera-matrix trajectory wobbles about the circular orbit."""
    r = np.random.Generator(np.random.PCG64(c["views"]))
    out = []
    for v in range(c["views"]):
        lam = v * math.radians(c["arc"]) / c["views"]
        D, f, dz, yaw, o1, o2, q = c["sid"], c["sdd"], 0.0, 0.0, 0.0, 0.0, 1.0
        if c["matrices"]:
            u = r.uniform(-1.0, 1.0, size=7)
            D, f, dz, yaw = D * (1 + 0.01 * u[0]), f * (1 + 0.01 * u[1]), 2.0 * u[2], math.radians(u[3])
            o1, o2, q = 3.0 * u[4], 3.0 * u[5], 1 + 0.02 * u[6]
        cl, sl, cy, sy = math.cos(lam), math.sin(lam), math.cos(yaw), math.sin(yaw)
        d = (-cl * cy + sl * sy, -sl * cy - cl * sy)
        out.append(((D * cl, D * sl, dz), (d[1], -d[0]), d, f / (c["pitch"] * q), f / c["pitch"],
                    (c["cols"] - 1) / 2 + o1, (c["rows"] - 1) / 2 + o2))
    return out


def _params(c):
    p = dict(vol_dims=(c["n1"], c["n2"], c["n3"]), voxel_mm=(c["a1"], c["a2"], c["a3"]), vol_offset_mm=(0.0, 0.0, 0.0),
             det_cols=c["cols"], det_rows=c["rows"])
    if c["matrices"]:
        P = np.zeros((c["views"], 3, 4))
        for v, (s, e1, d, fb1, fb2, c1, c2) in enumerate(_frames(c)):
            K = np.array([[fb1, 0, c1], [0, fb2, c2], [0, 0, 1.0]])
            R = np.array([[e1[0], e1[1], 0], [0, 0, -1.0], [d[0], d[1], 0]])
            P[v, :, :3] = K @ R
            P[v, :, 3] = -(K @ R) @ np.array(s)
        p["matrices"] = P
    else:
        p.update(pitch_mm=(c["pitch"], c["pitch"]), principal_px=None, sid_mm=c["sid"], sdd_mm=c["sdd"],
                 angles_rad=np.arange(c["views"]) * (math.radians(c["arc"]) / c["views"]))
    return p


def _options(c):
    return cvp.Options(variant=c["variant"], ec=c["ec"], scaling=c["scaling"])


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _ellipsoids(c, seed, n=12):
    """(centre, semi-axes, attenuation) of axis-aligned ellipsoids."""
    r = np.random.Generator(np.random.PCG64([int(seed), 77]))
    box = np.array([c["n1"] * c["a1"], c["n2"] * c["a2"], c["n3"] * c["a3"]])
    return [(r.uniform(-0.28, 0.28, 3) * box, r.uniform(0.04, 0.17, 3) * box, r.uniform(0.001, 0.02)) for _ in range(n)]


def _axes(c, dtype=torch.float64):
    return [(torch.arange(c["n%d" % q], device=DEV, dtype=dtype) - (c["n%d" % q] - 1) / 2) * c["a%d" % q]
            for q in (1, 2, 3)]


def _phantom(c, seed):
    X, Y, Z = _axes(c, torch.float32)
    vol = torch.rand((c["n3"], c["n2"], c["n1"]), generator=_gen(seed), device=DEV).mul_(2e-4)
    for m, s, mu in _ellipsoids(c, seed):
        px, py, pz = (((A - float(m[q])) / float(s[q])) ** 2 for q, A in enumerate((X, Y, Z)))
        vol += float(mu) * ((pz[:, None] + py)[:, :, None] + px <= 1.0)
    return vol


def _uniform(shape, seed):
    return torch.rand(shape, generator=_gen(seed + 1), device=DEV)


def _measured(c, seed):
    """Line integrals of the ellipsoids at the pixel centres plus 1 % noise."""
    b = torch.empty((c["views"], c["rows"], c["cols"]), device=DEV)
    ells = _ellipsoids(c, seed)
    for v, (s, e1, d, fb1, fb2, c1, c2) in enumerate(_frames(c)):
        w1 = (torch.arange(c["cols"], device=DEV, dtype=torch.float64) - c1) / fb1
        w2 = (torch.arange(c["rows"], device=DEV, dtype=torch.float64) - c2) / fb2
        g = ((d[0] + w1 * e1[0])[None, :], (d[1] + w1 * e1[1])[None, :], -w2[:, None])
        ln = torch.sqrt(g[0] ** 2 + g[1] ** 2 + g[2] ** 2)
        acc = torch.zeros_like(ln)
        for m, sa, mu in ells:
            o = [(s[q] - m[q]) / sa[q] for q in range(3)]
            h = [g[q] / sa[q] for q in range(3)]
            A = h[0] ** 2 + h[1] ** 2 + h[2] ** 2
            B = o[0] * h[0] + o[1] * h[1] + o[2] * h[2]
            acc += 2 * mu * torch.sqrt((B * B - A * (o[0] ** 2 + o[1] ** 2 + o[2] ** 2 - 1)).clamp(min=0)) / A
        b[v] = (acc * ln).float()
    sigma = 0.01 * float(b.double().square().mean().sqrt())
    return b + sigma * torch.randn(b.shape, generator=_gen(seed + 2), device=DEV)


LAYERS = [("c1a", 16, 16), ("c1b", 16, 16), ("c2a", 16, 32), ("c2b", 32, 32), ("c3a", 32, 64), ("c3b", 64, 64),
          ("u2", 64, 32), ("d2a", 64, 32), ("d2b", 32, 32), ("u1", 32, 16), ("d1a", 32, 16), ("d1b", 16, 16)]


def _net_inputs(case, seed):
    """Weights (He-uniform), small biases, head, two iterates and a target."""
    g = _gen(seed)
    P = {}
    for n, ci, co in LAYERS:
        P[n] = (torch.empty((27, co, ci), device=DEV).uniform_(-1, 1, generator=g) * math.sqrt(6.0 / (27 * ci)),
                0.05 * torch.randn(co, generator=g, device=DEV))
    P["head"] = (torch.empty(16, device=DEV).uniform_(-0.25, 0.25, generator=g),
                 0.05 * torch.randn(1, generator=g, device=DEV))
    vol = dict(n1=case["w"], n2=case["h"], n3=case["d"], a1=1.0, a2=1.0, a3=1.0)
    t = _phantom(vol, seed)
    x1 = 0.5 * t + 0.001 * torch.randn(t.shape, generator=g, device=DEV)
    x2 = 0.8 * t + 0.001 * torch.randn(t.shape, generator=g, device=DEV)
    return P, x1, x2, t


def _conv_inputs(case, seed):
    g = _gen(seed)
    sh = (case["d"], case["h"], case["w"])
    ci, co = case["ci"], case["co"]
    x = torch.randn(sh + (ci,), generator=g, device=DEV).clamp(min=0).bfloat16()
    w = (torch.empty((27, co, ci), device=DEV).uniform_(-1, 1, generator=g) * math.sqrt(6.0 / (27 * ci))).bfloat16()
    return x, w, 0.1 * torch.randn(co, generator=g, device=DEV), \
        torch.randn(sh + (co,), generator=g, device=DEV).bfloat16()


# ------------------------------------------------------------ prepare and run

def _geometry(c, cached):
    G = cvp.Geometry(_params(c))
    if cached:
        G.cache_records()
    return G


def prepare(case, seed):
    k = case["kind"]
    if k in ("operators", "cgls", "ossart"):
        G, opts = _geometry(case, case["cached"]), _options(case)
        if k == "operators":
            x, b = _phantom(case, seed), _uniform(G.proj_shape, seed)
            if case["autograd"]:
                x.requires_grad_(True)
            return dict(case=case, G=G, opts=opts, x=x, b=b)
        b = _measured(case, seed)
        if k == "cgls":
            return dict(case=case, solver=cvp.CGLS(G, opts, b))
        S = solvers.OSSART(G, opts, b, case["subsets"])
        S.setup()
        return dict(case=case, solver=S)
    if k == "batch":
        cs = _batch_members(case)
        Gs = [_geometry(c, case["cached"]) for c in cs]
        return dict(case=case, batch=cvp.Batch(Gs), opts=cvp.Options(variant="relaxed", ec=True),
                    xs=[_phantom(c, seed + q) for q, c in enumerate(cs)],
                    bs=[_uniform(G.proj_shape, seed + q) for q, G in enumerate(Gs)])
    if k == "conv":
        x, w, bias, dy = _conv_inputs(case, seed)
        L = unet.lib()
        wt = torch.empty((27, case["ci"], case["co"]), dtype=torch.bfloat16, device=DEV)
        unet._check(L.cvp_nn_transpose_weights(unet._p(w), unet._p(wt), case["co"], case["ci"], unet._s()))
        n = ctypes.c_int64()
        unet._check(L.cvp_nn_wgrad_workspace(ctypes.byref(unet.desc(x)), ctypes.byref(unet.desc(dy)), ctypes.byref(n)))
        return dict(case=case, L=L, x=x, w=w, wt=wt, bias=bias, dy=dy, y=torch.empty_like(dy), dx=torch.empty_like(x),
                    dw=torch.empty((27, case["co"], case["ci"]), device=DEV), db=torch.empty(case["co"], device=DEV),
                    work=torch.empty(n.value + 65536, device=DEV))
    P, x1, x2, t = _net_inputs(case, seed)
    net = unet.UNet((case["d"], case["h"], case["w"]), seed=0)
    for n, ci, co in LAYERS:                               # a trained network's parameters
        c = net.convs[n]
        c.w.copy_(P[n][0])
        c.b.copy_(P[n][1])
        c.wb.copy_(P[n][0])
        c.refresh()
    net.hw.copy_(P["head"][0])
    net.hb.copy_(P["head"][1])
    return dict(case=case, net=net, x1=x1, x2=x2, t=t)


def run(state):
    case = state["case"]
    k = case["kind"]
    if k == "operators":
        G, opts, x = state["G"], state["opts"], state["x"]
        if case["autograd"]:
            x.grad = None
            y = autograd.project(x, G, opts)
            y.backward(state["b"])
            return y.detach(), x.grad
        return cvp.project(x, G, opts), cvp.backproject(state["b"], G, opts)
    if k == "cgls":
        S = state["solver"]
        S.reset()
        S.set_tolerance(0.0)
        S.start()
        S.iterate(case["iters"])
        return S.x, S.s
    if k == "ossart":
        S = state["solver"]
        S.x.zero_()
        S.iterate(1)
        return S.x
    if k == "batch":
        return (cvp.project_batched(state["xs"], state["batch"], state["opts"]),
                cvp.backproject_batched(state["bs"], state["batch"], state["opts"]))
    if k == "conv":
        s, L, d = state, state["L"], unet.desc
        ref, p, st = ctypes.byref, unet._p, unet._s()
        unet._check(L.cvp_nn_conv3d(ref(d(s["x"])), p(s["w"]), p(s["bias"]), ref(d(s["y"])), 1, 0, st))
        unet._check(L.cvp_nn_conv3d(ref(d(s["dy"])), p(s["wt"]), None, ref(d(s["dx"])), 0, 1, st))
        unet._check(L.cvp_nn_conv3d_wgrad(ref(d(s["x"])), ref(d(s["dy"])), p(s["dw"]), p(s["work"]),
                                          s["work"].numel(), st))
        unet._check(L.cvp_nn_channel_sum(ref(d(s["dy"])), p(s["db"]), p(s["work"]), s["work"].numel(), st))
        return s["y"], s["dx"], s["dw"], s["db"]
    net = state["net"]
    x0 = net.forward(state["x1"], state["x2"])
    if k == "unet_forward":
        return x0
    loss = net.mse(x0, state["t"])
    net.backward(net.gx0)
    return dict(x0=x0, loss=loss, gw=[c.gw for c in net.convs.values()], gb=[c.gb for c in net.convs.values()],
                ghead=net.ghead)


# ----------------------------------------------------------------------- work

def _voxel_views(c):
    return c["n1"] * c["n2"] * c["n3"] * c["views"]


def _pair_work(c, pairs):
    # operands once each; about 100 operations per voxel-view (a voxel meets
    # about two detector columns and three pixels)
    nv, npx = c["n1"] * c["n2"] * c["n3"], c["views"] * c["cols"] * c["rows"]
    return pairs * 8.0 * (nv + npx), pairs * 200.0 * _voxel_views(c)


def work(case):
    k = case["kind"]
    if k == "operators":
        b, f = _pair_work(case, 1)
    elif k == "cgls":
        b, f = _pair_work(case, case["iters"] + 1)
    elif k == "ossart":
        b, f = _pair_work(case, 1)
        nv, npx = case["n1"] * case["n2"] * case["n3"], case["views"] * case["cols"] * case["rows"]
        b += 4.0 * npx + (case["subsets"] - 1) * 12.0 * nv      # b once; per subset x, x and the column sums
    elif k == "batch":
        ws = [_pair_work(c, 1) for c in _batch_members(case)]
        b, f = sum(w[0] for w in ws), sum(w[1] for w in ws)
    elif k == "conv":
        v = case["d"] * case["h"] * case["w"]
        b = 2.0 * v * (2 * case["ci"] + 2 * case["co"]) + 27 * case["ci"] * case["co"] * 8
        f = 3 * 54.0 * v * case["ci"] * case["co"]
    else:
        v = case["d"] * case["h"] * case["w"]
        res = dict(zip([n for n, _, _ in LAYERS], (1, 1, 8, 8, 64, 64, 8, 8, 8, 1, 1, 1)))
        f = sum(54.0 * v / res[n] * (2 if n == "c1a" else ci) * co for n, ci, co in LAYERS)
        b = 12.0 * v + 2 * sum(27 * ci * co for _, ci, co in LAYERS)
        if k == "unet_gradients":
            f, b = 3 * f, b + 4.0 * v + 4 * sum(27 * ci * co for _, ci, co in LAYERS)
    return {"bytes": float(b), "flops": float(f)}


# ---------------------------------------------------- the results in 64 bits

def _clip(h1, h2, gx, gy, c):
    """Integrals of 1, x, y, x^2, xy, y^2 over the rectangle [-h1, h1] x
    [-h2, h2] where gx x + gy y + c <= 0 (Green's theorem along the clipped
    boundary)."""
    px, py = (-h1, h1, h1, -h1), (-h2, -h2, h2, h2)
    f = [gx * px[q] + gy * py[q] + c for q in range(4)]
    z = torch.zeros_like(c)
    m = [z.clone() for _ in range(6)]

    def edge(x0, y0, x1, y1, on):
        cr = torch.where(on, x0 * y1 - x1 * y0, z)
        for q, t in enumerate((0.5, (x0 + x1) / 6, (y0 + y1) / 6, (x0 * x0 + x0 * x1 + x1 * x1) / 12,
                               (2 * x0 * y0 + x0 * y1 + x1 * y0 + 2 * x1 * y1) / 24,
                               (y0 * y0 + y0 * y1 + y1 * y1) / 12)):
            m[q] += t * cr

    ex, ey, nx, ny = z, z, z, z
    for a in range(4):
        b = (a + 1) % 4
        ia, ib = f[a] <= 0, f[b] <= 0
        t = f[a] / torch.where(ia != ib, f[a] - f[b], torch.ones_like(z))
        cx, cy = px[a] + t * (px[b] - px[a]), py[a] + t * (py[b] - py[a])
        X0, Y0 = torch.where(ia, px[a] + z, cx), torch.where(ia, py[a] + z, cy)
        X1, Y1 = torch.where(ib, px[b] + z, cx), torch.where(ib, py[b] + z, cy)
        edge(X0, Y0, X1, Y1, ia | ib)
        out, into = ia & ~ib, ib & ~ia
        ex, ey = torch.where(out, cx, ex), torch.where(out, cy, ey)
        nx, ny = torch.where(into, cx, nx), torch.where(into, cy, ny)
    cut = ((f[0] <= 0) != (f[1] <= 0)) | ((f[1] <= 0) != (f[2] <= 0)) | ((f[2] <= 0) != (f[3] <= 0))
    edge(ex, ey, nx, ny, cut)
    return m


def _hinge(c, e):
    """Mean of max(c + e t, 0) over t uniform in [-1, 1]."""
    return torch.where(c >= e, c, torch.where(c <= -e, torch.zeros_like(c),
                                              (c + e) ** 2 / (4 * torch.where(e > 0, e, torch.ones_like(e)))))


def _sigma(c, fr, scaling):
    _, _, _, fb1, fb2, c1, c2 = fr
    u = torch.arange(c["cols"], device=DEV, dtype=torch.float64)
    v = torch.arange(c["rows"], device=DEV, dtype=torch.float64)
    if scaling == "cos":
        R2 = ((u - c1) / fb1)[None, :] ** 2 + ((v - c2) / fb2)[:, None] ** 2 + 1
        return fb1 * fb2 * R2 ** 1.5

    def corner(x, y):
        X, Y = x[None, :], y[:, None]
        return torch.atan(X * Y / torch.sqrt(X * X + Y * Y + 1))
    x0, x1, y0, y1 = (u - 0.5 - c1) / fb1, (u + 0.5 - c1) / fb1, (v - 0.5 - c2) / fb2, (v + 0.5 - c2) / fb2
    return 1.0 / (corner(x1, y1) - corner(x0, y1) - corner(x1, y0) + corner(x0, y0))


def _weights(c, fr):
    """Yields (index, weight, voxels) blocks of one view: flat pixel index and
    weight, [n3, n2, n1], for each (column piece, row) slot -- the cutting
    voxel estimate area times mean row extent over r^2, or the TT footprint."""
    s, e1, d, fb1, fb2, c1, c2 = fr
    X, Y, Z = _axes(c)
    M, N, a1, a2, a3 = c["cols"], c["rows"], c["a1"], c["a2"], c["a3"]
    rx, ry = (X - s[0])[None, :].expand(c["n2"], -1), (Y - s[1])[:, None].expand(-1, c["n1"])
    P, D = e1[0] * rx + e1[1] * ry, d[0] * rx + d[1] * ry
    corner = []
    for sx in (-0.5, 0.5):
        for sy in (-0.5, 0.5):
            corner.append((c1 + fb1 * (P + e1[0] * sx * a1 + e1[1] * sy * a2) / (D + d[0] * sx * a1 + d[1] * sy * a2),
                           D + d[0] * sx * a1 + d[1] * sy * a2))
    chi = torch.stack([q[0] for q in corner])
    ulo, uhi = torch.floor(chi.amin(0) + 0.5), torch.floor(chi.amax(0) + 0.5)
    z0, z1 = (Z - 0.5 * a3 - s[2])[:, None, None], (Z + 0.5 * a3 - s[2])[:, None, None]
    zc = (Z - s[2])[:, None, None]
    tt = c["variant"] == "tt"
    if tt:
        Dn, Df = torch.stack([q[1] for q in corner]).amin(0), torch.stack([q[1] for q in corner]).amax(0)
        t = chi.sort(0).values
        amp = torch.minimum(a1 / rx.abs(), a2 / ry.abs()) * torch.sqrt(rx ** 2 + ry ** 2 + zc ** 2)

    def trapezoid(x, v):
        def h(a, b):
            return _hinge(x - 0.5 * (a + b), 0.5 * (b - a))
        return h(v[0], v[1]) - h(v[2], v[3])
    for p in range(int((uhi - ulo).max()) + 1):
        u = ulo + p
        ok = (u <= uhi) & (u >= 0) & (u < M)
        if tt:
            F1 = trapezoid(u + 0.5, t) - trapezoid(u - 0.5, t)
            ax = torch.stack(torch.broadcast_tensors(c2 - fb2 * z1 / Dn, c2 - fb2 * z1 / Df, c2 - fb2 * z0 / Dn,
                                                     c2 - fb2 * z0 / Df)).sort(0).values
            vlo, vhi = torch.floor(ax[0] + 0.5), torch.floor(ax[3] + 0.5)
        else:
            lo = _clip(a1 / 2, a2 / 2, (fb1 * e1[0] - (u - 0.5 - c1) * d[0]) / D,
                       (fb1 * e1[1] - (u - 0.5 - c1) * d[1]) / D, c1 + fb1 * P / D - (u - 0.5))
            hi = _clip(a1 / 2, a2 / 2, (fb1 * e1[0] - (u + 0.5 - c1) * d[0]) / D,
                       (fb1 * e1[1] - (u + 0.5 - c1) * d[1]) / D, c1 + fb1 * P / D - (u + 0.5))
            A, Sx, Sy, Sxx, Sxy, Syy = (h - q for h, q in zip(hi, lo))
            ok = ok & (A > 1e-12 * a1 * a2)
            A = torch.where(ok, A, torch.ones_like(A))
            cx, cy = Sx / A, Sy / A
            var = (d[0] ** 2 * (Sxx / A - cx * cx) + 2 * d[0] * d[1] * (Sxy / A - cx * cy)
                   + d[1] ** 2 * (Syy / A - cy * cy)).clamp(min=0)
            Du = D + d[0] * cx + d[1] * cy
            h = torch.sqrt(3 * var) if c["ec"] else torch.zeros_like(var)
            ends = [c2 - fb2 * z / q for z in (z0, z1) for q in (Du - h, Du + h)]
            vlo = torch.floor(torch.stack(ends).amin(0) + 0.5)
            vhi = torch.floor(torch.stack(ends).amax(0) + 0.5)
            R2 = (rx + cx) ** 2 + (ry + cy) ** 2

        def below(v):
            # mean x3 extent of the voxel above the plane of row boundary v - 1/2 ... per unit depth box
            zt = -(v - 0.5 - c2) / fb2 * Du
            e = ((v - 0.5 - c2) / fb2 * h).abs()
            return _hinge(zt - z0, e) - _hinge(zt - z1, e)
        for r in range(int((vhi - vlo).max()) + 1):
            v = vlo + r
            on = ok & (v <= vhi) & (v >= 0) & (v < N)
            if tt:
                w = F1 * amp * (trapezoid(v + 0.5, ax) - trapezoid(v - 0.5, ax))
            else:
                w = A * (below(v) - below(v + 1))
                if c["variant"] == "exact":
                    top, bot = -(v - 0.5 - c2) / fb2 * Du, -(v + 0.5 - c2) / fb2 * Du
                    zb = 0.5 * (torch.maximum(z0, bot) + torch.minimum(z1, top))
                    w = w / (R2 + torch.minimum(torch.maximum(zb, z0), z1) ** 2)
                else:
                    w = w / (rx ** 2 + ry ** 2 + zc ** 2)
            on = on.expand_as(w)
            idx = torch.where(on, v * M + u, torch.zeros_like(w)).long()
            yield idx, torch.where(on, w, torch.zeros_like(w))


def _apply(c, x=None, b=None, views=None):
    """(A x, A^T b) over `views` in 64 bits; A x for the other views is 0."""
    frames = _frames(c)
    npx = c["rows"] * c["cols"]
    Ax = torch.zeros((c["views"], npx), device=DEV, dtype=torch.float64) if x is not None else None
    Atb = torch.zeros((c["n3"], c["n2"], c["n1"]), device=DEV, dtype=torch.float64) if b is not None else None
    for v in range(c["views"]) if views is None else views:
        sg = 1.0 if c["variant"] == "tt" else _sigma(c, frames[v], c["scaling"]).reshape(-1)
        sb = (sg * b[v].double().reshape(-1)) if b is not None else None
        for idx, w in _weights(c, frames[v]):
            if x is not None:
                Ax[v].index_add_(0, idx.reshape(-1), (w * x).reshape(-1))
            if b is not None:
                Atb += w * sb[idx]
        if x is not None:
            Ax[v] *= sg
    return (None if x is None else Ax.reshape(c["views"], c["rows"], c["cols"])), Atb


def _conv64(x, w, b=None, relu=True):
    """3x3x3 convolution, zero padding: x [D, H, W, Ci], w [27, Co, Ci]."""
    D, H, W, ci = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    y = 0
    for t in range(27):
        z, r, q = t // 9, t // 3 % 3, t % 3
        y = y + (p[z:z + D, r:r + H, q:q + W].reshape(-1, ci) @ w[t].t()).reshape(D, H, W, -1)
    y = y if b is None else y + b
    return y.clamp(min=0) if relu else y


def _net64(P, x1, x2):
    def conv(n, x):
        return _conv64(x, P[n][0], P[n][1])

    def pool(x):
        D, H, W, C = x.shape
        return x.reshape(D // 2, 2, H // 2, 2, W // 2, 2, C).mean((1, 3, 5))

    def up(x):
        return x.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)
    x = torch.zeros(tuple(x1.shape) + (16,), device=DEV, dtype=torch.float64)
    x[..., 0], x[..., 1] = 100.0 * x1, 100.0 * x2
    s1 = conv("c1b", conv("c1a", x))
    s2 = conv("c2b", conv("c2a", pool(s1)))
    y = conv("u2", up(conv("c3b", conv("c3a", pool(s2)))))
    y = conv("d2b", conv("d2a", torch.cat([y, s2], -1)))
    y = conv("u1", up(y))
    y = conv("d1b", conv("d1a", torch.cat([y, s1], -1)))
    return x2 + (y @ P["head"][0] + P["head"][1]) / 100.0


def exact(case, seed):
    k = case["kind"]
    if k in ("operators", "cgls", "ossart"):
        applications = {"operators": 1, "cgls": 1 + case.get("iters", 0), "ossart": 2}[k]
        if applications * _voxel_views(case) > 1.2 * EXACT_LIMIT:
            return None
        if k == "operators":
            x, b = _phantom(case, seed), _uniform((case["views"], case["rows"], case["cols"]), seed)
            return _apply(case, x.double(), b)
        b = _measured(case, seed).double()
        if k == "cgls":
            x = torch.zeros((case["n3"], case["n2"], case["n1"]), device=DEV, dtype=torch.float64)
            r = b
            s = _apply(case, b=r)[1]
            p, gam = s.clone(), (s * s).sum()
            for _ in range(case["iters"]):
                q = _apply(case, x=p)[0]
                al = gam / (q * q).sum()
                x = x + al * p
                r = r - al * q
                s = _apply(case, b=r)[1]
                g2 = (s * s).sum()
                p, gam = s + g2 / gam * p, g2
            return x, s
        T = case["subsets"]
        x = torch.zeros((case["n3"], case["n2"], case["n1"]), device=DEV, dtype=torch.float64)
        one_x, one_b = torch.ones_like(x), torch.ones_like(b)

        def ratio(n, m):
            return torch.where(m != 0, n / torch.where(m != 0, m, torch.ones_like(m)), torch.zeros_like(n))
        for t in range(T):
            vs = range(t, case["views"], T)
            R, C = _apply(case, one_x, one_b, vs)
            Ax = _apply(case, x=x, views=vs)[0]
            x = x + ratio(_apply(case, b=ratio(b - Ax, R), views=vs)[1], C)
        return x
    if k == "batch":
        cs = _batch_members(case)
        if sum(_voxel_views(c) for c in cs) > EXACT_LIMIT:
            return None
        got = [_apply(c, _phantom(c, seed + q).double(), _uniform((c["views"], c["rows"], c["cols"]), seed + q))
               for q, c in enumerate(cs)]
        return [g[0] for g in got], [g[1] for g in got]
    if k == "conv":
        x, w, bias, dy = (t.double() for t in _conv_inputs(case, seed))
        D, H, W, ci = x.shape
        y = _conv64(x, w, bias)
        dx = _conv64(dy, w.flip(0).transpose(1, 2), relu=False)
        p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
        g = dy.reshape(-1, case["co"]).t().contiguous()
        dw = torch.stack([g @ p[t // 9:t // 9 + D, t // 3 % 3:t // 3 % 3 + H, t % 3:t % 3 + W].reshape(-1, ci)
                          for t in range(27)])
        return y, dx, dw, dy.sum((0, 1, 2))
    P, x1, x2, t = _net_inputs(case, seed)
    P = {n: (w.bfloat16().double() if n != "head" else w.double(), b.double()) for n, (w, b) in P.items()}
    x1, x2, t = x1.double(), x2.double(), t.double()
    if k == "unet_forward":
        with torch.no_grad():
            return _net64(P, x1, x2)
    for w, b in P.values():
        w.requires_grad_(True)
        b.requires_grad_(True)
    x0 = _net64(P, x1, x2)
    loss = ((x0 - t) ** 2).mean()
    loss.backward()
    return dict(x0=x0.detach(), loss=loss.detach().reshape(1), gw=[P[n][0].grad for n, _, _ in LAYERS],
                gb=[P[n][1].grad for n, _, _ in LAYERS], ghead=torch.cat([P["head"][0].grad, P["head"][1].grad]))
