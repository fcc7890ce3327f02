"""The work a program gives this library, as cases whose speed is measured.

A case is one pass through the public Python API: a stencil sweep, a few time steps of
one of the wave equations, or a whole adjoint gradient.  `listed()` names the cases that
are followed, `draw()` gives more of the same ranges, `prepare()` makes what a program
has in hand before the call, `run()` is the pass, `work()` its unavoidable bytes and
operations, and `exact()` the same results from plain torch in 64 bits.

Sizes are those of the repository's benchmark and tests (64^3 and 512^3 sweeps, 400^3
modelling, the 256^3 gradient) and ragged ones between them; time loops are cut to a few
steps, since every step does the same work.
"""
from __future__ import annotations

import math

import numpy as np
import torch

DEV = "cuda"
HALO = 4
# centre, k = 1..r: second derivative of order 4 (r = 2) and 8 (r = 4)
LAP = {2: (-5 / 2, 4 / 3, -1 / 12), 4: (-205 / 72, 8 / 5, -1 / 5, 8 / 315, -1 / 560)}
D1 = {2: (2 / 3, -1 / 12), 4: (4 / 5, -1 / 5, 4 / 105, -1 / 280)}
FACES = 1 | 2 | 4 | 8 | 32          # lateral faces and the bottom; the top is the free surface
ALPHA = 0.015
H, VMAX = 10.0, 4500.0 * 1.05       # metres, metres per second
DT = 0.4 * H / VMAX


# ------------------------------------------------------------------ the cases

def listed():
    sweep = dict(kind="sweep", precision="fp32", layout="aligned")
    cube = lambda n: dict(nx=n, ny=n, nz=n)
    return [
        # smallest call: one sweep of the 64^3 correctness grid; host and launch latency
        dict(sweep, name="star4-64", shape="star", radius=4, layout="packed", **cube(64)),
        # the three sweeps of the headline step at their size
        dict(sweep, name="star4-512", shape="star", radius=4, **cube(512)),
        dict(sweep, name="box2-512", shape="box", radius=2, **cube(512)),
        dict(sweep, name="box4-512", shape="box", radius=4, **cube(512)),
        # the split-precision box on the matrix cores, at the headline size
        dict(sweep, name="box4-512-bf16x3", shape="box", radius=4, **dict(cube(512),
             precision="bf16x3")),
        # an ordinary grid of odd extents, in the default layout, in the other split
        dict(sweep, name="box3-ragged-fp16x3s", shape="box", radius=3, nx=237, ny=203, nz=171,
             precision="fp16x3s", layout="packed"),
        # a stack of images: the 2-D box on every plane, odd extents
        dict(sweep, name="box2d3-stack", shape="box2d", radius=3, nx=1003, ny=701, nz=40,
             layout="packed"),
        # forward modelling of a small model: 50 steps of 64^3 in one call
        dict(kind="forward", name="forward-64", radius=4, steps=50, image=False, sponge=8,
             **cube(64)),
        # reverse-time migration's forward pass with its illumination image, 8 steps of 400^3
        dict(kind="forward", name="rtm-400", radius=4, steps=8, image=True, sponge=32,
             **cube(400)),
        # anisotropic modelling at the same size
        dict(kind="vti", name="vti-400", radius=4, steps=3, sponge=32, **cube(400)),
        dict(kind="tti", name="tti-400", radius=4, steps=2, sponge=32, **cube(400)),
        # waveform inversion: misfit, checkpointed adjoint and gradient, 256^3
        dict(kind="gradient", name="gradient-256", radius=4, steps=32, checkpoint=16, sponge=32,
             **cube(256)),
    ]


def _extents(rng, lo, hi, most):
    """Three extents spread over [lo, hi] in their logarithm, at most `most` points."""
    while True:
        n = [int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) for _ in range(3)]
        if n[0] * n[1] * n[2] <= most:
            return dict(nx=n[0], ny=n[1], nz=n[2])


def draw(rng):
    kind = rng.choice(["star", "box", "box", "split", "split", "plane", "forward", "forward", "vti",
                       "tti", "gradient"])
    layout = rng.choice(["aligned", "packed"])
    if kind == "star":
        return dict(kind="sweep", shape="star", radius=rng.choice([2, 4]), precision="fp32",
                    layout=layout, **_extents(rng, 40, 640, 512 ** 3))
    if kind == "box":
        return dict(kind="sweep", shape="box", radius=rng.choice([1, 2, 3, 4]), precision="fp32",
                    layout=layout, **_extents(rng, 40, 640, 512 ** 3))
    if kind == "split":
        return dict(kind="sweep", shape="box", radius=rng.choice([2, 3, 4]),
                    precision=rng.choice(["bf16x3", "fp16x3s"]), layout=layout,
                    **_extents(rng, 40, 640, 512 ** 3))
    if kind == "plane":
        e = _extents(rng, 100, 2000, 2 ** 27)
        e["nz"] = rng.randint(1, 64)
        return dict(kind="sweep", shape=rng.choice(["star2d", "box2d"]),
                    radius=rng.choice([2, 3, 4]), precision="fp32", layout=layout, **e)
    if kind == "gradient":
        e = _extents(rng, 24, 300, 256 ** 3)
        return dict(kind="gradient", radius=rng.choice([2, 4]), steps=rng.randint(6, 32),
                    checkpoint=rng.choice([5, 16, 50]), sponge=_sponge(e), **e)
    e = _extents(rng, 40, 480, 400 ** 3)
    radius = rng.choice([2, 4])
    if kind == "forward":
        return dict(kind=kind, radius=radius, steps=rng.randint(3, 8), image=rng.random() < 0.5,
                    sponge=_sponge(e), **e)
    return dict(kind=kind, radius=radius, steps=rng.randint(1, 3 if kind == "vti" else 2),
                sponge=_sponge(e), **e)


def _sponge(e):
    return 32 if min(e["nx"], e["ny"], e["nz"]) >= 128 else 8


# ------------------------------------------------------------------ inputs, from the seed alone

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1000003 + 17)


def _dims(case):
    return case["nz"], case["ny"], case["nx"]


def _noise(g, dims):
    """Dense [nz][ny][nx] FP32 field uniform in [-1, 1)."""
    return torch.rand(dims, generator=g, device=DEV).mul_(2.0).sub_(1.0)


def _smooth(g, dims, cells=8):
    """Dense FP32 field that varies over about `cells` cells, |values| of order one."""
    coarse = [max(2, n // cells + 2) for n in dims]
    f = torch.randn([1, 1] + coarse, generator=g, device=DEV)
    f = torch.nn.functional.interpolate(f, size=list(dims), mode="trilinear", align_corners=True)
    return f[0, 0].contiguous()


def _weights(case, seed):
    """Star weights are the Laplacian's (or, at radius 3, generic); box weights are uniform
    with the mean removed."""
    r, w = case["radius"], 2 * case["radius"] + 1
    rng = np.random.default_rng(seed + 7)
    if case["shape"].startswith("star"):
        axes = 3 if case["shape"] == "star" else 2
        if r in LAP:
            one = np.array(LAP[r][:0:-1] + LAP[r])
        else:
            one = rng.uniform(-1.0, 1.0, w)
        return np.stack([one] * axes).astype(np.float32)
    c = rng.uniform(-1.0, 1.0, (w,) * (2 if case["shape"] == "box2d" else 3))
    return (c - c.mean()).astype(np.float32)


def _velocity(g, dims):
    """Five depth layers from 1500 to 4500 m/s with a smooth 5 % perturbation."""
    nz = dims[0]
    layer = (1500.0 + 750.0 * ((5 * torch.arange(nz, device=DEV)) // nz)).view(nz, 1, 1)
    p = _smooth(g, dims, 16)
    return layer * (1.0 + 0.05 * (p / p.abs().max()))


def _ricker(nt):
    t = np.arange(nt) * DT - 0.25 / 15.0
    a = (np.pi * 15.0 * t) ** 2
    return (0.05 * (1.0 - 2.0 * a) * np.exp(-a)).astype(np.float32)


def _source(case):
    return min(5, case["nz"] - 1), case["ny"] // 2, case["nx"] // 2


def _levels(g, dims, n):
    """n pairs of consecutive levels of a smooth wavefield."""
    out = []
    for _ in range(n):
        u0 = _smooth(g, dims)
        out += [u0, u0 + 0.1 * _smooth(g, dims)]
    return out


def _inputs(case, seed):
    """Every dense input of a case (FP32, on the GPU) and its weights."""
    g, dims = _gen(seed), _dims(case)
    if case["kind"] == "sweep":
        return dict(x=_noise(g, dims), c=_weights(case, seed))
    d = dict(v=_velocity(g, dims), src=_ricker(case["steps"] + 1))
    if case["kind"] == "gradient":
        d["m"] = d.pop("v") ** 2
        d["u"] = [0.1 * u for u in _levels(g, dims, 1)]
        d["d_obs"] = _smooth(g, (case["steps"] + 1, dims[1], dims[2]))
        return d
    d["c2"] = (d.pop("v") * (DT / H)) ** 2
    if case["kind"] == "forward":
        d["u"] = _levels(g, dims, 1)
        return d
    d["u"] = _levels(g, dims, 2)
    eps = 0.15 + 0.05 * torch.tanh(_smooth(g, dims, 16))
    delta = 0.06 + 0.04 * torch.tanh(_smooth(g, dims, 16))
    d["c2"] = d["c2"] / 1.4
    if case["kind"] == "vti":
        return dict(d, a=1.0 + 2.0 * eps, b=torch.sqrt(1.0 + 2.0 * delta))
    theta = (math.pi / 8) * (1.0 + torch.tanh(_smooth(g, dims, 16)))
    phi = math.pi * (1.0 + torch.tanh(_smooth(g, dims, 16)))
    return dict(d, eps=eps, delta=delta, theta=theta, phi=phi)


# ------------------------------------------------------------------ one pass through the API

def _grid(case):
    import paper_2507_11067_amd as mms
    make = mms.Grid.aligned if case.get("layout") == "aligned" else mms.Grid
    return make(case["nx"], case["ny"], case["nz"], HALO)


def _put(grid, dense):
    t = grid.zeros(DEV)
    grid.interior(t).copy_(dense)
    return t


def prepare(case, seed):
    import paper_2507_11067_amd as mms
    grid, d, kind = _grid(case), _inputs(case, seed), case["kind"]
    s = dict(case=case, grid=grid)
    if kind == "sweep":
        return dict(s, x=_put(grid, d["x"]), out=grid.zeros(DEV), c=d["c"])
    lap, nt = LAP[case["radius"]], case["steps"] + 1
    src = torch.from_numpy(d["src"]).to(DEV)
    if kind == "gradient":
        from paper_2507_11067_amd.autograd import Problem
        prob = Problem(grid=grid, lap=lap, nt=nt, h=H, dt=DT, src=_source(case), src_dt2f=src,
                       sponge_width=case["sponge"], sponge_alpha=ALPHA, sponge_faces=FACES,
                       checkpoint_every=case["checkpoint"])
        return dict(s, problem=prob, d_obs=d["d_obs"],
                    leaves=[_put(grid, t).requires_grad_() for t in [d["m"]] + d["u"]])
    traces = torch.zeros((nt, grid.ny, grid.nx), device=DEV)
    w = mms.Wave(grid, _put(grid, d["c2"]), lap, nt, sponge_width=case["sponge"],
                 sponge_alpha=ALPHA, sponge_faces=FACES, src=_source(case), src_dt2f=src,
                 traces=traces)
    u = [_put(grid, t) for t in d["u"]]
    s.update(wave=w, traces=traces, u=u, work=[grid.zeros(DEV) for _ in range(len(u) // 2 * 3)])
    if kind == "forward" and case["image"]:
        w.set_image(torch.zeros(_dims(case), dtype=torch.float64, device=DEV),
                    torch.empty(_dims(case), device=DEV), 8)
    if kind == "vti":
        s.update(a=_put(grid, d["a"]), b=_put(grid, d["b"]))
    if kind == "tti":
        s.update(tti=mms.Tti(grid, *(_put(grid, d[k]) for k in ("eps", "delta", "theta", "phi")),
                             sigma=0.1, alpha=1.0, d1=D1[case["radius"]]))
    return s


def run(state):
    import paper_2507_11067_amd as mms
    case, kind = state["case"], state["case"]["kind"]
    if kind == "sweep":
        return mms.stencil_apply(state["x"], state["out"], state["grid"], case["shape"],
                                 case["radius"], state["c"], precision=case["precision"])
    if kind == "gradient":
        from paper_2507_11067_amd.autograd import misfit, propagate
        traces = propagate(*state["leaves"], state["problem"])
        J = misfit(traces, state["d_obs"])
        return [traces.detach(), J.detach()] + list(torch.autograd.grad(J, state["leaves"]))
    w, steps, work = state["wave"], case["steps"], state["work"]
    # the two initial levels are kept; later ones go round three buffers of each field
    first = state["u"][:2] + [work[i % 3] for i in range(steps)]
    if kind == "forward":
        w.record(0, first[0])
        w.forward(1, steps + 1, first)
        return [first[-2], first[-1], state["traces"]] + ([w.image] if case["image"] else [])
    second = state["u"][2:] + [work[3 + i % 3] for i in range(steps)]
    w.record(0, first[0])
    for n in range(1, steps + 1):
        if kind == "vti":
            w.vti_step(n, state["a"], state["b"], *first[n - 1:n + 2], *second[n - 1:n + 2])
        else:
            w.tti_step(n, state["tti"], *first[n - 1:n + 2], *second[n - 1:n + 2])
    return first[-2:] + second[-2:] + [state["traces"]]


# ------------------------------------------------------------------ unavoidable work

def work(case):
    """Bytes of each operand once per sweep or time step (a field does not fit the caches
    between two steps of the large cases), and the method's operations."""
    pts, r = case["nx"] * case["ny"] * case["nz"], case["radius"]
    star = 2 * (6 * r + 1)
    if case["kind"] == "sweep":
        w = 2 * r + 1
        taps = {"star": 6 * r + 1, "star2d": 4 * r + 1, "box": w ** 3, "box2d": w ** 2}
        return dict(bytes=8.0 * pts, flops=2.0 * pts * taps[case["shape"]])
    n, plane = case["steps"], 4.0 * case["nx"] * case["ny"] * case["steps"]
    if case["kind"] == "forward":
        # u^n, u^{n-1}, C2 read and u^{n+1} written; the image once per pass (8 B read and written)
        image = 16.0 * pts if case["image"] else 0.0
        return dict(bytes=16.0 * pts * n + plane + image, flops=(star + 7.0) * pts * n)
    if case["kind"] == "vti":
        return dict(bytes=36.0 * pts * n + plane, flops=(star + 20.0) * pts * n)
    if case["kind"] == "tti":
        return dict(bytes=44.0 * pts * n + plane, flops=(2.0 * (star + 6 * 4 * r) + 80.0) * pts * n)
    # forward and adjoint steps 16 B each, the gradient's operands u^n and the adjoint level 8 B;
    # the FP64 gradient is written once and three results come back
    return dict(bytes=(16.0 + 16.0 + 8.0) * pts * n + 3 * plane + 20.0 * pts,
                flops=(3.0 * star + 20.0) * pts * n)


# ------------------------------------------------------------------ the same results in 64 bits

def _pad(t, r):
    return torch.nn.functional.pad(t, (r,) * 6)


def _along(f, axis, weights, sign):
    """sum_k weights[k-1] (f(i+k) + sign f(i-k)) along an axis, zero outside the grid."""
    out = torch.zeros_like(f)
    for k, c in enumerate(weights, 1):
        n = f.shape[axis] - k
        if n <= 0:
            continue
        lo, hi = f.narrow(axis, 0, n), f.narrow(axis, k, n)
        out.narrow(axis, 0, n).add_(hi, alpha=c)
        out.narrow(axis, k, n).add_(lo, alpha=sign * c)
    return out


def _d2(f, axis, lap):
    return _along(f, axis, lap[1:], 1.0).add_(f, alpha=lap[0])


def _lap(f, lap):
    return _d2(f, 0, lap).add_(_d2(f, 1, lap)).add_(_d2(f, 2, lap))


def _sponge_field(case):
    def axis(n, lo, hi):
        i, f = torch.arange(n, device=DEV, dtype=torch.float64), 1.0
        for on, d in ((lo, i), (hi, n - 1 - i)):
            t = float(np.float32(ALPHA)) * (case["sponge"] - d).clamp(min=0.0)
            f = f * (torch.exp(-t * t) if on else torch.ones_like(d))
        return f
    nz, ny, nx = _dims(case)
    return (axis(nz, FACES & 16, FACES & 32).view(nz, 1, 1) *
            axis(ny, FACES & 4, FACES & 8).view(1, ny, 1) *
            axis(nx, FACES & 1, FACES & 2).view(1, 1, nx))


def _store(case, dense):
    """A dense interior in the padded layout the results come in."""
    nz, ny, nx = _dims(case)
    pitch = (nx + 3) // 4 * 4 + 2 * HALO
    if case.get("layout") == "aligned":
        pitch = (pitch + 31) // 32 * 32
    t = torch.zeros((nz + 2 * HALO, ny + 2 * HALO, pitch), dtype=torch.float64, device=DEV)
    t[HALO:HALO + nz, HALO:HALO + ny, HALO:HALO + nx] = dense
    return t


def exact(case, seed):
    d, kind, r = _inputs(case, seed), case["kind"], case["radius"]
    if kind == "sweep":
        x, c = d["x"].double(), d["c"].astype(np.float64)
        if case["shape"].startswith("star"):
            out = torch.zeros_like(x)
            axes = (0, 1, 2) if case["shape"] == "star" else (1, 2)
            for a, row in zip(axes, c):
                out.add_(_d2(x, a, [row[r]] + list(row[r + 1:])))
            return _store(case, out)
        nz, ny, nx = _dims(case)
        out, p = torch.zeros_like(x), _pad(x, r)
        for i in np.ndindex(c.shape):
            z, y, xo = ((r,) if len(i) == 2 else ()) + i
            out.add_(p[z:z + nz, y:y + ny, xo:xo + nx], alpha=float(c[i]))
        return _store(case, out)
    lap = [float(np.float32(v)) for v in LAP[r]]
    G, src, (sz, sy, sx) = _sponge_field(case), d["src"].astype(np.float64), _source(case)
    u = [t.double() for t in d["u"]]
    n_steps = case["steps"]
    if kind == "gradient":
        scale = float(np.float32((DT / H) ** 2))
        C2 = d["m"].double() * scale
        for n in range(1, n_steps + 1):
            un = G * (2 * u[n] - G * u[n - 1] + C2 * _lap(u[n], lap))
            un[sz, sy, sx] += src[n]
            u.append(un)
        traces = torch.stack([t[0] for t in u[:n_steps + 1]])
        resid = traces - d["d_obs"].double()
        J = 0.5 * (resid * resid).sum().view(1)
        l1, l2, grad = torch.zeros_like(C2), torch.zeros_like(C2), torch.zeros_like(C2)
        for n in range(n_steps, 0, -1):
            grad += scale * G * l1 * _lap(u[n], lap)
            l0 = 2 * G * l1 - G * G * l2 + _lap(C2 * G * l1, lap)
            l0[0] += resid[n]
            l1, l2 = l0, l1
        l0 = -G * G * l2
        l0[0] += resid[0]
        return [traces, J] + [_store(case, t) for t in (grad, l0, l1)]
    C2 = d["c2"].double()
    traces = [u[0][0]]
    if kind == "forward":
        image = torch.zeros_like(C2)
        for n in range(1, n_steps + 1):
            traces.append(u[1][0])
            un = G * (2 * u[1] - G * u[0] + C2 * _lap(u[1], lap))
            un[sz, sy, sx] += src[n]
            image += un * un
            u = [u[1], un]
        return ([_store(case, t) for t in u] + [torch.stack(traces)] +
                ([image] if case["image"] else []))
    p, q = u[:2], u[2:]
    if kind == "vti":
        a, b = d["a"].double(), d["b"].double()
        for n in range(1, n_steps + 1):
            traces.append(p[1][0])
            sxy, szz = _d2(p[1], 1, lap).add_(_d2(p[1], 2, lap)), _d2(q[1], 0, lap)
            pn = G * (2 * p[1] - G * p[0] + C2 * (a * sxy + b * szz))
            qn = G * (2 * q[1] - G * q[0] + C2 * (b * sxy + szz))
            for t in (pn, qn):
                t[sz, sy, sx] += src[n]
            p, q = [p[1], pn], [q[1], qn]
    else:
        d1 = [float(np.float32(v)) for v in D1[r]]
        sigma = float(np.float32(0.1))
        th, ph = d["theta"].double(), d["phi"].double()
        nx, ny, nz = th.sin() * ph.cos(), th.sin() * ph.sin(), th.cos()
        ex, ed = 1 + 2 * d["eps"].double(), 1 + 2 * d["delta"].double()

        def operators(f):
            dz, dy = _along(f, 0, d1, -1.0), _along(f, 1, d1, -1.0)
            xx, yy, zz = _d2(f, 2, lap), _d2(f, 1, lap), _d2(f, 0, lap)
            h1 = (nx * nx * xx + ny * ny * yy + nz * nz * zz +
                  2 * nx * ny * _along(dy, 2, d1, -1.0) + 2 * ny * nz * _along(dz, 1, d1, -1.0) +
                  2 * nx * nz * _along(dz, 2, d1, -1.0))
            return h1, xx + yy + zz - h1

        for n in range(1, n_steps + 1):
            traces.append(p[1][0])
            (p1, p2), (q1, q2) = operators(p[1]), operators(q[1])
            pn = G * (2 * p[1] - G * p[0] + C2 * (ex * p2 + q1 + sigma * (p1 - q1)))
            qn = G * (2 * q[1] - G * q[0] + C2 * (ed * p2 + q1 - sigma * (p2 - q2)))
            for t in (pn, qn):
                t[sz, sy, sx] += src[n]
            p, q = [p[1], pn], [q[1], qn]
    return [_store(case, t) for t in p + q] + [torch.stack(traces)]
