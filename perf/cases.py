"""The work that users of this library have it do, as measurable cases.

Every case goes through the public entry points as a program calls them: a
plan made once, gradients (or velocities, or network activations) on the GPU,
one call per pass.  A case is a dict of plain values; ``kind`` names the path:

* ``solve``   Algorithm 1 on one grid (``Plan.solve``): 2-D and 3-D, with and
  without missing data, FP32 and FP64, both schemes; to a tolerance, or for a
  fixed number of outer steps where the whole solve takes longer than a pass
  should (every outer step does the same work, so its time is the solve's
  time over the number of steps).
* ``flowsolve``  one snapshot of a velocity sequence: the source field from
  velocity (``pi_flow_source``), then its solve.
* ``flow``    the velocity-to-source stage alone.
* ``guess``   the coarse-grid warm start (``WarmStart.guess``): block means,
  the coarse solve with the fixed-point variant, upsampling.
* ``batch``   many uneven grids in one call (``solve_batched``).
* ``conv``    one decoder stage of the warm-start network, forward.
* ``convbwd`` one convolution of that network, backward: ReLU mask, weight and
  bias gradients, data gradient.

Inputs are Gaussian pressure wells (the solver's own recipes' fields) with
their exact gradients and seeded noise, Taylor and ABC flows, and normal
network activations and weights.
"""

import math
import random

import torch

import paper_2311_16935_amd as pi
from paper_2311_16935_amd import flow as pf
from paper_2311_16935_amd import unet as U
from paper_2311_16935_amd.warmstart import NEG3, TAPS3, UP8, ZERO1, WarmStart

DEV = "cuda:0"
BF16 = torch.bfloat16


# --------------------------------------------------------------------------- cases
def _solve(nx, ny, nz=1, **kw):
    c = dict(kind="solve", nx=nx, ny=ny, nz=nz, field="wells", noise=0.05, mask=0.0, fp64=False, cell=False,
             variant=False, tune=False, tol=1e-6, outer=10**7)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest configuration: 64^2 sin/cos field, 5 % noise, a whole solve; latency and launches
        dict(_solve(64, 64, field="sincos"), name="sin64"),
        # one snapshot of the 101^2 Taylor-vortex sequence, velocity to pressure (odd sides)
        dict(kind="flowsolve", nx=101, ny=101, tol=1e-6, name="taylor101"),
        # a planar PIV field with missing data in the paper's own precision, ragged sides
        dict(_solve(386, 301, mask=0.05, fp64=True, tol=0.0, outer=60), name="piv386"),
        # the 2-D configuration: 2048^2, 10 % noise, 5 % missing, autotuned; 40 of its outer steps
        dict(_solve(2048, 2048, mask=0.05, noise=0.10, tune=True, tol=0.0, outer=40), name="lamb2048"),
        # the same field in the cell-centred scheme
        dict(_solve(2048, 2048, mask=0.05, noise=0.10, cell=True, tune=True, tol=0.0, outer=40), name="cell2048"),
        # the headline volume, 256^3, autotuned; 40 of its outer steps
        dict(_solve(256, 256, 256, tune=True, tol=0.0, outer=40), name="blobs256"),
        # the largest volume, 500^3, autotuned; 10 of its outer steps
        dict(_solve(500, 500, 500, tune=True, tol=0.0, outer=10), name="blobs500"),
        # the coarse-grid warm start of a 256^3 solve (coarse grid 128^3), solved well below the fine tolerance
        dict(kind="guess", nx=256, ny=256, nz=256, factor=2, tol=1e-8, name="coarse256"),
        # an uneven batch of the batched recipe's sides, 2-D (some with missing data) and 3-D
        dict(kind="batch", n2=24, n3=2, lo2=128, hi2=1024, lo3=64, hi3=128, sizes=4000, fp64=False, outer=24,
             name="batch26"),
        # the last decoder stage of the 128^3 network on one field: inference for a 256^3 solve
        dict(kind="conv", n=1, d=128, h=128, w=128, ch=32, name="decode128"),
        # a 64 -> 32 channel convolution of the 64^3 network, training batch of four: backward
        dict(kind="convbwd", n=4, d=64, h=64, w=64, cin=64, cout=32, name="convbwd64"),
        # the source of a 256^3 unsteady Navier-Stokes snapshot
        dict(kind="flow", model=pf.PI_FLOW_NS, nx=256, ny=256, nz=256, steady=False, stress=False, name="flow256"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sides(rng, lo, hi, nd):
    """nd sides around one size of the range, within a factor of 1.5 of each other; one in three a multiple of 4."""
    s = _log(rng, lo, hi)
    out = [max(lo, min(hi, int(s * rng.uniform(0.8, 1.25)))) for _ in range(nd)]
    if rng.random() < 0.34:
        out[0] = max(4, out[0] // 4 * 4)
    return out


def draw(rng):
    kind = rng.choice(["solve2", "solve2", "solve3", "solve3", "cell", "flowsolve", "flow", "guess", "batch", "conv",
                       "convbwd"])
    if kind in ("solve2", "cell"):
        nx, ny = _sides(rng, 32, 2000, 2)
        fp64 = rng.random() < 0.3
        # small fields are solved to their tolerance, larger ones for a number of outer steps
        whole = nx * ny < 20000 and kind == "solve2" and rng.random() < 0.5
        return _solve(nx, ny, mask=rng.choice([0.0, 0.05]), fp64=fp64, cell=kind == "cell",
                      noise=rng.choice([0.05, 0.10]), tol=1e-6 if whole else 0.0,
                      outer=10**7 if whole else rng.randint(10, 40))
    if kind == "solve3":
        nx, ny, nz = _sides(rng, 16, 300, 3)
        return _solve(nx, ny, nz, mask=rng.choice([0.0, 0.0, 0.05]), fp64=rng.random() < 0.25,
                      tune=nx * ny * nz > 4_000_000, tol=0.0, outer=rng.randint(10, 30))
    if kind == "flowsolve":
        nx, ny = _sides(rng, 48, 160, 2)
        return dict(kind="flowsolve", nx=nx, ny=ny, tol=1e-6)
    if kind == "flow":
        nd3 = rng.random() < 0.6
        nx, ny, nz = _sides(rng, 24, 320, 3) if nd3 else _sides(rng, 64, 2048, 2) + [1]
        model = rng.choice([pf.PI_FLOW_NS, pf.PI_FLOW_NS, pf.PI_FLOW_RANS, pf.PI_FLOW_COMPRESSIBLE])
        return dict(kind="flow", model=model, nx=nx, ny=ny, nz=nz, steady=rng.random() < 0.3,
                    stress=rng.random() < 0.7)
    if kind == "guess":
        f = rng.choice([2, 2, 4])
        nx, ny, nz = (f * max(8, v // f) for v in _sides(rng, 48, 224, 3))
        return dict(kind="guess", nx=nx, ny=ny, nz=nz, factor=f, tol=1e-8)
    if kind == "batch":
        lo = _log(rng, 32, 256)
        return dict(kind="batch", n2=rng.randint(3, 24), n3=rng.randint(0, 3), lo2=lo, hi2=min(1024, 4 * lo), lo3=16,
                    hi3=96, sizes=rng.randint(1, 10**6), fp64=rng.random() < 0.25, outer=rng.randint(10, 30))
    if kind == "conv":
        ch = rng.choice([32, 32, 64, 128])
        d, h, w = (max(4, v // 2 * 2) for v in _sides(rng, 8, 3072 // ch, 3))
        return dict(kind="conv", n=rng.randint(1, 3), d=d, h=h, w=w, ch=ch)
    cin, cout = rng.choice([(4, 32), (32, 32), (64, 32), (32, 64), (64, 64), (128, 64), (128, 128), (256, 256)])
    d, h, w = _sides(rng, 8, 64 if cin * cout <= 4096 else 32, 3)
    return dict(kind="convbwd", n=rng.randint(1, 4), d=d, h=h, w=w, cin=cin, cout=cout)


# --------------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7FFFFFFF)


def _dims(c):
    return (c["nx"], c["ny"]) if c["nz"] == 1 else (c["nx"], c["ny"], c["nz"])


def _wells(dims, rng, dtype, count=16):
    """Gradient of a sum of Gaussian wells on the unit box, per component in storage order."""
    nd = len(dims)
    x = [(torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) / n for n in dims]
    shape = tuple(reversed(dims))
    g = [torch.zeros(shape, dtype=dtype, device=DEV) for _ in dims]
    for _ in range(count):
        s, amp = rng.uniform(0.03, 0.15), rng.gauss(0.0, 1.0)
        e, de = [], []
        for a in range(nd):
            t = x[a] - rng.random()
            ea = torch.exp(-t * t / (2 * s * s))
            view = [1] * nd
            view[nd - 1 - a] = dims[a]
            e.append(ea.to(dtype).view(view))
            de.append((-t / (s * s) * ea).to(dtype).view(view))
        for a in range(nd):
            f = [de[b] if b == a else e[b] for b in range(nd)]
            outer = f[0] * f[1] * amp
            if nd == 3:
                g[a].addcmul_(outer.expand(shape), f[2].expand(shape))
            else:
                g[a].add_(outer)
    return g


def _noise(g, level, gen):
    rms = math.sqrt(sum(float(x.double().square().mean()) for x in g))
    for x in g:
        x.add_(torch.randn(x.shape, generator=gen, device=DEV, dtype=torch.float32).to(x.dtype), alpha=level * rms)
    return g


def _disks(dims, rng, frac):
    """Missing data: disks (balls) until the fraction is reached; 1 = data, on the host."""
    shape = tuple(reversed(dims))
    m = torch.ones(shape, dtype=torch.uint8)
    small, total, nd = min(dims), m.numel(), len(dims)
    lo, hi = (0.01, 0.04) if nd == 2 else (0.03, 0.1)
    missing = 0
    for _ in range(400):
        if missing >= frac * total:
            break
        r = max(1.0, rng.uniform(lo, hi) * small)
        c = [rng.random() * n for n in dims]
        a = [max(0, int(c[k] - r)) for k in range(nd)]
        b = [min(dims[k], int(c[k] + r) + 2) for k in range(nd)]
        box = m[tuple(slice(a[k], b[k]) for k in reversed(range(nd)))]
        d2 = 0.0
        for k in range(nd):
            t = (torch.arange(a[k], b[k], dtype=torch.float64) + 0.5 - c[k]) ** 2
            view = [1] * nd
            view[nd - 1 - k] = t.numel()
            d2 = d2 + t.view(view)
        hit = (d2 <= r * r).to(torch.uint8)
        missing += int((hit * box).sum())
        box.mul_(1 - hit)
    return m


def _field(dims, seed, dtype, noise, mask_frac, kind="wells"):
    rng, gen = random.Random(seed), _gen(seed)
    if kind == "sincos":
        h = 1.0 / dims[0]
        x = ((torch.arange(dims[0], device=DEV, dtype=torch.float64) + 0.5) * h).view(1, -1)
        y = ((torch.arange(dims[1], device=DEV, dtype=torch.float64) + 0.5) * h).view(-1, 1)
        k = 2 * math.pi
        g = [h * k * torch.cos(k * x) * torch.cos(k * y), -h * k * torch.sin(k * x) * torch.sin(k * y)]
        g = [t.to(dtype).contiguous() for t in g]
    else:
        g = _wells(dims, rng, dtype)
    _noise(g, noise, gen)
    mask = _disks(dims, rng, mask_frac) if mask_frac > 0 else None
    if mask is not None:
        bad = (mask == 0).to(DEV)
        for t in g:
            t[bad] = float("nan")
    return g, mask


def _spacing(c, dims):
    return (1.0,) * len(dims) if c.get("field") == "sincos" else tuple(1.0 / n for n in dims)


def _taylor(c, seed):
    """Snapshots at t - dt, t, t + dt of the decaying Taylor vortex on [-3, 3]^2 (nu = rho = 1), t from the seed."""
    t0, dt = 0.05 + 0.25 * random.Random(seed).random(), 1e-3
    hx, hy = 6.0 / c["nx"], 6.0 / c["ny"]
    x = (-3 + (torch.arange(c["nx"], device=DEV, dtype=torch.float64) + 0.5) * hx).view(1, -1)
    y = (-3 + (torch.arange(c["ny"], device=DEV, dtype=torch.float64) + 0.5) * hy).view(-1, 1)

    def at(t):
        w = torch.exp(-(x * x + y * y) / (4 * t)) / (8 * math.pi * t * t)
        return [(-y * w).float().contiguous(), (x * w).float().contiguous()]

    return [at(t) for t in (t0 - dt, t0, t0 + dt)], dt, (hx, hy)


def _velocity(c, seed):
    """A smooth velocity, two neighbouring snapshots, and stresses of a plausible size."""
    rng, gen, dims = random.Random(seed), _gen(seed), _dims(c)
    shape, nd = tuple(reversed(dims)), len(dims)
    ax = []
    for a in range(nd):
        view = [1] * nd
        view[nd - 1 - a] = dims[a]
        ax.append((2 * math.pi * (torch.arange(dims[a], device=DEV, dtype=torch.float64) + 0.5) / dims[a]).view(view))
    ph = [rng.uniform(0, 2 * math.pi) for _ in range(2 * nd)]

    def snap(s):
        return [(s * (torch.sin(ax[(a + 1) % nd] + ph[a]) + 0.8 * torch.cos(ax[(a + 2) % nd] + ph[nd + a]))
                 ).float().expand(shape).contiguous() for a in range(nd)]

    u = snap(1.0)
    for t in u:
        t.add_(torch.randn(shape, generator=gen, device=DEV), alpha=0.01)
    R = None
    if c["stress"] and c["model"] != pf.PI_FLOW_NS:
        R = [0.05 * torch.rand(shape, generator=gen, device=DEV) for _ in range(3 if nd == 2 else 6)]
    return u, snap(1.0005), snap(0.9995), R, tuple(2 * math.pi / n for n in dims)


_GAS = dict(gas_R=287.0, gamma=1.4, T_inf=160.0, M_inf=0.4, V_inf=2.0)


def _batch_shapes(c):
    rng = random.Random(c["sizes"])
    out = [(rng.randint(c["lo2"], c["hi2"]), rng.randint(c["lo2"], c["hi2"])) for _ in range(c["n2"])]
    masks = [rng.choice([0.0, 0.04]) for _ in out]
    out3 = [tuple(rng.randint(c["lo3"], c["hi3"]) for _ in range(3)) for _ in range(c["n3"])]
    return list(zip(out, masks)) + [(d, 0.0) for d in out3]


def _act(shape, gen, relu):
    x = torch.randn(shape, generator=gen, device=DEV)
    return (x.relu_() if relu else x).to(BF16)


def _weights(taps, cin, cout, gen):
    """Layer weights [tap][cin][cout] in BF16 with the He scale, and their per-tap transposes."""
    w = (torch.randn((taps, cin, cout), generator=gen, device=DEV) * math.sqrt(2.0 / (taps * cin))).to(BF16)
    return w.contiguous(), w.transpose(1, 2).contiguous()


def prepare(case, seed):
    c, k = case, case["kind"]
    if k == "solve":
        dims = _dims(c)
        dtype = torch.float64 if c["fp64"] else torch.float32
        g, mask = _field(dims, seed, dtype, c["noise"], c["mask"], c["field"])
        plan = pi.Plan(dims, _spacing(c, dims), mask=mask, fp64=c["fp64"], cell_centered=c["cell"],
                       fixed_point=c["variant"])
        if c["tune"]:
            plan.autotune()
        return dict(kind=k, plan=plan, g=g, P=torch.empty(plan.shape, dtype=dtype, device=DEV), tol=c["tol"],
                    outer=c["outer"])
    if k == "flowsolve":
        (um, u, up), dt, h = _taylor(c, seed)
        plan = pi.Plan((c["nx"], c["ny"]), h)
        return dict(kind=k, plan=plan, um=um, u=u, up=up, dt=dt, h=h, f=[torch.empty_like(t) for t in u],
                    P=torch.empty(plan.shape, dtype=torch.float32, device=DEV), tol=c["tol"])
    if k == "flow":
        u, up, un, R, h = _velocity(c, seed)
        kw = dict(R=R)
        if c["model"] == pf.PI_FLOW_NS:
            kw = dict(mu=0.5) if c["steady"] else dict(mu=0.5, u_prev=up, u_next=un, dt=1e-3)
        elif c["model"] == pf.PI_FLOW_COMPRESSIBLE:
            kw.update(_GAS)
        return dict(kind=k, model=c["model"], u=u, h=h, kw=kw, f=[torch.empty_like(t) for t in u])
    if k == "guess":
        dims = _dims(c)
        g, _ = _field(dims, seed, torch.float32, 0.05, 0.0)
        plan = pi.Plan(dims, tuple(1.0 / n for n in dims))
        ws = WarmStart(None, c["factor"], coarse=True, coarse_tol=c["tol"])
        P = torch.empty(plan.shape, dtype=torch.float32, device=DEV)
        ws.guess(plan, g, P)  # a program's first guess makes the coarse plan that the later ones use
        return dict(kind=k, plan=plan, ws=ws, g=g, P=P)
    if k == "batch":
        dtype = torch.float64 if c["fp64"] else torch.float32
        plans, grads, Ps = [], [], []
        for i, (dims, frac) in enumerate(_batch_shapes(c)):
            g, mask = _field(dims, seed * 1000 + i, dtype, 0.05, frac)
            plans.append(pi.Plan(dims, tuple(1.0 / n for n in dims), mask=mask, fp64=c["fp64"]))
            grads.append(g)
            Ps.append(torch.empty(plans[-1].shape, dtype=dtype, device=DEV))
        return dict(kind=k, plans=plans, g=grads, P=Ps, outer=c["outer"])
    gen = _gen(seed)
    if k == "conv":
        n, d, h, w, ch = c["n"], c["d"], c["h"], c["w"], c["ch"]
        cat = torch.zeros((n, d, h, w, 2 * ch), dtype=BF16, device=DEV)
        cat[..., ch:] = _act((n, d, h, w, ch), gen, True)
        wu, wut = _weights(8, 2 * ch, ch, gen)
        wa, wat = _weights(27, 2 * ch, ch, gen)
        wb, wbt = _weights(27, ch, ch, gen)
        z = lambda: torch.zeros((n, d, h, w, ch), dtype=BF16, device=DEV)  # noqa: E731
        return dict(kind=k, src=_act((n, d // 2, h // 2, w // 2, 2 * ch), gen, True), cat=cat, wu=wu, wut=wut, wa=wa,
                    wat=wat, wb=wb, wbt=wbt, ba=0.1 * torch.randn(ch, generator=gen, device=DEV),
                    bb=0.1 * torch.randn(ch, generator=gen, device=DEV), ua=z(), ub=z(), m=(d, h, w), ch=ch)
    n, d, h, w, cin, cout = c["n"], c["d"], c["h"], c["w"], c["cin"], c["cout"]
    wl, _ = _weights(27, cin, cout, gen)
    work = U.pu_wgrad_work_floats(27, cin, cout, n * d * h * w)
    return dict(kind=k, x=_act((n, d, h, w, cin), gen, True), y=_act((n, d, h, w, cout), gen, True),
                g=_act((n, d, h, w, cout), gen, False), w=wl, m=(d, h, w),
                dw=torch.empty(27 * cin * cout, dtype=torch.float32, device=DEV),
                db=torch.empty(cout, dtype=torch.float32, device=DEV),
                gx=torch.empty((n, d, h, w, cin), dtype=BF16, device=DEV),
                work=torch.empty(work, dtype=torch.float32, device=DEV))


# --------------------------------------------------------------------------- one pass
def run(state):
    s, k = state, state["kind"]
    if k == "solve":
        return s["plan"].solve(s["g"], P=s["P"], tol=s["tol"], max_iter=s["outer"]).P
    if k == "flowsolve":
        f = pf.pi_flow_source(pf.PI_FLOW_NS, s["u"], s["h"], out=s["f"], u_prev=s["um"], u_next=s["up"], rho=1.0,
                              mu=1.0, dt=s["dt"])
        return f + [s["plan"].solve(f, P=s["P"], tol=s["tol"]).P]
    if k == "flow":
        return pf.pi_flow_source(s["model"], s["u"], s["h"], out=s["f"], **s["kw"])
    if k == "guess":
        return s["ws"].guess(s["plan"], s["g"], s["P"])
    if k == "batch":
        return pi.solve_batched(s["plans"], s["g"], s["P"], tol=0.0, max_iter=s["outer"])[1]
    T = U.tensor
    if k == "conv":
        ch, m = s["ch"], s["m"]
        half = tuple(v // 2 for v in m)
        for q, oo in enumerate(UP8):
            U.pu_conv(T(s["src"]), s["wut"][q], 1, ZERO1, None, T(s["cat"], 0, ch), half, 1, 2, oo)
        U.pu_conv(T(s["cat"]), s["wat"], 27, TAPS3, s["ba"], T(s["ua"]), m, relu=True)
        U.pu_conv(T(s["ua"]), s["wbt"], 27, TAPS3, s["bb"], T(s["ub"]), m, relu=True)
        return [s["cat"], s["ua"], s["ub"]]
    U.pu_relu_backward(T(s["y"]), T(s["g"]))
    U.pu_conv_wgrad(T(s["x"]), T(s["g"]), 27, TAPS3, s["dw"], s["db"], s["m"], 1, 1, (0, 0, 0), s["work"])
    U.pu_conv(T(s["g"]), s["w"], 27, NEG3, None, T(s["gx"]), s["m"])
    return [s["g"], s["dw"], s["db"], s["gx"]]


# --------------------------------------------------------------------------- what a pass cannot do without
def _inner(dims):
    lg = max(1, math.ceil(math.log2(max(dims))))
    return min(24, max(4, 3 * lg - 12)) if len(dims) == 3 else min(32, max(4, 4 * lg - 24))


def _solve_work(dims, fp64, outer, masked, inner=None):
    """Gradients, mask and field once.  The vectors of an inner iteration (residual, direction, correction) and of
    an outer step (field, source) count where the iteration's do not fit on the chip (about 160 MB of registers and
    LDS): then each is read and written once per iteration.  Operations: stencil, three updates, four dot products."""
    n = math.prod(dims)
    t = 8 if fp64 else 4
    inner = _inner(dims) if inner is None else inner
    by = n * (t * (len(dims) + 1) + (1 if masked else 0))
    if n * 3 * t > 160e6:
        by += n * outer * (inner * 6 * t + 24)
    return {"bytes": by, "flops": n * outer * (inner * (14 + 4 * len(dims)) + 20)}


def work(case):
    c, k = case, case["kind"]
    if k == "solve":
        dims = _dims(c)
        # about 16 outer steps per cell of the longest side to 1e-6
        return _solve_work(dims, c["fp64"], min(c["outer"], 16 * max(dims)), c["mask"] > 0)
    if k == "flowsolve":
        w = _solve_work((c["nx"], c["ny"]), False, 10 * max(c["nx"], c["ny"]), False)
        return {"bytes": w["bytes"] + 24 * c["nx"] * c["ny"], "flops": w["flops"]}
    if k == "flow":
        dims = _dims(c)
        n, nd = math.prod(dims), len(dims)
        arrays = 2 * nd + (0 if c["model"] == pf.PI_FLOW_NS or not c["stress"] else 3 * (nd - 1))
        if c["model"] == pf.PI_FLOW_NS and not c["steady"]:
            arrays += 2 * nd
        return {"bytes": 4 * n * arrays, "flops": n * nd * (9 * nd + 6)}
    if k == "guess":
        dims = _dims(c)
        n, f = math.prod(dims), c["factor"]
        w = _solve_work([v // f for v in dims], False, 1, False, 7 * max(dims) // f)
        return {"bytes": 16 * n + w["bytes"], "flops": w["flops"] + 12 * n}
    if k == "batch":
        ws = [_solve_work(d, c["fp64"], c["outer"], m > 0) for d, m in _batch_shapes(c)]
        return {"bytes": sum(w["bytes"] for w in ws), "flops": sum(w["flops"] for w in ws)}
    if k == "conv":
        p, ch = c["n"] * c["d"] * c["h"] * c["w"], c["ch"]
        return {"bytes": 2 * p * (2 * ch / 8 + 2 * ch + 2 * ch) + 2 * ch * ch * (16 + 54 + 27),
                "flops": 2 * p * ch * ch * (2 + 54 + 27)}
    p, cin, cout = c["n"] * c["d"] * c["h"] * c["w"], c["cin"], c["cout"]
    return {"bytes": 2 * p * (2 * cin + 3 * cout) + 6 * 27 * cin * cout, "flops": 2 * 2 * p * 27 * cin * cout}


# --------------------------------------------------------------------------- the same in 64 bits
def _diff(v, a, h, second=False):
    """Central differences along axis a; second-order one-sided ones at its ends (n >= 4 here)."""
    n = v.shape[a]
    t = lambda i, m=1: v.narrow(a, i, m)  # noqa: E731
    if second:
        mid = t(2, n - 2) - 2 * t(1, n - 2) + t(0, n - 2)
        lo = 2 * t(0) - 5 * t(1) + 4 * t(2) - t(3)
        hi = 2 * t(n - 1) - 5 * t(n - 2) + 4 * t(n - 3) - t(n - 4)
        return torch.cat([lo, mid, hi], a) / (h * h)
    mid = t(2, n - 2) - t(0, n - 2)
    return torch.cat([-3 * t(0) + 4 * t(1) - t(2), mid, 3 * t(n - 1) - 4 * t(n - 2) + t(n - 3)], a) / (2 * h)


def _flow_exact(model, u, h, rho=1.0, mu=0.0, u_prev=None, u_next=None, dt=0.0, R=None, **gas):
    nd = len(u)
    u = [t.double() for t in u]
    ax = [nd - 1 - a for a in range(nd)]
    pos = {(0, 1): nd, (0, 2): 4, (1, 2): 5} if nd == 3 else {(0, 1): 2}
    st = lambda i, j: 0.0 if R is None else R[i if i == j else pos[(min(i, j), max(i, j))]].double()  # noqa: E731
    if model != pf.PI_FLOW_COMPRESSIBLE:
        f = []
        for i in range(nd):
            acc = sum(u[j] * _diff(u[i], ax[j], h[j]) for j in range(nd))
            if R is not None:
                acc = acc + sum(_diff(st(i, j), ax[j], h[j]) for j in range(nd))
            if u_prev is not None:
                acc = acc + (u_next[i].double() - u_prev[i].double()) / (2 * dt)
            out = -rho * acc
            if model == pf.PI_FLOW_NS:
                out = out + mu * sum(_diff(u[i], ax[j], h[j], True) for j in range(nd))
            f.append(out)
        return f
    q = 0.5 * (gas["gamma"] - 1) * gas["M_inf"] ** 2
    T = gas["T_inf"] * (1 + q * (1 - sum(t * t for t in u) / gas["V_inf"] ** 2))
    W = [[u[i] * u[j] + st(i, j) for j in range(nd)] for i in range(nd)]
    dT = [_diff(T, ax[j], h[j]) for j in range(nd)]
    RT = gas["gas_R"] * T
    A = [[W[i][j] / RT + (1.0 if i == j else 0.0) for j in range(nd)] for i in range(nd)]
    b = [-(sum(_diff(W[i][j], ax[j], h[j]) - W[i][j] / T * dT[j] for j in range(nd))) / RT for i in range(nd)]

    def det(m):
        if nd == 2:
            return m[0][0] * m[1][1] - m[0][1] * m[1][0]
        return sum(m[0][j] * (m[1][(j + 1) % 3] * m[2][(j + 2) % 3] - m[1][(j + 2) % 3] * m[2][(j + 1) % 3])
                   for j in range(3))

    # Cramer's rule
    return [det([[b[r] if j == i else A[r][j] for j in range(nd)] for r in range(nd)]) / det(A) for i in range(nd)]


def _field_exact(g, h):
    """The fixed point on a grid without missing data: sum_j a_j (P_C - P_J) = S over neighbours inside the grid,
    S from the trapezoid rule, diagonal in the cosine basis of every axis; zero mean."""
    nd = len(g)
    g = [t.double() for t in g]
    n = [g[0].shape[nd - 1 - a] for a in range(nd)]
    face = [math.prod(h[b] for b in range(nd) if b != a) for a in range(nd)]
    S, lam = torch.zeros_like(g[0]), torch.zeros_like(g[0])
    C = []
    for a in range(nd):
        ax = nd - 1 - a
        step = 0.5 * h[a] * (g[a].narrow(ax, 1, n[a] - 1) + g[a].narrow(ax, 0, n[a] - 1)) * face[a]
        S.narrow(ax, 0, n[a] - 1).sub_(step)
        S.narrow(ax, 1, n[a] - 1).add_(step)
        i = torch.arange(n[a], device=DEV, dtype=torch.float64)
        m = torch.cos(math.pi * i.view(-1, 1) * (i.view(1, -1) + 0.5) / n[a]) * math.sqrt(2.0 / n[a])
        m[0] *= math.sqrt(0.5)
        C.append(m)
        view = [1] * nd
        view[ax] = n[a]
        lam = lam + (face[a] * (2 - 2 * torch.cos(math.pi * i / n[a]))).view(view)

    def along(v, m, ax):
        return (v.movedim(ax, -1).contiguous() @ m.t().contiguous()).movedim(-1, ax).contiguous()

    for a in range(nd):
        S = along(S, C[a], nd - 1 - a)
    lam.view(-1)[0] = 1.0
    S = S / lam
    S.view(-1)[0] = 0.0
    for a in range(nd):
        S = along(S, C[a].t(), nd - 1 - a)
    return S


def _upsample_exact(v, f):
    for ax in range(v.dim()):
        n = v.shape[ax]
        if n == 1 or f == 1:
            continue
        u = (torch.arange(n * f, device=DEV, dtype=torch.float64) + 0.5) / f - 0.5
        i = u.floor().long().clamp(0, n - 2)
        view = [1] * v.dim()
        view[ax] = n * f
        t = (u - i).view(view)
        v = v.index_select(ax, i) * (1 - t) + v.index_select(ax, i + 1) * t
    return v


def _conv_exact(x, w, offs, relu=False, bias=None):
    """sum over taps of x shifted by the tap's offset times w[tap] ([cin][cout]); zero outside."""
    x, w = x.double(), w.double()
    n, d, h, wd, _ = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    out = torch.zeros((n * d * h * wd, w.shape[2]), dtype=torch.float64, device=DEV)
    for t, (dz, dy, dx) in enumerate(offs):
        v = xp[:, 1 + dz:1 + dz + d, 1 + dy:1 + dy + h, 1 + dx:1 + dx + wd]
        out.addmm_(v.reshape(out.shape[0], -1), w[t])
    if bias is not None:
        out += bias.double()
    return (out.relu_() if relu else out).view(n, d, h, wd, -1)


def exact(case, seed):
    c, k = case, case["kind"]
    if k == "batch" or (k == "solve" and (c["mask"] > 0 or c["tol"] == 0.0 or c["cell"])):
        return None  # an iterate after a number of outer steps, or a field without a closed form
    if k == "solve":
        dims = _dims(c)
        g, _ = _field(dims, seed, torch.float64 if c["fp64"] else torch.float32, c["noise"], 0.0, c["field"])
        return _field_exact(g, _spacing(c, dims))
    if k == "flowsolve":
        (um, u, up), dt, h = _taylor(c, seed)
        f = _flow_exact(pf.PI_FLOW_NS, u, h, mu=1.0, u_prev=um, u_next=up, dt=dt)
        return f + [_field_exact(f, h)]
    if k == "guess":
        dims, f = _dims(c), c["factor"]
        g, _ = _field(dims, seed, torch.float32, 0.05, 0.0)
        nx, ny, nz = (v // f for v in dims)
        g = [t.double().view(nz, f, ny, f, nx, f).mean((1, 3, 5)) for t in g]
        return _upsample_exact(_field_exact(g, tuple(f / n for n in dims)), f)
    s = prepare(c, seed)
    if k == "flow":
        return _flow_exact(c["model"], s["u"], s["h"], **s["kw"])
    if k == "conv":
        ch, (d, h, w) = s["ch"], s["m"]
        cat = s["cat"].double()
        src = s["src"].double()
        for q, (oz, oy, ox) in enumerate(UP8):
            cat[:, oz::2, oy::2, ox::2, :ch] = (src.reshape(-1, 2 * ch) @ s["wu"][q].double()).view(
                src.shape[:4] + (ch,))
        ua = _conv_exact(cat, s["wa"], TAPS3, True, s["ba"])
        return [cat, ua, _conv_exact(ua, s["wb"], TAPS3, True, s["bb"])]
    g = s["g"].double() * (s["y"].double() > 0)
    n, d, h, w, cin = s["x"].shape
    xp = torch.nn.functional.pad(s["x"].double(), (0, 0, 1, 1, 1, 1, 1, 1))
    gf = g.reshape(-1, g.shape[-1])
    dw = [xp[:, 1 + dz:1 + dz + d, 1 + dy:1 + dy + h, 1 + dx:1 + dx + w].reshape(-1, cin).t().contiguous() @ gf
          for dz, dy, dx in TAPS3]
    return [g, torch.stack(dw).reshape(-1), gf.sum(0),
            _conv_exact(g, s["w"].transpose(1, 2).contiguous(), NEG3)]
