"""The calls this library is used for, as measurable cases.

Every case is one call of a public entry point of paper_1504_01380_amd on
inputs that are already on the GPU, with the default (untuned) settings:

* ``advance``   swept.advance of one periodic field in place: heat (float64
  and float32), Kuramoto-Sivashinsky, 1D Euler and the contraction-on forms;
* ``batch``     swept.advance_batch of many independent fields, half heat and
  half KS, of uneven sizes and step counts;
* ``window``    J = swept.WindowMeanSquare of a field and dJ/du0 (one
  gradient evaluation of an optimisation over initial fields);
* ``pullback``  swept.SweptAdvance forward and the gradient of its result's
  inner product with a given cotangent.

Sizes, step counts, parameters and input distributions are those of the
repository's own workloads (workloads.py) and tests, or lie between them.
"""
import math

import torch

import paper_1504_01380_amd as swept

DT, DX = 0.005, 0.5             # KS time step and grid spacing
GAMMA, CFL = 1.4, 0.2           # Euler gas constant and dt/dx
R = 0.25                        # heat r = dt/dx^2

# floating-point operations of one point and time step of each scheme as it is
# defined (heat: 5; KS: 2 x (4 + 9 + 2); Euler: 2 x (slopes 9, one face 66,
# update 12)), and bytes of one point's field value
FLOPS = {"heat": 5, "heat_f32": 5, "heat_fma": 5, "heat_f32_fma": 5, "ks": 30, "ks_fma": 30,
         "euler": 174}
BYTES = {"heat": 8, "heat_f32": 4, "heat_fma": 8, "heat_f32_fma": 4, "ks": 8, "ks_fma": 8,
         "euler": 24}


def listed():
    return [
        # a short call from an interactive program or a solver that couples
        # a small 1D grid to something else: latency and launches only
        dict(name="heat_call", kind="advance", stencil="heat", n=1000, nsteps=100),
        # the small heat workload: a grid far too small for the GPU, long run
        dict(name="heat_small", kind="advance", stencil="heat", n=4096, nsteps=10000),
        # the headline workload, heat on 2^24 points
        dict(name="heat_large", kind="advance", stencil="heat", n=1 << 24, nsteps=20000),
        # single precision on a mid-size grid
        dict(name="heat_f32", kind="advance", stencil="heat_f32", n=1 << 22, nsteps=5000),
        # an odd grid (a domain with both end points counted)
        dict(name="heat_odd", kind="advance", stencil="heat", n=(1 << 20) + 1, nsteps=4000),
        # KS on a small domain, as in studies of its dynamics
        dict(name="ks_small", kind="advance", stencil="ks", n=4096, nsteps=1000),
        # the KS workload (a tenth of its run)
        dict(name="ks", kind="advance", stencil="ks", n=1 << 20, nsteps=5000),
        # contraction-on KS on an even grid without a good even divisor
        # (299,998 = 2 x 149,999)
        dict(name="ks_fma_ragged", kind="advance", stencil="ks_fma", n=299998, nsteps=1000),
        # shock tubes: a small grid, and the 2^20-cell workload (a twentieth)
        dict(name="euler_small", kind="advance", stencil="euler", n=4096, nsteps=500),
        dict(name="euler", kind="advance", stencil="euler", n=1 << 20, nsteps=500),
        # the ensemble workload: an eighth of its instances, a tenth of its steps
        dict(name="ensemble", kind="batch", count=512, nmin=256, nmax=65536, smin=100, smax=2000),
        # objective and gradient of the KS adjoint workload (a tenth of its run)
        dict(name="ks_gradient", kind="window", stencil="ks", n=1 << 16, nsteps=2000, window=200),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# per stencil: the range of sizes and step counts of a drawn single-field case
_RANGES = {
    "heat": (256, 1 << 22, 64, 8000),
    "heat_f32": (256, 1 << 22, 64, 8000),
    "heat_fma": (256, 1 << 22, 64, 8000),
    "heat_f32_fma": (256, 1 << 22, 64, 8000),
    "ks": (256, 1 << 20, 32, 2000),
    "ks_fma": (256, 1 << 20, 32, 2000),
    "euler": (256, 1 << 20, 16, 500),
}


def draw(rng):
    kind = rng.choice(["advance"] * 7 + ["batch"] + ["window", "pullback"])
    if kind == "advance":
        st = rng.choice(["heat", "heat", "heat_f32", "heat_fma", "heat_f32_fma", "ks", "ks",
                         "ks_fma", "euler", "euler"])
        n0, n1, s0, s1 = _RANGES[st]
        return dict(kind=kind, stencil=st, n=_log_int(rng, n0, n1), nsteps=_log_int(rng, s0, s1))
    if kind == "batch":
        smax = _log_int(rng, 200, 2000)
        return dict(kind=kind, count=_log_int(rng, 4, 512), nmin=256,
                    nmax=_log_int(rng, 1024, 65536), smin=max(1, smax // 20), smax=smax)
    # the adjoint takes grids with an even divisor: multiples of 8
    st = rng.choice(["ks", "ks", "heat"])
    n = 8 * _log_int(rng, 32, 1 << 13)
    nsteps = _log_int(rng, 64, 2000)
    case = dict(kind=kind, stencil=st, n=n, nsteps=nsteps)
    if kind == "window":
        case["window"] = max(1, nsteps // rng.choice([4, 10, 30]))
    return case


# ---------------------------------------------------------------- inputs

def _params(stencil, n):
    if stencil.startswith("heat"):
        return [R]
    if stencil.startswith("ks"):
        return [DT, DX]
    return [CFL / n, 1.0 / n, GAMMA]


def _name(stencil):
    return {"heat_f32": "heat", "heat_f32_fma": "heat_fma"}.get(stencil, stencil)


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _ks_noise(n, g):
    """9-point periodic box filter of 0.1 N(0, 1) noise."""
    y = 0.1 * torch.randn(n, generator=g, dtype=torch.float64, device="cuda")
    acc = torch.zeros_like(y)
    for d in range(-4, 5):
        acc += torch.roll(y, -d)
    return acc / 9.0


def _sod(n, g):
    """Periodic shock tube: rho, p = (0.125, 0.1) on one half and (1, 1) on
    the other, u = 0, the low half's left end at a seeded position."""
    x = (torch.arange(n, dtype=torch.float64, device="cuda") + 0.5) / n
    at = torch.rand((), generator=g, dtype=torch.float64, device="cuda")
    low = torch.remainder(x - at, 1.0) < 0.5
    rho = torch.where(low, 0.125, 1.0).to(torch.float64)
    p = torch.where(low, 0.1, 1.0).to(torch.float64)
    return torch.stack([rho, torch.zeros_like(rho), p / (GAMMA - 1.0)], dim=1).contiguous()


def _field(stencil, n, g):
    if stencil.startswith("heat"):
        u = 2.0 * torch.rand(n, generator=g, dtype=torch.float64, device="cuda") - 1.0
        return u.float() if "f32" in stencil else u
    return _ks_noise(n, g) if stencil.startswith("ks") else _sod(n, g)


def _instances(case, seed):
    """Sizes log-uniform, steps uniform, half heat and half KS, shuffled."""
    g = torch.Generator().manual_seed(20250 + int(case["count"]) + 7 * int(seed))
    c = int(case["count"])
    lo, hi = math.log(case["nmin"]), math.log(case["nmax"])
    sizes = torch.exp(lo + (hi - lo) * torch.rand(c, generator=g, dtype=torch.float64))
    sizes = [int(v) for v in torch.round(sizes)]
    steps = torch.randint(case["smin"], case["smax"] + 1, (c,), generator=g).tolist()
    heat = torch.randperm(c, generator=g).lt(c // 2).tolist()
    return sizes, steps, ["heat" if h else "ks" for h in heat]


def prepare(case, seed):
    g = _generator(seed)
    if case["kind"] == "batch":
        # the sizes belong to the case, the values to the seed
        sizes, steps, kinds = _instances(case, 0)
        flat = 2.0 * torch.rand(sum(sizes), generator=g, dtype=torch.float64, device="cuda") - 1.0
        return dict(kind="batch", flat=flat, us=list(torch.split(flat, sizes)), steps=steps,
                    kinds=kinds, params=[[R] if k == "heat" else [DT, DX] for k in kinds])
    st, n = case["stencil"], case["n"]
    state = dict(kind=case["kind"], stencil=_name(st), nsteps=case["nsteps"],
                 params=_params(st, n))
    u = _field(st, n, g)
    if case["kind"] == "advance":
        state["u"] = u
    else:
        state["u0"] = u.requires_grad_(True)
        if case["kind"] == "window":
            state["window"] = case["window"]
        else:
            state["cot"] = torch.randn(n, generator=g, dtype=torch.float64, device="cuda")
    return state


def run(state):
    if state["kind"] == "advance":
        return swept.advance(state["u"], state["nsteps"], state["stencil"], state["params"])
    if state["kind"] == "batch":
        swept.advance_batch(state["us"], state["steps"], state["kinds"], state["params"])
        return state["flat"]
    u0 = state["u0"]
    if state["kind"] == "window":
        J = swept.WindowMeanSquare.apply(u0, state["nsteps"], state["stencil"], state["params"],
                                         state["window"])
        return {"J": J.detach(), "grad": torch.autograd.grad(J, u0)[0]}
    u = swept.SweptAdvance.apply(u0, state["nsteps"], state["stencil"], state["params"])
    return {"u": u.detach(), "grad": torch.autograd.grad(u, u0, state["cot"])[0]}


def work(case):
    if case["kind"] == "batch":
        sizes, steps, kinds = _instances(case, 0)
        return {"bytes": 16.0 * sum(sizes),
                "flops": float(sum(n * s * FLOPS[k] for n, s, k in zip(sizes, steps, kinds)))}
    st, n, s = case["stencil"], case["n"], case["nsteps"]
    if case["kind"] == "advance":
        return {"bytes": 2.0 * BYTES[st] * n, "flops": float(FLOPS[st]) * n * s}
    # forward for the value, and a reverse sweep of about twice its operations
    # beside the forward values it needs; u0 (and the cotangent) in, the
    # gradient (and the final field) out
    return {"bytes": (16.0 if case["kind"] == "window" else 32.0) * n,
            "flops": 3.0 * FLOPS[st] * n * s}


# ------------------------------------------------- the schemes in plain torch

def _d2(a, l, r):
    return (l + r) - 2.0 * a


def _heat_step(u, left, right, r):
    return u + r * _d2(u, left(u), right(u))


def _ks_step(u, left, right):
    c1, c2 = 1.0 / (2.0 * DX), 1.0 / (DX * DX)

    def rhs(a, b):
        return -(a * ((right(a) - left(a)) * c1) + b + _d2(b, left(b), right(b)) * c2)

    w = _d2(u, left(u), right(u)) * c2
    v = u + 0.5 * DT * rhs(u, w)
    z = _d2(v, left(v), right(v)) * c2
    return u + DT * rhs(v, z)


def _euler_step(q, n):
    """q: (3, n) = (rho, m, E)."""
    gm1, c = GAMMA - 1.0, (CFL / n) / (1.0 / n)

    def roll(a, d):
        return torch.roll(a, d, dims=1)

    def slope(v):
        a, b = v - roll(v, 1), roll(v, -1) - v
        s = torch.where(a.abs() < b.abs(), a, b)
        return torch.where(a * b > 0, s, torch.zeros_like(s))

    def flux(v):
        u = v[1] / v[0]
        p = gm1 * (v[2] - 0.5 * v[1] * u)
        return torch.stack([v[1], v[1] * u + p, (v[2] + p) * u]), u, (v[2] + p) / v[0]

    def diff(v, s):
        ql, qr = v + 0.5 * s, roll(v - 0.5 * s, -1)
        fl, ul, hl = flux(ql)
        fr, ur, hr = flux(qr)
        a, b = torch.sqrt(ql[0]), torch.sqrt(qr[0])
        um, hm = (a * ul + b * ur) / (a + b), (a * hl + b * hr) / (a + b)
        c2 = gm1 * (hm - 0.5 * um * um)
        lam = um.abs() + torch.sqrt(torch.clamp(c2, min=0.0))
        f = 0.5 * (fl + fr) - 0.5 * lam * (qr - ql)
        return f - roll(f, 1)

    r = q - 0.5 * c * diff(q, slope(q))
    return q - c * diff(r, slope(r))


def _left(u):
    return torch.roll(u, 1)


def _right(u):
    return torch.roll(u, -1)


def exact(case, seed):
    state = prepare(case, seed)
    if case["kind"] == "batch":
        if sum(n for n in _instances(case, 0)[0]) * case["smax"] > 4e10:
            return None
        return _exact_batch(state)
    st, n, nsteps = state["stencil"], case["n"], case["nsteps"]

    def step(u):
        return _heat_step(u, _left, _right, R) if st.startswith("heat") else \
            _ks_step(u, _left, _right)

    if case["kind"] == "advance":
        # about 25 passes over the field a heat step, 120 a KS one, 500 an Euler one
        passes = {"heat": 25, "heat_fma": 25, "ks": 120, "ks_fma": 120, "euler": 500}[st]
        if nsteps * (passes * n * 8 / 2.5e12 + passes * 2.5e-6) > 18.0:
            return None
        if st == "euler":
            q = state["u"].t().contiguous()
            for _ in range(nsteps):
                q = _euler_step(q, n)
            return q.t().contiguous()
        u = state["u"].double()
        for _ in range(nsteps):
            u = step(u)
        return u
    # gradients: reverse-mode differentiation of the plain steps, from a
    # stored field every `seg` steps
    u0 = state["u0"].detach()
    first = nsteps - case["window"] + 1 if case["kind"] == "window" else nsteps + 1
    wgt = 1.0 / (case["window"] * n) if case["kind"] == "window" else 0.0
    fields, seg = [u0], 50
    u = u0
    J = torch.zeros((), dtype=torch.float64, device="cuda")
    for j in range(1, nsteps + 1):
        u = step(u)
        if j >= first:
            J = J + wgt * (u * u).sum()
        if j % seg == 0:
            fields.append(u)
    cot = torch.zeros_like(u0) if case["kind"] == "window" else state["cot"]
    for b in range((nsteps - 1) // seg, -1, -1):
        x = fields[b].clone().requires_grad_(True)
        y, acc = x, 0.0
        for j in range(b * seg + 1, min(nsteps, (b + 1) * seg) + 1):
            y = step(y)
            if j >= first:
                acc = acc + wgt * (y * y).sum()
        cot = torch.autograd.grad((y * cot).sum() + acc, x)[0]
    return {"J": J, "grad": cot} if case["kind"] == "window" else {"u": u, "grad": cot}


def _exact_batch(state):
    """All instances at once: neighbours by index, fields that have finished
    their steps held."""
    flat = state["flat"].clone()
    sizes = [u.numel() for u in state["us"]]
    start = torch.tensor([0] + sizes[:-1], device="cuda").cumsum(0)
    size = torch.tensor(sizes, device="cuda")
    own = torch.repeat_interleave(torch.arange(len(sizes), device="cuda"), size)
    i = torch.arange(flat.numel(), device="cuda") - start[own]
    il = torch.remainder(i - 1, size[own]) + start[own]
    ir = torch.remainder(i + 1, size[own]) + start[own]
    steps = torch.tensor(state["steps"], device="cuda")[own]
    heat = torch.tensor([k == "heat" for k in state["kinds"]], device="cuda")[own]
    for which, step in ((heat, lambda u, le, ri: _heat_step(u, le, ri, R)), (~heat, _ks_step)):
        at = torch.nonzero(which).flatten()
        if not at.numel():
            continue
        place = torch.empty_like(i)
        place[at] = torch.arange(at.numel(), device="cuda")
        pl, pr, s, u = place[il[at]], place[ir[at]], steps[at], flat[at]
        for j in range(int(s.max())):
            u = torch.where(s > j, step(u, lambda a: a[pl], lambda a: a[pr]), u)
        flat[at] = u
    return flat
