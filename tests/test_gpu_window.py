"""The register-window schedule (the automatic schedule of swept_advance)
against the oracle, bit for bit, where it can go wrong: rings smaller than a
window (which then holds the ring several times over), owned parts and windows
that end on, just before or just after the ring's seam, runs of one to a few
steps (stages of zero steps), every evaluation form of heat and the
conditions that choose between them."""
import numpy as np
import pytest

import workloads
from tests.conftest import gpu_available, same_bits

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

TINY = {np.float64: 2.0 ** -1022, np.float32: 2.0 ** -126}


@pytest.fixture(scope="module")
def sw():
    import paper_1504_01380_amd as swept
    swept.init(0)
    swept.set_tuning(0, 0, swept.MODE_AUTO)
    swept.clear_tuning()
    yield swept


def run(sw, u0, nsteps, stencil, params):
    import torch
    u = torch.from_numpy(np.ascontiguousarray(u0)).to("cuda")
    sw.advance(u, nsteps, stencil, params)
    torch.cuda.synchronize()
    sw.sync()
    return u.cpu().numpy()


def same_up_to_nan(a, b):
    na, nb = np.isnan(a), np.isnan(b)
    return np.array_equal(na, nb) and same_bits(a[~na], b[~nb])


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("r", [0.25, 0.3, 0.5, 0.6])
@pytest.mark.parametrize("n,nsteps", [
    (3, 1), (3, 2), (5, 7), (31, 64), (64, 129), (127, 1), (128, 3), (257, 200), (1000, 100),
    (4095, 301), (4096, 1), (4097, 777), (65536 + 48, 150), (300000, 97), (1 << 20, 33),
])
def test_heat_bitwise(sw, oracle_mod, n, nsteps, r, dtype):
    """r = 1/4 and 1/2: the exact-product form; 0.3: the fused Laplacian;
    0.6: the operations as written."""
    u0 = workloads.white_noise(n, seed=n + nsteps, dtype=dtype)
    got = run(sw, u0, nsteps, "heat", [r])
    assert sw.last_heat_form() == (sw.FORM_FUSED if r <= 0.5 else sw.FORM_CANONICAL)
    assert same_up_to_nan(got, oracle_mod.heat(u0, nsteps, r))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_heat_tiny_values(sw, oracle_mod, dtype):
    """Values down to the subnormals: products r*lap underflow, so a window
    that holds one must not take the exact-product form; zeros may."""
    n, nsteps = 5000, 300
    u0 = workloads.white_noise(n, seed=3, dtype=dtype)
    u0[1000:1400] = (u0[1000:1400] * 4 * TINY[dtype]).astype(dtype)
    u0[3000:3500] = 0
    got = run(sw, u0, nsteps, "heat", [0.25])
    assert sw.last_heat_form() == sw.FORM_FUSED
    assert same_bits(got, oracle_mod.heat(u0, nsteps, 0.25))
    small = (workloads.white_noise(n, seed=4, dtype=dtype) * 8 * TINY[dtype]).astype(dtype)
    assert same_bits(run(sw, small, 40, "heat", [0.25]), oracle_mod.heat(small, 40, 0.25))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_heat_range_check(sw, oracle_mod, dtype):
    """A value above MAX/16 sends its windows to the operations as written and
    is reported; values of 0.4..0.6 MAX overflow there as in the oracle; the
    next call is fused again."""
    big = np.finfo(dtype).max
    u0 = workloads.white_noise(6001, seed=9, dtype=dtype)
    lim = dtype(big / 16)
    for at, form in ((lim, sw.FORM_FUSED), (np.nextafter(lim, dtype(np.inf)), sw.FORM_CANONICAL),
                     (dtype(0.55) * big, sw.FORM_CANONICAL), (dtype(np.inf), sw.FORM_FUSED),
                     (dtype(1), sw.FORM_FUSED)):
        v = u0.copy()
        v[2500:2503] = at
        got = run(sw, v, 90, "heat", [0.25])
        assert sw.last_heat_form() == form
        assert same_up_to_nan(got, oracle_mod.heat(v, 90, 0.25))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n,nsteps", [(7, 5), (999, 250), (70001, 60)])
def test_heat_fma_bitwise(sw, oracle_mod, n, nsteps, dtype):
    u0 = workloads.white_noise(n, seed=n, dtype=dtype)
    assert same_bits(run(sw, u0, nsteps, "heat_fma", [0.3]), oracle_mod.heat_fma(u0, nsteps, 0.3))


KS_P = [workloads.KS_DT, workloads.KS_DX]


@pytest.mark.parametrize("fma", [False, True])
@pytest.mark.parametrize("par", [KS_P, [0.005, 0.7], [1e-4, 0.25]])
@pytest.mark.parametrize("n,nsteps", [
    (3, 1), (3, 2), (5, 7), (33, 20), (127, 3), (128, 1), (257, 55), (1000, 100), (4097, 64),
    (65536 + 16, 41), (300000, 30), (1 << 20, 9),
])
def test_ks_bitwise(sw, oracle_mod, n, nsteps, par, fma):
    """dx = 1/2 and 1/4: the exact-product form (1/dx^2 a power of two); 0.7:
    the fused Laplacian."""
    u0 = workloads.smoothed_noise(n, seed=n + nsteps)
    got = run(sw, u0, nsteps, "ks_fma" if fma else "ks", par)
    want = (oracle_mod.ks_fma if fma else oracle_mod.ks)(u0, nsteps, *par)
    assert same_bits(got, want)


@pytest.mark.parametrize("fma", [False, True])
@pytest.mark.parametrize("par", [KS_P, [0.005, 0.7]])
def test_ks_leaves_the_fused_range(sw, oracle_mod, par, fma):
    """Zeros, subnormals and a localised pulse whose tails underflow as they
    spread (below the exact-product form's range), values that start above
    1e30, and a run that grows past it inside a stage and overflows: each as
    the oracle computes it."""
    oracle = oracle_mod.ks_fma if fma else oracle_mod.ks
    name = "ks_fma" if fma else "ks"
    n = 3000
    zero = np.zeros(n)
    pulse = zero.copy()
    pulse[1500:1520] = 0.3
    mixed = workloads.smoothed_noise(n, seed=2)
    mixed[700:900] *= 2.0 ** -1015
    mixed[1200:1210] = 0.0
    huge = workloads.smoothed_noise(n, seed=3)
    huge[50] = 3e200
    growing = workloads.smoothed_noise(n, seed=4)
    growing[2000:2003] = [3e3, -2e3, 5e3]
    inf = workloads.smoothed_noise(n, seed=5)
    inf[10] = np.inf
    for u0, nsteps in ((zero, 20), (pulse, 260), (mixed, 90), (huge, 6), (growing, 12),
                       (growing, 40), (inf, 5)):
        want = oracle(u0, nsteps, *par)
        assert same_up_to_nan(run(sw, u0, nsteps, name, par), want)
    assert not np.all(np.isfinite(oracle(growing, 40, *par)))   # the case does leave the range


@pytest.mark.parametrize("smooth", [False, True])
@pytest.mark.parametrize("n,nsteps", [
    (3, 1), (3, 2), (7, 9), (63, 3), (64, 1), (129, 25), (1000, 60), (4097, 33),
    (65536 + 16, 21), (1 << 18, 7),
])
def test_euler_bitwise(sw, oracle_mod, n, nsteps, smooth):
    q0 = workloads.euler_smooth(n, seed=n) if smooth else workloads.euler_mirrored_sod(n)
    par = [workloads.EULER_CFL / n, 1.0 / n, workloads.EULER_GAMMA]
    assert same_bits(run(sw, q0, nsteps, "euler", par), oracle_mod.euler(q0, nsteps, *par))


def euler_states(kind, n, seed):
    """Fields on both sides of the ranges the fast Euler step needs."""
    q = workloads.euler_smooth(n, seed=seed)
    g = workloads.rng(seed)
    at = slice(n // 3, n // 3 + n // 8)
    if kind == "negative_zero":          # gas at rest with m = -0.0
        q = workloads.euler_mirrored_sod(n)
        q[:, 1] = -0.0
    elif kind == "random":               # strong random jumps, many limiter branches
        q = workloads.euler_state(g.uniform(0.1, 2.0, n), g.uniform(-1, 1, n), g.uniform(0.1, 2, n))
    elif kind == "blast":
        q = workloads.euler_state(1.0, 0.0, np.where(np.arange(n) % 97 < 9, 1e4, 1e-3))
    elif kind == "tiny_momentum":        # below the range, subnormal, and zero
        q[:, 1] = 0.0
        q[at, 1] = 1e-200
        q[at.start + 3, 1], q[at.start + 5, 1] = 5e-324, -1e-310
    elif kind == "scaled_up":            # density and energy above it
        q[:, :] *= 1e60
    elif kind == "scaled_down":
        q[:, :] *= 1e-70
    elif kind == "near_vacuum":
        q[at] = workloads.euler_state(1e-35, 0.3, 1e-36)
    elif kind == "unphysical":           # negative pressure, then negative density
        q[at, 2] = 0.01 * q[at, 2]
        q[n // 2, 0] = -0.3
    elif kind == "nan":
        q[n // 2, 1] = np.nan
    elif kind == "inf":
        q[n // 2, 2] = np.inf
    return np.ascontiguousarray(q)


@pytest.mark.parametrize("kind", ["smooth", "negative_zero", "random", "blast", "tiny_momentum",
                                  "scaled_up", "scaled_down", "near_vacuum", "unphysical", "nan",
                                  "inf"])
@pytest.mark.parametrize("n,nsteps", [(300, 24), (5000, 13)])
def test_euler_ranges(sw, oracle_mod, kind, n, nsteps):
    """The fast Euler step where its ranges hold, and windows that start outside
    them or leave them during a stage: the oracle's bits (NaNs by place)."""
    q0 = euler_states(kind, n, seed=n + nsteps)
    par = [0.05 / n, 1.0 / n, workloads.EULER_GAMMA]
    got = run(sw, q0, nsteps, "euler", par)
    want = oracle_mod.euler(q0, nsteps, *par)
    assert same_up_to_nan(got, want)


@pytest.mark.parametrize("spread", [False, True])
def test_batch_bitwise(sw, oracle_mod, spread):
    """Batches on windows: rings far smaller than a window and larger ones,
    odd and even, runs of no, one, a few and many steps (so instances leave the
    stages at different times), every form of either stencil."""
    import torch
    sizes = [3, 4, 5, 63, 64, 65, 255, 1000, 4097] + ([20000, 65537] if spread else [])
    insts = []
    for q, n in enumerate(sizes):
        for steps in (0, 1, 2, 3, 17, 150) + ((700,) if spread else ()):
            st = "heat" if (q + steps) % 2 else "ks"
            par = [[0.25, 0.3, 0.5][q % 3]] if st == "heat" else [KS_P, [0.004, 0.7]][q % 2]
            u0 = workloads.white_noise(n, seed=n + steps)
            insts.append((st, n, steps, par, u0 if st == "heat" else 0.2 * u0))
    us = [torch.from_numpy(i[4].copy()).cuda() for i in insts]
    for rep in range(3):      # the tables' host buffers are used in turn
        for u, i in zip(us, insts):
            u.copy_(torch.from_numpy(i[4]))
        sw.advance_batch(us, [i[2] for i in insts], [i[0] for i in insts], [i[3] for i in insts])
    torch.cuda.synchronize()
    sw.sync()
    assert sw.last_heat_form() == sw.FORM_FUSED
    for (st, n, steps, par, u0), u in zip(insts, us):
        want = oracle_mod.heat(u0, steps, *par) if st == "heat" else oracle_mod.ks(u0, steps, *par)
        assert same_bits(u.cpu().numpy(), want), (st, n, steps, par)


@pytest.mark.parametrize("heat,ks", [
    ([(700001, 40), (300, 90), (200000, 7)], []),
    ([], [(400002, 20), (64, 50), (300000, 1)]),
    ([(500000, 30), (5, 3)], [(300001, 31), (4, 60)]),
    ([(900000, 25), (300000, 60)], [(100, 9)]),
    ([(4096, 100)], [(4096, 30)]),
])
@pytest.mark.parametrize("stream", [False, True])
def test_batch_chains(sw, heat, ks, stream):
    """The batch's two chains of launches: one stencil alone, KS and heat cut in
    halves at different places, and a batch of few tiles.  What the caller's
    stream does just before and after is ordered with both chains."""
    import torch
    insts = [("heat", n, k, [0.25]) for n, k in heat] + [("ks", n, k, KS_P) for n, k in ks]
    u0 = [torch.from_numpy(workloads.white_noise(n, seed=n)).cuda() for _, n, _, _ in insts]
    us = [torch.zeros_like(u) for u in u0]
    want = [sw.advance(u.clone(), k, st, p) for u, (st, n, k, p) in zip(u0, insts)]
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream() if stream else torch.cuda.current_stream()):
        for rep in range(3):
            for u, a in zip(us, u0):
                u.copy_(a)
            sw.advance_batch(us, [i[2] for i in insts], [i[0] for i in insts], [i[3] for i in insts])
            got = [u.clone() for u in us]
            for u in us:
                u.zero_()
    torch.cuda.synchronize()
    for g, w, i in zip(got, want, insts):
        assert same_bits(g.cpu().numpy(), w.cpu().numpy()), i


def test_batch_of_nothing(sw):
    import torch
    us = [torch.ones(10, dtype=torch.float64, device="cuda") for _ in range(3)]
    sw.advance_batch(us, [0, 0, 0], ["heat", "ks", "heat"], [[0.25], KS_P, [0.3]])
    torch.cuda.synchronize()
    assert all(bool((u == 1).all()) for u in us)


@pytest.mark.parametrize("n,nsteps,first", [
    (8, 1, 2), (8, 3, 0), (64, 2, 2), (64, 40, 41), (130, 65, 30), (1000, 33, 1), (4098, 120, 121),
    (20000, 50, 50),
])
@pytest.mark.parametrize("stencil", ["heat", "ks"])
@pytest.mark.parametrize("with_cot", [False, True])
def test_adjoint_bitwise(sw, oracle_mod, stencil, n, nsteps, first, with_cot):
    """Gradients on windows: no window, one that starts at step 0, inside and
    at the last step, with and without a final cotangent, rings smaller than
    the halo."""
    import torch
    u0 = workloads.white_noise(n, seed=n) if stencil == "heat" else \
        5 * workloads.smoothed_noise(n, seed=n)
    cot = workloads.white_noise(n, seed=1) if with_cot else None
    par = [0.3] if stencil == "heat" else KS_P
    g = sw.adjoint(torch.from_numpy(u0).cuda(), nsteps, stencil, par, window_first=first,
                   window_weight=0.01, cot_final=None if cot is None else torch.from_numpy(cot).cuda())
    torch.cuda.synchronize()
    oracle = oracle_mod.heat_adjoint if stencil == "heat" else oracle_mod.ks_adjoint
    assert same_bits(g.cpu().numpy(), oracle(u0, nsteps, *par, first, 0.01, cot))


@pytest.mark.parametrize("field,cot,weight", [
    ("noise", "noise", 0.01), ("noise", "spikes", 0.0), ("noise", "subnormal", 0.0),
    ("noise", "huge", 0.01), ("noise", "mixed", 0.01), ("noise", "noise", 1e300),
    ("zeros", "noise", 0.01), ("tiny", "noise", 0.01), ("large", "noise", 0.01),
    ("noise", "nan", 0.01),
])
@pytest.mark.parametrize("dx", [0.25, 0.5, 1.0, 0.7])
def test_ks_adjoint_forms(sw, oracle_mod, field, cot, weight, dx):
    """The adjoint's shorter form (c1 and c2 powers of two, c1 >= 1: dx = 1/4
    and 1/2) and the operations as written, over fields and cotangents inside
    and outside of its range: zeros, subnormals, 1e250 and NaN in some or all
    windows."""
    import torch
    n, nsteps = 4098, 33
    dt = 0.005 * min(1.0, (dx / 0.5) ** 4)
    u0 = workloads.smoothed_noise(n, seed=5)
    if field == "zeros":
        u0[700:1500] = 0.0
    elif field == "tiny":
        u0[700:1500] *= 2.0 ** -380
    elif field == "large":
        u0[1000] = 1e31
    c = workloads.white_noise(n, seed=6)
    if cot == "spikes":
        c[:] = 0.0
        c[[0, 2000, n - 1]] = 1.0
    elif cot == "subnormal":
        c *= 2.0 ** -1060
    elif cot == "huge":
        c *= 1e250
    elif cot == "mixed":
        c[1000:1100] *= 1e250
        c[3000:3100] *= 2.0 ** -1060
    elif cot == "nan":
        c[1234] = np.nan
    g = sw.adjoint(torch.from_numpy(u0).cuda(), nsteps, "ks", [dt, dx], window_first=20,
                   window_weight=weight, cot_final=torch.from_numpy(c).cuda())
    torch.cuda.synchronize()
    want = oracle_mod.ks_adjoint(u0, nsteps, dt, dx, 20, weight, c)
    assert same_up_to_nan(g.cpu().numpy(), want)


@pytest.mark.parametrize("stencil,n,nsteps,first", [
    ("heat", 1000, 40, 30), ("ks", 4099, 2100, 2), ("ks_fma", 300, 9, 0), ("heat_fma", 65536, 400, 100),
])
def test_objective_bits_do_not_depend_on_the_schedule(sw, stencil, n, nsteps, first):
    """The sums over steps kept by windows equal those formed one naive step at
    a time (a tile width asks for the swept and naive schedules)."""
    import torch
    u0 = torch.from_numpy(workloads.smoothed_noise(n, seed=3)).cuda()
    par = [0.3] if stencil.startswith("heat") else KS_P
    kw = dict(window_first=first, window_weight=0.5, cot_final=u0.flip(0).contiguous())
    a = sw.objective(u0, nsteps, stencil, par, **kw)
    sw.set_tuning(0, 0, sw.MODE_NAIVE)
    try:
        b = sw.objective(u0, nsteps, stencil, par, **kw)
    finally:
        sw.set_tuning(0, 0, sw.MODE_AUTO)
    torch.cuda.synchronize()
    assert float(a) == float(b)


@pytest.mark.parametrize("n,W", [(4096, 128), (65536, 1024)])
def test_profiled_stages_are_reported(sw, n, W):
    import torch
    u = torch.from_numpy(workloads.white_noise(n, seed=1)).cuda()
    sw.set_profiling(True)
    try:
        sw.advance(u, 500, "heat", [0.25])
        ms, kind = sw.stage_times()
        assert set(kind) == {4} and len(kind) % 2 == 0 and min(ms) > 0
        sw.set_tuning(W, 0, sw.MODE_AUTO)      # a tile width asks for the swept stages
        sw.advance(u, 500, "heat", [0.25])
        assert 4 not in sw.stage_times()[1]
    finally:
        sw.set_tuning(0, 0, sw.MODE_AUTO)
        sw.set_profiling(False)


@pytest.mark.parametrize("stencil", ["heat", "ks"])
@pytest.mark.parametrize("with_cot", [False, True])
@pytest.mark.parametrize("nsteps", [1, 9])
def test_adjoint_of_a_window_beyond_the_run(sw, oracle_mod, stencil, nsteps, with_cot):
    """window_first > nsteps leaves out the window term, however far beyond the
    last step it lies; without a final cotangent either the gradient is zero."""
    import torch
    n = 130
    u0 = workloads.white_noise(n, seed=n) if stencil == "heat" else workloads.smoothed_noise(n, seed=n)
    cot = workloads.white_noise(n, seed=1) if with_cot else None
    par = [0.3] if stencil == "heat" else KS_P
    oracle = oracle_mod.heat_adjoint if stencil == "heat" else oracle_mod.ks_adjoint
    want = oracle(u0, nsteps, *par, nsteps + 1, 0.01, cot)
    for first in (nsteps + 1, nsteps + 2, nsteps + 3, nsteps + 10 ** 6, 2 ** 62, 2 ** 63 - 1):
        g = sw.adjoint(torch.from_numpy(u0).cuda(), nsteps, stencil, par, window_first=first,
                       window_weight=0.01,
                       cot_final=None if cot is None else torch.from_numpy(cot).cuda())
        torch.cuda.synchronize()
        assert same_bits(g.cpu().numpy(), want), first
        assert with_cot or not g.any()


@pytest.mark.parametrize("stencil,n,nsteps,first", [
    ("ks", 20000, 1, 2), ("ks", 20000, 1, 0), ("ks", 70000, 40, 20), ("ks", 64, 3, 4),
    ("heat", 20000, 1, 0), ("heat", 70000, 60, 0), ("heat", 70000, 60, 30), ("heat", 20000, 9, 10),
])
@pytest.mark.parametrize("over", ["u0", "cot"])
@pytest.mark.parametrize("tile_w", [0, 32])
def test_adjoint_in_place(sw, stencil, n, nsteps, first, over, tile_w):
    """The C entry takes u0 or the final cotangent as the gradient's own memory:
    the same bits as into a field of its own (on windows, and on the swept
    adjoint, which a tile width asks for)."""
    import ctypes
    import torch
    u0 = torch.from_numpy(workloads.white_noise(n, seed=n)).cuda()
    cot = torch.from_numpy(workloads.white_noise(n, seed=2)).cuda()
    par = [0.3] if stencil == "heat" else KS_P
    want = sw.adjoint(u0, nsteps, stencil, par, window_first=first, window_weight=0.01, cot_final=cot)
    grad = u0 if over == "u0" else cot
    arr = (ctypes.c_double * len(par))(*par)
    sw.set_tuning(tile_w, 0, sw.MODE_AUTO)
    try:
        rc = sw.lib().swept_adjoint(u0.data_ptr(), grad.data_ptr(), n, nsteps,
                                    sw.stencil_id(stencil), arr, len(par), first, 0.01,
                                    cot.data_ptr())
    finally:
        sw.set_tuning(0, 0, sw.MODE_AUTO)
    assert rc == 0, sw.last_error()
    torch.cuda.synchronize()
    assert same_bits(grad.cpu().numpy(), want.cpu().numpy())


@pytest.mark.parametrize("n,nsteps,first", [
    (64, 2, 1), (64, 2, 2), (64, 23, 23), (64, 24, 24), (64, 32, 31), (64, 33, 32), (1000, 10, 5),
    (1000, 33, 20), (4096, 60, 53), (4096, 60, 54), (65536, 60, 33), (65536, 60, 34),
    (1 << 20, 9, 4), (1 << 20, 9, 5), (1 << 20, 17, 2), (4096, 700, 20),
])
@pytest.mark.parametrize("with_cot", [False, True])
def test_heat_adjoint_of_short_runs(sw, oracle_mod, n, nsteps, first, with_cot):
    """Windows that start after a few steps, whose fields are all kept, and ones
    just late enough that the steps below them run apart."""
    import torch
    u0 = workloads.white_noise(n, seed=n)
    cot = workloads.white_noise(n, seed=1) if with_cot else None
    g = sw.adjoint(torch.from_numpy(u0).cuda(), nsteps, "heat", [0.3], window_first=first,
                   window_weight=0.01, cot_final=None if cot is None else torch.from_numpy(cot).cuda())
    torch.cuda.synchronize()
    assert same_bits(g.cpu().numpy(), oracle_mod.heat_adjoint(u0, nsteps, 0.3, first, 0.01, cot))


def captured_launches(fn):
    """Nodes of the graph that fn's work on a stream of its own makes."""
    import ctypes
    import torch
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
    hip = ctypes.CDLL(path)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        fn()            # sizes the scratch
        torch.cuda.synchronize()
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(s.cuda_stream), 1) == 0   # thread-local
        try:
            fn()
        finally:
            graph = ctypes.c_void_p()
            rc = hip.hipStreamEndCapture(ctypes.c_void_p(s.cuda_stream), ctypes.byref(graph))
    assert rc == 0
    count = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return count.value


@pytest.mark.parametrize("stencil", ["heat", "ks"])
@pytest.mark.parametrize("n,nsteps,first", [
    (64, 1, 0), (64, 2, 1), (64, 2, 2), (1000, 10, 2), (1000, 10, 5), (4096, 5, 4), (65536, 20, 10),
])
def test_short_adjoints_take_few_launches(sw, stencil, n, nsteps, first):
    """A gradient of a few steps takes no more launches than on the swept
    adjoint, whose two passes are two stages each."""
    import ctypes
    import torch
    u0 = torch.from_numpy(workloads.smoothed_noise(n, seed=n)).cuda()
    cot, grad = torch.ones_like(u0), torch.empty_like(u0)
    par = [0.3] if stencil == "heat" else KS_P
    arr = (ctypes.c_double * len(par))(*par)

    def call():
        sw._prepare(u0, sw.stencil_id(stencil))
        rc = sw.lib().swept_adjoint(u0.data_ptr(), grad.data_ptr(), n, nsteps,
                                    sw.stencil_id(stencil), arr, len(par), first, 0.01,
                                    cot.data_ptr())
        assert rc == 0, sw.last_error()

    windows = captured_launches(call)
    sw.set_tuning(0, 0, sw.MODE_STAGE)
    try:
        swept = captured_launches(call)
    finally:
        sw.set_tuning(0, 0, sw.MODE_AUTO)
    assert windows <= swept, (windows, swept)


@pytest.mark.parametrize("stencil,n,nsteps,first", [
    ("heat", 4096, 300, 200), ("heat", 4096, 20, 15), ("ks", 4096, 120, 90), ("ks", 1000, 40, 41),
])
def test_captured_gradient_and_objective_replay(sw, stencil, n, nsteps, first):
    """adjoint() and objective() in a captured graph, once their scratch is
    sized: every replay, on new inputs in the same memory and with eager work
    and synchronisations between them, equals the eager result."""
    import torch
    par = [0.3] if stencil == "heat" else KS_P
    kw = dict(window_first=first, window_weight=0.01)
    inputs = [torch.from_numpy(workloads.smoothed_noise(n, seed=s)).cuda() for s in (1, 2, 3)]
    cot = torch.from_numpy(workloads.white_noise(n, seed=4)).cuda()
    want = [(sw.adjoint(u, nsteps, stencil, par, cot_final=cot, **kw),
             sw.objective(u, nsteps, stencil, par, cot_final=cot, **kw)) for u in inputs]
    torch.cuda.synchronize()
    u = torch.zeros_like(cot)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(graph, stream=s):
            g = sw.adjoint(u, nsteps, stencil, par, cot_final=cot, **kw)
            J = sw.objective(u, nsteps, stencil, par, cot_final=cot, **kw)
    torch.cuda.synchronize()
    for rep in range(2):
        for v, (wg, wJ) in zip(inputs, want):
            u.copy_(v)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert same_bits(g.cpu().numpy(), wg.cpu().numpy()), rep
            assert float(J) == float(wJ), rep
            # eager work in the library's own scratch between the replays
            sw.advance(v.clone(), 7, stencil, par)
            torch.cuda.synchronize()
