"""The swept schedules under settings that choose them.  Calls with every setting
at its default run on register windows; a mode, a tile width or a batch setting
asks for the swept kernels (paper, Section 3), which tunings and the autotuner
use as well.  Each case here names its schedule, checks by the profiled stages
that it ran where the library reports them, and compares bits with the oracle or
the naive schedule."""
import numpy as np
import pytest

import workloads
from tests.conftest import gpu_available, same_bits
from tests.test_gpu_heat_form import batch_oracle, mixed_batch, run_batch, same_bits_up_to_nan
from tests.test_gpu_ragged import case

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

KS_P = [workloads.KS_DT, workloads.KS_DX]
DMAX = np.finfo(np.float64).max
RAGGED, WINDOW = 3, 4      # stage_times' kinds


@pytest.fixture(scope="module")
def sw():
    import paper_1504_01380_amd as swept
    swept.init(0)
    swept.clear_tuning()
    yield swept


@pytest.fixture(autouse=True)
def _reset(sw):
    def defaults():
        sw.set_tuning(0, 0, sw.MODE_AUTO)
        sw.set_heat_form(sw.FORM_AUTO)
        sw.set_batch_schedule(sw.BATCH_PERSISTENT, 0, 0, 0)
        sw.set_profiling(False)
    defaults()
    yield
    defaults()


def run(sw, u0, nsteps, stencil, params):
    """The advanced field and the kinds of the stages that advanced it."""
    import torch
    u = torch.from_numpy(np.ascontiguousarray(u0)).cuda()
    sw.set_profiling(True)
    sw.advance(u, nsteps, stencil, params)
    kinds = set(sw.stage_times()[1])
    sw.set_profiling(False)
    sw.sync()
    return u.cpu().numpy(), kinds


def choose_ragged(sw, n, nsteps, name, dtype):
    """The unequal tiling the untuned swept plan takes for this grid."""
    import torch
    p = sw.plan(n, nsteps, name, torch.float32 if dtype == np.float32 else torch.float64)
    assert p["mode"] == sw.MODE_STAGE_RAGGED
    sw.set_tuning(p["tile_w"], 0, sw.MODE_STAGE_RAGGED)
    q = sw.plan(n, nsteps, name, torch.float32 if dtype == np.float32 else torch.float64)
    assert q == p
    return p


@pytest.mark.parametrize("stencil,n,nsteps", [
    ("heat", 1001, 333), ("heat", 8198, 1000), ("heat", 65537, 1200), ("heat", 129, 41),
    ("heat_f32", 1001, 400), ("heat_f32", 8198, 900), ("heat_fma", 4099, 700),
    ("ks", 1001, 120), ("ks", 8198, 250), ("ks", 65537, 100), ("ks_fma", 8198, 150),
    ("euler", 1001, 60), ("euler", 8198, 41),
])
def test_unequal_tiling(sw, oracle_mod, stencil, n, nsteps):
    name = "heat" if stencil == "heat_f32" else stencil
    u0, par, want = case(oracle_mod, stencil, n, nsteps)
    choose_ragged(sw, n, nsteps, name, u0.dtype)
    got, kinds = run(sw, u0, nsteps, name, par)
    assert kinds == {RAGGED}
    assert same_bits(got, want)


def test_unequal_tiling_of_a_large_awkward_grid(sw, oracle_mod):
    """2^24 + 2 points (= 2 x 3 x 2796203): 16,385 tiles, the last of 2 points."""
    import torch
    n, nsteps = (1 << 24) + 2, 3000
    u0 = workloads.white_noise(n, seed=77)
    p = choose_ragged(sw, n, nsteps, "heat", u0.dtype)
    assert p["depth_k"] >= 256
    got, kinds = run(sw, u0, nsteps, "heat", [0.25])
    assert kinds == {RAGGED}
    v = torch.from_numpy(u0).cuda()
    sw.naive_advance(v, nsteps, "heat", [0.25])
    assert same_bits(got, v.cpu().numpy())
    idx = np.array([0, 1, 1023, 1024, n // 2, n - 3, n - 2, n - 1], dtype=np.int64)
    assert same_bits(got[idx], oracle_mod.heat_points(u0, nsteps, 0.25, idx))


def test_noalloc_on_the_unequal_tiling(sw, oracle_mod):
    import torch
    n, nsteps = 100001, 500
    u0 = workloads.white_noise(n, seed=3)
    choose_ragged(sw, n, nsteps, "heat", u0.dtype)
    u = torch.from_numpy(u0).cuda()
    sw.advance_noalloc(u, nsteps, "heat", [0.25])
    assert same_bits(u.cpu().numpy(), oracle_mod.heat(u0, nsteps, 0.25))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n,nsteps,mode", [(1001, 700, 5), (8198, 513, 5), (5000, 300, 1),
                                           (5000, 300, 3)])
def test_heat_forms_on_the_swept_stages(sw, oracle_mod, n, nsteps, mode, dtype):
    """The fused form where the range check allows it, the operations as written
    where a value is too large or the caller asks for them."""
    u0 = workloads.white_noise(n, seed=n + 3, dtype=dtype)
    big = u0.copy()
    big[n // 3] = np.finfo(dtype).max / 4
    want = oracle_mod.heat(u0, nsteps, 0.25)
    sw.set_tuning(0, 0, mode)
    got, kinds = run(sw, u0, nsteps, "heat", [0.25])
    assert WINDOW not in kinds and sw.last_heat_form() == sw.FORM_FUSED
    assert same_bits(got, want)
    got, kinds = run(sw, big, nsteps, "heat", [0.25])
    assert WINDOW not in kinds and sw.last_heat_form() == sw.FORM_CANONICAL
    assert same_bits_up_to_nan(got, oracle_mod.heat(big, nsteps, 0.25))
    sw.set_heat_form(sw.FORM_CANONICAL)
    got, kinds = run(sw, u0, nsteps, "heat", [0.25])
    assert WINDOW not in kinds and sw.last_heat_form() == sw.FORM_CANONICAL
    assert same_bits(got, want)


@pytest.mark.parametrize("stencil,n,nsteps", [("heat", 1 << 28, 256), ("ks", 1 << 26, 100),
                                              ("euler", 1 << 24, 50)])
def test_swept_stages_at_the_largest_sizes(sw, stencil, n, nsteps):
    """The whole field against the naive schedule, compared on the device."""
    import torch
    if stencil == "euler":
        a = torch.from_numpy(workloads.euler_mirrored_sod(n)).cuda()
        par = [workloads.EULER_CFL / n, 1.0 / n, workloads.EULER_GAMMA]
    else:
        g = torch.Generator(device="cuda").manual_seed(n)
        a = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) - 0.5
        par = [0.25] if stencil == "heat" else KS_P
    b = a.clone()
    sw.set_tuning(0, 0, sw.MODE_STAGE)
    sw.set_profiling(True)
    sw.advance(a, nsteps, stencil, par)
    assert WINDOW not in sw.stage_times()[1]
    sw.naive_advance(b, nsteps, stencil, par)
    torch.cuda.synchronize()
    assert torch.equal(a.view(torch.int64), b.view(torch.int64))


@pytest.mark.parametrize("stencil,n,nsteps", [("heat", 1 << 16, 700), ("ks", 1 << 14, 150)])
def test_captured_swept_stages_replay(sw, stencil, n, nsteps):
    """Swept stages inside a captured graph: every replay, with eager work and
    synchronisations between them, equals the eager result."""
    import torch
    par = [0.25] if stencil == "heat" else KS_P
    u0 = workloads.white_noise(n, seed=5) if stencil == "heat" else \
        workloads.smoothed_noise(n, seed=5)
    sw.set_tuning(0, 0, sw.MODE_STAGE)
    src = torch.from_numpy(u0).cuda()
    ref = src.clone()
    sw.advance(ref, nsteps, stencil, par)          # sizes the scratch
    torch.cuda.synchronize()
    u = src.clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(graph, stream=s):
            sw.advance(u, nsteps, stencil, par)
    torch.cuda.synchronize()
    for rep in range(3):
        u.copy_(src)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(u.view(torch.int64), ref.view(torch.int64)), rep
        junk = (torch.randn(1 << 16, device="cuda") * 2).cpu()   # unrelated eager work
        del junk


@pytest.mark.parametrize("stencil,n,nsteps,first,with_cot", [
    ("heat", 64, 1, 0, True), ("heat", 64, 37, 20, True), ("heat", 128, 100, 1, False),
    ("heat", 1024, 333, 300, True), ("heat", 1 << 16, 400, 401, True), ("ks", 64, 1, 0, True),
    ("ks", 64, 9, 5, True), ("ks", 128, 40, 1, False), ("ks", 1024, 120, 100, True),
    ("ks", 1 << 16, 300, 200, False),
])
def test_swept_adjoint(sw, oracle_mod, stencil, n, nsteps, first, with_cot):
    """The adjoint at its deepest tiles (k = 32 where the grid allows it)."""
    import torch
    u0 = workloads.white_noise(n, seed=n + nsteps) if stencil == "heat" else \
        5 * workloads.smoothed_noise(n, seed=n + nsteps)
    cot = workloads.white_noise(n, seed=5) if with_cot else None
    par = [0.3] if stencil == "heat" else KS_P
    sw.set_tuning(0, 0, sw.MODE_STAGE)
    g = sw.adjoint(torch.from_numpy(u0).cuda(), nsteps, stencil, par, window_first=first,
                   window_weight=0.01, cot_final=None if cot is None else torch.from_numpy(cot).cuda())
    torch.cuda.synchronize()
    oracle = oracle_mod.heat_adjoint if stencil == "heat" else oracle_mod.ks_adjoint
    assert same_bits(g.cpu().numpy(), oracle(u0, nsteps, *par, first, 0.01, cot))


# ------------------------------------------------------------------ batches
# a number of tasks per claim, the library's own default here, asks for the
# persistent launch

def choose_persistent(sw):
    sw.set_batch_schedule(sw.BATCH_PERSISTENT, 0, 2, 0)


def test_persistent_batch(sw, oracle_mod):
    """Odd and even lengths, both stencils, no steps; then the same pointers
    again, which launches the captured graph a second time."""
    choose_persistent(sw)
    g = workloads.rng(2024)
    insts = []
    for q, n in enumerate([256, 257, 300, 1001, 2048, 3, 4, 999, 4096, 777, 513, 64]):
        st = "heat" if q % 2 == 0 else "ks"
        insts.append((st, int(g.integers(1, 120 if st == "ks" else 400)), g.uniform(-1, 1, n),
                      [0.25] if st == "heat" else KS_P))
    insts.append(("ks", 0, g.uniform(-1, 1, 100), KS_P))
    want = batch_oracle(oracle_mod, insts)
    us = run_batch(sw, insts)
    for rep in range(3):
        for u, w, i in zip(us, want, insts):
            assert same_bits(u.cpu().numpy(), w), (rep, i[0], i[1], w.size)
        run_batch(sw, insts, us)


def test_persistent_batch_heat_forms(sw, oracle_mod):
    """One decision for all heat instances, made anew at every launch of the
    captured graph: a field of values near MAX/2 sends that launch to the
    operations as written, and the next good one is fused again."""
    choose_persistent(sw)
    good = mixed_batch(32)
    bad = list(good)
    st, ns, u0, p = bad[2]
    rng = np.random.default_rng(6)
    bad[2] = (st, ns, DMAX * (0.5 + 0.1 * rng.uniform(-1.0, 1.0, u0.size)), p)
    runs = [(i, batch_oracle(oracle_mod, i), f) for i, f in ((good, sw.FORM_FUSED),
                                                            (bad, sw.FORM_CANONICAL))]
    assert not np.all(np.isfinite(runs[1][1][2]))
    us = None
    for insts, want, form in runs + runs:
        us = run_batch(sw, insts, us)
        assert sw.last_heat_form() == form
        for u, w in zip(us, want):
            assert same_bits_up_to_nan(u.cpu().numpy(), w)
    sw.set_heat_form(sw.FORM_CANONICAL)
    us = run_batch(sw, good)
    assert sw.last_heat_form() == sw.FORM_CANONICAL
    for u, w in zip(us, runs[0][1]):
        assert same_bits(u.cpu().numpy(), w)


def test_persistent_batch_of_few_large_instances(sw):
    """Instances that one queue per XCD cannot spread evenly (one launch per
    stage then) equal their own runs on the naive schedule."""
    import torch
    choose_persistent(sw)
    specs = [("heat", 1 << 20, 700), ("ks", 1 << 18, 150), ("heat", 3 * 65536 + 2, 301)]
    u0 = [torch.from_numpy(workloads.smoothed_noise(n, seed=n)).cuda() for _, n, _ in specs]
    us = [u.clone() for u in u0]
    pars = [[0.25] if st == "heat" else KS_P for st, _, _ in specs]
    sw.advance_batch(us, [ns for _, _, ns in specs], [st for st, _, _ in specs], pars)
    for u, v, (st, n, ns), p in zip(us, u0, specs, pars):
        sw.naive_advance(v, ns, st, p)
        assert torch.equal(u.view(torch.int64), v.view(torch.int64)), (st, n)
    sw.sync()


def test_persistent_batch_after_a_wait_that_gave_up(sw, oracle_mod):
    """A spin limit of one microsecond, set from the host, ends the launch early
    and is reported once; with the default's 60 seconds the batch is whole."""
    import torch
    g = workloads.rng(5)
    u0s = [g.uniform(-1, 1, size=8192 + 2 * q) for q in range(64)]
    us = [torch.from_numpy(u0.copy()).cuda() for u0 in u0s]
    args = ([3000] * 64, ["heat"] * 64, [[0.25]] * 64)
    sw.set_batch_schedule(sw.BATCH_PERSISTENT, 1, 0, 0)
    sw.advance_batch(us, *args)
    torch.cuda.synchronize()
    with pytest.raises(sw.SweptError) as err:
        sw.sync()
    assert err.value.code == -6
    sw.set_batch_schedule(sw.BATCH_PERSISTENT, 60 * 1000 * 1000, 0, 0)
    for u, u0 in zip(us, u0s):
        u.copy_(torch.from_numpy(u0))
    sw.advance_batch(us, *args)
    torch.cuda.synchronize()
    sw.sync()
    for q in (0, 63):
        assert same_bits(us[q].cpu().numpy(), oracle_mod.heat(u0s[q], 3000, 0.25))


def test_persistent_full_ensemble(sw):
    """The ensemble workload at full size against the naive batch."""
    import torch
    choose_persistent(sw)
    insts = workloads.batch()
    ns, kinds = [i.nsteps for i in insts], [i.stencil for i in insts]
    pars = [[0.25] if k == "heat" else KS_P for k in kinds]
    us = [torch.from_numpy(i.u0).cuda() for i in insts]
    vs = [u.clone() for u in us]
    print("swept batch", flush=True)
    sw.advance_batch(us, ns, kinds, pars)
    print("naive batch", flush=True)
    sw.naive_advance_batch(vs, ns, kinds, pars)
    torch.cuda.synchronize()
    sw.sync()
    for q, (a, b) in enumerate(zip(us, vs)):
        assert torch.equal(a.view(torch.int64), b.view(torch.int64)), q
