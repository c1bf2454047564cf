"""The window schedule's stage arithmetic (csrc/stages.hpp), compiled here with
the host compiler and walked through for whole runs: the reverse sweep takes
every step once, starts from the objective's cotangent once, and reads no field
that was not kept (paper, Section 3: what a stage computes follows from what it
holds)."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "stages.hpp"
using namespace swept;
extern "C" {
int64_t start_of(int64_t nsteps, int64_t stages, int64_t s) { return stage_start(nsteps, stages, s); }
void run_of(int every, int64_t nsteps, int64_t win_first, int64_t* out)
{
    const AdjointRun r = adjoint_run(every != 0, nsteps, win_first);
    const int64_t v[6] = {r.win_first, r.windowed, r.kept0, r.nkept, r.reverse, r.stop};
    for (int i = 0; i < 6; ++i)
        out[i] = v[i];
}
void stage_of(int every, int64_t nsteps, int64_t win_first, int64_t stages, int64_t s, int64_t* out)
{
    const AdjointRun r = adjoint_run(every != 0, nsteps, win_first);
    const AdjointStage a = adjoint_stage_at(r, nsteps, stages, s);
    out[0] = a.first, out[1] = a.steps, out[2] = a.seed, out[3] = a.empty;
    adjoint_stage_reads(r, a, out + 4, out + 5);
}
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("stages")
    src, lib = d / "stages.cpp", d / "libstages.so"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_1504_01380_amd", "csrc"), str(src), "-o", str(lib)])
    L = ctypes.CDLL(str(lib))
    i64, p = ctypes.c_int64, ctypes.POINTER(ctypes.c_int64)
    L.start_of.argtypes, L.start_of.restype = [i64, i64, i64], i64
    L.run_of.argtypes, L.run_of.restype = [ctypes.c_int, i64, i64, p], None
    L.stage_of.argtypes, L.stage_of.restype = [ctypes.c_int, i64, i64, i64, i64, p], None
    return L


@pytest.mark.parametrize("every", [False, True])
@pytest.mark.parametrize("nsteps", [1, 2, 3, 7, 40])
def test_reverse_sweep_reads_kept_fields_only(host, every, nsteps):
    """`every`: KS, which reads all steps' fields; else heat, which reads those
    of the objective's window.  Windows from before the first step to far
    beyond the last one."""
    firsts = list(range(-2, nsteps + 6)) + [nsteps + 1000, 2 ** 62, 2 ** 63 - 1, -2 ** 63]
    for win_first in firsts:
        out = (ctypes.c_int64 * 6)()
        host.run_of(every, nsteps, win_first, out)
        first, windowed, kept0, nkept, reverse, stop = list(out)
        sources = [j for j in range(nsteps + 1) if j >= win_first]
        assert windowed == bool(sources)
        assert [j for j in range(nsteps + 1) if j >= first] == sources
        kept = range(kept0, kept0 + nkept)
        assert nkept == 0 or kept[-1] == nsteps
        assert all(0 < j for j in kept) and nkept <= nsteps
        assert set(j for j in sources if j > 0) <= set(kept)
        assert reverse == (every or windowed)
        if not reverse:      # no stage is launched
            assert nkept == 0 and stop == nsteps
            continue
        if every:
            assert set(kept) == set(range(1, nsteps + 1)) and stop == 0
        else:   # nothing is read below `stop`
            assert all(j >= stop for j in sources)
        for stages in (1, 2, 3, 4, 5, 6, 2 * nsteps):
            taken, seeds = [], 0
            for s in range(stages):
                host.stage_of(every, nsteps, win_first, stages, s, out)
                at, steps, seed, empty, lo, hi = list(out)
                if empty:
                    assert steps == 0
                    continue
                seeds += seed
                assert seed == (not taken)
                taken += range(at + steps - 1, at - 1, -1)
                reads = range(lo, hi + 1)
                assert set(range(at, at + steps)) | {at} <= set(reads)
                assert all(j == 0 or j in kept for j in reads), (win_first, stages, s)
            assert seeds == 1 and taken == list(range(nsteps - 1, stop - 1, -1))


@pytest.mark.parametrize("nsteps,stages", [
    (1, 2), (7, 4), (40, 6), (20000, 180), (10 ** 12 + 7, 4 * 10 ** 9), (10 ** 15 - 1, 8 * 10 ** 12 + 2),
    (2 ** 60 - 1, 2 ** 59 + 2),
])
def test_stages_share_the_steps_evenly(host, nsteps, stages):
    """Stage s starts after floor(nsteps * s / stages) steps, also where the
    product of the two does not fit 64 bits."""
    at = sorted({0, 1, 2, stages // 3, stages // 2, stages - 2, stages - 1, stages})
    for s in at:
        assert host.start_of(nsteps, stages, s) == nsteps * s // stages
