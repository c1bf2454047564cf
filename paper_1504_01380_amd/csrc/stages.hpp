// stages.hpp -- host arithmetic of the window schedule's stages: which time
// steps each stage of a run takes and, for the adjoint, which kept fields it
// reads.  No HIP in it, so that a test compiles it with the host compiler and
// walks through whole schedules.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace swept {

// time steps done before stage s of a plan: the run spread evenly over its
// stages (the product passes 64 bits from 3e9 stages on)
inline int64_t stage_start(int64_t nsteps, int64_t stages, int64_t s)
{
    return nsteps / stages * s + (int64_t)((__int128)(nsteps % stages) * s / stages);
}

// What the window adjoint keeps of the forward pass and how far its reverse
// sweep goes: with `every` (KS, and heat where that saves launches) all steps'
// fields and all steps; else (heat) those of the objective's window, below
// which, or without one, heat's transposed step reads no field and is the
// forward step itself.
struct AdjointRun {
    int64_t win_first;   // first step with a source; nsteps + 1 if no step has one
    bool windowed;       // some step of the run has a source
    int64_t kept0;       // the fields of steps kept0 .. kept0 + nkept - 1 are kept
    int64_t nkept;
    bool reverse;        // there is a reverse sweep (else the cotangent runs all the way)
    int64_t stop;        // it goes from nsteps down to this step
};

inline AdjointRun adjoint_run(bool every, int64_t nsteps, int64_t win_first)
{
    AdjointRun r;
    // any window beyond the last step is the same as one just beyond it
    r.win_first = std::min(std::max<int64_t>(win_first, 0), nsteps + 1);
    r.windowed = r.win_first <= nsteps;
    r.kept0 = every ? 1 : std::max<int64_t>(r.win_first, 1);
    r.reverse = every || r.windowed;
    r.nkept = r.reverse ? nsteps - r.kept0 + 1 : 0;
    r.stop = every ? 0 : std::min(r.win_first, nsteps);
    return r;
}

// Heat: whether all fields are kept.  Running the steps below the window apart
// takes four launches more (two forward and two back; one or two where the
// window itself takes no or one step), about 3.5 us each.  Keeping those fields
// as well costs a step 0.1 to 0.25 us, or 2.6 us more at 2^20 points, for which
// their traffic counts, as long as the Infinity Cache holds them all (half of
// its 256 MB; 2^20 points, window from step 2: 66 us apart and 44 together for 10
// steps, 220 and 246 for 50).  So a window that starts that early is treated as
// one of all steps (4096 points, window from step 5 of 10: 31 us apart, 18
// together; from step 50 of 100: 34 and 35).
inline bool adjoint_keeps_all(int64_t nx, int64_t nsteps, int64_t win_first)
{
    if (win_first > nsteps || 8.0 * (double)nx * (double)nsteps > 134217728.0)
        return false;
    const double apart = win_first == nsteps ? 6000.0 : (win_first == nsteps - 1 ? 8000.0 : 14000.0);
    return (double)win_first * (250.0 + 2.6e-3 * (double)nx) <= apart;
}

// Stage s of the reverse sweep: from step first + steps down to step `first`.
struct AdjointStage {
    int64_t first, steps;
    bool seed;    // starts from the objective's cotangent of the last field
    bool empty;   // neither steps nor the seed: nothing to launch
};

inline AdjointStage adjoint_stage_at(const AdjointRun& r, int64_t nsteps, int64_t stages, int64_t s)
{
    const int64_t total = nsteps - r.stop;
    const int64_t done = stage_start(total, stages, s), upto = stage_start(total, stages, s + 1);
    AdjointStage a;
    a.first = nsteps - upto;
    a.steps = upto - done;
    // the seed goes with the first steps, or, without any, with the first stage
    a.seed = done == 0;
    a.empty = a.steps == 0 && (total > 0 || s > 0);
    return a;
}

// The steps lo .. hi whose fields a stage reads: those it takes back, the last
// one where the seed has a source, and in any case `first` (adjoint_stage's loads).
inline void adjoint_stage_reads(const AdjointRun& r, const AdjointStage& a, int64_t* lo, int64_t* hi)
{
    const int64_t last = a.first + a.steps;
    const bool source = a.seed && last >= r.win_first;
    *lo = a.first;
    *hi = std::max(a.first, source ? last : last - 1);
}

}  // namespace swept
