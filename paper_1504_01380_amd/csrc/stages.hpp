// stages.hpp -- host arithmetic of the window schedule's stages: which time
// steps each stage of a run takes and, for the adjoint, which kept fields it
// reads.  No HIP in it, so that a test compiles it with the host compiler and
// walks through whole schedules.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace swept {

// time steps done before stage s of a plan: the run spread evenly over its stages
inline int64_t stage_start(int64_t nsteps, int64_t stages, int64_t s)
{
    return nsteps / stages * s + nsteps % stages * s / stages;
}

// What the window adjoint keeps of the forward pass and how far its reverse
// sweep goes: KS (`every` true) reads every step's field; heat those of the
// objective's window, and below it (or without one) none, since its transposed
// step is the forward step itself.
struct AdjointRun {
    int64_t win_first;   // first step with a source; nsteps + 1 if no step has one
    bool windowed;       // some step of the run has a source
    int64_t kept0;       // the fields of steps kept0 .. kept0 + nkept - 1 are kept
    int64_t nkept;
    int64_t stop;        // the reverse sweep goes from nsteps down to this step
};

inline AdjointRun adjoint_run(bool every, int64_t nsteps, int64_t win_first)
{
    AdjointRun r;
    // any window beyond the last step is the same as one just beyond it
    r.win_first = std::min(std::max<int64_t>(win_first, 0), nsteps + 1);
    r.windowed = r.win_first <= nsteps;
    r.kept0 = every ? 1 : std::max<int64_t>(r.win_first, 1);
    r.nkept = every || r.windowed ? nsteps - r.kept0 + 1 : 0;
    r.stop = every ? 0 : std::min(r.win_first, nsteps);
    return r;
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

// The steps lo .. hi whose fields a stage reads (none if lo > hi): those it
// takes back, and the last one where the seed has a source.
inline void adjoint_stage_reads(const AdjointRun& r, const AdjointStage& a, int64_t* lo, int64_t* hi)
{
    const int64_t last = a.first + a.steps;
    const bool source = a.seed && last >= r.win_first;
    *lo = a.steps > 0 ? a.first : last;
    *hi = source ? last : last - 1;
}

}  // namespace swept
