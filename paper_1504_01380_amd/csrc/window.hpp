// window.hpp -- the register-window schedule: the automatic schedule of
// swept_advance.  Like the swept stages of kernels.hpp it advances a field many
// time steps per launch, so that tiles exchange data through HBM once per
// stage instead of once per step (paper, Sections 1 and 3), and it applies
// the same per-point operations, so the bits are the same.
//
// Geometry.  A stage advances the ring by `steps` time steps from one field
// buffer to another.  Tile t owns the points [t*own, t*own + own) (the last
// one the rest).  Its wavefront holds a window of 64*M consecutive points in
// registers -- lane l the M points from column l*M on -- that reaches `halo`
// = (stencil radius per time step) x steps points beyond the owned ones on
// either side, and advances all of them together: inside a lane the
// neighbours are registers, between lanes the outermost points move by one
// DPP wave shift per sub-timestep.  The columns whose dependence reaches
// outside the window go wrong from the two ends inwards by one point per
// sub-timestep, which the halo absorbs exactly.
//
// What bounds it, and why this shape.  A row costs M point updates and two DPP
// moves of one point per lane; nothing touches LDS and there is no pipeline to
// fill, so almost every issued instruction is an update.  The price is the
// halo, 2*halo of 64*M columns: deep registers (M up to 48 for heat) keep it at
// 10 to 23% of the owned points on grids that fill the chip.  On small grids it
// is most of a window (4096 points: 8 times the points for heat, 12 for KS),
// run by SIMDs that would idle, for stages that are deeper.  Against the diamonds of swept_diamond_cont_kernel, whose
// fill and drain idle a fifth of its slots and whose lane-0 chain, band
// changes and hand-on moves take another 16% of the issue (point-steps/s, or
// time of a step, on MI355X):
//   heat f64, 2^24 points   6.2e12 -> 7.8e12 with the same four operations per
//                           update, 1.0e13 with three (HeatExact below)
//   heat f64, 4096 points   225 -> 54 ns (one wave per SIMD, no two-rows-per-
//                           level diamond)
//   heat f32, 2^22 points   6.6e12 -> 1.4e13
//   KS, 2^20 points         4.8e11 -> 1.08e12;  4096 points 1.21 -> 0.26 us
//   Euler, 2^20 cells       2.3e10 -> 8.8e10;  4096 cells 8.7 -> 1.04 us
// What is left, by the counters: heat at 2^24 points issues vector
// instructions in 90% of its clocks, 96% of them FP64.  KS at 2^20 points is one
// wave a SIMD: a wave lives 68 thousand clocks and issues in 52 of them (0.77),
// and no other wave's rows cover its start, its first loads and its last stores
// (0.75 of a launch of 29 us in a run; 0.56 of the launches that the counters
// serialise).  Two waves of half the window cover them, but the halo is twice
// the part of a window: 1.08 us a step against 1.00.  Small grids are the
// latency of a row (M points and two DPP moves in a chain) and 2.2 us a launch.
#pragma once

#include <limits>

#include "kernels.hpp"

namespace swept {

template <class S>
using WindowBound = std::conditional_t<has_faces<S>::value, double, typename S::T>;

template <class S>
struct WindowArgs {
    const typename S::T* in;
    typename S::T* out;
    int64_t n;       // points of the ring
    int64_t own;     // points a tile owns
    int tiles;       // ceil(n / own)
    int halo;        // points on either side of them
    int steps;       // time steps of this stage
    typename S::Consts c;
    // the evaluation forms this stage may take and their conditions on the
    // values of a window (heat: heat_advance; KS: ks_advance)
    int fused;                  // 0: the operations as written only
    WindowBound<S> big;         // largest |u| of the fused forms
    WindowBound<S> tiny;        // smallest |u| of the exact-product form (0: not allowed)
    int rows;                   // heat: rows `tiny` is good for
    unsigned long long guard;   // heat: the call's id on its first stage (marks the call), else 0
};

// heat: the fused Laplacian (HeatLap) where r is a power of two, r = 2^-e.
// Then r*lap is exact unless it underflows, and u + r*lap rounds once either
// way: fma(r, lap, u) gives the canonical bits from three operations.  No
// product underflows inside a stage of h steps if every nonzero |u| at its
// start is at least 2^(emin + e*h) (emin: exponent of the smallest normal
// value): all values are then multiples of 2^g, g >= emin - p + 1 + e*h for a
// p-bit significand; sums and differences of such multiples stay multiples
// when rounded (a rounded result's unit exceeds 2^g), a step lowers g by e,
// so every lap*2^-e is a multiple of the smallest subnormal: exact.
template <class TT>
struct HeatExact : Heat<TT> {
};

// One row of heat: u' from u and s = u[left] + u[right].
template <class S>
__device__ __forceinline__ typename S::T heat_point(typename S::T u, typename S::T s,
                                                    const typename S::Consts& k)
{
    using T = typename S::T;
    if constexpr (std::is_base_of_v<HeatExact<T>, S> || std::is_base_of_v<HeatFma<T>, S>)
        return fmad(k.r, fmad(T(-2), u, s), u);
    else if constexpr (std::is_base_of_v<HeatLap<T>, S>)
        return u + k.r * fmad(T(-2), u, s);
    else
        return u + k.r * (s - T(2) * u);
}

// The sums of the next point are formed before a point is overwritten, so the
// row updates in place and needs no register copies (a plain left-to-right
// update cost one v_mov_b64 per point, 19% of the row).
// each(j): called with the window at row j = 0, 1, ... done.
template <class S, int M, class Each>
__device__ __forceinline__ void heat_rows(typename S::T (&u)[M], int first, int rows,
                                          const typename S::Consts& k, Each&& each)
{
    using T = typename S::T;
    auto row = [&](int j) {
        const T left = dpp_record<kWaveShr1>(u[M - 1]);
        const T right = dpp_record<kWaveShl1>(u[0]);
        T s = left + (M > 1 ? u[M > 1 ? 1 : 0] : right);
#pragma unroll
        for (int q = 0; q < M; ++q) {
            T sn = T(0);
            if (q + 1 < M)
                sn = u[q] + (q + 2 < M ? u[q + 2 < M ? q + 2 : 0] : right);
            u[q] = heat_point<S>(u[q], s, k);
            s = sn;
        }
        each(j);
    };
    int j = first;
    if constexpr (M <= 8) {   // short rows: the loop's own instructions are a fifth of them
        for (; j + 4 <= rows; j += 4) {
            row(j);
            row(j + 1);
            row(j + 2);
            row(j + 3);
        }
    }
    for (; j < rows; ++j)
        row(j);
}

// Heat's evaluation of a window for one stage.  The conditions of the fused
// forms are checked on the window itself, so that no launch reads the field
// beforehand and every stage is judged on its own data: no finite |u| above
// `big` (HeatLap: with 0 <= r <= 1/2 the values cannot come near the
// overflow of 2u inside a stage; the host passes MAX/16 for the initial field
// and MAX/8, which the run-length bound keeps out of reach, afterwards), and
// for the exact-product form no nonzero |u| below `tiny`, which holds for
// `rows` rows: a deeper stage (binary32) looks again after each of them.  A
// wave decides for itself; all forms give the same bits.
template <class S, int M, class Each>
__device__ __forceinline__ void heat_advance(typename S::T (&u)[M], const WindowArgs<S>& g,
                                             Each&& each)
{
    using T = typename S::T;
    if constexpr (has_fused_form<S>) {
        if (g.fused != 0) {
            // one maximum and one minimum a point settle nearly every window;
            // infinities and zeros, which are allowed, take the exact look
            T mx = T(0);
#pragma unroll
            for (int q = 0; q < M; ++q)
                mx = __builtin_fmax(mx, __builtin_fabs(u[q]));
            bool bad = mx > g.big;
            if (__any(bad)) {
                bad = false;
#pragma unroll
                for (int q = 0; q < M; ++q) {
                    const T a = __builtin_fabs(u[q]);
                    bad = bad || (a > g.big && __builtin_isfinite(a));
                }
            }
            if (!__any(bad)) {
                int j = 0;
                while (g.tiny > T(0) && j < g.steps) {
                    T mn = __builtin_fabs(u[0]);
#pragma unroll
                    for (int q = 1; q < M; ++q)
                        mn = __builtin_fmin(mn, __builtin_fabs(u[q]));
                    bool sub = mn < g.tiny;
                    if (__any(sub)) {
                        sub = false;
#pragma unroll
                        for (int q = 0; q < M; ++q) {
                            const T a = __builtin_fabs(u[q]);
                            sub = sub || (a < g.tiny && a != T(0));
                        }
                        if (__any(sub))
                            break;
                    }
                    const int upto = min(j + g.rows, g.steps);
                    heat_rows<HeatExact<T>, M>(u, j, upto, g.c, each);
                    j = upto;
                }
                if (j < g.steps)
                    heat_rows<HeatLap<T>, M>(u, j, g.steps, g.c, each);
                return;
            }
            if (g.guard != 0 && threadIdx.x == 0)
                atomicMax(&g_form_mark, g.guard);
        }
    }
    heat_rows<S, M>(u, 0, g.steps, g.c, each);
}

// ------------------------------------------------------------------- KS
// Three evaluations of the KS step with the same bits.
//  kKsWritten  the operations as written (30 a point and step; 22 on KSFmaF64).
//  kKsLap      D2's (l + r) - 2c as fma(-2, c, l + r), as in HeatLap (26).
//              Needs |a| <= MAX/2 for every a that D2 is applied to.
//  kKsExact    for c1 = 1/(2dx) and c2 = 1/dx^2 powers of two: multiplications
//              by them are exact, so they move into the operation that takes
//              the product (fma), and b = D2(a) is kept as b/c2, which saves
//              its multiplication (20; KSFmaF64 18).  With X = -F(a, b) and
//              B = b/c2: X/c2 = (a*(ra - la)*(c1/c2) + B) + D2(B), every
//              operation the written one scaled by a power of two.  Needs no
//              underflow: a scaled result below the smallest normal number
//              would round where the written one does not.
// 2^20 points: 1.00 us a step in kKsExact, 1.16 in kKsLap; KSFmaF64 0.97 in
// kKsExact, 1.03 as written.
// Both hold for a whole step if 2^-400 <= |u| <= 1e30 at its start and the
// constants are moderate (window_form: all at most 1e10, and for kKsExact
// c2 in [1, 2^8], c1 in [2^-8, 2^8]).  From above: |w| <= 4e40, |F| <= 3e70,
// |v| <= 3e80, |z| <= 2e91, |F| <= 2e171, |u'| <= 2e181.  From below, by
// the units the values are multiples of (rounding never makes one finer): u of
// 2^-452, and so is u[i+1] - u[i-1], so a product of two is 0 or at least
// 2^-852; v = u - h*X is 0 or at least 2^-54 |u| (what cancellation leaves is
// half a unit of u or more), so a multiple of 2^-506, and a product of v and
// a difference of two v is 0 or at least 2^-960, a multiple of 2^-1012.
// Divided by the powers of two above that is a multiple of 2^-1036, so every
// scaled sum is exact where the smallest subnormal, 2^-1074, could matter.
// So the wave checks u at every step of a stage: the largest and the smallest
// magnitude of all points' high words, compared as binary32 bit patterns (a
// high word's top bits order like the number; patterns of binary32 NaNs start
// at 2^1017, which a step that starts below 1e30 cannot reach): one v_max3 and
// one v_min3 per two points.  A window that leaves the range is loaded again
// and runs the stage as written (its input is intact: stages go from one
// buffer to the other).
enum { kKsWritten = 0, kKsLap = 1, kKsExact = 2 };

template <class S>
constexpr bool is_ks = std::is_base_of_v<KSF64, S>;
template <class S>
constexpr bool is_ks_fma = std::is_base_of_v<KSFmaF64, S>;

// One Runge-Kutta half of a step for all points: out = u + coef*F(a, D2(a))
// (out may be u)
template <class S, int FORM, int M>
__device__ __forceinline__ void ks_half(const double (&a)[M], const double (&u)[M],
                                        double (&out)[M], double coef, const KSF64::Consts& k,
                                        double c1s)
{
    constexpr bool kFma = is_ks_fma<S>;
    auto lap = [](double l, double c, double r) {
        if constexpr (FORM == kKsWritten && !kFma)
            return (l + r) - 2.0 * c;
        else
            return fmad(-2.0, c, l + r);
    };
    double b[M];
    {
        const double la = dpp_record<kWaveShr1>(a[M - 1]), ra = dpp_record<kWaveShl1>(a[0]);
#pragma unroll
        for (int q = 0; q < M; ++q) {
            b[q] = lap(q > 0 ? a[q > 0 ? q - 1 : 0] : la, a[q],
                       q + 1 < M ? a[q + 1 < M ? q + 1 : 0] : ra);
            if constexpr (FORM != kKsExact)
                b[q] = b[q] * k.c2;
        }
        const double lb = dpp_record<kWaveShr1>(b[M - 1]), rb = dpp_record<kWaveShl1>(b[0]);
#pragma unroll
        for (int q = 0; q < M; ++q) {
            const double al = q > 0 ? a[q > 0 ? q - 1 : 0] : la;
            const double ar = q + 1 < M ? a[q + 1 < M ? q + 1 : 0] : ra;
            const double bl = q > 0 ? b[q > 0 ? q - 1 : 0] : lb;
            const double br = q + 1 < M ? b[q + 1 < M ? q + 1 : 0] : rb;
            const double d2 = lap(bl, b[q], br);
            if constexpr (FORM == kKsExact) {
                // c1s = c1/c2, coef = h*c2 or dt*c2
                double t;
                if constexpr (kFma)
                    t = fmad(a[q], (ar - al) * c1s, b[q]);
                else
                    t = fmad(a[q] * (ar - al), c1s, b[q]);
                const double x = fmad(d2, k.c2, t);
                out[q] = kFma ? fmad(-coef, x, u[q]) : u[q] - coef * x;
            } else {
                const double d1 = (ar - al) * k.c1;
                const double t = kFma ? fmad(a[q], d1, b[q]) : a[q] * d1 + b[q];
                const double f = -(t + d2 * k.c2);
                out[q] = kFma ? fmad(coef, f, u[q]) : u[q] + coef * f;
            }
        }
    }
}

// `steps` KS steps of the window; returns (kKsLap, kKsExact) whether every
// step's u stayed in the form's range
template <class S, int FORM, int M, class Each>
__device__ __forceinline__ bool ks_rows(double (&u)[M], int steps, const KSF64::Consts& k,
                                        Each&& each)
{
    const double c1s = k.c1 / k.c2;   // exact where it is used (kKsExact)
    const double ch = FORM == kKsExact ? k.h * k.c2 : k.h;
    const double cf = FORM == kKsExact ? k.dt * k.c2 : k.dt;
    float hi = 0.0f, lo = __int_as_float(0x7f7fffff);
    double v[M];
    for (int s = 0; s < steps; ++s) {
        ks_half<S, FORM, M>(u, u, v, ch, k, c1s);
        ks_half<S, FORM, M>(v, u, u, cf, k, c1s);
        each(s);
        if constexpr (FORM != kKsWritten) {
#pragma unroll
            for (int q = 0; q < M; q += 2) {
                const int x = __double2hiint(u[q]), y = __double2hiint(u[q + 1 < M ? q + 1 : q]);
                asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(hi) : "v"(x), "v"(y));
                if constexpr (FORM == kKsExact)
                    asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(lo) : "v"(x), "v"(y));
            }
        }
    }
    if constexpr (FORM == kKsWritten)
        return true;
    // high words: 1e30 = 0x46293e59..., 2^-400 = 0x26f00000
    const bool ok = hi < __int_as_float(0x46293e59) &&
                    (FORM != kKsExact || lo > __int_as_float(0x26f00000));
    return __all(ok);
}

// ---------------------------------------------------------------- Euler
// One flux or slope sub-timestep of all M cells of the lanes.  In a flux
// sub-timestep every cell computes the face to its right once and takes the
// one to its left from the cell before (in the next lane by DPP).  A row is
// about 480 instructions a cell, divisions and square roots most of them, so
// neither the halo moves (60 DPP a step) nor the field's traffic matter; M is
// bounded by the registers of nine values a cell.  Against the diamonds (two
// waves per SIMD, a fifth of the slots in fill and drain; 4096 cells: two rows
// a level): 2^20 cells 2.3e10 -> 5.7e10 cell-steps/s untuned (4.2e10 tuned),
// 4096 cells 8.7 -> 1.7 us a step (euler_half below takes both further).
template <class S, int PH, int M>
__device__ __forceinline__ void window_phase(typename S::Pt (&P)[M], const typename S::Consts& c)
{
    using Pt = typename S::Pt;
    const Pt right = dpp_record<kWaveShl1>(P[0]);
    if constexpr (face_phase<S, PH>()) {
        using Face = typename S::Face;
        Face F[M];
#pragma unroll
        for (int q = 0; q < M; ++q)
            F[q] = S::template face_of<PH>(P[q], q + 1 < M ? P[q + 1 < M ? q + 1 : 0] : right, c);
        Face prev = dpp_record<kWaveShr1>(F[M - 1]);
#pragma unroll
        for (int q = 0; q < M; ++q) {
            P[q] = S::template step_faces<PH>(P[q], prev, F[q], c);
            prev = F[q];
        }
    } else {
        Pt prev = dpp_record<kWaveShr1>(P[M - 1]);
#pragma unroll
        for (int q = 0; q < M; ++q) {
            const Pt cur = P[q];
            P[q] = S::template step<PH>(prev, cur, q + 1 < M ? P[q + 1 < M ? q + 1 : 0] : right, c);
            prev = cur;
        }
    }
}

// The same step with the same bits from 300 instruction slots a cell instead of
// 490 (2^20 cells: 19.1 -> 12.6 us a step in 384-cell windows of 3 steps, 11.9
// in windows of 256 cells and 6 steps; 4096: 1.56 -> 1.04), for states far from
// the ends of the exponent range (EulerRange):
//  - halvings are exact, so 0.5*x + y is fma(0.5, x, y), and faces are kept as
//    2F with the half moved into the step's coefficient;
//  - a/b and sqrt(x) are the sequences the compiler emits for them (Newton steps
//    on the hardware's estimates and a fused residual, Markstein's method)
//    without the scalings and special cases, which do nothing for such
//    operands; the two quotients by one density, and by one Roe weight, share
//    their reciprocal;
//  - minmod(a, b) = max(0, min(a, b)) + min(0, max(a, b)), +0 where the written
//    one returns 0; for NaNs it differs, which the ranges exclude.
// Ranges, checked at every half step of a stage: density and energy in
// [2^-100, 2^100], |m| <= 2^100 and 0 or at least 2^-400, and a positive Roe
// sound speed squared (constants moderate: window_form).  Then velocities are 0
// or 2^-555..2^201, quotients' operands differ by less than 2^768 and are 0 or at
// least 2^-660 (no scaling), sums that cancel leave multiples of 2^-959 or
// more (halvings exact), and nothing overflows.  A zero momentum's sign may
// change in its velocity, which only multiplies by zero from there.  The ring
// of lanes is closed (wave rotations), so that the columns that go wrong at a
// window's ends stay ordinary gas states instead of leaving the ranges.  A
// window that does leave them is loaded again and runs the stage as written.
constexpr int kWaveRor1 = 0x13C;   // lane i receives lane i-1, lane 0 lane 63
constexpr int kWaveRol1 = 0x134;

struct Recip {
    double d, y;
    __device__ __forceinline__ explicit Recip(double x) : d(x), y(__builtin_amdgcn_rcp(x))
    {
        y = fmad(y, fmad(-d, y, 1.0), y);
        y = fmad(y, fmad(-d, y, 1.0), y);
    }
    __device__ __forceinline__ double times(double n) const   // n / d
    {
        const double q = n * y;
        return fmad(fmad(-d, q, n), y, q);
    }
};

__device__ __forceinline__ double plain_sqrt(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = y * 0.5;
    const double r = fmad(-h, g, 0.5);
    g = fmad(g, r, g);
    h = fmad(h, r, h);
    g = fmad(fmad(-g, g, x), h, g);
    return fmad(fmad(-g, g, x), h, g);
}

// smallest and largest high words seen of what has to stay in range
struct EulerRange {
    int lo, hi;        // density and energy
    unsigned mlo;      // twice |m|'s high word, less one (0: the largest)
    int mhi;           // |m|'s high word
    int c2;            // the sound speed squared
    __device__ __forceinline__ void see(const Cons& v)
    {
        const int r = __double2hiint(v.r), e = __double2hiint(v.e), m = __double2hiint(v.m);
        lo = min(min(lo, r), e);
        hi = max(max(hi, r), e);
        mlo = min(mlo, ((unsigned)m << 1) - 1u);
        mhi = max(mhi, m & 0x7fffffff);
    }
    // high words: 2^-100 = 0x39b00000, 2^100 = 0x46300000, 2^-400 = 0x26f00000
    __device__ __forceinline__ bool ok() const
    {
        return lo >= 0x39b00000 && hi < 0x46300000 && mlo >= 2u * 0x26f00000u - 1u &&
               mhi < 0x46300000 && c2 > 0;
    }
};

// one side of a face: state, the rest of its flux, velocity, enthalpy, root density
struct EulerSide {
    Cons q;
    double f1, f2, u, H, a;
    __device__ __forceinline__ EulerSide(const Cons& v, double gm1) : q(v)
    {
        const Recip y(q.r);
        u = y.times(q.m);
        const double mu = q.m * u;
        const double p = gm1 * fmad(-0.5, mu, q.e);
        const double ep = q.e + p;
        f1 = mu + p;
        f2 = ep * u;
        H = y.times(ep);
        a = plain_sqrt(q.r);
    }
};

// twice the face flux
__device__ __forceinline__ Cons euler_face2(const EulerSide& L, const EulerSide& R, double gm1,
                                            int& c2min)
{
    const Recip w(L.a + R.a);
    const double ur = w.times(L.a * L.u + R.a * R.u);
    const double Hr = w.times(L.a * L.H + R.a * R.H);
    const double c2 = gm1 * fmad(-0.5, ur * ur, Hr);
    c2min = min(c2min, __double2hiint(c2));
    const double lam = __builtin_fabs(ur) + plain_sqrt(c2);
    return Cons{(L.q.m + R.q.m) - lam * (R.q.r - L.q.r), (L.f1 + R.f1) - lam * (R.q.m - L.q.m),
                (L.f2 + R.f2) - lam * (R.q.e - L.q.e)};
}

__device__ __forceinline__ double quick_minmod(double a, double b)
{
    return __builtin_fmax(0.0, __builtin_fmin(a, b)) + __builtin_fmin(0.0, __builtin_fmax(a, b));
}

// out = base - 2*half_coef * dF(v, slope(v)) for the lane's M cells (out may be base)
template <int M>
__device__ __forceinline__ void euler_half(const Cons (&v)[M], const Cons (&base)[M],
                                           Cons (&out)[M], double half_coef, double gm1,
                                           EulerRange& rng)
{
    const Cons vl = dpp_record<kWaveRor1>(v[M - 1]), vr = dpp_record<kWaveRol1>(v[0]);
    Cons s[M];
    Cons dl{v[0].r - vl.r, v[0].m - vl.m, v[0].e - vl.e};
#pragma unroll
    for (int q = 0; q < M; ++q) {
        const Cons n = q + 1 < M ? v[q + 1 < M ? q + 1 : 0] : vr;
        const Cons dr{n.r - v[q].r, n.m - v[q].m, n.e - v[q].e};
        s[q] = Cons{quick_minmod(dl.r, dr.r), quick_minmod(dl.m, dr.m), quick_minmod(dl.e, dr.e)};
        dl = dr;
    }
    const Cons sr = dpp_record<kWaveRol1>(s[0]);
    auto face = [&](int q) {   // between cell q and the one to its right
        const Cons& a = v[q];
        const Cons b = q + 1 < M ? v[q + 1 < M ? q + 1 : 0] : vr;
        const Cons t = q + 1 < M ? s[q + 1 < M ? q + 1 : 0] : sr;
        const EulerSide L(Cons{fmad(0.5, s[q].r, a.r), fmad(0.5, s[q].m, a.m), fmad(0.5, s[q].e, a.e)},
                          gm1);
        const EulerSide R(Cons{fmad(-0.5, t.r, b.r), fmad(-0.5, t.m, b.m), fmad(-0.5, t.e, b.e)}, gm1);
        return euler_face2(L, R, gm1, rng.c2);
    };
    const Cons last = face(M - 1);
    Cons prev = dpp_record<kWaveRor1>(last);
#pragma unroll
    for (int q = 0; q < M; ++q) {
        const Cons F = q + 1 < M ? face(q) : last;
        out[q] = Cons{base[q].r - half_coef * (F.r - prev.r), base[q].m - half_coef * (F.m - prev.m),
                      base[q].e - half_coef * (F.e - prev.e)};
        rng.see(out[q]);
        prev = F;
    }
}

// How a window passes between HBM and the lanes' blocks of M points.  Reading a
// block per lane straight from HBM spreads every 16-byte access of a wave over
// 64 cache lines.  Where one wave fills its SIMD (blocks of 128 to 208 bytes,
// the windows of about 2^20 points) nothing hides that: a stage of heat
// (M = 20) took 8 us beside its rows, 4.5 us when the wave reads and writes
// 16-byte quads in order (1 KB an instruction) and turns them through LDS:
// lane l's block starts at quad l*(kQuads + kPad), kPad making the stride odd
// against bank conflicts.  Smaller blocks spread less, and with several waves
// on a SIMD (larger blocks, at 2^24 points) the turn costs more than it saves
// (heat M = 48: 219 us a stage without, 237 with it).
template <class T, int M>
struct WindowTurn {
    static constexpr int kBytes = M * (int)sizeof(T);
    static constexpr bool kUse =
        16 % sizeof(T) == 0 && kBytes >= 128 && kBytes <= 208 && kBytes % 16 == 0;
    static constexpr int kQuads = kBytes / 16;
    static constexpr int kPad = kQuads % 2 == 0 ? 1 : 0;
};
struct alignas(16) Quad {
    unsigned w[4];
};
// a quad of field values wherever it starts (values are aligned to themselves)
template <class T>
struct alignas(sizeof(T) % 8 == 0 ? 8 : 4) LooseQuad {
    unsigned w[4];
};

template <class T, int M>
__device__ __forceinline__ Quad* window_lds()
{
    using Turn = WindowTurn<T, M>;
    __shared__ Quad buf[64 * (Turn::kQuads + Turn::kPad)];
    return buf;
}

// A lane's M points of the window that starts at point x0 of the ring
// (-n < x0 < n where n >= 64*M).
template <class T, int M>
__device__ __forceinline__ void window_load(T (&u)[M], const T* in, int64_t n, int64_t x0)
{
    constexpr int W = 64 * M;
    const int lane = threadIdx.x;
    if (x0 >= 0 && x0 + W <= n) {
        if constexpr (WindowTurn<T, M>::kUse) {
            constexpr int Q = WindowTurn<T, M>::kQuads, pad = WindowTurn<T, M>::kPad;
            const auto* p = reinterpret_cast<const LooseQuad<T>*>(in + x0);
            Quad* lds = window_lds<T, M>();
            LooseQuad<T> r[Q];   // all loads in flight before the first is turned
#pragma unroll
            for (int i = 0; i < Q; ++i)
                r[i] = p[i * 64 + lane];
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const int e = i * 64 + lane;
                __builtin_memcpy(&lds[e + pad * (e / Q)], &r[i], 16);
            }
            __syncthreads();
            Quad w[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i)
                w[i] = lds[lane * (Q + pad) + i];
            __builtin_memcpy(u, w, sizeof(u));
            __syncthreads();
        } else {
            const T* p = in + (x0 + lane * M);
#pragma unroll
            for (int q = 0; q < M; ++q)
                u[q] = p[q];
        }
    } else {   // the window crosses the ring's seam, perhaps more than once
        int64_t x = x0 + lane * M;
        if (n >= W) {
            x = x < 0 ? x + n : (x >= n ? x - n : x);
        } else {
            const int y = (int)x % (int)n;
            x = y < 0 ? y + n : y;
        }
#pragma unroll
        for (int q = 0; q < M; ++q) {
            u[q] = in[x];
            x = x + 1 == n ? 0 : x + 1;
        }
    }
}

// A KS stage of the window: the cheapest form its values allow, and the
// operations as written where a value leaves the form's range on the way.
template <class S, int M, class Each>
__device__ __forceinline__ void ks_advance(double (&u)[M], const WindowArgs<S>& g, int64_t x0,
                                           Each&& each)
{
    if (g.fused != 0) {
        // (a NaN passes as itself: its results are NaNs in every form)
        double mx = 0.0, mn = __builtin_fabs(u[0]);
#pragma unroll
        for (int q = 0; q < M; ++q) {
            mx = __builtin_fmax(mx, __builtin_fabs(u[q]));
            mn = __builtin_fmin(mn, __builtin_fabs(u[q]));
        }
        if (__all(mx <= g.big)) {
            bool ok;
            if (g.tiny != 0.0 && !__any(mn < g.tiny))
                ok = ks_rows<S, kKsExact, M>(u, g.steps, g.c, each);
            else if constexpr (!is_ks_fma<S>)
                ok = ks_rows<S, kKsLap, M>(u, g.steps, g.c, each);
            else
                ok = ks_rows<S, kKsWritten, M>(u, g.steps, g.c, each);
            if (ok)
                return;
            window_load<double, M>(u, g.in, g.n, x0);
        }
    }
    ks_rows<S, kKsWritten, M>(u, g.steps, g.c, each);
}

template <class S, int M>
__device__ __forceinline__ void euler_advance(typename S::T (&u)[M], const WindowArgs<S>& g,
                                              int64_t x0)
{
    if (g.fused != 0) {
        EulerRange rng{0x7fffffff, 0, 0xffffffffu, 0, 0x7fffffff};
        bool in = true;
#pragma unroll
        for (int q = 0; q < M; ++q) {
            rng.see(u[q]);
            in = in && (u[q].m == 0.0 || __builtin_fabs(u[q].m) >= 0x1p-400);
        }
        if (__all(in && rng.ok())) {
            const double ch = 0.5 * g.c.ch, cf = 0.5 * g.c.cf;
            Cons r[M];
            for (int s = 0; s < g.steps; ++s) {
                euler_half<M>(u, u, r, ch, g.c.gm1, rng);
                euler_half<M>(r, u, u, cf, g.c.gm1, rng);
            }
            if (__all(rng.ok()))
                return;
            window_load<Cons, M>(u, g.in, g.n, x0);
        }
    }
    typename S::Pt P[M];
#pragma unroll
    for (int q = 0; q < M; ++q)
        P[q] = S::from_field(u[q]);
    for (int s = 0; s < g.steps; ++s) {
        window_phase<S, 0, M>(P, g.c);
        window_phase<S, 1, M>(P, g.c);
        window_phase<S, 2, M>(P, g.c);
        window_phase<S, 3, M>(P, g.c);
    }
#pragma unroll
    for (int q = 0; q < M; ++q)
        u[q] = S::to_field(P[q]);
}

// Store the owned points [t0, t0 + cnt) of a window whose column `halo` is t0.
template <class T, int M>
__device__ __forceinline__ void window_store(const T (&u)[M], T* out, int64_t t0, int halo, int cnt)
{
    const int lane = threadIdx.x;
    T* base = out + (t0 - halo);   // the window's column 0
    if constexpr (WindowTurn<T, M>::kUse) {
        constexpr int Q = WindowTurn<T, M>::kQuads, pad = WindowTurn<T, M>::kPad;
        constexpr int V = 16 / (int)sizeof(T);
        Quad* lds = window_lds<T, M>();
        Quad w[Q];
        __builtin_memcpy(w, u, sizeof(u));
#pragma unroll
        for (int i = 0; i < Q; ++i)
            lds[lane * (Q + pad) + i] = w[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int e = i * 64 + lane;
            T v[V];
            __builtin_memcpy(v, &lds[e + pad * (e / Q)], 16);
            const int c = e * V - halo;   // the quad's first column among the owned
            if (c >= 0 && c + V <= cnt) {
                LooseQuad<T> x;
                __builtin_memcpy(&x, v, 16);
                *reinterpret_cast<LooseQuad<T>*>(base + e * V) = x;
            } else {
#pragma unroll
                for (int q = 0; q < V; ++q)
                    if (c + q >= 0 && c + q < cnt)
                        base[e * V + q] = v[q];
            }
        }
    } else {
        const int c0 = lane * M - halo;   // this lane's first column among the owned
        T* o = base + lane * M;
        if (c0 >= 0 && c0 + M <= cnt) {
#pragma unroll
            for (int q = 0; q < M; ++q)
                o[q] = u[q];
        } else {
#pragma unroll
            for (int q = 0; q < M; ++q)
                if (c0 + q >= 0 && c0 + q < cnt)
                    o[q] = u[q];
        }
    }
}

// One tile's stage: load, advance, store the owned points.  ALL: every step's
// field is stored, step j of the stage (from 0) at out + j*n.
template <class S, int M, bool ALL = false>
__device__ __forceinline__ void window_tile(const WindowArgs<S>& g, unsigned tile)
{
    using T = typename S::T;
    const int64_t t0 = (int64_t)tile * g.own;
    const int64_t x0 = t0 - g.halo;
    const int64_t left = g.n - t0;
    const int cnt = (int)(left < g.own ? left : g.own);
    T u[M];
    window_load<T, M>(u, g.in, g.n, x0);
    auto each = [&](int j) {
        if constexpr (ALL)
            window_store<T, M>(u, g.out + j * g.n, t0, g.halo, cnt);
    };
    if constexpr (is_ks<S>) {
        ks_advance<S, M>(u, g, x0, each);
    } else if constexpr (has_faces<S>::value) {
        static_assert(!ALL, "the adjoint's stencils only");
        euler_advance<S, M>(u, g, x0);
    } else {
        heat_advance<S, M>(u, g, each);
    }
    if constexpr (!ALL)
        window_store<T, M>(u, g.out, t0, g.halo, cnt);
}

// Workgroups are dealt to the eight XCDs in turn: workgroup b of a launch of
// `count` takes an index such that each XCD has a contiguous run of them
// (count or more: none).
__device__ __forceinline__ unsigned xcd_run(unsigned b, unsigned count)
{
    const unsigned per = (count + 7) / 8, x = b & 7, i = b >> 3;
    return i < per ? x * per + i : count;
}

// One stage of one field: workgroup = one wave = one tile.  Neighbouring tiles
// run on one XCD, so that the halos they share are read through one L2.
// ALL: of every step's field (window_tile).
template <class S, int M, bool ALL>
__global__ __launch_bounds__(64) void window_kernel(WindowArgs<S> g)
{
    const unsigned tile = xcd_run(blockIdx.x, (unsigned)g.tiles);
    if (tile < (unsigned)g.tiles)
        window_tile<S, M, ALL>(g, tile);
}

// ------------------------------------------------------------------ batch
// One stage of every instance of one stencil that still has stages to go: the
// tasks (instance, tile) are sorted by their instance's stage count, so those
// of stage s are the first `count`.  Each instance has its own even number of
// stages, at most h steps each, and its own owned width (equal tiles); odd
// lengths need no cover.  Stages alternate between the instance's field and
// its spare copy.
template <class S>
struct WindowInst {
    typename S::T* u;
    typename S::T* spare;
    int64_t n;
    int own;
    int base, rem;     // stage s advances base + (s < rem) steps
    int fused;         // as WindowArgs::fused
    int e;             // heat: r = 2^-e (0: no exact-product form); KS: 1 for the exact-product form
    typename S::Consts c;
};

template <class S>
struct WindowBatchArgs {
    const WindowInst<S>* inst;
    const BatchTask* tasks;
    unsigned count;
    int stage;
    int halo;
    unsigned long long guard;
};

template <class S, int M>
__global__ __launch_bounds__(64) void window_batch_kernel(WindowBatchArgs<S> b)
{
    using T = typename S::T;
    const unsigned i = xcd_run(blockIdx.x, b.count);
    if (i >= b.count)
        return;
    const BatchTask task = b.tasks[i];
    const WindowInst<S>& I = b.inst[task.inst];
    const bool odd = (b.stage & 1) != 0;
    WindowArgs<S> g;
    g.in = odd ? I.spare : I.u;
    g.out = odd ? I.u : I.spare;
    g.n = I.n;
    g.own = I.own;
    g.steps = I.base + (b.stage < I.rem);
    g.halo = b.halo;
    g.c = I.c;
    g.fused = I.fused;
    if constexpr (is_ks<S>) {
        g.big = 1e30;
        g.tiny = I.e != 0 ? __hiloint2double(0x26f00000, 0) : 0.0;   // 2^-400
        g.guard = 0;
    } else {
        static_assert(sizeof(T) == 8, "the batch takes binary64 stencils");
        g.big = std::numeric_limits<T>::max() / (b.stage == 0 ? 16 : 8);
        g.tiny = I.e != 0 ? __hiloint2double((1 + I.e * g.steps) << 20, 0) : 0.0;   // 2^(e*steps - 1022)
        g.rows = g.steps;
        g.guard = b.stage == 0 ? b.guard : 0;
    }
    window_tile<S, M>(g, (unsigned)task.tile);
}

// ---------------------------------------------------------------- adjoint
// The discrete adjoint on windows: a stage takes the cotangent field of step
// first + steps back to step `first`, each step by the transposed
// sub-timesteps (S::adj) on the forward field the forward pass kept of that
// step, whose middle level (KS: v) is recomputed in registers.  A window's
// cotangents go wrong from its ends by the stencil's radius per step; the
// recomputed v by three columns whatever the depth, which its first step
// passes on: the halo is radius x steps, plus two for KS.
//
// What bounds it: the chain of a step, 40 operations a point (as written 54)
// with 28 DPP moves, one wave per SIMD on the grids this is used for.  Keeping
// every step's field (8 bytes a point and step; the lane-frame stages kept 6)
// costs no recomputation beyond v, no LDS and no halo for forward values:
// against swept_adjoint_kernel's stages of 8 KS steps (forward recomputed, then
// reversed, two rows a level) 2.2 -> 0.86 us a step at 2^16 points, with the
// operations as written and the next step's field loaded during a step.  That
// load is from HBM and takes longer than the step: with the shorter form below
// alone it stayed at 0.86, with the fields of four steps on their way as well
// 0.69.
//
// KS with powers of two for c1 and c2 (ks_adj_quick): the same bits from fewer
// operations.  2m, c2*x and c1*x are exact, so (l + r) - 2m = fma(-2, m, l + r),
// a + c2*x = fma(c2, x, a) and c1*x - b = fma(c1, x, -b): each rounds once where
// the written form does.  Nothing can underflow for c1, c2 >= 1 (a power of
// two scales up); nothing overflows if the cotangents are at most 1e60 at
// either end of each step, the source's weight is, and u is in kKsExact's range
// (|v| <= 3e80, and by the bounds on the constants no value passes 1e200).
// u's range also lets kKsExact recompute v.  Checked at every step like
// ks_rows's; a window that leaves the range runs the stage again as written.
template <class S>
struct WindowAdjArgs {
    const typename S::T* u0;      // field of step 0
    const typename S::T* kept;    // field of step j >= kept0 at kept + (j - kept0)*n
    int64_t kept0;
    const typename S::T* in;      // cotangent of step first + steps (null: zero)
    typename S::T* out;           // cotangent of step `first`
    int64_t n, own;
    int tiles, halo, steps;
    int seed;                     // `in` is the objective's cotangent of the final field
    int64_t first;                // time step of `out`
    int64_t win_first;            // first time step of the objective's window (stages.hpp)
    typename S::T two_w;          // 2 * objective weight
    int quick;                    // KS: the constants allow ks_adj_quick
    typename S::Consts c;
};

// the transposed sub-timestep PH of all points of the window; k: the forward
// values it reads
template <class S, int PH, int M>
__device__ __forceinline__ void adj_phase(typename S::Ad (&a)[M], const typename S::Kept (&k)[M],
                                          const typename S::Consts& c)
{
    using Ad = typename S::Ad;
    using Kept = typename S::Kept;
    Ad prev = dpp_record<kWaveShr1>(a[M - 1]);
    const Ad right = dpp_record<kWaveShl1>(a[0]);
    const Kept kl = dpp_record<kWaveShr1>(k[M - 1]), kr = dpp_record<kWaveShl1>(k[0]);
#pragma unroll
    for (int q = 0; q < M; ++q) {
        const Ad cur = a[q];
        a[q] = S::template adj<PH>(prev, cur, q + 1 < M ? a[q + 1 < M ? q + 1 : 0] : right,
                                   q > 0 ? k[q > 0 ? q - 1 : 0] : kl, k[q],
                                   q + 1 < M ? k[q + 1 < M ? q + 1 : 0] : kr, c);
        prev = cur;
    }
}

// The four transposed KS sub-timesteps of all points: a, the cotangents of u'
// in, of u out; u and v: the step's field and its middle level (KSF64::adj has
// the operations as written).
template <int M>
__device__ __forceinline__ void ks_adj_quick(double (&a)[M], const double (&u)[M],
                                             const double (&v)[M], const KSF64::Consts& k)
{
    // z[q]: the value of point q, from -1 (lane before) to M (lane after)
    struct Row {
        double l, r;
        const double (&z)[M];
        __device__ __forceinline__ explicit Row(const double (&x)[M])
            : l(dpp_record<kWaveShr1>(x[M - 1])), r(dpp_record<kWaveShl1>(x[0])), z(x)
        {
        }
        __device__ __forceinline__ double at(int q) const { return q < 0 ? l : q < M ? z[q] : r; }
        __device__ __forceinline__ double lap(int q) const
        {
            return fmad(-2.0, z[q], at(q - 1) + at(q + 1));
        }
    };
    // c1*(g[i+1]*f[i+1] - g[i-1]*f[i-1]) - g*((f[i+1] - f[i-1])*c1)
    auto cross = [&](const Row& g, const Row& f, int q) {
        const double d = (f.at(q + 1) - f.at(q - 1)) * k.c1;
        return fmad(k.c1, g.at(q + 1) * f.at(q + 1) - g.at(q - 1) * f.at(q - 1), -(g.z[q] * d));
    };
    double g[M], x[M], y[M];
#pragma unroll
    for (int q = 0; q < M; ++q)
        g[q] = k.dt * a[q];
    {
        const Row gr(g), vr(v);
#pragma unroll
        for (int q = 0; q < M; ++q) {
            x[q] = cross(gr, vr, q);
            y[q] = -fmad(k.c2, gr.lap(q), g[q]);
        }
    }
    {
        const Row yr(y);
#pragma unroll
        for (int q = 0; q < M; ++q) {
            x[q] = fmad(k.c2, yr.lap(q), x[q]);
            g[q] = k.h * x[q];
        }
    }
    {
        const Row gr(g), ur(u);
#pragma unroll
        for (int q = 0; q < M; ++q) {
            a[q] = (a[q] + x[q]) + cross(gr, ur, q);
            y[q] = -fmad(k.c2, gr.lap(q), g[q]);
        }
    }
    {
        const Row yr(y);
#pragma unroll
        for (int q = 0; q < M; ++q)
            a[q] = fmad(k.c2, yr.lap(q), a[q]);
    }
}

// The steps of a stage; lam: the cotangents of step `first`.  load(x, p): the
// window of the field p; field(j): the kept field of step j.  False: a value
// left the range of ks_adj_quick.
template <class S, int M, bool kQuick, class Load, class Field>
__device__ __forceinline__ bool adjoint_stage(typename S::T (&lam)[M], const WindowAdjArgs<S>& g,
                                              Load&& load, Field&& field)
{
    using T = typename S::T;
    using Ad = typename S::Ad;
    using Kept = typename S::Kept;
    const int64_t last = g.first + g.steps;
    // fields on their way while a step is computed
    constexpr int kSlots = 4;
    T f[kSlots][M];
    if (g.in != nullptr) {
        load(lam, g.in);
    } else {
#pragma unroll
        for (int q = 0; q < M; ++q)
            lam[q] = T(0);
    }
    Ad a[M];
    if (g.seed != 0 && last >= g.win_first) {
        load(f[0], field(last));
#pragma unroll
        for (int q = 0; q < M; ++q)
            a[q] = S::seed(lam[q], g.two_w, f[0][q], true);
    } else {
#pragma unroll
        for (int q = 0; q < M; ++q)
            a[q] = S::seed(lam[q], g.two_w, T(0), false);
    }
    if constexpr (kQuick) {
        bool in = true;
#pragma unroll
        for (int q = 0; q < M; ++q) {
            lam[q] = S::grad(a[q]);
            in = in && !(__builtin_fabs(lam[q]) > 1e60);   // (a NaN passes as itself)
        }
        if (!__all(in))
            return false;
    }
    float big_a = 0.0f, tiny_u = __int_as_float(0x7f7fffff);
    bool big_u = false;
    auto step = [&](const T (&u)[M], bool source) {
        if constexpr (kQuick) {
            double v[M];
            ks_half<S, kKsExact, M>(u, u, v, g.c.h * g.c.c2, g.c, g.c.c1 / g.c.c2);
            ks_adj_quick<M>(lam, u, v, g.c);
            if (source) {
#pragma unroll
                for (int q = 0; q < M; ++q)
                    lam[q] = lam[q] + g.two_w * u[q];
            }
#pragma unroll
            for (int q = 0; q < M; q += 2) {
                const int q1 = q + 1 < M ? q + 1 : q;
                const int x = __double2hiint(lam[q]), y = __double2hiint(lam[q1]);
                const int z = __double2hiint(u[q]), w = __double2hiint(u[q1]);
                asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(big_a) : "v"(x), "v"(y));
                // (u is loaded anew at each step: its high word may be any)
                big_u = big_u || __builtin_fabs(u[q]) > 1e30 || __builtin_fabs(u[q1]) > 1e30;
                asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(tiny_u) : "v"(z), "v"(w));
            }
        } else {
            Kept k[M];
#pragma unroll
            for (int q = 0; q < M; ++q)
                k[q] = u[q];
            if constexpr (S::NPHASE == 4) {
                typename S::Pt P[M];
#pragma unroll
                for (int q = 0; q < M; ++q)
                    P[q] = S::from_field(u[q]);
                window_phase<S, 0, M>(P, g.c);
                window_phase<S, 1, M>(P, g.c);
                Kept kv[M];
#pragma unroll
                for (int q = 0; q < M; ++q)
                    kv[q] = S::template keep<3>(P[q]);
                adj_phase<S, 3, M>(a, kv, g.c);
                adj_phase<S, 2, M>(a, kv, g.c);
                adj_phase<S, 1, M>(a, k, g.c);
            }
            adj_phase<S, 0, M>(a, k, g.c);
            if (source) {
#pragma unroll
                for (int q = 0; q < M; ++q)
                    a[q] = S::source(a[q], k[q], g.two_w);
            }
        }
    };
    // (a field below the stage's steps is not read: the loads stop at `first`.
    // A stage without steps, the seed alone, loads the field of `first` too:
    // a branch around these loads costs the heat stages 12%)
    auto fetch = [&](T (&u)[M], int64_t j) { load(u, field(j > g.first ? j : g.first)); };
#pragma unroll
    for (int i = 0; i < kSlots; ++i)
        fetch(f[i], last - 1 - i);
    int64_t j = last - 1;
    for (; j - (kSlots - 1) >= g.first; j -= kSlots) {
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            step(f[i], j - i >= g.win_first);
            fetch(f[i], j - i - kSlots);
        }
    }
#pragma unroll
    for (int i = 0; i < kSlots - 1; ++i)
        if (j - i >= g.first)
            step(f[i], j - i >= g.win_first);
    if constexpr (kQuick) {
        // high words: 1e60 = 0x4c63e9e4..., 2^-400 as in ks_rows
        const bool in = big_a < __int_as_float(0x4c63e9e4) && !big_u &&
                        tiny_u > __int_as_float(0x26f00000);
        return (bool)__all(in);
    } else {
#pragma unroll
        for (int q = 0; q < M; ++q)
            lam[q] = S::grad(a[q]);
        return true;
    }
}

template <class S, int M>
__global__ __launch_bounds__(64) void window_adjoint_kernel(WindowAdjArgs<S> g)
{
    using T = typename S::T;
    const unsigned tile = xcd_run(blockIdx.x, (unsigned)g.tiles);
    if (tile >= (unsigned)g.tiles)
        return;
    const int64_t t0 = (int64_t)tile * g.own;
    const int64_t x0 = t0 - g.halo;
    const int64_t left = g.n - t0;
    const int cnt = (int)(left < g.own ? left : g.own);
    auto field = [&](int64_t j) { return j == 0 ? g.u0 : g.kept + (j - g.kept0) * g.n; };
    // byte offsets of the lane's points in a field (n < 2^28: 32 bits): the
    // loads of the loop then have no branch for windows across the seam, which
    // would make each wait for its data at once
    unsigned off[M];
    {
        int64_t x = (x0 + (int)threadIdx.x * M) % g.n;
        x = x < 0 ? x + g.n : x;
#pragma unroll
        for (int q = 0; q < M; ++q) {
            off[q] = (unsigned)x * (unsigned)sizeof(T);
            x = x + 1 == g.n ? 0 : x + 1;
        }
    }
    auto load = [&](T (&v)[M], const T* p) {
#pragma unroll
        for (int q = 0; q < M; ++q)
            v[q] = *reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(p) + off[q]);
    };
    T lam[M];
    bool done = false;
    if constexpr (is_ks<S>)
        done = g.quick != 0 && adjoint_stage<S, M, true>(lam, g, load, field);
    if (!done)
        adjoint_stage<S, M, false>(lam, g, load, field);
    window_store<T, M>(lam, g.out, t0, g.halo, cnt);
}

}  // namespace swept
