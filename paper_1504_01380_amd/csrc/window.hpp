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
// halo, 2*halo of 64*M columns, which deep registers (M up to 48 for heat)
// make small.  Against the diamonds of swept_diamond_cont_kernel, whose
// fill and drain idle a fifth of its slots and whose lane-0 chain, band
// changes and hand-on moves take another 16% of the issue: heat f64 at 2^24
// points 6.2e12 -> 7.8e12 point-updates/s with the same four operations per
// update, 9.9e12 with three (HeatExact below); 4096 points 225 -> 67 ns per
// step (one wave per SIMD and no two-rows-per-level diamond).
#pragma once

#include "kernels.hpp"

namespace swept {

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
    // heat: the forms this stage may take (window_form) and their conditions
    typename S::T big;          // largest finite |u| of the fused forms
    typename S::T tiny;         // smallest nonzero |u| of the exact-product form (0: not allowed)
    unsigned long long guard;   // the call's id on its first stage (marks the call), else 0
    int fused;                  // 0: the canonical form only
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
template <class S, int M>
__device__ __forceinline__ void heat_rows(typename S::T (&u)[M], int rows,
                                          const typename S::Consts& k)
{
    using T = typename S::T;
    for (int j = 0; j < rows; ++j) {
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
    }
}

// Heat's evaluation of a window for one stage.  The conditions of the fused
// forms are checked on the window itself, so that no launch reads the field
// beforehand and every stage is judged on its own data: no finite |u| above
// `big` (HeatLap: with 0 <= r <= 1/2 the values cannot come near the
// overflow of 2u inside a stage; the host passes MAX/16 for the initial field
// and MAX/8, which the run-length bound keeps out of reach, afterwards), and
// for the exact-product form no nonzero |u| below `tiny`.  A wave decides for
// itself; all forms give the same bits.
template <class S, int M>
__device__ __forceinline__ void window_advance(typename S::T (&u)[M], const WindowArgs<S>& g)
{
    using T = typename S::T;
    if constexpr (has_fused_form<S>) {
        if (g.fused != 0) {
            bool bad = false, sub = g.tiny == T(0);
#pragma unroll
            for (int q = 0; q < M; ++q) {
                const T a = __builtin_fabs(u[q]);
                bad = bad || (a > g.big && __builtin_isfinite(a));
                sub = sub || (a < g.tiny && a != T(0));
            }
            if (!__any(bad)) {
                if (!__any(sub))
                    heat_rows<HeatExact<T>, M>(u, g.steps, g.c);
                else
                    heat_rows<HeatLap<T>, M>(u, g.steps, g.c);
                return;
            }
            if (g.guard != 0 && threadIdx.x == 0)
                atomicMax(&g_form_mark, g.guard);
        }
    }
    heat_rows<S, M>(u, g.steps, g.c);
}

// One stage: workgroup = one wave = one tile.  Consecutive tiles go to the
// same XCD (workgroups are dealt to the eight XCDs in turn), so that the
// halos neighbouring tiles share are read through one L2.
template <class S, int M>
__global__ __launch_bounds__(64) void window_kernel(WindowArgs<S> g)
{
    using T = typename S::T;
    constexpr int W = 64 * M;
    const int lane = threadIdx.x;
    const unsigned per = (unsigned)(g.tiles + 7) / 8;
    const unsigned tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (tile >= (unsigned)g.tiles)
        return;
    const int64_t t0 = (int64_t)tile * g.own;
    const int64_t x0 = t0 - g.halo;
    T u[M];
    if (x0 >= 0 && x0 + W <= g.n) {
        const T* p = g.in + (x0 + lane * M);
#pragma unroll
        for (int q = 0; q < M; ++q)
            u[q] = p[q];
    } else {   // the window crosses the ring's seam, perhaps more than once
        int64_t x = x0 + lane * M;
        if (g.n >= W) {
            x = x < 0 ? x + g.n : (x >= g.n ? x - g.n : x);
        } else {
            const int n = (int)g.n;
            const int y = (int)x % n;
            x = y < 0 ? y + n : y;
        }
#pragma unroll
        for (int q = 0; q < M; ++q) {
            u[q] = g.in[x];
            x = x + 1 == g.n ? 0 : x + 1;
        }
    }
    window_advance<S, M>(u, g);
    const int64_t left = g.n - t0;
    const int cnt = (int)(left < g.own ? left : g.own);
    const int c0 = lane * M - g.halo;   // this lane's first column among the owned points
    T* o = g.out + (t0 + c0);
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

}  // namespace swept
