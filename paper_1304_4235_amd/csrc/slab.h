// The polychromatic near slab of the near/far scheme: device code of the rate
// kernel, whose lanes share a march.
#pragma once

#include "physics.h"

namespace rrt {

constexpr int kSlabMaxSteps = 4096;

// ln of the rate at the bottom of a uniform slab (density nH, coefficients
// alpha, gcoll at its temperature) of total hydrogen column Nn, lit by the
// binned spectrum (attenuation table sp) after a far column Nf: the
// polychromatic near slab.  With HI column u below the surface the rate is
// Gamma(Nf + u), the neutral fraction x(u) = x_-(Gamma), and the hydrogen
// column down to u is
// H(u) = int_0^u du' / x(u'); the bottom is where H = Nn.  The march takes
// steps that lower ln Gamma by about 1/2 (6-point Gauss-Legendre on each,
// nodes glx and weights glw on [-1, 1]); inside the step where H passes Nn,
// Newton's method on the depth, kept to a bracket (dH/du = 1/x).  Once x is
// within 1e-13 of x_ce, 1/x stays constant and the rest of the slab is linear.
//
// A march is one long serial chain, so kSlabLanes lanes of a wave share it: the
// first six evaluate a step's nodes at once, the next its far end, and every
// lane of the group sums the nodes in their order (all hold the same values and
// take the same branches).  All lanes of a group call it together.
constexpr int kSlabLanes = 8;
__device__ inline double slab_ln_rate_poly(double Nf, double Nn, double nH, double alpha,
                                           double gcoll, const AttenuationTable& sp,
                                           const double* glx, const double* glw)
{
    double sb = 0.0;
    double l = ln_rate_after(Nf, sp, &sb);
    if (!(Nn > 0.0) || l == -INFINITY) return l;
    const double xce = alpha / (alpha + gcoll);
    const int role = threadIdx.x & (kSlabLanes - 1);
    double gx = 0.0, gw = 0.0;
    for (int q = 0; q < 6; ++q)
        if (role == q) gx = glx[q], gw = glw[q];
    // int_{u0}^{u1} du / x, and ln Gamma, its slope and x at u1
    double le = 0.0, se = 0.0, xe = 0.0;
    auto piece = [&](double u0, double u1) {
        const double c = 0.5 * (u0 + u1), h = 0.5 * (u1 - u0);
        double sl = 0.0;
        const double lv = ln_rate_after(Nf + (role < 6 ? c + h * gx : u1), sp, &sl);
        const double xv = x_minus(exp(lv), nH, alpha, gcoll);
        const double t = gw / xv;
        double acc = 0.0;
        for (int q = 0; q < 6; ++q) acc += __shfl(t, q, kSlabLanes);
        le = __shfl(lv, 6, kSlabLanes);
        se = __shfl(sl, 6, kSlabLanes);
        xe = __shfl(xv, 6, kSlabLanes);
        return acc * h;
    };
    double u = 0.0, H = 0.0, x = x_minus(exp(l), nH, alpha, gcoll);
    for (int step = 0; step < kSlabMaxSteps; ++step) {
        if (xce / x - 1.0 < 1e-13) break;             // neutral from here on
        const double du = 0.5 / sb;
        const double I = piece(u, u + du);
        if (H + I >= Nn) {
            double lo = 0.0, hi = du, t = du * ((Nn - H) / I);
            for (int it = 0; it < 60; ++it) {
                const double F = H + piece(u, u + t) - Nn;
                if (fabs(F) <= 1e-15 * Nn) break;     // t is the bottom
                if (F > 0.0) hi = t;
                else lo = t;
                double tn = t - F * xe;
                if (!(tn > lo && tn < hi)) tn = 0.5 * (lo + hi);
                const bool done = fabs(tn - t) <= 1e-15 * (u + t);
                t = tn;
                if (done) break;
            }
            return ln_rate_after(Nf + u + t, sp, nullptr);
        }
        H += I;
        u += du;
        sb = se;
        x = xe;
    }
    return ln_rate_after(Nf + u + (Nn - H) * xce, sp, nullptr);
}

}  // namespace rrt
