// The pair arithmetic of the ray paths, shared by the traversal (trace.hip) and
// the recorded paths (paths.hip): the canonical hit predicate's operation
// order, the kernel chord integral and small wave helpers.
#pragma once

#include "internal.h"
#include "quotient.h"

namespace rrt {

__device__ __forceinline__ float tab_eval(const float4* __restrict__ tb, float x)
{
    float s = x * (float)kTabIntervals;
    int i = (int)s;
    i = i < 0 ? 0 : (i > kTabIntervals - 1 ? kTabIntervals - 1 : i);
    float u = s - (float)i;
    float4 c = tb[i];
    return fmaf(fmaf(fmaf(c.w, u, c.z), u, c.y), u, c.x);
}

__device__ __forceinline__ float erf_t_odd(const float4* __restrict__ tb, float z)
{
    float a = fminf(fabsf(z), 1.0f);
    float v = tab_eval(tb, a);
    return z < 0.f ? -v : v;
}

// sign bit of a recorded factor: the hit is near (factors are >= 0)
constexpr uint32_t kNearBit = 0x80000000u;

// The canonical predicate (shared operation order with the FP64 reference):
// d = (r_j - r_p) + s B ; s_par = d.u ; t = clamp(s_par, 0, L) ; c = d - t u ;
// hit <=> |c|^2 < h^2, with the dot products and c in fused multiply-adds as
// written below (dot_u, norm2) and no other contraction.
#pragma clang fp contract(off)
// K/h^2 of one intersection: the chord integral of the kernel (eq. Gt) in
// units of h, over h^2, C e^{-t^2 q^2} [erf(t z2) - erf(t z1)] / h^2.  sp = d.u
// locates the point of the ray nearest the particle, b2 is the squared impact
// parameter and h2 = h^2, all FP64; hf = h.  z1, z2 are the chord's ends in
// units of h, clipped to the sphere and to the segment [0, L].  0 for a
// tangent touch.
//  * The Gaussian: the exponent -a q^2 (a = t^2 log2 e, q^2 = b2 / h2) is
//    formed in FP64; its integer part is applied exactly and its fraction by
//    the hardware 2^x (about 1 ulp).
//  * erf from the LDS table; a chord that spans the whole sphere (z1 = -z2)
//    needs one lookup, erf being odd.
//  * Reciprocals and the square root are the hardware's single instructions
//    (about 1 ulp).
__device__ __forceinline__ float chord_factor(double sp, double b2, double h2, double L,
                                              float hf, const float4* __restrict__ t_erf,
                                              double gc, double ga)
{
    const double l2 = h2 - b2;
    if (!(l2 > 0.0)) return 0.0f;
    const float ih2 = __builtin_amdgcn_rcpf((float)h2);
    const float lh = __builtin_amdgcn_sqrtf(fminf((float)l2 * ih2, 1.0f));
    const float ih = __builtin_amdgcn_rcpf(hf);
    const float z1 = fmaxf((float)(-sp) * ih, -lh);
    const float z2 = fminf((float)(L - sp) * ih, lh);
    if (!(z2 > z1)) return 0.0f;
    const double e = -ga * quotient_from(b2, h2, __builtin_amdgcn_rcp(h2));
    const double en = floor(e);
    const float g = (float)gc * ldexpf(__builtin_amdgcn_exp2f((float)(e - en)), (int)en);
    const float e2 = erf_t_odd(t_erf, z2);
    float e1;
    if (z1 == -z2) e1 = -e2;
    else e1 = erf_t_odd(t_erf, z1);
    return ih2 * (g * (e2 - e1));
}

// The canonical operation order of the pair arithmetic (the same wherever a
// pair is evaluated): a dot product with u, or a squared norm, starts with the
// x product and adds y, then z, by fused multiply-add; a component of d - t u
// is one fused multiply-add.  fma rounds once, as IEEE 754 defines it.
__device__ __forceinline__ double dot_u(double d0, double d1, double d2, const double u[3])
{
    return fma(d2, u[2], fma(d1, u[1], d0 * u[0]));
}

__device__ __forceinline__ double norm2(double c0, double c1, double c2)
{
    return fma(c2, c2, fma(c1, c1, c0 * c0));
}

// The pair's geometry: d = (r_j - r_p) + s B and sp = d.u.
struct PairGeom {
    double d0, d1, d2, sp;
};

// From coordinates already in FP64; for an unshifted image (kShifted false,
// s = 0) the adds of zero are left out, which changes no bit.
template <bool kShifted>
__device__ __forceinline__ PairGeom pair_geom_d(double qx, double qy, double qz, double o0,
                                                double o1, double o2, const double sh[3],
                                                const double u[3])
{
    PairGeom pg;
    pg.d0 = qx - o0;
    pg.d1 = qy - o1;
    pg.d2 = qz - o2;
    if (kShifted) {
        pg.d0 = pg.d0 + sh[0];
        pg.d1 = pg.d1 + sh[1];
        pg.d2 = pg.d2 + sh[2];
    }
    pg.sp = dot_u(pg.d0, pg.d1, pg.d2, u);
    return pg;
}

// K/h^2 of a hit: the squared impact parameter from d - sp u, then the chord.
__device__ __forceinline__ float hit_factor(const PairGeom& pg, const double u[3], float hf,
                                            double L, const float4* __restrict__ t_erf,
                                            double gc, double ga)
{
    const double px = fma(-pg.sp, u[0], pg.d0), py = fma(-pg.sp, u[1], pg.d1),
                 pz = fma(-pg.sp, u[2], pg.d2);
    const double b2 = norm2(px, py, pz);
    const double hj = (double)hf;
    return chord_factor(pg.sp, b2, hj * hj, L, hf, t_erf, gc, ga);
}

#pragma clang fp contract(fast)

// lanes where b holds (the HIP __ballot takes an int and re-tests it)
__device__ __forceinline__ uint64_t wave_ballot(bool b)
{
    return __builtin_amdgcn_ballot_w64(b);
}

// LDS written by some lanes of a wave and read by others: order the accesses
// within the wave (no block barrier needed, the wave runs in lockstep)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace rrt
