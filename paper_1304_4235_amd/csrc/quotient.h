// The quotient b / a from an approximate reciprocal of a (host code too).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace rrt {

// b / a for normal a and 0 <= b < a, from a reciprocal r0 to 2^-24 relative (the
// hardware's is 2^-24.4 at worst): a Newton step takes it to the last bits, and one
// correction of the quotient by its remainder to the correctly rounded quotient (equal
// to the division for each of 2.7e8 pairs of the chord factor; without the Newton step
// up to 19 ulp off).  The division's scaling and special cases, a dozen instructions
// more, have no use for such operands.
__host__ __device__ inline double quotient_from(double b, double a, double r0)
{
    const double r = fma(fma(-r0, a, 1.0), r0, r0), q = b * r;
    return fma(fma(-q, a, b), r, q);
}

}  // namespace rrt
