// Division by a quantity whose reciprocal is at hand, for host and device code.
#pragma once

#include <math.h>

#if defined(__HIPCC__)
#define LX_QHD __host__ __device__ inline
#else
#define LX_QHD inline
#endif

namespace lx {

// x / d with r = 1 / d rounded: the product x r, corrected once by its
// residual.  The residual is exact, and the result has the division's
// rounding, while neither x r overflows nor the residual underflows
// (|x| above about 1e-290).  A product that is not finite is returned as it is:
// its correction would turn an infinity into NaN.
LX_QHD double quotient_rcp(const double x, const double d, const double r) {
    const double q = x * r;
    const double c = fma(fma(-q, d, x), r, q);
    return __builtin_isfinite(q) ? c : q;
}

}  // namespace lx
