// FP64 quotients, rounded as the IEEE operation.  A reciprocal starts from the
// hardware estimate (about 24 bits) and takes Newton steps; a quotient is then
// a y corrected once by its exact residual, which rounds it correctly but for
// ties within about 2^-50, also where y is a product of reciprocals and a few
// units in the last place off.  So several quotients by one divisor, and
// divisors that are products of geometry factors, share their reciprocals: a
// compiled FP64 division is about eleven instructions, a quotient three, a
// reciprocal five.  Divisors are normal numbers with normal reciprocals.
#pragma once

#include <hip/hip_runtime.h>

namespace ffpic {

__device__ __forceinline__ double rcp64(double b) {
    double y = __builtin_amdgcn_rcp(b);
    y = __builtin_fma(__builtin_fma(-b, y, 1.0), y, y);
    return __builtin_fma(__builtin_fma(-b, y, 1.0), y, y);
}
// a / b with y the reciprocal of b
__device__ __forceinline__ double quot(double a, double b, double y) {
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-b, q, a), y, q);
}
// whether b is a divisor that rcp64 and quot take (0, tiny, huge and
// non-finite ones are left to the division)
__device__ __forceinline__ bool quot_ok(double b) { return b >= 0x1p-900 && b <= 0x1p900; }

}  // namespace ffpic
