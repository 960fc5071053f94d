// ln(1 + y) in FP64 for the rate quadrature, y >= 0.
//
// The quadrature is bound by its logarithms (36 per rate, GL_SUM), and the library
// log1p serves every argument at about 120 FP64 operations.  Here y >= 0 and
// the terms share one table in LDS, so about 18 do, by the table-driven method
// of Tang (1990, ACM TOMS 16, 378): u = fl(1 + y) = 2^e m
// with m in [1, 2), the table interval i of m (top 7 mantissa bits) gives
// invc_i ~ 1/m and ln(c_i) = -ln(invc_i), and
//   ln(1 + y) = e ln 2 + ln(c_i) + ln(1 + t),  t = m invc_i - 1 + 2^-e (y - (u - 1)) invc_i,
// the last term restoring what rounding 1 + y lost.  Interval 0 has c = 1, so a
// small y returns ln(1 + t), t = y, with full relative accuracy; every term
// is >= 0 otherwise and nothing cancels.  |t| < 2^-7: the Taylor series to t^8
// leaves 2^-59 of t.  Measured against 80-bit logarithms: at most 1.3 ulp, 0.28 in
// the mean (the library's 0.64 and 0.25).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace pic {

constexpr int LOG_N = 128;
constexpr double LOG_Y_MAX = 1e300;  // beyond it the callers take the library log1p

// {invc_i, ln c_i} of the intervals, host side.  Any invc_i near 1 / m serves, so
// of 64 neighbouring doubles the one whose logarithm (in 80 bits) lies closest
// to a double is taken: ln c_i then adds next to no rounding of its own where
// it is small and the terms differ in sign.
inline void log_table(double* t)
{
    for (int i = 0; i < LOG_N; ++i) {
        double invc = i == 0 ? 1.0 : 1.0 / (1.0 + (i + 0.5) / LOG_N), best = 1.0;
        t[2 * i] = invc;
        t[2 * i + 1] = 0.0;
        for (int k = 0; i > 0 && k < 64; ++k, invc = nextafter(invc, 0.0)) {
            const long double l = -logl((long double)invc);
            const double d = (double)l, miss = (double)fabsl(l - d);
            if (miss < best) {
                best = miss;
                t[2 * i] = invc;
                t[2 * i + 1] = d;
            }
        }
    }
}

// 0 <= y <= LOG_Y_MAX; tab: log_table's {invc, ln c} pairs
__host__ __device__ inline double log1p_pos(double y, const double2* tab)
{
    const double u = 1.0 + y;
    const double lost = y - (u - 1.0);
    uint64_t bits;
    __builtin_memcpy(&bits, &u, 8);
    const uint32_t hi = (uint32_t)(bits >> 32);
    const int e = (int)(hi >> 20) - 1023;
    const uint64_t mbits = (uint64_t)((hi & 0xFFFFFu) | 0x3FF00000u) << 32 | (uint32_t)bits;
    double m;
    __builtin_memcpy(&m, &mbits, 8);
    const double2 c = tab[(hi >> 13) & (LOG_N - 1)];
    const double t = fma(ldexp(lost, -e), c.x, fma(m, c.x, -1.0));
    double q = fma(t, -1.0 / 8.0, 1.0 / 7.0);
    q = fma(t, q, -1.0 / 6.0);
    q = fma(t, q, 1.0 / 5.0);
    q = fma(t, q, -1.0 / 4.0);
    q = fma(t, q, 1.0 / 3.0);
    q = fma(t, q, -1.0 / 2.0);
    const double p = fma(t * t, q, t);
    return fma((double)e, 0.693147180559945309417, c.y + p);
}

}  // namespace pic
