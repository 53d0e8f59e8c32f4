// julia_trap.h -- discs about an attracting cycle that no orbit leaves.  For host
// and device code alike; host compilers need nothing else.
#pragma once

#include <math.h>

#ifdef __HIPCC__
#define JR_HOST_DEVICE __host__ __device__
#else
#define JR_HOST_DEVICE
#endif

namespace jr {

// Traps.  A Julia image's bounded orbits end in an attracting cycle z_0 ..
// z_{p-1} of Z^d + C, if there is one, and the critical point 0 leads to it.
// Discs about the cycle, radii r_k with
//     r_{k+1} >= (|z_k| + r_k)^d - |z_k|^d + eps   and   r_p <= r_0,
// trap orbits: |(z + h)^d - z^d| <= (|z| + |h|)^d - |z|^d, so an iterate within
// r_k of z_k is followed by one within r_{k+1} of z_{k+1}, as long as eps covers
// what the rounding of one step moves it by; and with |z_k| + r_k < 2 none of
// them ever escapes, so the count is the cap.  eps = 1e-5 d: a step in binary32
// moves Z' by at most d * 1e-6 (d - 1 products of relative error 3e-7 with
// |W| < 4, one sum, C rounded to binary32); binary64 and float-float by less.
constexpr int kTrapPeriodMax = 16;
constexpr double kTrapMinRadius = 0.004;
constexpr int kCriticalSteps = 512;

// Iterates the critical orbit of Z^degree + C.  Returns the period of a trap
// (its disc 0 in x, y, r), or 0: none was found within kCriticalSteps.  `steps`
// is the step at which the critical orbit escaped, kCriticalSteps if it did not: the higher,
// the longer the image's orbits take.
JR_HOST_DEVICE inline int find_trap(double cr, double ci, int degree, float* x, float* y,
                                    float* r, int* steps) {
    const double eps = 1e-5 * degree;
    double zx = 0.0, zy = 0.0, near = 0.02;
    int n = 0;
    auto next = [&](double& a, double& b) {
        double wr = a, wi = b;
        for (int k = 1; k < degree; ++k) {
            const double t = wr * a - wi * b;
            wi = wr * b + wi * a;
            wr = t;
        }
        a = wr + cr;
        b = wi + ci;
    };
    *steps = kCriticalSteps;
    for (int stop = 32; stop <= kCriticalSteps; stop *= 4, near *= 0.2) {
        for (; n < stop; ++n) {
            if (!(zx * zx + zy * zy <= 4.0)) {
                *steps = n;
                return 0;
            }
            next(zx, zy);
        }
        // the first near return is taken as the period
        double ux = zx, uy = zy, m[kTrapPeriodMax], off = 0.0;
        int p = 0;
        for (int k = 0; k < kTrapPeriodMax && p == 0; ++k) {
            m[k] = sqrt(ux * ux + uy * uy);
            next(ux, uy);
            off = sqrt((ux - zx) * (ux - zx) + (uy - zy) * (uy - zy));
            if (off < near) p = k + 1;
        }
        if (p == 0) continue;
        // the largest disc 0 of a falling sequence whose discs close
        for (double r0 = 1.0; r0 >= kTrapMinRadius; r0 *= 0.8) {
            double rk = r0, least = r0;
            bool ok = true;
            for (int k = 0; k < p && ok; ++k) {
                ok = m[k] + rk <= 1.99;
                double a = 1.0, b = 1.0;
                for (int j = 0; j < degree; ++j) {
                    a *= m[k] + rk;
                    b *= m[k];
                }
                least = least < rk ? least : rk;
                rk = a - b + eps;
            }
            if (ok && rk + off <= r0 && least >= kTrapMinRadius) {
                *x = (float)zx;
                *y = (float)zy;
                *r = (float)r0;
                return p;
            }
        }
    }
    return 0;
}

}  // namespace jr
