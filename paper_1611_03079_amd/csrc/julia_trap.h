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
constexpr int kCriticalSteps = 512, kCriticalShort = 32;

// A wider disc for cycles of Z^2 + C of period 1 or 2, whose points have closed
// forms.  About the cycle the map is h -> 2 z_k h + h^2; n steps of it are a
// polynomial of degree 2^n in h, and a disc that the sum of its terms' moduli
// does not leave is a trap of n steps.  Where the multiplier is near a root of
// unity the terms of n steps cancel and the disc is far wider than one step's
// (C = -0.7279 + 0.0612i: 0.24 against 0.014), which is where orbits take
// longest to come in.  Returns the largest radius of a falling sequence, 0 if
// none closes above kTrapMinRadius.  `at`: the cycle's point, of `p`, to start at.
inline double wide_radius(const double* zx, const double* zy, int p, int at, int n, double eps) {
    constexpr int kDegree = 16;
    double re[5][kDegree + 1] = {}, im[5][kDegree + 1] = {}, size[5][kDegree + 1];
    re[0][1] = 1.0;
    for (int j = 0; j <= n; ++j) {
        const int deg = 1 << j;
        for (int k = 1; k <= deg; ++k) size[j][k] = sqrt(re[j][k] * re[j][k] + im[j][k] * im[j][k]);
        if (j == n) break;
        const double mx = 2.0 * zx[(at + j) % p], my = 2.0 * zy[(at + j) % p];
        for (int k = 1; k <= deg; ++k) {
            re[j + 1][k] += mx * re[j][k] - my * im[j][k];
            im[j + 1][k] += mx * im[j][k] + my * re[j][k];
            for (int i = 1; i <= deg; ++i) {
                re[j + 1][k + i] += re[j][k] * re[j][i] - im[j][k] * im[j][i];
                im[j + 1][k + i] += re[j][k] * im[j][i] + im[j][k] * re[j][i];
            }
        }
    }
    for (double r = 0.7; r >= kTrapMinRadius; r *= 0.85) {
        double reach = r, drift = 0.0;  // of the disc, and of rounding, after j steps
        bool ok = true;
        for (int j = 0; j <= n && ok; ++j) {
            reach = 0.0;
            for (int k = 1 << j; k >= 1; --k) reach = (reach + size[j][k]) * r;
            if (j == n) break;
            const double x = zx[(at + j) % p], y = zy[(at + j) % p];
            const double m = sqrt(x * x + y * y);
            ok = m + reach + drift <= 1.99;
            drift = (2.0 * (m + reach) + drift) * drift + eps;
        }
        if (ok && reach + drift <= r) return r;
    }
    return 0.0;
}

// The cycle of Z^2 + C of period p = 1 or 2 in closed form, if it attracts.  `off`:
// what p rounded steps miss its first point by.
JR_HOST_DEVICE inline bool short_cycle(int p, double cr, double ci, double* zx, double* zy,
                                       double* off) {
    // period 1: z = (1 - sqrt(1 - 4 C)) / 2; period 2: (-1 + sqrt(-3 - 4 C)) / 2
    const double ax = (p == 1 ? 1.0 : -3.0) - 4.0 * cr, ay = -4.0 * ci;
    const double m = sqrt(ax * ax + ay * ay);
    double sx = sqrt(0.5 * (m + fabs(ax)));
    double sy = sx > 0.0 ? 0.5 * ay / sx : 0.0;
    if (ax < 0.0) {
        const double t = sx;
        sx = fabs(sy);
        sy = ay < 0.0 ? -t : t;
    }
    zx[0] = p == 1 ? 0.5 * (1.0 - sx) : 0.5 * (sx - 1.0);
    zy[0] = p == 1 ? -0.5 * sy : 0.5 * sy;
    zx[1] = zx[0] * zx[0] - zy[0] * zy[0] + cr;
    zy[1] = 2.0 * zx[0] * zy[0] + ci;
    double mult = 4.0 * (zx[0] * zx[0] + zy[0] * zy[0]);
    mult = p == 1 ? mult : mult * 4.0 * (zx[1] * zx[1] + zy[1] * zy[1]);
    if (!(mult < 0.9999)) return false;  // |multiplier|^2
    const double bx = p == 1 ? zx[1] - zx[0] : zx[1] * zx[1] - zy[1] * zy[1] + cr - zx[0];
    const double by = p == 1 ? zy[1] - zy[0] : 2.0 * zx[1] * zy[1] + ci - zy[0];
    *off = sqrt(bx * bx + by * by);
    return true;
}

// The trap of a cycle of Z^2 + C of period 1 or 2 whose discs close step by step:
// returns the period or 0.  A few hundred operations without arrays, for the frames
// whose constants are made on the device: there the whole search (find_trap) held
// 2.2 KB of stack memory a lane, and every launch of a path waited for it, 16 frames
// of 200x150 in FP32, cap 100, with C by the cardioid's rim 386 us for now 23.
JR_HOST_DEVICE inline int find_step_trap(double cr, double ci, float* x, float* y, float* r,
                                         float* r1) {
    for (int p = 1; p <= 2; ++p) {
        double zx[2], zy[2], off;
        if (!short_cycle(p, cr, ci, zx, zy, &off)) continue;
        const double eps = 2e-5 + off;
        const double m0 = sqrt(zx[0] * zx[0] + zy[0] * zy[0]);
        const double m1 = sqrt(zx[1] * zx[1] + zy[1] * zy[1]);
        for (double d = 0.7; d >= kTrapMinRadius; d *= 0.85) {
            const double d1 = (2.0 * m0 + d) * d + eps;
            const double back = p == 1 ? d1 : (2.0 * m1 + d1) * d1 + eps;
            if (back > d || m0 + d > 1.99) continue;
            if (p == 2 && (m1 + d1 > 1.99 || d1 < kTrapMinRadius)) continue;
            *x = (float)zx[0];
            *y = (float)zy[0];
            *r = (float)d;
            *r1 = p == 2 ? (float)(0.999 * d1) : 0.0f;
            return p;
        }
    }
    return 0;
}

// The same with the wider discs (wide_radius), for the host.
inline int find_short_trap(double cr, double ci, float* x, float* y, float* r, float* r1) {
    for (int p = 1; p <= 2; ++p) {
        double zx[2], zy[2], off;
        if (!short_cycle(p, cr, ci, zx, zy, &off)) continue;
        const double eps = 2e-5 + off;
        double best[2] = {0.0, 0.0};
        for (int at = 0; at < p; ++at)
            for (int n = p; n <= 4; n += p) {
                const double w = wide_radius(zx, zy, p, at, n, eps);
                best[at] = w > best[at] ? w : best[at];
                if (w >= 0.2) break;  // wide enough: orbits are in within a few steps
            }
        if (best[0] <= 0.0 || (p == 2 && best[1] <= 0.0)) continue;
        *x = (float)zx[0];
        *y = (float)zy[0];
        *r = (float)best[0];
        *r1 = (float)best[1];
        return p;
    }
    return 0;
}

// Iterates the critical orbit of Z^degree + C, on the host.  Returns the period of a
// trap (its disc 0 in x, y, r; the second disc's radius in r1 where the period is
// 2), or 0: none was found within kCriticalSteps.  `steps` is the step at which the
// critical orbit escaped, kCriticalSteps if it did not: the higher, the longer the
// image's orbits take.  `effort` 1: without the wide discs; 0: nor more than
// kCriticalShort steps.
inline int find_trap(double cr, double ci, int degree, float* x, float* y, float* r, float* r1,
                     int* steps, int effort = 2) {
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
    *r1 = 0.0f;
    if (degree == 2) {
        const int p = effort > 1 ? find_short_trap(cr, ci, x, y, r, r1)
                                 : find_step_trap(cr, ci, x, y, r, r1);
        if (p > 0) return p;
    }
    const int last = effort > 0 ? kCriticalSteps : kCriticalShort;
    for (int stop = kCriticalShort; stop <= last; stop *= 4, near *= 0.2) {
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
            double rk = r0, least = r0, second = 0.0;
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
                second = k == 0 ? rk : second;
            }
            if (ok && rk + off <= r0 && least >= kTrapMinRadius) {
                *x = (float)zx;
                *y = (float)zy;
                *r = (float)r0;
                *r1 = p == 2 ? (float)(0.999 * second) : 0.0f;
                return p;
            }
        }
    }
    return 0;
}

// Whether the critical orbit of Z^2 + C ends on a repelling cycle of a period up to
// kTrapPeriodMax that binary64 holds exactly (C = i, -2): the set has no interior then.
inline bool critical_orbit_repelled(double cr, double ci) {
    double x = 0.0, y = 0.0, ux = 0.0, uy = 0.0, m2 = 1.0;
    for (int n = 0; n < 64 + kTrapPeriodMax; ++n) {
        if (n >= 64) {
            if (n == 64) {
                ux = x;
                uy = y;
            } else if (x == ux && y == uy) {
                return m2 > 1.0;
            }
            m2 *= 4.0 * (x * x + y * y);  // |multiplier|^2
        }
        const double t = x * x - y * y + cr;
        y = 2.0 * x * y + ci;
        x = t;
    }
    return false;
}

// A disc of a trap as a kernel tests it (centre and squared radius), and the step
// from (x, y, r) to the next one.  1% + 1e-5 keeps it inside the true disc
// whatever binary32 did to the centre and to the test itself (a centre's error
// grows along the cycle no faster than the radii do, so it stays within
// 16 * 2e-7 / 0.004 of the radius).
JR_HOST_DEVICE inline void next_disc(int p, int degree, float cr, float ci, float& x, float& y,
                                     float& r, float r1, float& disc_x, float& disc_y,
                                     float& disc_r2) {
    const float rt = r * 0.99f - 1e-5f;
    disc_x = x;
    disc_y = y;
    disc_r2 = rt * rt;
    const float m = sqrtf(x * x + y * y);
    float wr = x, wi = y, p0 = m, p1 = m + r;
    for (int d = 1; d < degree; ++d) {
        const float t = wr * x - wi * y;
        wi = wr * y + wi * x;
        wr = t;
        p0 *= m;
        p1 *= m + r;
    }
    x = wr + cr;
    y = wi + ci;
    r = p == 2 ? r1 : p1 - p0;
}

#ifdef __HIP_DEVICE_COMPILE__
__device__ inline float near_sqrt(float v) { return __builtin_amdgcn_sqrtf(v); }  // 1 ulp
__device__ inline float near_reciprocal(float v) { return __builtin_amdgcn_rcpf(v); }
#else
JR_HOST_DEVICE inline float near_sqrt(float v) { return sqrtf(v); }
JR_HOST_DEVICE inline float near_reciprocal(float v) { return 1.0f / v; }
#endif

// Whether the orbit of Z^2 + C that is at z (binary32 parts of the iterate and of
// C) never escapes, for orbits whose frame has no trap, above all of Mandelbrot
// pixels, each with a C of its own.  One Newton step from z looks for a point w
// of a cycle of period 1 or 2, and a disc about w that two steps send into itself
// and that holds z is a trap: |f(w + h) - f(w)| <= 2 |w| |h| + |h|^2, twice.  eps =
// 2e-5 covers the rounding of one step in any arithmetic (2e-6 at most in
// binary32) and of the binary32 images of w and C; 0.002 more of radius what z
// and w are off by, and 0.1% of it the sums here.  An orbit that a cycle of period 1
// or 2 attracts gets there unless the multiplier's modulus is close to 1.  w need not be a cycle's point: the
// inequality alone is the proof.
JR_HOST_DEVICE inline bool settles(float x, float y, float cr, float ci) {
    const float eps = 2e-5f;
    float x1 = (x * x - y * y) + cr, y1 = 2.0f * x * y + ci;
    float x2 = (x1 * x1 - y1 * y1) + cr, y2 = 2.0f * x1 * y1 + ci;
    const float gx = x2 - x, gy = y2 - y;
    const float dx = 4.0f * (x * x1 - y * y1) - 1.0f, dy = 4.0f * (x * y1 + y * x1);
    const float q = near_reciprocal(dx * dx + dy * dy);
    const float hx = (gx * dx + gy * dy) * q, hy = (gy * dx - gx * dy) * q;
    const float wx = x - hx, wy = y - hy;
    x1 = (wx * wx - wy * wy) + cr;
    y1 = 2.0f * wx * wy + ci;
    x2 = (x1 * x1 - y1 * y1) + cr;
    y2 = 2.0f * x1 * y1 + ci;
    const float m0 = near_sqrt(wx * wx + wy * wy), m1 = near_sqrt(x1 * x1 + y1 * y1);
    const float off = near_sqrt((x2 - wx) * (x2 - wx) + (y2 - wy) * (y2 - wy));
    const float r = near_sqrt(hx * hx + hy * hy) + 0.002f;
    const float r1 = (2.0f * m0 + r) * r + eps;
    const float r2 = (2.0f * m1 + r1) * r1 + eps;
    return m0 + r < 1.99f && m1 + r1 < 1.99f && off + r2 <= 0.999f * r;
}

}  // namespace jr
