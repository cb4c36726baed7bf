// Coefficients of the coupled inverse p-th root iteration  T = a I - g M,  X <- X T,  M <- T^p M.
//
// Every eigenvalue mu of M moves by the scalar map f(mu) = (a - g mu)^p mu.  The classical
// Newton choice a = (p + 1) / p, g = 1 / p grows a small eigenvalue by only ((p + 1) / p)^p per
// step (2.44 for p = 4).  When the spectrum of M is known to lie in [lo, hi] the pair (a, g) can
// instead be chosen so that f maps the whole interval as close to 1 as possible: write
// f(mu) = g^p (c - mu)^p mu with c = a / g (the zero of T); the minimax choice equalises
// f(lo) = f(hi) = 1 - E and f(c / (p + 1)) = 1 + E (the interior maximum), which has the closed
// form below.  c is kept >= (1 + theta) hi so that T stays safely positive definite even if hi
// was underestimated.  As the interval contracts to {1} the pair tends to the Newton pair.
// The same routine runs on the host (iteration budget, precision switch) and on the device
// (per-factor coefficients).
#pragma once
#include <math.h>

#ifdef __HIPCC__
#define ASTERIA_HD __host__ __device__
#else
#define ASTERIA_HD
#endif

namespace asteria {

struct RootInterval { double lo, hi; };

ASTERIA_HD inline double ipow(double x, int p)
{
    double r = 1.0;
    for (int i = 0; i < p; ++i) r *= x;
    return r;
}

// (a, g) for a spectrum in [lo, hi]; adapted = false gives the classical Newton pair.
ASTERIA_HD inline void root_coefficients(double lo, double hi, int p, bool adapted, double theta,
                                         double &a, double &g)
{
    a = (p + 1.0) / p;
    g = 1.0 / p;
    if (!adapted || !(lo > 0.0) || !(hi > lo)) return;
    const double rho = pow(hi / lo, 1.0 / p);
    if (!(rho > 1.0 + 1e-9)) return;
    double c = (rho * hi - lo) / (rho - 1.0);
    if (c < hi * (1.0 + theta)) c = hi * (1.0 + theta);
    if (!(c < 1e6)) return;
    const double flo = ipow(c - lo, p) * lo, fhi = ipow(c - hi, p) * hi;
    double fmin = flo < fhi ? flo : fhi, fmax = flo > fhi ? flo : fhi;
    const double ms = c / (p + 1.0);
    if (ms > lo && ms < hi) {
        const double fm = ipow(c - ms, p) * ms;
        if (fm > fmax) fmax = fm;
        if (fm < fmin) fmin = fm;
    }
    g = pow(2.0 / (fmin + fmax), 1.0 / p);
    a = g * c;
}

// image of [lo, hi] under mu -> (a - g mu)^p mu
ASTERIA_HD inline RootInterval root_image(double lo, double hi, int p, double a, double g)
{
    const double flo = ipow(a - g * lo, p) * lo, fhi = ipow(a - g * hi, p) * hi;
    RootInterval r;
    r.lo = flo < fhi ? flo : fhi;
    r.hi = flo > fhi ? flo : fhi;
    const double ms = a / ((p + 1.0) * g);
    if (ms > lo && ms < hi) {
        const double fm = ipow(a - g * ms, p) * ms;
        if (fm > r.hi) r.hi = fm;
        if (fm < r.lo) r.lo = fm;
    }
    return r;
}

constexpr double ROOT_THETA = 0.1;   // safety margin of T's positivity: zero of T >= 1.1 hi

// ---- T of degree d <= 3 ---------------------------------------------------------------------------
// T = c0 I - c1 M (+ c2 M^2 - c3 M^3) moves every eigenvalue by f(mu) = T(mu)^4 mu.  The best T on [lo, hi]
// brings T(mu) mu^(1/4) as close to 1 as possible: the relative minimax approximation of mu^(-1/4), found by
// the Remez exchange.  Its extremes are lo, hi and the d roots of T + 4 mu T' in between; from Chebyshev nodes
// the exchange settles in at most 5 steps for every hi / lo up to 1e9.  T is scaled so that f ranges over
// 1 -+ E.  What a degree costs and lifts (ratio lo / hi per iteration, small lo): degree 1 4 products (T^2, T^4,
// T^4 M, X T), 12 x; degree 2 5 products, 36 x; degree 3 6 products, 74 x.
struct RootPoly {
    double c[4];          // T(mu) = c[0] + c[1] mu + c[2] mu^2 + c[3] mu^3
    RootInterval image;   // f([lo, hi])
};

// Degree as a template argument: every loop unrolls and the points stay in registers.  (Indexed at run time they lie in
// scratch memory, and the one thread that works on them takes 26 us instead of 4.)
template <int D>
ASTERIA_HD inline double root_t(const double (&c)[4], double x)
{
    double t = c[D];
#pragma unroll
    for (int i = D - 1; i >= 0; --i) t = t * x + c[i];
    return t;
}

template <int D>
ASTERIA_HD inline RootPoly root_poly_of(double lo, double hi)
{
    RootPoly P;
    P.c[0] = P.c[1] = P.c[2] = P.c[3] = 0.0;
    // a nearly flat spectrum: the polynomial of a wider interval is accurate enough (deviation 4e-6) and keeps
    // the exchange away from cancellation
    const double l = lo < 0.9 * hi ? lo : 0.9 * hi;
    double x[D + 2], w[D + 2];
    x[0] = l; x[D + 1] = hi;
#pragma unroll
    for (int j = 1; j <= D; ++j) {
        // cos(pi j / (D + 1)) for D = 2, 3
        const double cj = D == 2 ? (j == 1 ? 0.5 : -0.5) : (j == 1 ? 0.70710678118654752 : (j == 2 ? 0.0 : -0.70710678118654752));
        x[j] = l + (hi - l) * 0.5 * (1.0 - cj);
    }
    double dd[D + 1], e = 0.0;
    for (int it = 0; it < 6; ++it) {
        // T(x_i) = (1 + s_i e) w_i with s = -, +, -, ...: the divided difference over all D + 2 points vanishes
        double num = 0.0, den = 0.0, sg = -1.0;
#pragma unroll
        for (int i = 0; i <= D + 1; ++i) {
            w[i] = 1.0 / sqrt(sqrt(x[i]));
            double pr = 1.0;
#pragma unroll
            for (int j = 0; j <= D + 1; ++j)
                if (j != i) pr *= x[i] - x[j];
            const double q = w[i] / pr;
            num -= q; den += sg * q;
            sg = -sg;
        }
        const double before = e;
        e = num / den;
        sg = -1.0;
#pragma unroll
        for (int i = 0; i <= D; ++i) { dd[i] = (1.0 + sg * e) * w[i]; sg = -sg; }
        // Newton's form on x_0 .. x_D, then powers of mu
#pragma unroll
        for (int j = 1; j <= D; ++j)
#pragma unroll
            for (int i = D; i >= j; --i) dd[i] = (dd[i] - dd[i - 1]) / (x[i] - x[i - j]);
        double c[4] = {dd[D], 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = D - 1; i >= 0; --i) {
#pragma unroll
            for (int j = D - i; j > 0; --j) c[j] = c[j - 1] - c[j] * x[i];
            c[0] = dd[i] - c[0] * x[i];
        }
#pragma unroll
        for (int j = 0; j <= D; ++j) P.c[j] = c[j];
        // interior extremes of T mu^(1/4): roots of q(mu) = sum (1 + 4 j) c_j mu^j
        if constexpr (D == 2) {
            const double q0 = c[0], q1 = 5.0 * c[1], q2 = 9.0 * c[2];
            const double disc = q1 * q1 - 4.0 * q2 * q0;
            if (!(disc > 0.0)) break;
            const double s = sqrt(disc), big = -q1 + s;      // c1 < 0, c2 > 0
            x[2] = big / (2.0 * q2);
            x[1] = 2.0 * q0 / big;
        } else {
            // Newton from the points so far, each root deflated by nothing: they are well apart
            const double q[4] = {c[0], 5.0 * c[1], 9.0 * c[2], 13.0 * c[3]};
#pragma unroll
            for (int j = 1; j <= 3; ++j) {
                double y = x[j];
                for (int t = 0; t < 4; ++t) {
                    const double fv = ((q[3] * y + q[2]) * y + q[1]) * y + q[0], fd = (3.0 * q[3] * y + 2.0 * q[2]) * y + q[1];
                    if (fd == 0.0) break;
                    double z = y - fv / fd;
                    const double a = 0.5 * (x[j - 1] + y), b = 0.5 * (y + x[j + 1]);   // stay between the neighbours
                    z = z < a ? a : (z > b ? b : z);
                    y = z;
                }
                x[j] = y;
            }
        }
        // the deviation is stationary in the points: they are settled to about the root of this
        if (it > 0 && fabs(e - before) <= 1e-12 * fabs(e)) break;
    }
    // f at the ends and at the interior extremes, whatever the exchange has reached
    double fmin = 1e300, fmax = -1e300;
#pragma unroll
    for (int i = 0; i <= D + 1; ++i) {
        const double t = root_t<D>(P.c, x[i]), f = t * t * t * t * x[i];
        fmin = f < fmin ? f : fmin; fmax = f > fmax ? f : fmax;
    }
    const double s4 = 2.0 / (fmin + fmax), s = sqrt(sqrt(s4));
#pragma unroll
    for (int j = 0; j <= D; ++j) P.c[j] *= s;
    P.image.lo = fmin * s4; P.image.hi = fmax * s4;
    return P;
}

ASTERIA_HD inline RootPoly root_poly(double lo, double hi, int d)
{
    if (d == 2) return root_poly_of<2>(lo, hi);
    if (d == 3) return root_poly_of<3>(lo, hi);
    RootPoly P;
    double a, g;
    root_coefficients(lo, hi, 4, true, 0.1, a, g);
    P.c[0] = a; P.c[1] = -g; P.c[2] = P.c[3] = 0.0;
    P.image = root_image(lo, hi, 4, a, g);
    return P;
}

// The schedule starts from [lo0, ROOT_TOP]: an estimate of the largest eigenvalue up to 5 % low (beyond the scaling's
// own margin) stays inside the interval.  A T of even degree grows beyond it, 20-fold per iteration; Lanczos from one
// start vector is that low where the vector hardly meets the top eigenvector and the gap below it is a few per cent
// (one factor in about 1e4 at a gap of 1 %).
constexpr double ROOT_TOP = 1.05;

// Degrees of T by iteration for a spectrum of M_0 in [lo0, 1] (relative to its top): the sequence of least cost (a product counts 1,
// in the fp64 iterations, of degree 2 at most, 1.5) whose last image lies within 1 -+ 2.6e-3, from an exhaustive
// search.  `from`:
// the sequence holds from this lo0 up to the next entry's.  Below the first entry (three and more fp64
// iterations) T stays linear.
struct RootDegrees { double from; const char *deg; };
inline const char *root_degrees(double lo0)
{
    static const RootDegrees tab[] = {
        {1.3e-7, "112233"}, {2.0e-7, "22333"}, {4.0e-7, "22233"}, {8.0e-7, "22223"}, {2.0e-6, "22222"}, {2.6e-6, "12223"},
        {6.4e-6, "2333"}, {1.3e-5, "2233"}, {3.0e-5, "2223"}, {4.1e-5, "1233"}, {8.0e-5, "2222"}, {1.05e-4, "1223"},
        {2.0e-4, "1222"}, {2.6e-4, "333"}, {5.1e-4, "233"}, {1.05e-3, "223"}, {2.6e-3, "222"}, {3.3e-3, "123"},
        {6.4e-3, "122"}, {1.05e-2, "113"}, {1.6e-2, "33"}, {3.2e-2, "23"}, {6.4e-2, "22"}, {8.2e-2, "13"}, {0.17, "12"},
        {0.41, "3"}, {0.64, "2"}};
    const char *d = "";
    for (const RootDegrees &e : tab)
        if (lo0 >= e.from) d = e.deg;
    return d;
}

}  // namespace asteria
