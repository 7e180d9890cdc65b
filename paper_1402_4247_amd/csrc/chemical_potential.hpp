// The chemical potential of Band_DFT_Col Part 5: mu with count(mu) = nelec on a
// bracket [lo, hi], count(x) the number of electrons at x (not falling in x
// when no weight is negative).  Plain C++ with no HIP dependency besides the
// function attributes: the count is a template parameter, so the search can be
// exercised on the host.
//
// Where the slope of the count fixes mu: Newton steps inside the bracket
// (about 6) and a few more points around their limit leave bisection an
// interval of some ulps instead of the whole bracket's 60 halvings.  In a gap
// the count is flat to rounding, and mu is where bisection of the whole bracket
// ends: the steps stop at the first point there, and the halvings whose outcome
// the points so far decide are taken without an evaluation.  With one workgroup
// at n = 1040 x 16 (616 x 8): a metal 270 us (65 to 121), a gap 755 us (297);
// bisection alone 838 (324) and 763 us (296); steps that went on in the gap and
// were then thrown away 1370 us (556).
#pragma once

#include <math.h>

#ifdef __HIP__
#define KGEV_HOST_DEVICE __host__ __device__
#else
#define KGEV_HOST_DEVICE
#endif

namespace kgev {

// count(x, slope): the count at x and, unless slope is null, its derivative.
// rising: no weight is negative.
template <typename Count>
KGEV_HOST_DEVICE inline double chemical_potential(Count count, bool rising, double nelec, double kT, double lo, double hi)
{
    // the count is clearly (far beyond its rounding) less and more than nelec here
    double below = lo, above = hi;
    if (rising) {
        constexpr double CLEAR = 1e-12;
        double a = lo, c = hi, x = 0.5 * (lo + hi), slope = 0.0;
        bool good = false;
        int lost = 0;                            // points without a slope after one with
        for (int it = 0; it < 40; ++it) {
            const double cnt = count(x, &slope);
            if (cnt < nelec) a = x;
            else c = x;
            // (a point that is bisection's own needs no second evaluation)
            if (x == 0.5 * (lo + hi)) (cnt < nelec ? lo : hi) = x;
            const double scale = fmax(fabs(x), kT);
            good = slope * scale * 1e-9 > 1e-14 * nelec;
            if (cnt < nelec * (1.0 - CLEAR)) below = x;
            else if (cnt > nelec * (1.0 + CLEAR)) above = x;
            else if (!good) break;               // in a gap
            if (good) lost = 1;
            else if (lost > 0 && ++lost > 3) break;      // on the way into one
            const double step = (nelec - cnt) / slope;
            if (good && fabs(step) <= 8e-16 * scale) break;
            double y = x + step;
            if (!(y > a && y < c)) y = 0.5 * (a + c);
            if (!(y > a && y < c)) break;
            x = y;
        }
        // pinch: x - d and x + d with d from a few ulps up, until they bracket
        double d = 4e-16 * fmax(fabs(x), kT);
        for (int it = 0; good && it < 24; ++it, d *= 16.0) {
            const double y = x - d;
            if (y <= a) break;
            if (count(y, nullptr) < nelec) {
                a = y;
                break;
            }
            c = y;
        }
        d = 4e-16 * fmax(fabs(x), kT);
        for (int it = 0; good && it < 24; ++it, d *= 16.0) {
            const double y = x + d;
            if (y >= c) break;
            if (!(count(y, nullptr) < nelec)) {
                c = y;
                break;
            }
            a = y;
        }
        if (good && a < c) {
            lo = a;
            hi = c;
        }
    }
    for (int it = 0; it < 400; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (!(mid > lo && mid < hi)) break;
        if (mid <= below || (mid < above && count(mid, nullptr) < nelec)) lo = mid;
        else hi = mid;
    }
    return 0.5 * (lo + hi);
}

}  // namespace kgev
