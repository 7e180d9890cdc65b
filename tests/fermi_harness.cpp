// The library's search for the chemical potential on the host, and plain
// bisection of the whole bracket beside it; each counts its evaluations.
#include <math.h>

#include "chemical_potential.hpp"

namespace {

struct Spectrum {
    const double* w;
    const double* wk;
    int n, nk;
    double kT, g;
    int* evals;
    double operator()(double x, double* slope) const
    {
        ++*evals;
        double s = 0.0, t = 0.0;
        for (int k = 0; k < nk; ++k)
            for (int j = 0; j < n; ++j) {
                const double u = (w[k * n + j] - x) / kT;
                const double e = exp(-fabs(u)), f = u > 0.0 ? e / (1.0 + e) : 1.0 / (1.0 + e);
                s += wk[k] * f;
                t += wk[k] * f * (1.0 - f);
            }
        if (slope) *slope = g * t / kT;
        return g * s;
    }
};

}  // namespace

extern "C" double fh_search(const double* w, const double* wk, int n, int nk, double nelec, double kT, double g,
                            int rising, int plain, int* evals)
{
    double lo = w[0], hi = w[0];
    for (int q = 0; q < n * nk; ++q) {
        lo = fmin(lo, w[q]);
        hi = fmax(hi, w[q]);
    }
    lo -= 50.0 * kT;
    hi += 50.0 * kT;
    *evals = 0;
    const Spectrum count{w, wk, n, nk, kT, g, evals};
    if (!plain) return kgev::chemical_potential(count, rising != 0, nelec, kT, lo, hi);
    for (int it = 0; it < 400; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (!(mid > lo && mid < hi)) break;
        if (count(mid, nullptr) < nelec) lo = mid;
        else hi = mid;
    }
    return 0.5 * (lo + hi);
}
