// Host build of the parameter choice's filter factors and sums
// (paper_2511_09798_amd/csrc/filter.hpp), for CPU tests.
#include "../../paper_2511_09798_amd/csrc/filter.hpp"

using namespace mqh::filter;

// phi, psi, g (3 x n) of s^2, lambda^2, f^2
extern "C" void factors_host(const double* s2, const double* l2, const double* f2, int n, double* out) {
    for (int i = 0; i < n; ++i) {
        const Factors t = factors(s2[i], l2[i], f2[i]);
        out[i] = t.phi;
        out[n + i] = t.psi;
        out[2 * n + i] = t.g;
    }
}
// num, tr, then R, R1, R2, E, E1, E2 over a spectrum at one lambda
extern "C" void sums_host(const double* s, const double* f, int l, double lam, double* out) {
    CurveSums c;
    out[0] = out[1] = 0.0;
    for (int i = 0; i < l; ++i) {
        gcv_term(s[i], f[i], lam * lam, out[0], out[1]);
        lcurve_term(s[i], f[i], lam * lam, c);
    }
    const double v[6] = {c.R, c.R1, c.R2, c.E, c.E1, c.E2};
    for (int k = 0; k < 6; ++k) out[2 + k] = v[k];
}
