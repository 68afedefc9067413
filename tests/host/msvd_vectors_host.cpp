// Host build of the recurrences of k_msvd_setup and k_msvd_vectors
// (paper_2511_09798_amd/csrc/msvd.hpp), for CPU tests.
#include <float.h>
#include <math.h>

#include <vector>

#include "../../paper_2511_09798_amd/csrc/msvd.hpp"

using namespace mqh::msvd;

// The quotients s_k of a chain of n from its operands u, v (n - 1): by pair_chain, and by
// its steps one after another, the pair rescaled after each (a power of two, so
// the quotients' bits are the same).
extern "C" void chain_host(const double* u, const double* v, int n, double w0, double lam, double* s, double* plain) {
    std::vector<double> uv(2 * (size_t)n);
    for (int k = 0; k + 1 < n; ++k) {
        uv[2 * k] = u[k];
        uv[2 * k + 1] = v[k];
    }
    pair_chain(uv.data(), n, w0, lam);
    for (int k = 0; k < n; ++k) s[k] = pair_quotient(uv[2 * k], uv[2 * k + 1]);
    double w = w0, c = 1.0;
    for (int k = 0; k < n; ++k) {
        const double b = c;
        const double a = pair_step(w, c, k + 1 < n ? u[k] : 0.0, k + 1 < n ? v[k] : 0.0, lam);
        plain[k] = pair_quotient(a, b);
        const double sc = pair_scale(w, c);
        w *= sc;
        c *= sc;
    }
}

// One direction of the twisted solve into z (n, filled by the caller).
extern "C" void twisted_host(const double* mul, int st, int n, int r, int dir, double* z) {
    twisted_from(mul, st, n, r, dir, z);
}

// The unit singular vectors v, u of the upper bidiagonal (d, e) for the j-th largest
// value, with the value, as k_msvd_values and k_msvd_vectors form them: multisection
// of lambda_j (P points a round), operands, chains, twists and solves. Returns its
// residual over the acceptance bound.
extern "C" double triple_host(const double* d, const double* e, int l, int j, int P, double* v, double* u,
                              double* sigma) {
    const double bound = eig_bound(d, e, l);
    const int sh = pair_shift(bound);
    std::vector<double> D(l), E(l, 0.0), d2(l), e2(l), ch(8 * (size_t)l);
    for (int i = 0; i < l; ++i) {
        D[i] = ldexp(d[i], -sh);
        E[i] = i + 1 < l ? ldexp(e[i], -sh) : 0.0;
        d2[i] = D[i] * D[i];
        e2[i] = E[i] * E[i];
    }
    double lo = 0.0, hi = ldexp(bound, -2 * sh), s1 = 0.0;
    auto value = [&](int jj) {
        lo = 0.0;
        hi = ldexp(bound, -2 * sh);
        for (int round = 0; round < 64 && hi - lo > 2.0 * DBL_EPSILON * hi; ++round) {
            double nlo = lo, nhi = hi;
            for (int t = 0; t < P; ++t) {
                const double x = section_point(lo, hi, t, P);
                if (negcount(d2.data(), 1, e2.data(), 1, l, x, DBL_MIN) <= l - 1 - jj) {
                    nlo = x;
                } else {
                    nhi = x;
                    break;
                }
            }
            if (nlo == lo && nhi == hi) break;
            lo = nlo;
            hi = nhi;
        }
        return lo + 0.5 * (hi - lo);
    };
    s1 = sqrt(value(0));
    const double lam = value(j), sig = sqrt(lam);
    for (int k = 0; k + 1 < l; ++k) chain_operands(D.data(), E.data(), l, l, k, ch.data());
    unsigned quot = 0;
    for (int c = 0; c < 4; ++c) quot |= chain_pairs(D.data(), E.data(), l, l, c, lam, ch.data()) ? 1u << c : 0u;
    int tw[2];
    for (int side = 0; side < 2; ++side) {
        double best = INFINITY;
        tw[side] = l - 1;
        for (int i = 0; i < l; ++i) {
            const double g = twist_step(D.data(), E.data(), l, l, side, i, lam, quot, ch.data());
            if (g < best) {
                best = g;
                tw[side] = i;
            }
        }
    }
    for (int side = 0; side < 2; ++side)
        for (int dn = 0; dn < 2; ++dn)
            twisted_from(ch.data() + 2 * l * side + dn, 2, l, tw[side], dn ? 1 : -1, ch.data() + 2 * l * (side + 2));
    const double *zv = ch.data() + 4 * l, *zu = ch.data() + 6 * l;
    double nv = 0.0, nu = 0.0, t = 0.0, r1 = 0.0, r2 = 0.0;
    for (int k = 0; k < l; ++k) {
        nv += zv[k] * zv[k];
        nu += zu[k] * zu[k];
        t += zu[l - 1 - k] * (D[k] * zv[k] + (k + 1 < l ? E[k] * zv[k + 1] : 0.0));
    }
    for (int k = 0; k < l; ++k) {
        v[k] = zv[k] / sqrt(nv);
        u[k] = zu[l - 1 - k] / (t < 0.0 ? -sqrt(nu) : sqrt(nu));
    }
    for (int k = 0; k < l; ++k) {
        const double a = resid_row(D[k], v[k], E[k], k + 1 < l ? v[k + 1] : 0.0, sig, u[k]);
        const double b = resid_row(D[k], u[k], k > 0 ? E[k - 1] : 0.0, k > 0 ? u[k - 1] : 0.0, sig, v[k]);
        r1 += a * a;
        r2 += b * b;
    }
    *sigma = ldexp(sig, sh);
    return sqrt(r1 > r2 ? r1 : r2) / resid_bound(sig, s1, l);
}

// u / v = rhobar^2 after the rotations of steps 0 .. l - 2, the maps composed in pairs of
// neighbours (the order of a scan), from alpha (l), beta_2 .. (l - 1).
extern "C" double rhobar2_host(const double* alpha, const double* beta, int l) {
    std::vector<QMap> m(l > 1 ? l - 1 : 0);
    for (int i = 0; i + 1 < l; ++i) m[i] = QMap{alpha[i + 1] * alpha[i + 1], 1.0, beta[i] * beta[i]};
    while (m.size() > 1) {
        std::vector<QMap> h;
        for (size_t i = 0; i < m.size(); i += 2) h.push_back(i + 1 < m.size() ? after(m[i + 1], m[i]) : m[i]);
        m.swap(h);
    }
    const double u = alpha[0] * alpha[0];
    return m.empty() ? u : m[0].a * u / (m[0].c * u + m[0].b);
}
