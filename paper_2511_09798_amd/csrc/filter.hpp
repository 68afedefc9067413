// filter.hpp -- the Tikhonov filter factors of the parameter choice (Algorithm 4
// step 4): one term of the GCV sums and of the L-curve sums.  Usable on the host and on
// the device.
#pragma once

#include <math.h>

#ifdef __HIPCC__
#define MQH_HD __host__ __device__
#else
#define MQH_HD
#endif

namespace mqh {
namespace filter {

// phi = s^2 / (s^2 + lambda^2), psi = lambda^2 / (s^2 + lambda^2) and g = f^2 / (s^2 +
// lambda^2), by one reciprocal in place of three divisions.
struct Factors {
    double phi, psi, g;
};
// Sums s^2 + lambda^2 whose reciprocal is a normal number; outside (singular values
// near 1e-154 or 1e154, squares near the ends of the range) 1 / den over- or underflows
// where the quotients do not, and they are divided out.
constexpr double kDenMin = 0x1p-1000, kDenMax = 0x1p1000;

// a / den from q = 1 / den rounded: a q and one correction by its remainder, which
// rounds as the division does where nothing is subnormal.
MQH_HD inline double quotient(double a, double q, double den) {
    const double p = a * q;
    return fma(fma(-p, den, a), q, p);
}

MQH_HD inline Factors factors(double s2, double l2, double f2) {
    const double den = s2 + l2;
    if (den >= kDenMin && den <= kDenMax) {
        const double q = 1.0 / den;
        return Factors{quotient(s2, q, den), quotient(l2, q, den), quotient(f2, q, den)};
    }
    return Factors{s2 / den, l2 / den, f2 / den};
}

// GCV numerator (without f~_{l+1}) and trace terms of one singular value.
MQH_HD inline void gcv_term(double s, double f, double l2, double& num, double& tr) {
    const Factors t = factors(s * s, l2, 0.0);
    const double x = t.psi * f;
    num = fma(x, x, num);
    tr += t.phi;
}

// The L-curve's sums over the spectrum, without their constant factors: the residual R
// (without f~_{l+1}^2) and the solution norm E with their first two derivatives in log
// lambda (d phi / dt = -2 phi psi).
struct CurveSums {
    double R = 0.0, R1 = 0.0, R2 = 0.0, E = 0.0, E1 = 0.0, E2 = 0.0;
};
MQH_HD inline void lcurve_term(double s, double f, double l2, CurveSums& c) {
    const double f2 = f * f;
    const Factors t = factors(s * s, l2, f2);
    const double r = t.psi * t.psi * f2, r1 = t.phi * r;
    const double e = t.phi * t.g, e1 = t.psi * e;  // phi^2 f^2 / s^2 = phi f^2 / (s^2 + lambda^2)
    c.R += r;
    c.R1 += r1;
    c.R2 = fma(r1, fma(2.0, t.phi, -t.psi), c.R2);
    c.E += e;
    c.E1 += e1;
    c.E2 = fma(e1, fma(2.0, t.psi, -t.phi), c.E2);
}

}  // namespace filter
}  // namespace mqh
