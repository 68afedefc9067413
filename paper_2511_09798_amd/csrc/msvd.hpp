// msvd.hpp -- scalar recurrences of the projected SVD by multisection and
// twisted factorisations (the fast path of Algorithm 2 step 2 and
// Algorithm 4 step 2; the implicit QR iteration of bidiag_svd.hpp is the
// fallback).  Usable on the host and on the device.
//
// After the left rotations that reduce C_l to an upper bidiagonal B (d on
// the diagonal, e above it), the squared singular values of B are the
// eigenvalues of
//     B^T B = L D L^T,  D_i = d_i^2,  L_i = e_i / d_i   (so L_i^2 D_i = e_i^2,
//                                                          D_i L_i = d_i e_i),
// and of B B^T, which is the same form on the reversed sequences
// (d_{n-1}, .., d_0), (e_{n-2}, .., e_0).  A bidiagonal determines its
// singular values to high relative accuracy, and so do these factored forms;
// the differential qd transforms below work on them without forming B^T B:
//  * negcount: the number of negative pivots of the factorisation of L D L^T - x I
//    is the number of eigenvalues below x (Sylvester's law of inertia),
//    which drives the bisection of the values;
//  * chain_operands, chain_pairs: the top-down (L+ D+ L+^T) and bottom-up
//    (U- D- U-^T) factorisations of L D L^T - lambda I at an eigenvalue
//    lambda, D+_i = s_i + d_i^2, L+_i = d_i e_i / D+_i, s_{i+1} = e_i^2 s_i /
//    D+_i - lambda from s_0 = -lambda, and D-_{i+1} = e_i^2 + p_{i+1}, U-_i =
//    d_i e_i / D-_{i+1}, p_i = p_{i+1} d_i^2 / D-_{i+1} - lambda from
//    p_{n-1} = d_{n-1}^2 - lambda;
//  * twist_step, twisted_from: gamma_k = s_k + p_k + lambda is the pivot of the
//    factorisation twisted at k, and the k of least |gamma_k| (the smallest on
//    ties) gives the eigenvector by one step of inverse iteration with z_k = 1.
// Zero pivots (in the quotient form of the count pivots below pivmin in
// magnitude) are replaced by tiny negative ones (a perturbation of x within the
// rounding of the data), so no recurrence divides by zero; in the quotient
// form of the count a quotient that comes out NaN is taken as 1.
#pragma once

#include <math.h>
#include <stdint.h>

#ifndef __HIPCC__
#include <vector>
#endif

#ifdef __HIPCC__
#define MQH_HD __host__ __device__
#else
#define MQH_HD
#endif

namespace mqh {
namespace msvd {

// The transforms below carry s_i + x as a quotient w_i / c_i (and p_i + x alike),
// which leaves two dependent FMAs on a step's serial chain where the quotient
// itself puts a division there:
//     a = w - x c (s_i = a / c),  c' = a + u c (the pivot is c' / c),  w' = v a,
// u = d_i^2, v = e_i^2 from the top, u = e_i^2, v = d_i^2 from the bottom.  The
// roundings are relative perturbations of s_i, of the pivot and of v, one fewer
// than in the quotient form.  The pair is brought back near exponent zero every
// kRescale steps (exact); callers keep u, v and x at most about one, so no step
// in between overflows.
constexpr int kRescale = 4;
// Exponent fields (of 2^-300 and 2^300) beyond which a pair may lose range between
// two rescalings: seen halfway through a group and applied at its end, the scale
// lags by up to six steps, over which the pair then shrinks by no more than
// 2^-600 (and grows by 3^6); with x >= kCountFloor the product x c stays a normal
// number.
constexpr uint32_t kPairMin = (1023u - 300u) << 20, kPairMax = (1023u + 300u) << 20;
constexpr double kCountFloor = 0x1p-360;
constexpr double kZeroPivot = 0x1p-300;

MQH_HD inline uint32_t high_word(double x) {
#ifdef __HIP_DEVICE_COMPILE__
    return (uint32_t)__double2hiint(x);
#else
    uint64_t b;
    __builtin_memcpy(&b, &x, 8);
    return (uint32_t)(b >> 32);
#endif
}
// Keeps a value loaded ahead of its use where it was loaded: without it the
// compiler folds the load of the next group back to the start of that group,
// and its latency returns to the chain.
MQH_HD inline double kept(double x) {
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+v"(x));
#endif
    return x;
}
// The larger exponent field of a and b, and the power of two that takes
// max(|a|, |b|) into [1, 2) (a multiplication by it is exact).
MQH_HD inline uint32_t pair_exponent(double a, double b) {
    const uint32_t ea = high_word(a) & 0x7ff00000u, eb = high_word(b) & 0x7ff00000u;
    return ea > eb ? ea : eb;
}
MQH_HD inline double scale_of(uint32_t ex) {
    const uint32_t s = 0x7fe00000u - ex;
#ifdef __HIP_DEVICE_COMPILE__
    return __hiloint2double((int)s, 0);
#else
    const uint64_t v = (uint64_t)s << 32;
    double r;
    __builtin_memcpy(&r, &v, 8);
    return r;
#endif
}
MQH_HD inline double pair_scale(double a, double b) { return scale_of(pair_exponent(a, b)); }

// The map (u, v) -> (a u, c u + b v) up to a common factor, a, b, c >= 0, and the
// product of two (later after earlier); positive terms only, so every entry keeps
// its relative accuracy.
struct QMap {
    double a, c, b;
};
MQH_HD inline QMap after(const QMap& x, const QMap& y) {
    const double a = x.a * y.a, c = fma(x.c, y.a, x.b * y.c), b = x.b * y.b;
    const uint32_t ea = pair_exponent(a, b), ec = pair_exponent(c, 0.0);
    const double s = scale_of(ea > ec ? ea : ec);
    return QMap{a * s, c * s, b * s};
}

// acc with the sign of c shifted in, and the sign changes among its last m + 1 bits.
MQH_HD inline uint32_t push_sign(uint32_t acc, double c) {
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_alignbit(acc, high_word(c), 31);
#else
    return (acc << 1) | (high_word(c) >> 31);
#endif
}
MQH_HD inline uint32_t sign_changes(uint32_t acc, int m) {
    return (uint32_t)__builtin_popcount((acc ^ (acc >> 1)) & ((1u << m) - 1u));
}

// Number of eigenvalues of L D L^T below x, from d2 = d^2 (n) and e2 = e^2
// (n - 1), by the quotients s_i themselves (pivots below pivmin replaced).
// Elements are read at d2[i * ds], e2[i * es] (ds, es = +1 or -1 on suitably
// placed pointers give the reversed sequences).
MQH_HD inline int negcount_quotient(const double* d2, int ds, const double* e2, int es, int n, double x,
                                    double pivmin) {
    double s = -x;
    int neg = 0;
    for (int i = 0; i < n - 1; ++i) {
        double dp = s + d2[i * ds];
        dp = fabs(dp) < pivmin ? -pivmin : dp;
        neg += dp < 0.0 ? 1 : 0;
        double t = s / dp;
        t = t == t ? t : 1.0;
        s = t * e2[i * es] - x;
    }
    double dp = s + d2[(n - 1) * ds];
    dp = fabs(dp) < pivmin ? -pivmin : dp;
    return neg + (dp < 0.0 ? 1 : 0);
}

// A chain of the count: the pair, the signs of its last c's, the extreme exponents
// of its pairs, and the scale of the current group.
struct CountChain {
    double w, c, sc;
    uint32_t acc, lo, hi;
};
MQH_HD inline void count_step(CountChain& t, double u, double v, double x) {
    const double a = fma(-x, t.c, t.w);
    t.c = fma(u, t.c, a);
    t.w = v * a;
    t.acc = push_sign(t.acc, t.c);
}
MQH_HD inline void count_exponent(CountChain& t) {
    const uint32_t ex = pair_exponent(t.w, t.c);
    t.lo = ex < t.lo ? ex : t.lo;
    t.hi = ex > t.hi ? ex : t.hi;
    t.sc = scale_of(ex);
}
struct CountOperands {  // of kRescale steps of both chains
    double u[kRescale], v[kRescale], p[kRescale], r[kRescale];
};
MQH_HD inline void count_load(CountOperands& o, const double* d2, int ds, const double* e2, int es, const double* db,
                              const double* eb, int i) {
    for (int q = 0; q < kRescale; ++q) {
        o.u[q] = d2[(i + q) * ds];
        o.v[q] = e2[(i + q) * es];
        o.p[q] = eb[-(i + q) * es];
        o.r[q] = db[-(i + q) * ds];
    }
}
MQH_HD inline void count_keep(CountOperands& o) {
    for (int q = 0; q < kRescale; ++q) {
        o.u[q] = kept(o.u[q]);
        o.v[q] = kept(o.v[q]);
        o.p[q] = kept(o.p[q]);
        o.r[q] = kept(o.r[q]);
    }
}
// kRescale steps of both chains; the scale is formed halfway, off the chain.
MQH_HD inline void count_group(CountChain& t, CountChain& b, const CountOperands& o, double x) {
    for (int q = 0; q < kRescale; ++q) {
        count_step(t, o.u[q], o.v[q], x);
        count_step(b, o.p[q], o.r[q], x);
        if (q == kRescale / 2 - 1) {
            count_exponent(t);
            count_exponent(b);
        }
    }
    t.w *= t.sc;
    t.c *= t.sc;
    b.w *= b.sc;
    b.c *= b.sc;
}

// The same count from the pairs (a pivot is negative where c changes sign), by the
// factorisation twisted at the middle k: the pivots of the top-down transform
// above it, those of the bottom-up one below it, and gamma_k = s_k + (p_k + x).
// Two chains of half the length, independent of each other.  The c's are a Sturm
// sequence, so a zero among them counts rightly with either sign: its neighbours
// differ in sign.  An x below kCountFloor, a pair that left its range or one that
// vanished sends the count to the quotients.
MQH_HD inline int negcount(const double* d2, int ds, const double* e2, int es, int n, double x, double pivmin) {
    const int k = n / 2, nb = n - 1 - k;  // steps from the top (nb or nb + 1) and from the bottom
    const double* db = d2 + (n - 2) * ds;
    const double* eb = e2 + (n - 2) * es;
    CountChain t{0.0, 1.0, 1.0, 0u, kPairMax, kPairMin}, b{d2[(n - 1) * ds], 1.0, 1.0, 0u, kPairMax, kPairMin};
    uint32_t neg = 0;
    constexpr int kTwo = 2 * kRescale;
    const int full = nb / kTwo * kTwo;
    if (full > 0) {
        CountOperands A, B;
        count_load(A, d2, ds, e2, es, db, eb, 0);
        for (int i = 0; i < full; i += kTwo) {  // the other group's operands in flight during one
            count_load(B, d2, ds, e2, es, db, eb, i + kRescale);
            count_group(t, b, A, x);
            count_keep(B);
            count_load(A, d2, ds, e2, es, db, eb, i + kTwo < full ? i + kTwo : 0);
            count_group(t, b, B, x);
            count_keep(A);
            neg += sign_changes(t.acc, kTwo);
            neg += sign_changes(b.acc, kTwo);
        }
    }
    int i = full;
    if (nb - i >= kRescale) {
        CountOperands A;
        count_load(A, d2, ds, e2, es, db, eb, i);
        count_group(t, b, A, x);
        neg += sign_changes(t.acc, kRescale);
        neg += sign_changes(b.acc, kRescale);
        i += kRescale;
    }
    if (const int rem = nb - i) {
        double u[kRescale], v[kRescale], p[kRescale], r[kRescale];
        for (int q = 0; q < kRescale - 1; ++q) {
            const int j = q < rem ? i + q : i;
            u[q] = d2[j * ds];
            v[q] = e2[j * es];
            p[q] = eb[-j * es];
            r[q] = db[-j * ds];
        }
        for (int q = 0; q < kRescale - 1; ++q) {
            if (q < rem) {
                count_step(t, u[q], v[q], x);
                count_step(b, p[q], r[q], x);
            }
        }
        neg += sign_changes(t.acc, rem);
        neg += sign_changes(b.acc, rem);
    }
    if (k > nb) {
        count_step(t, d2[nb * ds], e2[nb * es], x);
        neg += sign_changes(t.acc, 1);
    }
    count_exponent(t);
    count_exponent(b);
    const double ct = t.c * t.sc;
    const double at = fma(-x, ct, t.w * t.sc);
    const double g = fma(at, b.c * b.sc, (b.w * b.sc) * ct);  // gamma_k times both c
    neg += (high_word(g) ^ high_word(t.c) ^ high_word(b.c)) >> 31;
    const uint32_t lo = t.lo < b.lo ? t.lo : b.lo, hi = t.hi > b.hi ? t.hi : b.hi;
    const bool ok = x >= kCountFloor && lo > kPairMin && hi < kPairMax && fabs(g) > 0.0;
    return ok ? (int)neg : negcount_quotient(d2, ds, e2, es, n, x, pivmin);
}

// One step of a transform's pair; s_i = a / (c before the step).
MQH_HD inline double pair_step(double& w, double& c, double u, double v, double lam) {
    const double a = fma(-lam, c, w);
    w = v * a;
    c = fma(u, c, a);
    return a;
}
// s_i of a stored pair; a zero c (a zero pivot before it) as a tiny negative pivot.
MQH_HD inline double pair_pivot(double c) { return c == 0.0 ? -kZeroPivot : c; }
MQH_HD inline double pair_quotient(double a, double b) { return a / pair_pivot(b); }

// The pairs of a transform, in place: uv holds (u_k, v_k), k < n - 1, and receives
// (a_k, c_k), s_k = a_k / c_k, k < n.  The top-down (stationary) transform has
// (u, v) = (d^2, e^2) from the top and w0 = 0; the bottom-up one (e^2, d^2) from
// the bottom and w0 = d_{n-1}^2 (then s_k is p_{n-1-k}).  False where the pairs may
// not tell, and quotient_chain takes the chain's place: one of them vanished (a zero
// pivot at a zero off-diagonal entry leaves (0, 0), and nothing follows from it) or
// fell by 2^-400 over four steps (an end of the chain may then lose range: over the six
// steps between two scales it falls by at most 2^-800); a pivot is zero where
// the pair is scaled (what stands for it, pair_pivot, is of one scale); or lam is below
// kChainFloor, so that what a quotient loses under 2^-222 could tell beside it.
constexpr double kChainFloor = 0x1p-170;
constexpr uint32_t kChainMin = (1023u - 400u) << 20;

MQH_HD inline bool pair_chain(double* uv, int n, double w0, double lam) {
    double w = w0, c = 1.0;
    uint32_t lo = kPairMax, hi = kPairMin;
    bool zero = false;
    double u[kRescale], v[kRescale];
    const int full = (n - 1) / kRescale * kRescale;
    for (int q = 0; q < kRescale && full > 0; ++q) {
        u[q] = uv[2 * q];
        v[q] = uv[2 * q + 1];
    }
    for (int k0 = 0; k0 < full; k0 += kRescale) {
        double un[kRescale], vn[kRescale];  // the next group's
        const double* nx = uv + (k0 + kRescale < full ? 2 * kRescale : 0);
        for (int q = 0; q < kRescale; ++q) {
            un[q] = nx[2 * q];
            vn[q] = nx[2 * q + 1];
        }
        double sc = 1.0;
        for (int q = 0; q < kRescale; ++q) {
            uv[2 * q + 1] = c;
            uv[2 * q] = pair_step(w, c, u[q], v[q], lam);
            if (q == kRescale / 2 - 1) {
                const uint32_t ex = pair_exponent(w, c);
                lo = ex < lo ? ex : lo;
                hi = ex > hi ? ex : hi;
                sc = scale_of(ex);
            }
        }
        zero = zero || c == 0.0;
        w *= sc;
        c *= sc;
        uv += 2 * kRescale;
        for (int q = 0; q < kRescale; ++q) {
            u[q] = kept(un[q]);
            v[q] = kept(vn[q]);
        }
    }
    for (int k = full; k < n - 1; ++k) {
        const double uk = uv[0], vk = uv[1];
        uv[1] = c;
        uv[0] = pair_step(w, c, uk, vk, lam);
        uv += 2;
    }
    uv[0] = fma(-lam, c, w);
    uv[1] = c;
    const uint32_t ex = pair_exponent(w, c);
    lo = ex < lo ? ex : lo;
    hi = ex > hi ? ex : hi;
    return lam >= kChainFloor && lo > kChainMin && hi < kPairMax && !zero;
}

// The same by the quotients themselves, from op(k, u, v) = (u_k, v_k): uv receives (s_k,
// D_k), D = s + u, s' = v s / D - lam, a pivot below the normal numbers replaced by a
// tiny negative one.  Where u is zero the pivot is s itself (the bottom-up transform
// at a zero off-diagonal entry).
template <class Operands>
MQH_HD inline void quotient_chain(double* uv, int n, double w0, double lam, const Operands& op) {
    double s = w0 - lam;
    for (int k = 0; k < n; ++k) {
        uv[2 * k] = s;
        uv[2 * k + 1] = 1.0;
        if (k + 1 == n) break;
        double u, v;
        op(k, u, v);
        double dp = s + u;
        dp = fabs(dp) < 0x1p-1022 ? -0x1p-1022 : dp;
        uv[2 * k + 1] = dp;
        double t = u == 0.0 ? 1.0 : s / dp;
        t = t == t ? t : 1.0;
        s = t * v - lam;
    }
}

// s_k of an entry of a chain, and d e / D for its pivot D = s + u: L+_i of the top-down
// transform (u = d^2) and U-_i of the bottom-up one (u = e^2).  quot: the entry is
// quotient_chain's.
MQH_HD inline double chain_s(const double* x, bool quot) { return quot ? x[0] : pair_quotient(x[0], x[1]); }
MQH_HD inline double pair_multiplier(double a, double b, double u, double de) {
    const double c = pair_pivot(b);
    return de * c / pair_pivot(fma(u, c, a));
}
MQH_HD inline double chain_multiplier(const double* x, bool quot, double u, double de) {
    return quot ? de / x[1] : pair_multiplier(x[0], x[1], u, de);
}

// The four chains of a singular triple: side 0 is B^T B on (d, e), side 1 B B^T on
// the reversed sequences, chain c = side + 2 bottom_up at ch + 2 ld c (ld >= l).
// Operands of step k of chain c, k < l - 1, those of every chain, and a chain's w0.
MQH_HD inline void chain_operand(const double* d, const double* e, int l, int c, int k, double& u, double& v) {
    const int i = c == 0 || c == 3 ? k : l - 2 - k;  // the chains 1 and 2 run from the end
    const double di = d[c & 1 ? i + 1 : i], ei = e[i];
    u = c < 2 ? di * di : ei * ei;
    v = c < 2 ? ei * ei : di * di;
}
MQH_HD inline void chain_operands(const double* d, const double* e, int l, int ld, int k, double* ch) {
    for (int c = 0; c < 4; ++c) {
        double* uv = ch + 2 * ld * c + 2 * k;
        chain_operand(d, e, l, c, k, uv[0], uv[1]);
    }
}
MQH_HD inline double chain_start(const double* d, int l, int c) {
    const double dn = c == 2 ? d[l - 1] : (c == 3 ? d[0] : 0.0);
    return dn * dn;
}

// The pairs of chain c in place of its operands; true: its quotients.
MQH_HD inline bool chain_pairs(const double* d, const double* e, int l, int ld, int c, double lam, double* ch) {
    double* uv = ch + 2 * ld * c;
    const double w0 = chain_start(d, l, c);
    if (pair_chain(uv, l, w0, lam)) return false;
    quotient_chain(uv, l, w0, lam, [&](int k, double& u, double& v) { chain_operand(d, e, l, c, k, u, v); });
    return true;
}

// |gamma_i| of a side from its two chains (bit c of quot: chain c holds quotients); the
// multipliers L+_i and U-_i (i < l - 1) take the place of the top-down entry.
MQH_HD inline double twist_step(const double* d, const double* e, int l, int ld, int side, int i, double lam,
                                unsigned quot, double* ch) {
    const bool qt = quot >> side & 1u, qb = quot >> (side + 2) & 1u;
    const double di = side ? d[l - 1 - i] : d[i];
    const double ei = i + 1 < l ? (side ? e[l - 2 - i] : e[i]) : 0.0;
    double* top = ch + 2 * ld * side + 2 * i;
    const double* bot = ch + 2 * ld * (side + 2) + 2 * (l - 1 - i);
    const double g = fabs(chain_s(top, qt) + chain_s(bot, qb) + lam);
    if (i + 1 < l) {
        const double lp = chain_multiplier(top, qt, di * di, di * ei);
        top[1] = chain_multiplier(bot - 2, qb, ei * ei, di * ei);
        top[0] = lp;
    }
    return g;
}

// One direction of the twisted solve from z_r = 1 (z_r included, so that both may run
// at once): dir < 0 takes mul[k st] = L+_k, dir > 0 U-_k.
MQH_HD inline void twisted_from(const double* mul, int st, int n, int r, int dir, double* zout) {
    constexpr int kAhead = 8;  // multipliers in flight ahead of the chain
    double z = 1.0;
    zout[r] = 1.0;
    const int steps = dir < 0 ? r : n - 1 - r;
    const int full = steps / kAhead * kAhead, sd = st * dir;
    const double* m = mul + st * (dir < 0 ? r - 1 : r);
    double* out = zout + r;
    double q[kAhead];
    for (int k = 0; k < kAhead && full > 0; ++k) q[k] = m[sd * k];
    for (int k0 = 0; k0 < full; k0 += kAhead) {
        double qn[kAhead];
        if (k0 + kAhead < full) m += sd * kAhead;
        for (int k = 0; k < kAhead; ++k) qn[k] = m[sd * k];
        for (int k = 0; k < kAhead; ++k) {
            z = -q[k] * z;
            out += dir;
            out[0] = z;
        }
        for (int k = 0; k < kAhead; ++k) q[k] = kept(qn[k]);
    }
    if (full > 0) m += sd * kAhead;
    for (int k = full; k < steps; ++k) {
        z = -m[0] * z;
        m += sd;
        out += dir;
        out[0] = z;
    }
}

#ifndef __HIPCC__
// The recurrences above on strided sequences, one transform at a time, for host
// programs: s and L+ of the top-down transform; the twist index and its gamma with U-
// in place of s (su); one direction of the twisted solve, z in place of L+ (z_r is the
// caller's).
template <class Operands>
inline bool host_chain(std::vector<double>& uv, int n, double w0, double lam, const Operands& op) {
    for (int k = 0; k + 1 < n; ++k) op(k, uv[2 * k], uv[2 * k + 1]);
    if (pair_chain(uv.data(), n, w0, lam)) return false;
    quotient_chain(uv.data(), n, w0, lam, op);
    return true;
}
inline void stationary(const double* d, int ds, const double* e, int es, int n, double lam, double, double* lp,
                       double* s) {
    std::vector<double> uv(2 * (size_t)n);
    const bool q = host_chain(uv, n, 0.0, lam, [&](int k, double& u, double& v) {
        u = d[k * ds] * d[k * ds];
        v = e[k * es] * e[k * es];
    });
    for (int i = 0; i < n; ++i) {
        s[i] = chain_s(&uv[2 * i], q);
        if (i + 1 < n) lp[i] = chain_multiplier(&uv[2 * i], q, d[i * ds] * d[i * ds], d[i * ds] * e[i * es]);
    }
}
inline int progressive_twist(const double* d, int ds, const double* e, int es, int n, double lam, double, double* su,
                             double* gamma_r) {
    std::vector<double> uv(2 * (size_t)n);  // entry k: index n - 1 - k
    const double w0 = d[(n - 1) * ds] * d[(n - 1) * ds];
    const bool q = host_chain(uv, n, w0, lam, [&](int k, double& u, double& v) {
        u = e[(n - 2 - k) * es] * e[(n - 2 - k) * es];
        v = d[(n - 2 - k) * ds] * d[(n - 2 - k) * ds];
    });
    int r = -1;
    for (int i = 0; i < n; ++i) {
        const double* bot = &uv[2 * (n - 1 - i)];
        const double g = su[i] + chain_s(bot, q) + lam;
        if (r < 0 || fabs(g) < fabs(*gamma_r)) {
            *gamma_r = g;
            r = i;
        }
        if (i + 1 < n) su[i] = chain_multiplier(bot - 2, q, e[i * es] * e[i * es], d[i * ds] * e[i * es]);
    }
    return r;
}
inline void twisted_solve(double* lp_z, const double* um, int n, int r, int dir) {
    std::vector<double> z(n);
    twisted_from(dir < 0 ? lp_z : um, 1, n, r, dir, z.data());
    for (int i = r + dir; i >= 0 && i < n; i += dir) lp_z[i] = z[i];
}
#endif

// d x + e y - s w for one row of B v - s u (or B^T u - s v) with the
// rounding error of e y added back (two-product by fma): near a singular
// triple d x + e y nearly cancels against s w, and without the correction
// the rounding of the products, eps (|d x| + |e y|), would swamp a residual
// that is small relative to a tiny s.
MQH_HD inline double resid_row(double d, double x, double e, double y, double s, double w) {
    const double p = e * y;
    const double pe = fma(e, y, -p);
    const double q = fma(d, x, p);
    return fma(-s, w, q) + pe;
}

// Multisection points: P points strictly inside (lo, hi), equally spaced in
// log2 while the bracket spans more than a factor of two (from max(lo, hi 2^-350) and
// the smallest normal number on; a value below hi 2^-350 is looked for from the next
// round's hi on), equally spaced otherwise.
MQH_HD inline double section_point(double lo, double hi, int t, int P) {
    const double f = (double)(t + 1) / (double)(P + 1);
    if (lo == 0.0 || hi > 2.0 * lo) {
        const double low = hi * 0x1p-350 > 0x1p-1022 ? hi * 0x1p-350 : 0x1p-1022;
        const double a = log2(lo > low ? lo : low);
        const double b = log2(hi);
        return exp2(a + (b - a) * f);
    }
    return lo + (hi - lo) * f;
}

// Upper bound of the eigenvalues of B^T B: the square of max_i (|d_i| + |e_i|, |d_i| + |e_{i-1}|),
// which bounds ||B||_2 by the geometric mean of the 1- and infinity-norms.
MQH_HD inline double eig_bound_row(const double* d, const double* e, int n, int i) {
    const double a = fabs(d[i]);
    const double r = a + (i < n - 1 ? fabs(e[i]) : 0.0);
    const double c = a + (i > 0 ? fabs(e[i - 1]) : 0.0);
    return r > c ? r : c;
}
MQH_HD inline double eig_bound_of(double m) { return m * m * (1.0 + 64.0 * 2.220446049250313e-16); }
MQH_HD inline double eig_bound(const double* d, const double* e, int n) {
    double m = 0.0;
    for (int i = 0; i < n; ++i) {
        const double r = eig_bound_row(d, e, n, i);
        m = r > m ? r : m;
    }
    return eig_bound_of(m);
}
// Half the power of two that brings B^T B's bound below one: d 2^-h, e 2^-h,
// lambda 2^-2h are the scaled operands of the pair recurrences (exact).
MQH_HD inline int pair_shift(double bound) {
    int ex;
    (void)frexp(bound, &ex);
    return (ex + 2) / 2;
}

// Thresholds of the fast path's acceptance test: the Gram matrices of the
// computed right and left vectors within kOrthTol of I, and for every
// triple max(||B v - s u||, ||B^T u - s v||) <= resid_bound(s, s_1, n).  The
// absolute term is the floor that rounding the vectors to double already
// puts under any residual (about eps sqrt(n) s_1), with a wide margin.
constexpr double kOrthTol = 1e-9;
constexpr double kResTol = 1e-9;
MQH_HD inline double resid_bound(double s, double s1, int n) {
    return kResTol * s + 64.0 * (double)n * 2.220446049250313e-16 * s1;
}
constexpr int kSections = 256;  // multisection points per round at most (64 to 256 on the device, by l)

}  // namespace msvd
}  // namespace mqh
