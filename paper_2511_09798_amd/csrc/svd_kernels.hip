// svd_kernels.hip -- SVD of the projected bidiagonal C_l (Algorithm 2 step 2,
// Algorithm 4 step 2) on the device, by multisection for the singular values
// and twisted factorisations for the vectors, with the implicit QR iteration
// (k_bidiag_svd) as the fallback for spectra the fast path does not resolve.
//
// Steps, one problem per grid row (blockIdx.y, or blockIdx.x for the
// per-problem kernels):
//  1. k_msvd_setup: the left rotations that take C_l to the upper bidiagonal
//     B (d, e) while carrying beta_1 e_1 (g, and f~_{l+1}); the eigenvalue
//     bound.
//  2. k_msvd_values: 64 to 256 threads per singular value s_j (the j-th
//     largest): as many counts of the eigenvalues of B^T B below as many points
//     of the current bracket per round (multisection), about eight rounds to a
//     bracket of two ulps.  Each s_j to high relative accuracy, independently of the others.
//  3. k_msvd_vectors: one wave per j: twisted factorisations of B^T B - s_j^2 I
//     (right vector v_j) and B B^T - s_j^2 I (left vector u_j), the sign of
//     u_j from u_j^T B v_j > 0, the residuals of both relations, h_j = u_j^T g.
//  4. k_msvd_gram: E = V^T V - I (kept), the largest |U^T U - I| (tile maxima)
//     and U h.
//  5. k_msvd_finish: the acceptance test (Gram matrices within 1e-9 of I,
//     residuals within 1e-9 s_j plus a rounding floor); on success V <- V (I - E/2) and
//     f~ = (I - E_U/2) h, which make the vectors orthonormal to second order
//     in E; otherwise the problem is flagged for the fallback.
//  6. k_bidiag_svd (QR) runs for flagged problems only.
// The vectors of singular values with relative gap g are determined by the
// data to about eps/g; the symmetric correction of step 5 restores the
// orthogonality without moving them further than that.
#include <float.h>

#include "bidiag_svd.hpp"
#include "kernels.hpp"
#include "msvd.hpp"

namespace mqh {

namespace {

constexpr int kFinRows = 4;    // rows of V updated per workgroup in k_msvd_finish
constexpr int kGramTile = 32;  // k_msvd_gram tile edge
constexpr int kGramK = 32;     // rows per chunk of its sums
constexpr int kGramRows = kGramK * kGramTile / kBlock;  // of them per thread

// |x| with NaN taken as +inf (a maximum that a NaN cannot hide in)
__device__ __forceinline__ double abs_or_inf(double x) { return x == x ? fabs(x) : INFINITY; }

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double w = __shfl_xor(v, o, kWave);
        v = w > v ? w : v;
    }
    return v;
}

template <int NT>
__device__ __forceinline__ double block_max(double v, double* lds) {
    v = wave_max(v);
    const int w = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) lds[w] = v;
    __syncthreads();
    double m = lds[0];
#pragma unroll
    for (int i = 1; i < NT / kWave; ++i) m = lds[i] > m ? lds[i] : m;
    __syncthreads();
    return m;
}

}  // namespace

// ---------------------------------------------------------------------------
// 1. Setup (one workgroup per problem)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_msvd_setup(const double* __restrict__ alpha,
                                                       const double* __restrict__ beta, int32_t L,
                                                       const int32_t* __restrict__ l_ptr, double* __restrict__ ws,
                                                       double* __restrict__ ftil, int32_t* __restrict__ status,
                                                       ProjBatch pb) {
    const int64_t z = blockIdx.x;
    alpha += z * pb.vec;
    beta += z * pb.vec;
    ftil += z * pb.vec;
    if (l_ptr != nullptr) l_ptr += z * pb.lstr;
    if (status != nullptr) status += z;
    const SvdWs w = svd_ws(ws + z * pb.ws, L);
    const int l = l_ptr != nullptr ? *l_ptr : L;
    __shared__ double sa[kMaxEll], sb[kMaxEll + 1], sd[kMaxEll], se[kMaxEll], sg[kMaxEll];
    __shared__ double red[kBlock / kWave];
    const int tid = threadIdx.x;
    if (l <= 0) {
        if (tid == 0) {
            ftil[0] = beta[0];
            w.flag[0] = 0;
            w.flag[1] = 0;
            if (status != nullptr) status[0] = 0;
        }
        return;
    }
    double plain = 0.0;
    for (int i = tid; i < l; i += kBlock) {
        const double a = alpha[i], b = beta[i + 1];
        sa[i] = a;
        sb[i + 1] = b;
        se[i] = 0.0;
        if (!(a >= 1e-30 && a <= 1e30 && (b == 0.0 || (b >= 1e-100 && b <= 1e30)))) plain = 1.0;
    }
    if (tid == 0) sb[0] = beta[0];
    plain = block_max<kBlock>(plain, red);
    if (plain == 0.0) {
        // Positive coefficients of moderate size (what the Golub-Kahan step writes): the
        // square of rhobar as a quotient of positive numbers,
        //     q_i = u / v,  v' = u + beta_{i+1}^2 v,  u' = alpha_{i+1}^2 u,
        // a linear map of (u, v) per step, so the chain of square roots and divisions
        // becomes a scan over one wave (7.5 us at l = 300, the chain 85).  The rotations,
        // c^2 = u / v', s^2 = beta^2 v / v', rho^2 = v' / v, are then formed by all
        // threads.  Where rhobar falls below 1e-120 the rotations themselves are run.
        if (tid < kWave) {
            // step i is the map [[a, 0], [c, b]] = [[alpha^2, 0], [1, beta^2]] of (u, v):
            // a chunk of steps per lane, a scan over the lanes, the chunks again
            const int per = (l - 1 + kWave - 1) / kWave;
            const int i0 = tid * per < l - 1 ? tid * per : l - 1, i1 = i0 + per < l - 1 ? i0 + per : l - 1;
            msvd::QMap m{1.0, 0.0, 1.0};
            for (int i = i0; i < i1; ++i) {
                const double a = sa[i + 1], b = sb[i + 1];
                m = msvd::after(msvd::QMap{a * a, 1.0, b * b}, m);
            }
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const msvd::QMap p{__shfl_up(m.a, o, kWave), __shfl_up(m.c, o, kWave), __shfl_up(m.b, o, kWave)};
                if (tid >= o) m = msvd::after(m, p);
            }
            const double pa = __shfl_up(m.a, 1, kWave), pc = __shfl_up(m.c, 1, kWave), pb1 = __shfl_up(m.b, 1, kWave);
            double u = sa[0] * sa[0], v = 1.0;
            if (tid == 0) {
                sd[0] = u;
                sg[0] = v;
            } else {
                v = fma(pc, u, pb1);
                u *= pa;
            }
            for (int i = i0; i < i1; ++i) {
                const double sc = msvd::pair_scale(u, v), a = sa[i + 1], b = sb[i + 1];
                u *= sc;
                v *= sc;
                v = fma(b * b, v, u);
                u *= a * a;
                sd[i + 1] = u;
                sg[i + 1] = v;
            }
        }
        __syncthreads();
        for (int i = tid; i < l; i += kBlock) {
            const double u = sd[i], v = sg[i];
            if (!(u > 1e-280 && v > 1e-280 && u < 1e280 && v < 1e280 && u > 1e-240 * v)) plain = 1.0;
        }
        plain = block_max<kBlock>(plain, red);
    }
    if (plain > 0.0) {
        if (tid == 0) ftil[l] = bsvd::reduce_lower(sa, sb, l, sd, se, sg);
    } else {
        for (int i = tid; i < l; i += kBlock) {
            const double u = sd[i], v = sg[i], b = sb[i + 1];
            const double vn = fma(b * b, v, u);
            const double sn = b * sqrt(v / vn);
            sd[i] = sqrt(vn / v);
            sg[i] = sqrt(u / vn);
            if (i + 1 < l) se[i] = sn * sa[i + 1];
            sb[i + 1] = sn;  // each entry is read above by this thread alone
        }
        __syncthreads();
        if (tid < kWave) {  // carry beta_1 e_1 (g_i = c_i phibar_i), by a scan of the products of -s_i
            const int per = (l + kWave - 1) / kWave;
            const int i0 = tid * per < l ? tid * per : l, i1 = i0 + per < l ? i0 + per : l;
            double p = 1.0;
            for (int i = i0; i < i1; ++i) p *= -sb[i + 1];
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const double q = __shfl_up(p, o, kWave);
                if (tid >= o) p *= q;
            }
            const double pre = __shfl_up(p, 1, kWave);
            double phibar = tid == 0 ? sb[0] : sb[0] * pre;
            for (int i = i0; i < i1; ++i) {
                sg[i] *= phibar;
                phibar *= -sb[i + 1];
            }
            if (tid == kWave - 1) ftil[l] = phibar;
        }
    }
    __syncthreads();
    double bad = 0.0, bnd = 0.0;
    for (int i = tid; i < l; i += kBlock) {
        w.d[i] = sd[i];
        w.e[i] = se[i];
        w.g[i] = sg[i];
        const double bi = msvd::eig_bound_row(sd, se, l, i);
        bnd = bi > bnd ? bi : bnd;
        // a zero or non-finite pivot of B (an exactly singular bidiagonal)
        // leaves the relative-accuracy transforms undefined: fallback
        bad = (!(sd[i] > 0.0) || !isfinite(sd[i]) || !isfinite(se[i]) || !isfinite(sg[i])) ? 1.0 : bad;
    }
    bad = block_max<kBlock>(bad, red);
    bnd = block_max<kBlock>(bnd, red);
    if (tid == 0) {
        w.misc[0] = msvd::eig_bound_of(bnd);
        w.flag[0] = bad > 0.0 ? 1 : 0;
        w.flag[1] = 0;
    }
}

// ---------------------------------------------------------------------------
// 2. Values: TPV threads bracket lambda_j = s_j^2, the j-th largest eigenvalue
// of B^T B, by rounds of TPV counts; kBlock / TPV values per workgroup.  Bound by
// the counts' serial chain (msvd::negcount), so one wave per SIMD is the right
// load: 256 threads a value up to l = 256, 128 up to 512, 64 beyond (a function
// of l alone: a problem's values do not depend on its batch).  At l = 300 70 us, nine
// rounds of a chain of 150 steps; with a division on a chain of 300 and 256
// threads a value 282.
// ---------------------------------------------------------------------------
template <int TPV>
__global__ __launch_bounds__(kBlock) void k_msvd_values(int32_t L, const int32_t* __restrict__ l_ptr,
                                                        double* __restrict__ ws, double* __restrict__ sv,
                                                        ProjBatch pb) {
    constexpr int kVals = kBlock / TPV, kWpv = TPV / kWave;
    const int64_t z = blockIdx.y;
    sv += z * pb.vec;
    if (l_ptr != nullptr) l_ptr += z * pb.lstr;
    const SvdWs w = svd_ws(ws + z * pb.ws, L);
    const int l = l_ptr != nullptr ? *l_ptr : L;
    if ((int)blockIdx.x * kVals >= l) return;
    __shared__ double d2[kMaxEll], e2[kMaxEll];
    __shared__ double xs[kBlock];
    __shared__ unsigned long long masks[kBlock / kWave];
    __shared__ int open[kVals];
    const int tid = threadIdx.x, v = tid / TPV, t = tid % TPV;
    const int j = (int)blockIdx.x * kVals + v;
    const bool live = j < l;
    const double bound = w.misc[0];
    const int sh = msvd::pair_shift(bound);
    for (int i = tid; i < l; i += kBlock) {
        const double di = ldexp(w.d[i], -sh), ei = ldexp(w.e[i], -sh);
        d2[i] = di * di;
        e2[i] = ei * ei;
    }
    double lo = 0.0, hi = ldexp(bound, -2 * sh);
    const int k = l - 1 - j;  // lambda_j is the k-th smallest (0-based)
    __syncthreads();
    for (int round = 0; round < 64; ++round) {
        const bool go = live && hi - lo > 2.0 * DBL_EPSILON * hi;
        double x = 0.0;
        unsigned long long m = 0ull;
        if (go) {  // uniform over the value's threads
            x = msvd::section_point(lo, hi, t, TPV);
            m = __ballot(msvd::negcount(d2, 1, e2, 1, l, x, DBL_MIN) <= k);
        }
        xs[tid] = x;
        if ((tid & (kWave - 1)) == 0) masks[tid / kWave] = m;
        if (t == 0) open[v] = go ? 1 : 0;
        __syncthreads();
        bool any = false;
        for (int q = 0; q < kVals; ++q) any = any || open[q] != 0;
        // the largest point with at most k eigenvalues below it
        int ts = -1;
        for (int q = kWpv - 1; q >= 0 && ts < 0; --q) {
            const unsigned long long mq = masks[v * kWpv + q];
            if (mq != 0ull) ts = q * kWave + 63 - __clzll(mq);
        }
        const double nlo = ts >= 0 ? xs[v * TPV + ts] : lo;
        const double nhi = ts + 1 < TPV ? xs[v * TPV + ts + 1] : hi;
        __syncthreads();
        if (!any) break;
        if (go) {
            if (nlo == lo && nhi == hi) {
                hi = lo + 0.5 * (hi - lo);  // cannot shrink further: the midpoint
                lo = hi;
            } else {
                lo = nlo;
                hi = nhi;
            }
        }
    }
    if (t == 0 && live) {
        const double lam = ldexp(lo + 0.5 * (hi - lo), 2 * sh);
        w.lam[j] = lam;
        sv[j] = sqrt(lam);
        // a value with no point below it: not bracketed
        if (!(lo > 0.0)) w.flag[0] = 1;
    }
}

// ---------------------------------------------------------------------------
// 3. Vectors: one wave per (j, problem), for the sides 0 = B^T B on (d, e) and
// 1 = B B^T on the reversed sequences.  Four lanes run the four chains (a side's
// top-down and bottom-up transform) at once, each over operands laid out in its
// order in LDS and overwritten by its pairs (or quotients); quotients, multipliers and twist
// indices are formed by the whole wave, and four lanes again run the two
// directions of both twisted solves.  Operands scaled by a power of two
// (msvd::pair_shift).  Bound by the issue of the chains' instructions by one wave.
// At l = 300 138 us with both transforms in sequence on two lanes and a division
// per step, 36 us now.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kWave) void k_msvd_vectors(int32_t L, const int32_t* __restrict__ l_ptr,
                                                        double* __restrict__ ws, const double* __restrict__ sv,
                                                        double* __restrict__ V, int64_t ldv, ProjBatch pb) {
    const int64_t z = blockIdx.y;
    sv += z * pb.vec;
    V += z * pb.mat;
    if (l_ptr != nullptr) l_ptr += z * pb.lstr;
    const SvdWs w = svd_ws(ws + z * pb.ws, L);
    const int l = l_ptr != nullptr ? *l_ptr : L;
    const int j = blockIdx.x;
    if (j >= l) return;
    extern __shared__ double arrays[];
    double* Ld = arrays;
    double* Le = arrays + L;
    // chain c (bit 0: side, bit 1: bottom-up) at 2 L c: its operands, then its
    // pairs; the top-down ones then (L+, U-), the bottom-up ones z
    double* Ch = arrays + 2 * L;
    const int lane = threadIdx.x;
    const int shf = msvd::pair_shift(w.misc[0]);
    for (int i = lane; i < l; i += kWave) {
        Ld[i] = ldexp(w.d[i], -shf);
        Le[i] = i + 1 < l ? ldexp(w.e[i], -shf) : 0.0;
    }
    const double lam = ldexp(w.lam[j], -2 * shf);
    const double sig = ldexp(sv[j], -shf);
    __syncthreads();
    for (int k = lane; k + 1 < l; k += kWave) msvd::chain_operands(Ld, Le, l, L, k, Ch);
    __syncthreads();
    const bool quot = lane < 4 && msvd::chain_pairs(Ld, Le, l, L, lane, lam, Ch);
    const unsigned quots = (unsigned)__ballot(quot);
    __syncthreads();
    int tw[2];
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        double best = INFINITY;
        int r = l - 1;
        for (int i = lane; i < l; i += kWave) {
            const double g = msvd::twist_step(Ld, Le, l, L, side, i, lam, quots, Ch);
            if (g < best) {  // ties to the smaller index
                best = g;
                r = i;
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double ob = __shfl_xor(best, o, kWave);
            const int orr = __shfl_xor(r, o, kWave);
            if (ob < best || (ob == best && orr < r)) {
                best = ob;
                r = orr;
            }
        }
        tw[side] = r;
    }
    __syncthreads();
    if (lane < 4) {
        const int side = lane & 1;
        const int r = side ? tw[1] : tw[0];
        const int dn = lane >> 1;  // 0: upwards by L+, 1: downwards by U-
        msvd::twisted_from(Ch + 2 * L * side + dn, 2, l, r, dn ? 1 : -1, Ch + 2 * L * (side + 2));
    }
    __syncthreads();
    // norms; side 1 holds u in reversed order: u_k = Zu[l - 1 - k]
    const double* Zv = Ch + 4 * L;
    const double* Zu = Ch + 6 * L;
    double nv = 0.0, nu = 0.0;
    for (int k = lane; k < l; k += kWave) {
        nv = fma(Zv[k], Zv[k], nv);
        nu = fma(Zu[k], Zu[k], nu);
    }
    nv = wave_sum(nv);
    nu = wave_sum(nu);
    const double iv = 1.0 / sqrt(nv), iu = 1.0 / sqrt(nu);
    // sign of u from u^T B v > 0
    double t = 0.0;
    for (int k = lane; k < l; k += kWave) {
        const double vk1 = k + 1 < l ? Le[k] * Zv[k + 1] : 0.0;
        t = fma(Zu[l - 1 - k], fma(Ld[k], Zv[k], vk1), t);
    }
    t = wave_sum(t);
    const double su = t < 0.0 ? -iu : iu;
    // residuals of B v = s u and B^T u = s v; h = u^T g
    double r1 = 0.0, r2 = 0.0, hg = 0.0;
    for (int k = lane; k < l; k += kWave) {
        const double vk = Zv[k] * iv;
        const double vk1 = k + 1 < l ? Zv[k + 1] * iv : 0.0;
        const double uk = Zu[l - 1 - k] * su;
        const double ukm = k > 0 ? Zu[l - k] * su : 0.0;
        const double a = msvd::resid_row(Ld[k], vk, k + 1 < l ? Le[k] : 0.0, vk1, sig, uk);
        const double b = msvd::resid_row(Ld[k], uk, k > 0 ? Le[k - 1] : 0.0, ukm, sig, vk);
        hg = fma(uk, w.g[k], hg);
        r1 = fma(a, a, r1);
        r2 = fma(b, b, r2);
        V[(int64_t)j * ldv + k] = vk;
        w.U[(int64_t)j * L + k] = uk;
    }
    r1 = wave_sum(r1);
    r2 = wave_sum(r2);
    hg = wave_sum(hg);
    if (lane == 0) {
        w.h[j] = hg;
        const double rr = sqrt(r1 > r2 ? r1 : r2) / msvd::resid_bound(sig, ldexp(sv[0], -shf), l);
        w.res[j] = rr == rr ? rr : INFINITY;
    }
}

// ---------------------------------------------------------------------------
// 4. Gram matrices on the FP64 matrix cores (v_mfma_f64_16x16x4f64: lane l
// supplies A[l%16][l/16] and B[l/16][l%16] and receives D[4r + l/16][l%16]):
// tile (bx, by) of V^T V - I (part 0, kept in E) or of U^T U - I (part 1, only its
// largest entry), one 16 x 16 quarter per wave, 11 us at l = 300 (36 with the sums on
// the vector units); part 2 forms w = U h (32 rows per
// bx, by = 0) into lam, which no later step reads as eigenvalues.
// ---------------------------------------------------------------------------
typedef double v4d __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kBlock) void k_msvd_gram(int32_t L, const int32_t* __restrict__ l_ptr,
                                                      double* __restrict__ ws, const double* __restrict__ V,
                                                      int64_t ldv, ProjBatch pb) {
    const int which = blockIdx.z % 3;
    const int64_t z = blockIdx.z / 3;
    V += z * pb.mat;
    if (l_ptr != nullptr) l_ptr += z * pb.lstr;
    const SvdWs w = svd_ws(ws + z * pb.ws, L);
    const int l = l_ptr != nullptr ? *l_ptr : L;
    const int ntl = (l + kGramTile - 1) / kGramTile;
    const int bi = blockIdx.x, bj = blockIdx.y;
    if (bi >= ntl || bj >= ntl) return;
    __shared__ double red[kBlock / kGramTile][kGramTile];
    const int tid = threadIdx.x;
    if (which == 2) {
        if (bj != 0) return;
        const int r = tid % kGramTile, g = tid / kGramTile;
        const int row = bi * kGramTile + r;
        double a = 0.0;
        if (row < l) {
#pragma unroll 16
            for (int q = g; q < l; q += kBlock / kGramTile) a = fma(w.U[(int64_t)q * L + row], w.h[q], a);
        }
        red[g][r] = a;
        __syncthreads();
        if (g == 0 && row < l) {
            for (int q = 1; q < kBlock / kGramTile; ++q) a += red[q][r];
            w.lam[row] = a;
        }
        return;
    }
    const double* M = which ? w.U : V;
    const int64_t ld = which ? (int64_t)L : ldv;
    // kGramK rows of the tile's two column sets at a time through LDS, the next ones
    // in registers; a stride of 2 past a multiple of 32 doubles keeps the operand
    // reads off each other's banks
    __shared__ double Ts[2][kGramTile][kGramK + 2];
    const int lane = tid & (kWave - 1), wv = tid / kWave, li = lane & 15, lk = lane >> 4;
    const int i0 = bi * kGramTile + 16 * (wv >> 1), j0 = bj * kGramTile + 16 * (wv & 1);
    // half a wave loads the kGramK rows of every eighth column
    const int sk = tid % kGramK, sc = tid / kGramK;
    double a[kGramRows], b[kGramRows];
    auto fetch = [&](int k0) {
        const int kc = k0 + sk < l ? k0 + sk : 0;
#pragma unroll
        for (int q = 0; q < kGramRows; ++q) {
            const int c = sc + kBlock / kGramK * q, ci = bi * kGramTile + c, cj = bj * kGramTile + c;
            a[q] = M[(int64_t)(ci < l ? ci : 0) * ld + kc];
            b[q] = M[(int64_t)(cj < l ? cj : 0) * ld + kc];
        }
    };
    v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
    fetch(0);
    for (int k0 = 0; k0 < l; k0 += kGramK) {
        __syncthreads();  // the previous chunk has been read
#pragma unroll
        for (int q = 0; q < kGramRows; ++q) {
            // what lies outside is dropped here: a choice at the load becomes a branch
            // around it, and the loads then follow one another
            const int c = sc + kBlock / kGramK * q;
            const bool in = k0 + sk < l;
            Ts[0][c][sk] = in && bi * kGramTile + c < l ? a[q] : 0.0;
            Ts[1][c][sk] = in && bj * kGramTile + c < l ? b[q] : 0.0;
        }
        __syncthreads();
        if (k0 + kGramK < l) fetch(k0 + kGramK);
#pragma unroll
        for (int k = 0; k < kGramK; k += 4)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Ts[0][16 * (wv >> 1) + li][k + lk],
                                                       Ts[1][16 * (wv & 1) + li][k + lk], acc, 0, 0, 0);
    }
    double m = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = i0 + 4 * r + lk, jj = j0 + li;
        if (i < l && jj < l) {
            const double v = acc[r] - (i == jj ? 1.0 : 0.0);
            if (!which) w.E[(int64_t)i * L + jj] = v;
            const double av = abs_or_inf(v);
            m = av > m ? av : m;
        }
    }
    m = block_max<kBlock>(m, &red[0][0]);
    if (tid == 0) w.tmax[which * kSvdTiles + bi * (kSvdTiles / 32) + bj] = m;
}

// ---------------------------------------------------------------------------
// 5. Acceptance test and the symmetric correction.  Workgroup b updates rows
// kFinRows b .. of V (all columns: V <- V - V E / 2, from a copy of the rows in
// LDS; a wave takes 256 columns and its share of the sum) and computes f~_j for the
// same j; every workgroup takes the same decision from the tile maxima and
// residuals.  Bound by the reads of E, which every workgroup makes in full; with
// four rows a workgroup there are 75 of them at l = 300: 26 us, against 31 with 16
// rows on the matrix cores (whose FP64 rate is that of the vector units), and 90
// with a serial sum per thread and U h formed by every workgroup.
// ---------------------------------------------------------------------------
constexpr int kFinThreads = 512;
constexpr int kFinCols = 4;  // columns per thread
constexpr int kFinWaves = kFinThreads / kWave;

__global__ __launch_bounds__(kFinThreads) void k_msvd_finish(int32_t L, const int32_t* __restrict__ l_ptr,
                                                             double* __restrict__ ws, double* __restrict__ V,
                                                             int64_t ldv, double* __restrict__ ftil,
                                                             int32_t* __restrict__ status, ProjBatch pb) {
    const int64_t z = blockIdx.y;
    V += z * pb.mat;
    ftil += z * pb.vec;
    if (l_ptr != nullptr) l_ptr += z * pb.lstr;
    if (status != nullptr) status += z;
    const SvdWs w = svd_ws(ws + z * pb.ws, L);
    const int l = l_ptr != nullptr ? *l_ptr : L;
    const int r0 = blockIdx.x * kFinRows;
    if (r0 >= l) return;
    __shared__ double Vr[kMaxEll][kFinRows];
    __shared__ double part[kFinWaves][kFinRows][kFinCols * kWave];
    __shared__ double red[kFinWaves];
    const int tid = threadIdx.x;
    const int ntl = (l + kGramTile - 1) / kGramTile;
    double mo = 0.0, mr = 0.0;
    for (int q = tid; q < 2 * ntl * ntl; q += kFinThreads) {
        const int which = q / (ntl * ntl), rem = q % (ntl * ntl);
        const double v = abs_or_inf(w.tmax[which * kSvdTiles + (rem / ntl) * (kSvdTiles / 32) + rem % ntl]);
        mo = v > mo ? v : mo;
    }
    for (int i = tid; i < l; i += kFinThreads) {
        const double v = abs_or_inf(w.res[i]);
        mr = v > mr ? v : mr;
    }
    mo = block_max<kFinThreads>(mo, red);
    mr = block_max<kFinThreads>(mr, red);
    const bool ok = w.flag[0] == 0 && mo <= msvd::kOrthTol && mr <= 1.0;
    if (!ok) {
        if (blockIdx.x == 0 && tid == 0) {
            w.flag[1] = 1;
            if (status != nullptr) status[0] = 2;
        }
        return;
    }
    const int lane = tid & (kWave - 1), wv = tid / kWave;
    const int rv = tid % kFinRows, rc = r0 + rv < l ? r0 + rv : r0;  // a row past l repeats the first
#pragma unroll 4
    for (int i = tid / kFinRows; i < l; i += kFinThreads / kFinRows) Vr[i][rv] = V[(int64_t)i * ldv + rc];
    __syncthreads();
    // strips of 256 columns (four a lane, so that a value of V read from LDS meets
    // four of E), the sum over i dealt to the waves of a strip
    constexpr int kStrip = kFinCols * kWave;
    const int nstrip = (l + kStrip - 1) / kStrip, ngrp = kFinWaves / nstrip;
    const int strip = wv % nstrip, grp = wv / nstrip;
    double acc[kFinRows][kFinCols] = {};
    if (grp < ngrp) {
        const double* Ec[kFinCols];
#pragma unroll
        for (int c = 0; c < kFinCols; ++c) {
            const int col = strip * kStrip + c * kWave + lane;
            Ec[c] = w.E + (col < l ? col : 0);
        }
#pragma unroll 8
        for (int i = grp; i < l; i += ngrp) {
            double e[kFinCols];
#pragma unroll
            for (int c = 0; c < kFinCols; ++c) e[c] = Ec[c][(int64_t)i * L];
#pragma unroll
            for (int r = 0; r < kFinRows; ++r)
#pragma unroll
                for (int c = 0; c < kFinCols; ++c) acc[r][c] = fma(Vr[i][r], e[c], acc[r][c]);
        }
    }
#pragma unroll
    for (int r = 0; r < kFinRows; ++r)
#pragma unroll
        for (int c = 0; c < kFinCols; ++c) part[wv][r][c * kWave + lane] = acc[r][c];
    __syncthreads();
    for (int q = tid; q < l * kFinRows; q += kFinThreads) {
        const int i = q / kFinRows, rr = q % kFinRows;
        double a = 0.0;
        for (int g = 0; g < ngrp; ++g) a += part[g * nstrip + i / kStrip][rr][i % kStrip];
        if (r0 + rr < l) V[(int64_t)i * ldv + r0 + rr] = fma(-0.5, a, Vr[i][rr]);
    }
    // f~_j = h_j - ((U^T U - I) h)_j / 2 = 1.5 h_j - u_j^T (U h) / 2, one wave per j
    const int jj = r0 + wv;
    if (wv < kFinRows && jj < l) {
        double a = 0.0;
#pragma unroll 4
        for (int r = lane; r < l; r += kWave) a = fma(w.U[(int64_t)jj * L + r], w.lam[r], a);
        a = wave_sum(a);
        if (lane == 0) ftil[jj] = fma(1.5, w.h[jj], -0.5 * a);
    }
    if (blockIdx.x == 0 && tid == 0 && status != nullptr) status[0] = 0;
}

// Steps 2 to 5.
static void launch_msvd_steps(int32_t l, const int32_t* l_ptr, double* ws, double* sv, double* ftil, double* V,
                              int64_t ldv, int32_t* status, hipStream_t s, int nz, const ProjBatch& pb) {
    if (l <= 256)
        k_msvd_values<256><<<dim3(l, nz), kBlock, 0, s>>>(l, l_ptr, ws, sv, pb);
    else if (l <= 512)
        k_msvd_values<128><<<dim3((l + 1) / 2, nz), kBlock, 0, s>>>(l, l_ptr, ws, sv, pb);
    else
        k_msvd_values<64><<<dim3((l + 3) / 4, nz), kBlock, 0, s>>>(l, l_ptr, ws, sv, pb);
    k_msvd_vectors<<<dim3(l, nz), kWave, 10 * (size_t)l * sizeof(double), s>>>(l, l_ptr, ws, sv, V, ldv, pb);
    const int nt = (l + kGramTile - 1) / kGramTile;
    k_msvd_gram<<<dim3(nt, nt, 3 * nz), kBlock, 0, s>>>(l, l_ptr, ws, V, ldv, pb);
    k_msvd_finish<<<dim3((l + kFinRows - 1) / kFinRows, nz), kFinThreads, 0, s>>>(l, l_ptr, ws, V, ldv, ftil, status,
                                                                                  pb);
}

// ---------------------------------------------------------------------------
// Host launcher: the fast path, then the QR iteration for flagged problems
// (mode 0); the QR iteration alone (mode 1); the fast path alone, a failed
// acceptance test leaving status 2 (mode 2).
// ---------------------------------------------------------------------------
void launch_bidiag_svd(const double* alpha, const double* beta, int32_t l, const int32_t* l_ptr, double* ws,
                       double* sv, double* ftil, double* V, int64_t ldv, int32_t* status, int mode, hipStream_t s,
                       int nz, ProjBatch pb) {
    if (mode != 1) {
        k_msvd_setup<<<nz, kBlock, 0, s>>>(alpha, beta, l, l_ptr, ws, ftil, status, pb);
        launch_msvd_steps(l, l_ptr, ws, sv, ftil, V, ldv, status, s, nz, pb);
    }
    if (mode != 2) launch_bidiag_qr(alpha, beta, l, l_ptr, ws, sv, ftil, V, ldv, status, mode == 0, s, nz, pb);
}

void launch_msvd_core(int32_t l, double* ws, double* sv, double* ftil, double* V, int64_t ldv, int32_t* status,
                      hipStream_t s) {
    launch_msvd_steps(l, nullptr, ws, sv, ftil, V, ldv, status, s, 1, ProjBatch{});
}

}  // namespace mqh
