// block_kernels.hip -- the block Golub-Kahan process for s <= 16 right-hand
// sides that share one Krylov space (Algorithm 1 with an n x s starting
// block) on gfx950, FP64.
//
// Two tall-skinny contractions carry the reorthogonalisation against a
// shared basis of m columns (m = s j at step j) and the block QR:
//   c = V^T P   (m x s, K = n rows)        -- k_blk_gemvt + k_blk_reduce
//   P -= V c, or P = V c                   -- k_blk_update (with P^T P on request)
// both on the FP64 matrix cores (v_mfma_f64_16x16x4f64: lane l supplies
// A[l%16][l/16] and B[l/16][l%16] and receives D[4r + l/16][l%16]).  The
// block QR is shifted Cholesky QR applied three times (the shift in the
// first pass keeps the Cholesky factorisation defined for nearly dependent
// columns; the two unshifted passes restore orthogonality to rounding):
// k_blk_chol adds the parts of one 16 x 16 Gram matrix and factors it.

#include <float.h>
#include <math.h>

#include "common.hpp"
#include "kernels.hpp"

namespace mqh {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kBt = 64;        // rows of a staged tile; basis columns per workgroup of k_blk_gemvt
constexpr int kBtLd = kBt + 1;  // padded LDS row of the basis tile
constexpr int kPLd = kBlkRhs + 1;

// part[(chunk m + col) 16 + k] = sum over the rows i of the chunk (i < n) of
// V[col][i] P[k][i], for col < m and all 16 k (zero for k >= s).  V: column
// col at V + col ldv; P: column k at P + k ldp.  Grid (chunks, ceil(m / 64)),
// chunk a multiple of 64; wave w forms columns 64 y + 16 w .. + 15.
__global__ __launch_bounds__(kBlock) void k_blk_gemvt(const double* __restrict__ V, const double* __restrict__ P,
                                                      int64_t n, int64_t chunk, int64_t ldv, int64_t ldp, int32_t m,
                                                      int32_t s, double* __restrict__ part) {
    __shared__ double tV[kBt * kBtLd];
    __shared__ double tP[kBt * kPLd];
    const int64_t r0 = (int64_t)blockIdx.x * chunk;
    const int64_t r1 = r0 + chunk < n ? r0 + chunk : n;
    const int c0 = blockIdx.y * kBt;
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int li = lane & 15, lk = lane >> 4;
    const int rr = threadIdx.x & (kBt - 1), rq = threadIdx.x / kBt;  // staging: row rr, column rq + 4 q
    v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
    for (int64_t rb = r0; rb < r1; rb += kBt) {
        const int64_t row = rb + rr;
        const bool rok = row < r1;
        const int64_t rl = rok ? row : rb;
        constexpr int kNv = kBt / (kBlock / kBt), kNp = kBlkRhs / (kBlock / kBt);
        // all loads in flight together (under conditions they wait one by one: 6.8 -> 5.6 us
        // at 20 000 rows, m = 16 .. 112)
        double tv[kNv], tp[kNp];
#pragma unroll
        for (int q = 0; q < kNv; ++q) {
            const int col = c0 + rq + (kBlock / kBt) * q;
            tv[q] = V[(int64_t)(col < m ? col : c0) * ldv + rl];
        }
#pragma unroll
        for (int q = 0; q < kNp; ++q) {
            const int k = rq + (kBlock / kBt) * q;
            tp[q] = P[(int64_t)(k < s ? k : 0) * ldp + rl];
        }
#pragma unroll
        for (int q = 0; q < kNv; ++q) arrived(tv[q]);
#pragma unroll
        for (int q = 0; q < kNp; ++q) arrived(tp[q]);
        __syncthreads();  // the previous tile's reads are done
#pragma unroll
        for (int q = 0; q < kNv; ++q) {
            const int cc = rq + (kBlock / kBt) * q;
            tV[rr * kBtLd + cc] = rok && c0 + cc < m ? tv[q] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < kNp; ++q) {
            const int k = rq + (kBlock / kBt) * q;
            tP[rr * kPLd + k] = rok && k < s ? tp[q] : 0.0;
        }
        __syncthreads();
#pragma unroll 4
        for (int kk = 0; kk < kBt; kk += 4) {
            // A[i][k'] = V[col 16 w + i][row kk + k'], B[k'][j] = P[rhs j][row kk + k']
            const double a = tV[(kk + lk) * kBtLd + 16 * w + li];
            const double b = tP[(kk + lk) * kPLd + li];
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int col = c0 + 16 * w + 4 * r + lk;
        if (col < m) part[((int64_t)blockIdx.x * m + col) * kBlkRhs + li] = acc[r];
    }
}

// c[col 16 + k] = sum over chunks of part[(chunk m + col) 16 + k]: one wave
// per entry, lane l summing chunks l, l + 64, ... in order, then a fixed
// shuffle tree (deterministic).
__global__ __launch_bounds__(kBlock) void k_blk_reduce(const double* __restrict__ part, int chunks, int32_t m,
                                                       double* __restrict__ c) {
    const int64_t e = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (e >= (int64_t)m * kBlkRhs) return;  // wave-uniform
    const int lane = threadIdx.x & (kWave - 1);
    double v = 0.0;
    for (int q = lane; q < chunks; q += kWave) v += part[(int64_t)q * m * kBlkRhs + e];
    v = wave_sum(v);
    if (lane == 0) c[e] = v;
}

// Rows of the s output columns, 16 per wave and turn:
//   sub = 1: P[k][i] -= sum_col V[col][i] c[col cs + k ks]
//   sub = 0: P[k][i]  = sum_col V[col][i] c[col cs + k ks]
// (V may be P itself for sub = 0: a wave reads all its rows before it
// writes them, and no two waves share a row).  Workgroup x takes rows
// [x chunk, (x + 1) chunk), chunk a multiple of the rows of a turn.  With GRAM it also leaves its part
// of the Gram matrix of the columns it writes, in the layout of k_blk_gemvt for m =
// s: the new values are the operands of the products as the lanes hold them, so
// the pass of k_blk_gemvt over P and its launch are saved (6.3 + 5.6 -> 6.5 us
// at 20 000 rows, m = s = 16).
// Products of four columns whose loads are in flight together (a load under a
// condition, one product at a time, waits for itself: 6.5 -> 5.7 us at 20 000 rows).
constexpr int kUpdU = 4;
constexpr int kGramThreads = 512;
constexpr int64_t kGramRowsPer = 16 * (kGramThreads / kWave);  // rows of a workgroup in one turn

template <bool GRAM, int NT>
__global__ __launch_bounds__(NT) void k_blk_update(const double* V, int64_t ldv, int64_t n, int32_t m,
                                                       const double* __restrict__ c, int64_t cs, int64_t ks,
                                                       double* P, int64_t ldp, int32_t s, int32_t sub, int64_t chunk,
                                                       double* __restrict__ part) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int li = lane & 15, lk = lane >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * chunk;
    const int64_t r1 = r0 + chunk < n ? r0 + chunk : n;
    v4d gram = v4d{0.0, 0.0, 0.0, 0.0};
    for (int64_t row0 = r0 + 16 * w; row0 < r1; row0 += 16 * (NT / kWave)) {
        const int64_t row = row0 + li;
        const bool rok = row < n;
        v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
        const double* vr = V + (rok ? row : row0);
        const double* cr = c + (int64_t)(li < s ? li : 0) * ks;
        for (int kk = 0; kk < m; kk += 4 * kUpdU) {
            // A[i][k'] = V[col kk + k'][row0 + i], B[k'][j] = c[col kk + k'][j]
            double a[kUpdU], b[kUpdU];  // the loads of kUpdU products in flight together
#pragma unroll
            for (int u = 0; u < kUpdU; ++u) {
                const int64_t col = kk + 4 * u + lk < m ? kk + 4 * u + lk : m - 1;
                a[u] = vr[col * ldv];
                b[u] = cr[col * cs];
            }
#pragma unroll
            for (int u = 0; u < kUpdU; ++u) {
                arrived(a[u]);
                arrived(b[u]);
            }
#pragma unroll
            for (int u = 0; u < kUpdU; ++u) {
                if (kk + 4 * u >= m) break;
                const bool cok = kk + 4 * u + lk < m;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(rok && cok ? a[u] : 0.0, cok && li < s ? b[u] : 0.0, acc, 0,
                                                           0, 0);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t rr = row0 + 4 * r + lk;
            const bool in = li < s && rr < n;
            double* dst = P + (int64_t)(in ? li : 0) * ldp + (in ? rr : row0);
            const double v = sub ? *dst - acc[r] : acc[r];
            if (in) *dst = v;
            acc[r] = in ? v : 0.0;
        }
        if (GRAM) {
#pragma unroll
            for (int r = 0; r < 4; ++r) gram = __builtin_amdgcn_mfma_f64_16x16x4f64(acc[r], acc[r], gram, 0, 0, 0);
        }
    }
    if (GRAM) {
        __shared__ double g[NT / kWave][kBlkRhs][kBlkRhs + 1];
#pragma unroll
        for (int r = 0; r < 4; ++r) g[w][4 * r + lk][li] = gram[r];
        __syncthreads();
        const int i = threadIdx.x / kBlkRhs, k = threadIdx.x % kBlkRhs;
        if (i >= s) return;
        double v = g[0][i][k];
#pragma unroll
        for (int q = 1; q < NT / kWave; ++q) v += g[q][i][k];
        part[((int64_t)blockIdx.x * s + i) * kBlkRhs + k] = v;
    }
}
static_assert(kGramThreads >= kBlkRhs * kBlkRhs, "one entry of the Gram matrix per thread");

// What the block QR's last pass does with the factor (no host round trip per step).
// kind 0: E_1 (the data's factor, kept in E1; a diagonal entry at most tau
// times its largest, or a failed factorisation, marks the sources invalid);
// kind 1: D_j = R^T of step j; kind 2: E_{j+1} = R.  For kinds 1 and 2 the
// running scale is the largest diagonal entry of the D and E blocks so far; a
// failed factorisation or a diagonal entry at most tau times the scale stops
// the run (ell_done = j - 1 at a D block, j at an E block, flag = kind).
// Otherwise the block goes into C (row-major, ld ldc) and its transpose (16 x
// 16, the update kernel's coefficient layout) into mat, the coefficients of
// the next shift.  Once stopped, nothing is written.  One wave; R: the factor in LDS.
__device__ void blk_check(const double (*R)[kBlkRhs + 1], bool bad, int32_t s, const BlkCheck& ck) {
    const int lane = threadIdx.x, j = ck.j;
    BlkState* bs = ck.bs;
    const double d = fabs(R[lane & 15][lane & 15]);
    double mn = (lane & 15) < s ? d : HUGE_VAL, mx = (lane & 15) < s ? d : 0.0;
    // NaN loses every comparison, as in a scan of the diagonal
    mn = mn < HUGE_VAL ? mn : HUGE_VAL;
    mx = mx > 0.0 ? mx : 0.0;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
        const double a = __shfl_xor(mn, o, kWave), b = __shfl_xor(mx, o, kWave);
        mn = a < mn ? a : mn;
        mx = b > mx ? b : mx;
    }
    const double scale = bs->scale;
    bool ok = bs->stopped == 0;
    if (!ok) return;
    if (ck.kind == 0) {
        ok = !bad && mn > ck.tau * mx;
        if (!ok && lane == 0) {
            bs->invalid = 1;
            bs->stopped = 1;
            bs->ell_done = 0;
        }
    } else {
        const double sc = mx > scale ? mx : scale;
        ok = !bad && mn > ck.tau * sc;
        if (lane == 0) {
            if (!ok) {
                bs->stopped = 1;
                bs->ell_done = ck.kind == 1 ? j - 1 : j;
                bs->flag = ck.kind;
            } else {
                bs->scale = sc;
            }
        }
    }
    if (!ok) return;
    for (int q = lane; q < kBlkRhs * kBlkRhs; q += kWave) {
        const int r = q / kBlkRhs, c = q % kBlkRhs;
        const double v = R[r][c];
        const bool in = r < s && c < s;
        ck.mat[c * kBlkRhs + r] = in ? v : 0.0;
        if (!in) continue;
        if (ck.kind == 0)
            ck.E1[r * s + c] = v;
        else if (ck.kind == 1)
            ck.C[(int64_t)((j - 1) * s + c) * ck.ldc + (j - 1) * s + r] = v;  // D_j = R^T
        else
            ck.C[(int64_t)(j * s + r) * ck.ldc + (j - 1) * s + c] = v;  // E_{j+1} = R
    }
}

// One pass (0, 1, 2) of (shifted) Cholesky QR on one workgroup.  All threads add the
// chunks' parts of G (c layout, G[i 16 + j] = P_i . P_j, i, j < s), thread group
// q the chunks q, q + kCholGroups, ..; one wave does the rest.  G plus, in pass 0,
// 11 (n s + s (s + 1)) eps trace(G) on the diagonal is factored as R^T R by row
// elimination, lane (j, g) = (l % 16, l / 16) with rows 4 g .. + 3 of column j; the
// same operations take the identity to R^{-T}, so no substitution follows.
// Rinv = R^{-1} in the c layout of k_blk_update (Rinv[col 16 + k]); Racc <- R Racc
// (row-major 16 x 16, the accumulated triangular factor, from the identity in pass
// 0).  status (0 at pass 0) <- 1 if a pivot is not positive and finite; Racc and Rinv
// are then left as they were.  Pass 2 ends with blk_check.
// 12.5 us with 157 parts, most of it their way to one compute unit and the columns'
// chain, in place of a reduction of 4.7, a factorisation of 13.3 (three barriers
// a column, a serial substitution) and a third of the launches for the identity
// (4.3) and the breakdown test (4.4).
constexpr int kCholGroups = 4;

__global__ __launch_bounds__(kCholGroups* kBlkRhs* kBlkRhs) void k_blk_chol(
    const double* __restrict__ part, int chunks, int32_t s, int64_t n, int32_t pass, double* __restrict__ Rinv,
    double* __restrict__ Racc, int32_t* __restrict__ status, BlkCheck ck) {
    __shared__ double G[kCholGroups][kBlkRhs * kBlkRhs];
    __shared__ double R[kBlkRhs][kBlkRhs + 1], Q[kBlkRhs][kBlkRhs + 1];
    {
        const int e = threadIdx.x % (kBlkRhs * kBlkRhs), q = threadIdx.x / (kBlkRhs * kBlkRhs);
        double v = 0.0;
        if (e < s * kBlkRhs) {
            const double* pe = part + e;
#pragma unroll 8
            for (int c = q; c < chunks; c += kCholGroups) v += pe[(int64_t)c * s * kBlkRhs];
        }
        G[q][e] = v;
    }
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    const int lane = threadIdx.x, j = lane & 15, g = lane >> 4;
    double m[4], y[4];  // entries (4 g + r, j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = 4 * g + r, e = i * kBlkRhs + j;
        double v = G[0][e];
#pragma unroll
        for (int q = 1; q < kCholGroups; ++q) v += G[q][e];
        m[r] = (i < s && j < s) ? v : 0.0;
        y[r] = i == j ? 1.0 : 0.0;
        Q[i][j] = pass == 0 ? y[r] : Racc[e];
    }
    bool bad = pass != 0 && *status != 0;
    if (pass == 0) {
        double tr = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) tr += 4 * g + r == j ? m[r] : 0.0;
        tr = wave_sum(tr);
        const double shift = 11.0 * ((double)n * s + (double)s * (s + 1)) * DBL_EPSILON * tr;
#pragma unroll
        for (int r = 0; r < 4; ++r) m[r] += (4 * g + r == j && j < s) ? shift : 0.0;
    }
    bool fail = false;
    // a rolled loop: the code is fetched once, and cold
#pragma unroll 1
    for (int c = 0; c < s; ++c) {
        const int rc = c & 3;
        if (g == c >> 2) {  // row c to every lane
            R[0][j] = rc == 0 ? m[0] : rc == 1 ? m[1] : rc == 2 ? m[2] : m[3];
            R[1][j] = rc == 0 ? y[0] : rc == 1 ? y[1] : rc == 2 ? y[2] : y[3];
        }
        wave_sync();
        const double d = R[0][c];
        double rj = R[0][j], yj = R[1][j], ri[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) ri[r] = R[0][4 * g + r];
        const bool pos = d > 0.0 && isfinite(d);
        fail = fail || !pos;
        const double inv = pos ? rsqrt_f64(d) : 1.0;
        rj *= inv;
        yj *= inv;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * g + r;
            const double f = i > c ? -ri[r] * inv : 0.0;
            m[r] = i == c ? rj : fma(f, rj, m[r]);
            y[r] = i == c ? yj : fma(f, yj, y[r]);
        }
        wave_sync();
    }
    if (!fail) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * g + r;
            R[i][j] = i <= j ? m[r] : 0.0;
            // row i of R^{-T} is column i of R^{-1}
            Rinv[j * kBlkRhs + i] = (j <= i && i < s) ? y[r] : 0.0;
        }
        wave_sync();
        v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < kBlkRhs; k += 4)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(R[j][k + g], Q[k + g][j], acc, 0, 0, 0);
        wave_sync();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * r + g;
            if (i < s && j < s) Q[i][j] = j >= i ? acc[r] : 0.0;
        }
    }
    wave_sync();
    if (!fail || pass == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * g + r;
            Racc[i * kBlkRhs + j] = Q[i][j];
        }
    }
    bad = bad || fail;
    if (lane == 0 && (pass == 0 || fail)) *status = bad ? 1 : 0;
    if (pass == 2) blk_check(Q, bad, s, ck);
}

}  // namespace

int blk_chunks(int64_t n, int32_t m, int64_t* chunk) {
    const int64_t tiles = (m + kBt - 1) / kBt;
    int64_t want = (1024 + tiles - 1) / tiles;
    const int64_t cmax = (n + kBt - 1) / kBt;
    if (want > cmax) want = cmax;
    if (want < 1) want = 1;
    int64_t ch = (n + want - 1) / want;
    ch = (ch + kBt - 1) / kBt * kBt;
    *chunk = ch;
    return (int)((n + ch - 1) / ch);
}

void launch_blk_gemvt(const double* V, int64_t ldv, int64_t n, int32_t m, const double* P, int64_t ldp, int32_t s,
                      double* part, double* c, hipStream_t st) {
    int64_t chunk;
    const int chunks = blk_chunks(n, m, &chunk);
    k_blk_gemvt<<<dim3((unsigned)chunks, (unsigned)((m + kBt - 1) / kBt)), kBlock, 0, st>>>(V, P, n, chunk, ldv, ldp, m, s, part);
    const int64_t waves = (int64_t)m * kBlkRhs, per = kBlock / kWave;
    k_blk_reduce<<<(unsigned)((waves + per - 1) / per), kBlock, 0, st>>>(part, chunks, m, c);
}

void launch_blk_update(const double* V, int64_t ldv, int64_t n, int32_t m, const double* c, int64_t cs, int64_t ks,
                       double* P, int64_t ldp, int32_t s, int32_t sub, hipStream_t st) {
    const int64_t rows_per_block = 16 * (kBlock / kWave);
    k_blk_update<false, kBlock><<<(unsigned)((n + rows_per_block - 1) / rows_per_block), kBlock, 0, st>>>(
        V, ldv, n, m, c, cs, ks, P, ldp, s, sub, rows_per_block, nullptr);
}

// Workgroups (and rows of each) of an update that leaves the Gram matrix: at most
// 256 parts for the next k_blk_chol to add.
static int gram_chunks(int64_t n, int64_t* chunk) {
    int64_t ch = (n + 255) / 256;
    ch = (ch + kGramRowsPer - 1) / kGramRowsPer * kGramRowsPer;
    *chunk = ch;
    return (int)((n + ch - 1) / ch);
}

int launch_blk_update_gram(const double* V, int64_t ldv, int64_t n, int32_t m, const double* c, int64_t cs, int64_t ks,
                           double* P, int64_t ldp, int32_t s, int32_t sub, double* part, hipStream_t st) {
    int64_t chunk;
    const int chunks = gram_chunks(n, &chunk);
    k_blk_update<true, kGramThreads>
        <<<(unsigned)chunks, kGramThreads, 0, st>>>(V, ldv, n, m, c, cs, ks, P, ldp, s, sub, chunk, part);
    return chunks;
}

int launch_blk_gram(const double* P, int64_t ldp, int64_t n, int32_t s, double* part, hipStream_t st) {
    int64_t chunk;
    const int chunks = blk_chunks(n, s, &chunk);
    k_blk_gemvt<<<dim3((unsigned)chunks, 1), kBlock, 0, st>>>(P, P, n, chunk, ldp, ldp, s, s, part);
    return chunks;
}

void launch_blk_chol(const double* part, int chunks, int32_t s, int64_t n, int32_t pass, double* Rinv, double* Racc,
                     int32_t* status, const BlkCheck& ck, hipStream_t st) {
    k_blk_chol<<<1, kCholGroups * kBlkRhs * kBlkRhs, 0, st>>>(part, chunks, s, n, pass, Rinv, Racc, status, ck);
}

// The Jacobi route's work matrix of the projected problem from the device
// copies: G[i][j] = C[i][j] (m x ls, leading dimension ldc) and the data
// columns G[i][m + k] = E1[i][k] for i < s (rows i >= s stay zero).  G is
// zero on entry (full_reset).
__global__ __launch_bounds__(kBlock) void k_blk_fill_g(const double* __restrict__ C, int64_t ldc, int64_t m,
                                                       int64_t ls, const double* __restrict__ E1, int32_t s,
                                                       double* __restrict__ G, int64_t ldg) {
    const int64_t i = blockIdx.y;
    const double* ci = C + i * ldc;
    double* gi = G + i * ldg;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < ls; j += (int64_t)gridDim.x * kBlock) gi[j] = ci[j];
    if (blockIdx.x == 0 && i < s && (int)threadIdx.x < s) gi[m + threadIdx.x] = E1[i * s + threadIdx.x];
}

void launch_blk_fill_g(const double* C, int64_t ldc, int64_t m, int64_t ls, const double* E1, int32_t s, double* G,
                       int64_t ldg, hipStream_t st) {
    const unsigned gx = (unsigned)((ls + kBlock - 1) / kBlock);
    k_blk_fill_g<<<dim3(gx, (unsigned)m), kBlock, 0, st>>>(C, ldc, m, ls, E1, s, G, ldg);
}

}  // namespace mqh
