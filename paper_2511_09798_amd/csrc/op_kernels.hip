// op_kernels.hip -- the matrix-free Kansa operator on gfx950: products with
// FP64 entries or FP32 entries and FP64 accumulation (single vectors and
// blocks of right-hand sides), the deterministic split-K reduction, the rows
// of A as the products generate them and the evaluation of the RBF
// expansion.  (The stored matrix is in stored_kernels.hip.)
//
// Layout: n nodes as double4/float4 records (centred, scaled by eps; the
// 4th lane is padding).  Vectors have a leading dimension ldn (multiple of
// 64, >= n) and are zero past n.
#include "kernels.hpp"

namespace mqh {

// ---------------------------------------------------------------------------
// FP32-evaluated matrix-free products: the squared distances on the matrix
// cores.
//
// Nodes are visited in a spatially sorted order (Morton order within each
// class, interior first) and cut into blocks of kMfmFixed "fixed" nodes, each
// with a frame centre c among its nodes.  With d = P - c (P the eps-scaled
// node, in FP32),
//     t_ij = 1 + |d_i - d_j|^2 = |d_i|^2 + sum_k a_ik b_kj,
//     a_i = (-2 d_i, 1),  b_j = (d_j, 1 + |d_j|^2),
// a K = 4 contraction per 16 x 16 tile of entries.  Each FP32 factor is split
// exactly into three bf16 parts by truncation (h = top 8 significant bits,
// m = next 8, l = the last 8), and the eight cross products that matter at
// FP32 precision (all but l*l, 2^-32 relative) are laid out along K = 32 of
// one v_mfma_f32_16x16x32_bf16: t comes out with FP32 accuracy at half the
// matrix-core time of the FP32 MFMA.  Close pairs have small |d_i|, |d_j|
// (the frame sits among the fixed nodes), so t keeps its relative accuracy
// where 1 + eps^2 r^2 is near 1.  The entries are evaluated on the VALU from
// t: by the pair products (one vector) and the block products (16 vectors)
// below.
//
// Lane layout of v_mfma_f32_16x16x32_bf16 (wave64): lane l holds A[l%16][k]
// and B[k][l%16] for k = 8(l/16) .. 8(l/16)+7, and D[4(l/16)+r][l%16],
// r = 0..3.  Lane group g = l/16 carries coordinate g (g < 3) or the
// 1 * (1 + |d_j|^2) term (g = 3).
// ---------------------------------------------------------------------------

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));


// Exact split x = h + m + l of a finite FP32 value into three bf16 values,
// returned as FP32 bit patterns with zero low halves: h keeps the top 16 bits
// of x, m those of x - h (exact), l = x - h - m (exact, at most 8 significant
// bits).
__device__ __forceinline__ void split_bf16x3(float x, unsigned& h, unsigned& m, unsigned& l) {
    h = __float_as_uint(x) & 0xFFFF0000u;
    const float r1 = x - __uint_as_float(h);
    m = __float_as_uint(r1) & 0xFFFF0000u;
    l = __float_as_uint(r1 - __uint_as_float(m));
}

// Two bf16 values in one dword: lo's high half in bits 0..15, hi's in 16..31.
__device__ __forceinline__ unsigned pack_bf16(unsigned lo, unsigned hi) {
    return __builtin_amdgcn_perm(hi, lo, 0x07060302u);
}

// Eight K slots of one coordinate: the cross products
// (h,h) (h,m) (m,h) (h,l) (l,h) (m,m) (m,l) (l,m) of a (fixed side) and b.
__device__ __forceinline__ v4u fixed_terms(float a) {
    unsigned h, m, l;
    split_bf16x3(a, h, m, l);
    v4u r;
    r[0] = pack_bf16(h, h);
    r[1] = pack_bf16(m, h);
    r[2] = pack_bf16(l, m);
    r[3] = pack_bf16(m, l);
    return r;
}
__device__ __forceinline__ v4u loop_terms(float b) {
    unsigned h, m, l;
    split_bf16x3(b, h, m, l);
    v4u r;
    r[0] = pack_bf16(h, m);
    r[1] = pack_bf16(h, l);
    r[2] = pack_bf16(h, m);
    r[3] = pack_bf16(l, m);
    return r;
}

// ---------------------------------------------------------------------------
// FP32-evaluated products over unordered pairs of nodes.
//
// The entry of A depends on t_ij = 1 + eps^2 r_ij^2 and on the kind of its
// row only, so A_ij and A_ji share t and s = t^(-1/2): for an interior row
// the entry is (kappa^2 t + 2 eps^2 + eps^2 s^2) s, for a boundary row
// t s = sqrt(t).  A product y = A x (or A^T x) therefore needs each
// unordered pair {i, j} once: y_i += A_ij x_j and y_j += A_ji x_i (A^T: the
// two entries swap).  On this GPU the rsqrt of an entry costs as much as all
// its other VALU work together and overlaps none of it, so halving the
// pairs halves the dominant cost.
//
// Work item (k, s) of the SymLayout: fixed blocks fb of super-row k one
// after another; for each, the loop blocks c >= fb of segment s in chunks
// of at most two blocks of one class (the block's own square fb == fb on its
// own, row sums only).  Per 16 x 16 tile the MFMA above gives t (frame of
// the fixed block); a lane holds 4 fixed rows x 1 loop column per tile and
// kMfmFt tiles.  Row sums stay per lane in FP32 over a chunk, then FP64;
// a tile's column sums (a lane's 8 rows in FP32) are added over pairs of
// lane groups by a swizzle and stored to LDS, and after the chunk the 8
// partials of each loop node are added in FP64 and collected in LDS over the
// item's fixed blocks.  Weights come
// from XS[q].w (w = x[perm[q]] in FP32).  Work items are launched largest
// first and write their partials at their place in (super-row, segment) order.
// ---------------------------------------------------------------------------

// B: nodes per block of the layout.
template <int B = kMfmFixed>
__device__ __forceinline__ int64_t sym_blk_start(int b, const SymLayout& L) {
    return b < L.nb_int ? (int64_t)b * B : L.n_int + (int64_t)(b - L.nb_int) * B;
}
template <int B = kMfmFixed>
__device__ __forceinline__ int64_t sym_blk_end(int b, const SymLayout& L) {
    const int64_t e = sym_blk_start<B>(b, L) + B;
    const int64_t lim = b < L.nb_int ? L.n_int : L.n;
    return e < lim ? e : lim;
}

// A work item, the run's state and the layout's sizes by one wait: left to itself the
// compiler reads the layout from the arguments after the item has come.
__device__ __forceinline__ void arrived_with_layout(int& item, int& stop, SymLayout& L) {
    asm volatile(""
                 : "+s"(item), "+s"(stop), "+s"(L.n), "+s"(L.n_int), "+s"(L.nb_int), "+s"(L.nb), "+s"(L.F),
                   "+s"(L.Lb));
}

// Sum of a row's 16 lane partials by four neighbouring lanes (part p takes 4p ..
// 4p + 3), in a fixed order; every lane gets the sum.
__device__ __forceinline__ double row_sum16(const double* __restrict__ row, int p) {
    double s = (row[4 * p] + row[4 * p + 1]) + (row[4 * p + 2] + row[4 * p + 3]);
    s = add_xor<2>(add_xor<1>(s));
    return s;
}

// NT staged tiles of 16 loop nodes against the lane's fixed rows.  RI / CI:
// the row sums / column sums take the interior formula (else the boundary
// one); SYM: column sums wanted (off the block's own square).
template <bool RI, bool CI, bool SYM, int NT>
__device__ __forceinline__ void mfs_tiles(const v4u* __restrict__ lds_b, const float* __restrict__ lds_w,
                                          const v4u (&a)[kMfmFt], const v4f (&C)[kMfmFt],
                                          const float (&xi)[kMfmFt][4], float k2, float e2x2, float e2,
                                          double (&acc)[kMfmFt][4], float* __restrict__ colw) {
    const int lane = threadIdx.x & (kWave - 1), g = lane >> 4, jj = lane & 15;
    float s32[kMfmFt][4];
#pragma unroll
    for (int f = 0; f < kMfmFt; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) s32[f][r] = 0.f;
    v4f t[kMfmFt];
    float wl = lds_w[jj];
    {
        const v8bf bk = __builtin_bit_cast(v8bf, lds_b[jj * 4 + g]);
#pragma unroll
        for (int f = 0; f < kMfmFt; ++f)
            t[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a[f]), bk, C[f], 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        if (u < NT) {
            v4f tn[kMfmFt];
            float wn = wl;
            if (u + 1 < NT) {
                const v8bf bn = __builtin_bit_cast(v8bf, lds_b[((u + 1) * 16 + jj) * 4 + g]);
                wn = lds_w[(u + 1) * 16 + jj];
#pragma unroll
                for (int f = 0; f < kMfmFt; ++f)
                    tn[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a[f]), bn, C[f], 0, 0, 0);
            }
            float cp = 0.f;
#pragma unroll
            for (int f = 0; f < kMfmFt; ++f) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float tt = t[f][r];
                    if (RI && CI) {
                        const float sv = __builtin_amdgcn_rsqf(tt);
                        const float e = fmaf(e2, sv * sv, fmaf(k2, tt, e2x2)) * sv;
                        s32[f][r] = fmaf(e, wl, s32[f][r]);
                        if (SYM) cp = fmaf(e, xi[f][r], cp);
                    } else if (!RI && !CI) {
                        const float e = __builtin_amdgcn_sqrtf(tt);
                        s32[f][r] = fmaf(e, wl, s32[f][r]);
                        if (SYM) cp = fmaf(e, xi[f][r], cp);
                    } else {
                        const float sv = __builtin_amdgcn_rsqf(tt);
                        const float ei = fmaf(e2, sv * sv, fmaf(k2, tt, e2x2)) * sv;
                        const float eb = tt * sv;
                        s32[f][r] = fmaf(RI ? ei : eb, wl, s32[f][r]);
                        cp = fmaf(CI ? ei : eb, xi[f][r], cp);
                    }
                }
            }
            // keep the row and column sums at their tile: left to itself the
            // compiler sinks them to their uses after the loop and holds every
            // tile's entries live until then
#pragma unroll
            for (int f = 0; f < kMfmFt; ++f)
                asm volatile("" : "+v"(s32[f][0]), "+v"(s32[f][1]), "+v"(s32[f][2]), "+v"(s32[f][3]));
            if (SYM) {
                // lanes l and l ^ 16 hold the same loop node: add them (ds_swizzle,
                // xor 16 within each half-wave) and let the lower lane store
                const float o = __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(cp), 0x401F));
                cp += o;
                if ((lane & 16) == 0) colw[u * 16] = cp;
            }
            if (u + 1 < NT) {
#pragma unroll
                for (int f = 0; f < kMfmFt; ++f) t[f] = tn[f];
                wl = wn;
            }
        }
    }
#pragma unroll
    for (int f = 0; f < kMfmFt; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[f][r] += (double)s32[f][r];
}

template <int NT>
__device__ __forceinline__ void mfs_dispatch(bool ri, bool ci, const v4u* lds_b, const float* lds_w,
                                             const v4u (&a)[kMfmFt], const v4f (&C)[kMfmFt],
                                             const float (&xi)[kMfmFt][4], float k2, float e2x2, float e2,
                                             double (&acc)[kMfmFt][4], float* colw) {
    if (ri && ci)
        mfs_tiles<true, true, true, NT>(lds_b, lds_w, a, C, xi, k2, e2x2, e2, acc, colw);
    else if (!ri && !ci)
        mfs_tiles<false, false, true, NT>(lds_b, lds_w, a, C, xi, k2, e2x2, e2, acc, colw);
    else if (ri)
        mfs_tiles<true, false, true, NT>(lds_b, lds_w, a, C, xi, k2, e2x2, e2, acc, colw);
    else
        mfs_tiles<false, true, true, NT>(lds_b, lds_w, a, C, xi, k2, e2x2, e2, acc, colw);
}

// One work item (blockIdx.x) of the SymLayout.  TRANS: y = A^T x.
// RowP[item][(fb - kF) kMfmFixed + row], ColP[sym_col_base(c) + k][node].
template <bool TRANS>
__global__ __launch_bounds__(kBlock) void k_mfs(const PairItem* __restrict__ items, const GkbState* __restrict__ st,
                                                const float4* __restrict__ XS, const float4* __restrict__ frames,
                                                double* __restrict__ RowP, double* __restrict__ ColP, SymLayout L,
                                                EntryConst c) {
    __shared__ v4u lds_b[4 * kMfmChunk];
    __shared__ float lds_w[kMfmChunk];
    __shared__ float lds_col[2 * (kBlock / kWave)][kMfmChunk];  // per (wave, lane-group pair)
    __shared__ double colacc[kSymMaxLb * kMfmFixed];
    PairItem item = items[blockIdx.x];  // launch order: the largest items first
    int stop = st != nullptr ? st->stopped : 0;
    arrived_with_layout(item.x, stop, L);
    if (stop) return;
    const int64_t slot = item.z;
    const int b0 = item.x * L.F;
    const int b1 = b0 + L.F < L.nb ? b0 + L.F : L.nb;
    const int c0 = b0 + item.y * L.Lb;
    const int c1 = c0 + L.Lb < L.nb ? c0 + L.Lb : L.nb;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), g = lane >> 4, jj = lane & 15, wv = tid / kWave;
    for (int i = tid; i < L.Lb * kMfmFixed; i += kBlock) colacc[i] = 0.0;
    // the entry constants in vector registers: an FP32 instruction with a
    // scalar operand does not pair with another in one issue cycle
    float k2 = c.k2f, e2x2 = c.e2x2f, e2 = c.e2f;
    asm volatile("" : "+v"(k2), "+v"(e2x2), "+v"(e2));
    double* red = reinterpret_cast<double*>(lds_b);  // 64 rows x 17 (padded) doubles, between chunks
    // a chunk: two whole blocks of one class, or one (the own square, a short block)
    auto chunk_end = [&](int cb, int fb) {
        const bool two = cb != fb && cb + 1 < c1 && (cb + 1 < L.nb_int) == (cb < L.nb_int) &&
                         sym_blk_end(cb, L) - sym_blk_start(cb, L) == kMfmFixed;
        return cb + (two ? 2 : 1);
    };
    for (int fb = b0; fb < b1; ++fb) {
        const int64_t fs = sym_blk_start(fb, L), fe = sym_blk_end(fb, L);
        const bool fint = fb < L.nb_int;
        const float4 fr = frames[fb];
        int cb = c0 > fb ? c0 : fb;
        float4 qn;  // this thread's node of the next chunk
        {
            const int64_t k = sym_blk_start(cb < c1 ? cb : fb, L) + tid;
            qn = XS[k < L.n ? k : L.n - 1];
        }
        // the lane's fixed nodes, all in flight together (rows past the block read
        // its first): loads under a condition wait one by one, ten latencies a
        // fixed block (1 800 nodes, one block a workgroup: 9.9 -> 9.0 us)
        float4 qa[kMfmFt], qc[kMfmFt][4];
#pragma unroll
        for (int f = 0; f < kMfmFt; ++f) {
            const int64_t base = fs + (int64_t)(wv * kMfmFt + f) * 16;
            qa[f] = XS[base + jj < fe ? base + jj : fs];
#pragma unroll
            for (int r = 0; r < 4; ++r) qc[f][r] = XS[base + 4 * g + r < fe ? base + 4 * g + r : fs];
        }
#pragma unroll
        for (int f = 0; f < kMfmFt; ++f) {
            arrived(qa[f]);
#pragma unroll
            for (int r = 0; r < 4; ++r) arrived(qc[f][r]);
        }
        v4u a[kMfmFt];
        v4f C[kMfmFt];
        float xi[kMfmFt][4];
        double acc[kMfmFt][4];
#pragma unroll
        for (int f = 0; f < kMfmFt; ++f) {
            const int64_t base = fs + (int64_t)(wv * kMfmFt + f) * 16;
            const int64_t i = base + jj;
            float d[3] = {0.f, 0.f, 0.f};
            if (i < fe) {
                d[0] = qa[f].x - fr.x;
                d[1] = qa[f].y - fr.y;
                d[2] = qa[f].z - fr.z;
            }
            if (g < 3) {
                a[f] = fixed_terms(-2.0f * d[g]);
            } else {
                const unsigned one = 0x3F80u;  // bf16 1.0
                a[f][0] = one | (one << 16);
                a[f][1] = one;
                a[f][2] = 0u;
                a[f][3] = 0u;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t i2 = base + 4 * g + r;
                float d2 = 0.f, w = 0.f;
                if (i2 < fe) {
                    const float4 q = qc[f][r];
                    const float ex = q.x - fr.x, ey = q.y - fr.y, ez = q.z - fr.z;
                    d2 = fmaf(ez, ez, fmaf(ey, ey, ex * ex));
                    w = q.w;
                }
                C[f][r] = d2;
                xi[f][r] = w;
                acc[f][r] = 0.0;
            }
        }
        while (cb < c1) {
            const bool diag = cb == fb;
            const bool cint = cb < L.nb_int;
            const int ce = chunk_end(cb, fb);
            const int64_t j0 = sym_blk_start(cb, L), j1 = sym_blk_end(ce - 1, L);
            // stage the chunk's loop nodes in the fixed block's frame: B
            // operand (4 lane groups x 8 bf16) and weight; past j1: d = 0, w = 0
            const float4 q = qn;
            if (ce < c1) {  // the next chunk's nodes, in flight during this one
                const int64_t k = sym_blk_start(ce, L) + tid;
                qn = XS[k < L.n ? k : L.n - 1];
            }
            float dx = 0.f, dy = 0.f, dz = 0.f, w = 0.f;
            if (j0 + tid < j1) {
                w = q.w;
                dx = q.x - fr.x;
                dy = q.y - fr.y;
                dz = q.z - fr.z;
            }
            const v4u bb0 = loop_terms(dx), bb1 = loop_terms(dy), bb2 = loop_terms(dz);
            unsigned h, m, l;
            split_bf16x3(fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, 1.0f))), h, m, l);
            v4u bb3;
            bb3[0] = pack_bf16(h, m);
            bb3[1] = l >> 16;
            bb3[2] = 0u;
            bb3[3] = 0u;
            __syncthreads();  // the previous chunk (or the row reduction) is done with LDS
            lds_b[tid * 4 + 0] = bb0;
            lds_b[tid * 4 + 1] = bb1;
            lds_b[tid * 4 + 2] = bb2;
            lds_b[tid * 4 + 3] = bb3;
            lds_w[tid] = w;
            __syncthreads();
            // row sums: formula of the rows of A the fixed nodes stand for
            // (A x: the fixed rows; A^T x: the loop rows); column sums: the other
            const bool ri = TRANS ? cint : fint, ci = TRANS ? fint : cint;
            float* colw = &lds_col[2 * wv + (g >> 1)][jj];
            if (diag) {
                if (fint)
                    mfs_tiles<true, true, false, 8>(lds_b, lds_w, a, C, xi, k2, e2x2, e2, acc, colw);
                else
                    mfs_tiles<false, false, false, 8>(lds_b, lds_w, a, C, xi, k2, e2x2, e2, acc, colw);
            } else if (ce == cb + 2) {
                mfs_dispatch<16>(ri, ci, lds_b, lds_w, a, C, xi, k2, e2x2, e2, acc, colw);
            } else {
                mfs_dispatch<8>(ri, ci, lds_b, lds_w, a, C, xi, k2, e2x2, e2, acc, colw);
            }
            if (!diag) {
                // the chunk's column sums: the 8 (wave, lane-group pair) partials of each loop node
                __syncthreads();
                if (tid < (int)(j1 - j0)) {
                    double v = 0.0;
#pragma unroll
                    for (int q = 0; q < 2 * (kBlock / kWave); ++q) v += (double)lds_col[q][tid];
                    colacc[(cb - c0) * kMfmFixed + tid] += v;
                }
            }
            cb = ce;
        }
        // the fixed block's row sums: each row's 16 lane partials in a fixed order
        double* rp = RowP + slot * L.F * kMfmFixed + (int64_t)(fb - b0) * kMfmFixed;
#pragma unroll
        for (int f = 0; f < kMfmFt; ++f) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(wv * 16 + 4 * g + r) * 17 + jj] = acc[f][r];
            __syncthreads();
            const int node = tid >> 2;
            const double sum = row_sum16(red + node * 17, tid & 3);
            const int row = ((node >> 4) * kMfmFt + f) * 16 + (node & 15);
            if ((tid & 3) == 0) rp[row] = fs + row < fe ? sum : 0.0;
        }
    }
    __syncthreads();
    for (int i = tid; i < (c1 - c0) * kMfmFixed; i += kBlock)
        ColP[(sym_col_base(c0 + i / kMfmFixed, L.F) + item.x) * kMfmFixed + i % kMfmFixed] = colacc[i];
}

// ---------------------------------------------------------------------------
// FP64 products over unordered pairs of nodes: the work items, lane layout
// and partials of k_mfs with every quantity in FP64.  A lane holds the
// coordinates and weights of 4 fixed rows (4g + r) of each of its kMfmFt
// tiles and takes loop node jj of each staged tile of 16; t = 1 + |P_i -
// P_j|^2 comes from the coordinate differences (FP64 VALU; the matrix cores
// at FP64 would save little and leave t exposed to the rank-4 form's
// cancellation), s = t^(-1/2) from the FP64 estimate and one third-order step,
// the entry as in the single-entry FP64 products.  Row sums stay per lane in
// FP64 and are reduced over the 16 lanes of a row at the end of the fixed
// block; column sums are added over the lane's 8 rows, over lane groups g by
// a swizzle and LDS, and collected per item as in k_mfs.  XS64: sorted
// coordinates, the weight x[perm[q]] in .w (written by k_gather_w64).
// ---------------------------------------------------------------------------

__device__ __forceinline__ double swizzle_xor16(double v) {
    const int lo = __builtin_amdgcn_ds_swizzle(__double2loint(v), 0x401F);
    const int hi = __builtin_amdgcn_ds_swizzle(__double2hiint(v), 0x401F);
    return __hiloint2double(hi, lo);
}

// nt tiles of 16 staged loop nodes against the lane's 4 FT fixed rows.
template <bool RI, bool CI, bool SYM, int FT>
__device__ __forceinline__ void mfs64_tiles(const double4* __restrict__ lds_p, int nt, const double (&px)[FT][4],
                                            const double (&py)[FT][4], const double (&pz)[FT][4],
                                            const double (&xi)[FT][4], double k2, double e2x2, double e2,
                                            double (&acc)[FT][4], double* __restrict__ colw) {
    const int lane = threadIdx.x & (kWave - 1), jj = lane & 15;
    for (int u = 0; u < nt; ++u) {
        const double4 q = lds_p[u * 16 + jj];
        double cp = 0.0;
#pragma unroll
        for (int f = 0; f < FT; ++f) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double dx = px[f][r] - q.x, dy = py[f][r] - q.y, dz = pz[f][r] - q.z;
                const double t = fma(dz, dz, fma(dy, dy, fma(dx, dx, 1.0)));
                const double sv = rsqrt_f64(t);
                if (RI && CI) {
                    const double e = fma(e2, sv * sv, fma(k2, t, e2x2)) * sv;
                    acc[f][r] = fma(e, q.w, acc[f][r]);
                    if (SYM) cp = fma(e, xi[f][r], cp);
                } else if (!RI && !CI) {
                    const double e = t * sv;
                    acc[f][r] = fma(e, q.w, acc[f][r]);
                    if (SYM) cp = fma(e, xi[f][r], cp);
                } else {
                    const double ei = fma(e2, sv * sv, fma(k2, t, e2x2)) * sv;
                    const double eb = t * sv;
                    acc[f][r] = fma(RI ? ei : eb, q.w, acc[f][r]);
                    cp = fma(CI ? ei : eb, xi[f][r], cp);
                }
            }
        }
        // keep the row sums at their tile (left to itself the compiler sinks
        // them past the loop and holds every tile's entries live)
#pragma unroll
        for (int f = 0; f < FT; ++f)
            asm volatile("" : "+v"(acc[f][0]), "+v"(acc[f][1]), "+v"(acc[f][2]), "+v"(acc[f][3]));
        if (SYM) {
            // lanes l and l ^ 16 hold the same loop node: add them and let the lower lane store
            cp += swizzle_xor16(cp);
            if ((lane & 16) == 0) colw[u * 16] = cp;
        }
    }
}

// One work item of the layout, blocks of B = 64 FT nodes.
template <bool TRANS, int FT>
__global__ __launch_bounds__(kBlock) void k_mfs64(const PairItem* __restrict__ items, const GkbState* __restrict__ st,
                                                  const double4* __restrict__ XS64, double* __restrict__ RowP,
                                                  double* __restrict__ ColP, SymLayout L, EntryConst c) {
    constexpr int B = 64 * FT;
    __shared__ double4 lds_p[kMfmChunk];
    __shared__ double lds_col[2 * (kBlock / kWave)][kMfmChunk];  // per (wave, lane-group pair)
    __shared__ double colacc[kSymMaxLb * B];
    double* red = &lds_col[0][0];  // 64 rows x 17 (padded), between chunks (four workgroups fit a CU's LDS)
    PairItem item = items[blockIdx.x];
    int stop = st != nullptr ? st->stopped : 0;
    arrived_with_layout(item.x, stop, L);
    if (stop) return;
    const int64_t slot = item.z;
    const int b0 = item.x * L.F;
    const int b1 = b0 + L.F < L.nb ? b0 + L.F : L.nb;
    const int c0 = b0 + item.y * L.Lb;
    const int c1 = c0 + L.Lb < L.nb ? c0 + L.Lb : L.nb;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), g = lane >> 4, jj = lane & 15, wv = tid / kWave;
    for (int i = tid; i < L.Lb * B; i += kBlock) colacc[i] = 0.0;
    const double k2 = c.k2, e2x2 = c.e2x2, e2 = c.e2;
    for (int fb = b0; fb < b1; ++fb) {
        const int64_t fs = sym_blk_start<B>(fb, L), fe = sym_blk_end<B>(fb, L);
        const bool fint = fb < L.nb_int;
        double px[FT][4], py[FT][4], pz[FT][4], xi[FT][4], acc[FT][4];
        int cb = c0 > fb ? c0 : fb;
#pragma unroll
        for (int f = 0; f < FT; ++f) {
            const int64_t base = fs + (int64_t)(wv * FT + f) * 16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t i2 = base + 4 * g + r;
                const double4 q = XS64[i2 < fe ? i2 : fs];
                const bool in = i2 < fe;
                px[f][r] = q.x;
                py[f][r] = q.y;
                pz[f][r] = q.z;
                xi[f][r] = in ? q.w : 0.0;
                acc[f][r] = 0.0;
            }
        }
        while (cb < c1) {
            const bool diag = cb == fb;
            const bool cint = cb < L.nb_int;
            // a chunk: as many whole blocks of one class as the staging holds (the own square alone)
            int ce = cb + 1;
            while (!diag && ce < c1 && (ce - cb) < kMfmChunk / B && (ce < L.nb_int) == cint) ++ce;
            const int64_t j0 = sym_blk_start<B>(cb, L), j1 = sym_blk_end<B>(ce - 1, L);
            const int nt = (int)((j1 - j0 + 15) / 16);
            // stage the chunk's loop nodes (coordinates and weight); past j1 the
            // first node with weight 0 (its column sums are not collected)
            const int64_t j = j0 + tid;
            double4 q = XS64[j < j1 ? j : j0];
            if (!(j < j1)) q.w = 0.0;
            __syncthreads();  // the previous chunk (or the row reduction) is done with LDS
            lds_p[tid] = q;
            __syncthreads();
            const bool ri = TRANS ? cint : fint, ci = TRANS ? fint : cint;
            double* colw = &lds_col[2 * wv + (g >> 1)][jj];
            if (diag) {
                if (fint)
                    mfs64_tiles<true, true, false, FT>(lds_p, nt, px, py, pz, xi, k2, e2x2, e2, acc, colw);
                else
                    mfs64_tiles<false, false, false, FT>(lds_p, nt, px, py, pz, xi, k2, e2x2, e2, acc, colw);
            } else {
                if (ri && ci)
                    mfs64_tiles<true, true, true, FT>(lds_p, nt, px, py, pz, xi, k2, e2x2, e2, acc, colw);
                else if (!ri && !ci)
                    mfs64_tiles<false, false, true, FT>(lds_p, nt, px, py, pz, xi, k2, e2x2, e2, acc, colw);
                else if (ri)
                    mfs64_tiles<true, false, true, FT>(lds_p, nt, px, py, pz, xi, k2, e2x2, e2, acc, colw);
                else
                    mfs64_tiles<false, true, true, FT>(lds_p, nt, px, py, pz, xi, k2, e2x2, e2, acc, colw);
                // the chunk's column sums: the 8 (wave, lane-group pair) partials of each loop node
                __syncthreads();
                if (tid < (int)(j1 - j0)) {
                    double v = 0.0;
#pragma unroll
                    for (int qq = 0; qq < 2 * (kBlock / kWave); ++qq) v += lds_col[qq][tid];
                    colacc[(cb - c0) * B + tid] += v;
                }
            }
            cb = ce;
        }
        // the fixed block's row sums: each row's 16 lane partials in a fixed order
        double* rp = RowP + slot * L.F * B + (int64_t)(fb - b0) * B;
#pragma unroll
        for (int f = 0; f < FT; ++f) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(wv * 16 + 4 * g + r) * 17 + jj] = acc[f][r];
            __syncthreads();
            const int node = tid >> 2;
            const double sum = row_sum16(red + node * 17, tid & 3);
            const int row = ((node >> 4) * FT + f) * 16 + (node & 15);
            if ((tid & 3) == 0) rp[row] = fs + row < fe ? sum : 0.0;
        }
    }
    __syncthreads();
    for (int i = tid; i < (c1 - c0) * B; i += kBlock)
        ColP[(sym_col_base(c0 + i / B, L.F) + item.x) * B + i % B] = colacc[i];
}

// XS64[q].w = x[perm[q]]: the weights of a FP64 pair product in the sorted order.
__global__ __launch_bounds__(kBlock) void k_gather_w64(const double* __restrict__ x, const int32_t* __restrict__ perm,
                                                       int64_t n, double4* __restrict__ XS64,
                                                       const GkbState* __restrict__ st) {
    if (st != nullptr && st->stopped) return;
    const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= n) return;
    XS64[q].w = x[perm[q]];
}

// y_o = (row partials of the items of q's super-row + column partials of
// the items whose segment holds q's block) - shift z_o, o = perm[q].  One
// workgroup per block of B nodes, kSymRedThreads / B groups of B threads taking
// every so-many-th row partial (item order) and column partial (super-row
// order), the groups' sums added in group order.  Bound by the latency of the
// strided reads: with a thread per node taking them all one product's
// reduction took 7.1 us at 4 000 nodes and 15 us at 20 000.
constexpr int kSymRedThreads = 1024;

template <int B>
__global__ __launch_bounds__(kSymRedThreads) void k_mfs_reduce(const int32_t* __restrict__ item_first,
                                                               const GkbState* __restrict__ st,
                                                               const double* __restrict__ RowP,
                                                               const double* __restrict__ ColP,
                                                               const int32_t* __restrict__ perm, int F, SymLayout L,
                                                               const double* __restrict__ shift_ptr, double shift_val,
                                                               const double* __restrict__ z, double* __restrict__ y) {
    constexpr int kGroups = kSymRedThreads / B;
    __shared__ double part[kGroups][B];
    const int beta = blockIdx.x;
    const int off = threadIdx.x % B, grp = threadIdx.x / B;
    const int k = beta >> sym_shift(F);
    const int64_t rs = (int64_t)F * B;
    int i0 = item_first[k];
    int stop = st != nullptr ? st->stopped : 0;
    arrived_with_layout(i0, stop, L);
    if (stop) return;
    const int nrow = (L.nb - k * F + L.Lb - 1) / L.Lb;
    const double* rp = RowP + i0 * rs + (int64_t)(beta - k * F) * B + off;
    const double* cp = ColP + sym_col_base(beta, F) * B + off;
    // the output's place and its shift term, while the partials are on their way
    const int64_t q = sym_blk_start<B>(beta, L) + off;
    const bool out = grp == 0 && q < sym_blk_end<B>(beta, L);
    int o = 0;
    if (out) o = perm[q];
    double sc = batched_sum<4>(0.0, cp, grp, k + 1, kGroups, B);
    double zo = 0.0, sh = 0.0;
    if (out && z != nullptr) {
        sh = shift_ptr != nullptr ? *shift_ptr : shift_val;
        zo = z[o];
    }
    double s = batched_sum<4>(0.0, rp, grp, nrow, kGroups, rs);
    s += sc;
    part[grp][off] = s;
    __syncthreads();
    if (!out) return;
    s = 0.0;
#pragma unroll
    for (int g = 0; g < kGroups; ++g) s += part[g][off];
    if (z != nullptr) s -= sh * zo;
    y[o] = s;
}

// XS[q].w = x[perm[q]] in FP32: the weights of a FP32 pair product in the sorted order.
__global__ __launch_bounds__(kBlock) void k_gather_w32(const double* __restrict__ x, const int32_t* __restrict__ perm,
                                                       int64_t n, float4* __restrict__ XS,
                                                       const GkbState* __restrict__ st) {
    if (st != nullptr && st->stopped) return;
    const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= n) return;
    XS[q].w = (float)x[perm[q]];
}

// ---------------------------------------------------------------------------
// Block products for kBlkRhs right-hand sides at once (lockstep Golub-Kahan
// runs sharing each pass over A): P[slice][k][q] = sum over the slice's loop
// nodes j of A(q, j) v_k[j] (rows) or A(j, q) v_k[j] (columns), in sorted
// node order.
//
// Per 16 x 16 tile the squared distances come from the same bf16x3 MFMA as
// in the pair products with the operands swapped (A = loop nodes, B = fixed
// nodes), so a lane holds t for 4 loop nodes j = 4g + r and one fixed node.
// The contraction E (16 fixed x 16 loop) V (16 loop x 16 rhs) runs on the
// matrix cores in FP16 with both operands split in two: the entries, scaled
// by 2^se, as e = e_h + e_l (e_h = fp16(e) to nearest, e_l = fp16(e - e_h)),
// the right-hand sides, each column scaled by its own power of two, as v =
// v_h + v_l alike, and E V ~ E_h V_h + E_l V_h + E_h V_l: three
// v_mfma_f32_16x16x16_f16 (a lane group's 4 K slots are its 4 loop nodes).  e_h + e_l keeps e to 2^-22
// relative (the FP32 entries carry an error of that order from their rsqrt
// already), and the dropped E_l V_l is below 2^-22 |e v|.  Products of two
// fp16 values are exact in FP32; sums are FP32 over one 256-node chunk,
// FP64 across chunks and slices, and the scales are taken out exactly in
// FP64.  On this GPU the FP32 matrix instructions do not overlap VALU work
// while the FP16 ones largely do: four v_mfma_f32_16x16x4_f32 per tile
// (128 cycles, exposed) become three FP16 ones (24 cycles, mostly hidden)
// and 8 VALU instructions for the split of 4 entries.
// ---------------------------------------------------------------------------

typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));

constexpr float kBlkRange = 16384.0f;  // scaled entries and right-hand sides stay below this (fp16 max 65504)

// Two FP32 values as fp16 pairs: H = (fp16(a), fp16(b)) rounded to nearest,
// L = the same of the remainders a - H.lo, b - H.hi (exact in FP32).
__device__ __forceinline__ void split_f16x2(float a, float b, unsigned& H, unsigned& L) {
    const v2h h = __builtin_convertvector((v2f){a, b}, v2h);
    const v2h l = __builtin_convertvector((v2f){a - (float)h[0], b - (float)h[1]}, v2h);
    H = __builtin_bit_cast(unsigned, h);
    L = __builtin_bit_cast(unsigned, l);
}

// Entries of the lane's 4 loop nodes x FT fixed nodes from their squared
// distances, scaled by 2^se, split into (H01, H23, L01, L23).  MIX = 1: the
// interior formula, 0: the boundary one, 2: by the loop node's class
// (node jb + r interior when below n_int; the chunk of a column product that
// straddles the classes).
template <int MIX, int FT>
__device__ __forceinline__ void block_split(const v4f (&t)[FT], const BlockEntry& c, int64_t jb, int64_t n_int,
                                            unsigned (&h)[FT][4]) {
#pragma unroll
    for (int f = 0; f < FT; ++f) {
        float e[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float tt = t[f][r];
            if (MIX == 1) {
                const float sv = __builtin_amdgcn_rsqf(tt);
                e[r] = fmaf(c.e2, sv * sv, fmaf(c.k2, tt, c.e2x2)) * sv;
            } else if (MIX == 0) {
                e[r] = __builtin_amdgcn_sqrtf(tt) * c.bsc;
            } else {
                const float sv = __builtin_amdgcn_rsqf(tt);
                const float ei = fmaf(c.e2, sv * sv, fmaf(c.k2, tt, c.e2x2)) * sv;
                const float eb = tt * sv * c.bsc;
                e[r] = jb + r < n_int ? ei : eb;
            }
        }
        split_f16x2(e[0], e[1], h[f][0], h[f][2]);
        split_f16x2(e[2], e[3], h[f][1], h[f][3]);
    }
}

// Squared distances of tile u (16 staged loop nodes) to the lane's fixed nodes.
template <int FT>
__device__ __forceinline__ void block_tdist(const v4u* __restrict__ lds_a, int u, int jj, int g, const v4u (&bf)[FT],
                                            const v4f (&Cf)[FT], v4f (&t)[FT]) {
    const v8bf ak = __builtin_bit_cast(v8bf, lds_a[(u * 16 + jj) * 4 + g]);
#pragma unroll
    for (int f = 0; f < FT; ++f)
        t[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ak, __builtin_bit_cast(v8bf, bf[f]), Cf[f], 0, 0, 0);
}

// The 16 staged tiles of one chunk (first loop node t0) against the lane's
// fixed tiles, as a three-stage pipeline, fully unrolled: the squared
// distances of tile u + 2, the entries and their split of tile u + 1 and
// the contraction of tile u are in flight together.
template <int MIX, int FT>
__device__ __forceinline__ void mfh_chunk(const v4u* __restrict__ lds_a, const uint4* __restrict__ lds_v, int64_t t0,
                                          int64_t n_int, const BlockEntry& c, const v4u (&bf)[FT],
                                          const v4f (&Cf)[FT], double (&acc)[FT][4]) {
    const int lane = threadIdx.x & (kWave - 1), g = lane >> 4, jj = lane & 15;
    constexpr int kTiles = kMfmChunk / 16;
    // one instruction shape on each accumulator: a chain feeding its own
    // result back as C is the case the matrix cores forward without waiting
    // (a 16x16x16 reading the fresh result of a 16x16x32 as C is not)
    v4f d2[FT];
#pragma unroll
    for (int f = 0; f < FT; ++f) d2[f] = v4f{0.f, 0.f, 0.f, 0.f};
    v4f tc[FT], tn[FT];
    unsigned hc[FT][4];
    block_tdist<FT>(lds_a, 0, jj, g, bf, Cf, tc);
    block_tdist<FT>(lds_a, 1, jj, g, bf, Cf, tn);
    block_split<MIX, FT>(tc, c, t0 + 4 * g, n_int, hc);
#pragma unroll
    for (int u = 0; u < kTiles; ++u) {
        // the lane group's 4 loop nodes, split, for right-hand side jj
        const uint4 bv = lds_v[(u * 4 + g) * kBlkRhs + jj];
        v4f tnn[FT];
        if (u + 2 < kTiles) block_tdist<FT>(lds_a, u + 2, jj, g, bf, Cf, tnn);
        unsigned hn[FT][4];
        if (u + 1 < kTiles) block_split<MIX, FT>(tn, c, t0 + (u + 1) * 16 + 4 * g, n_int, hn);
        // the lane group's 4 loop nodes in the K slots: e_h v_h, e_l v_h, e_h v_l
        const v2u vhi = {bv.x, bv.y}, vlo = {bv.z, bv.w};
#pragma unroll
        for (int f = 0; f < FT; ++f) {
            const v2u ehi = {hc[f][0], hc[f][1]}, elo = {hc[f][2], hc[f][3]};
            d2[f] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(v4h, ehi), __builtin_bit_cast(v4h, vhi),
                                                          d2[f], 0, 0, 0);
            d2[f] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(v4h, elo), __builtin_bit_cast(v4h, vhi),
                                                          d2[f], 0, 0, 0);
            d2[f] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(v4h, ehi), __builtin_bit_cast(v4h, vlo),
                                                          d2[f], 0, 0, 0);
        }
        if (u + 1 < kTiles) {
#pragma unroll
            for (int f = 0; f < FT; ++f) {
#pragma unroll
                for (int q = 0; q < 4; ++q) hc[f][q] = hn[f][q];
                tn[f] = tnn[f];
            }
        }
    }
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[f][r] += (double)d2[f][r];
}

// One slice [j0, j1) of loop nodes (block-uniform; contains barriers; j0 a
// multiple of kMfmChunk).  ROWS: the fixed nodes' class (fint) picks the
// formula; columns: each chunk's loop nodes do.
template <bool ROWS, int FT>
__device__ __forceinline__ void mfh_span(const float4* __restrict__ XS, const uint4* __restrict__ Vh, int64_t j0,
                                         int64_t j1, int64_t n_int, bool fint, const float4& fr, const BlockEntry& c,
                                         const v4u (&bf)[FT], const v4f (&Cf)[FT], double (&acc)[FT][4],
                                         v4u* __restrict__ lds_a, uint4* __restrict__ lds_v) {
    for (int64_t t0 = j0; t0 < j1; t0 += kMfmChunk) {
        const int64_t j = t0 + threadIdx.x;
        float dx = 0.f, dy = 0.f, dz = 0.f;
        if (j < j1) {
            const float4 q = XS[j];
            dx = q.x - fr.x;
            dy = q.y - fr.y;
            dz = q.z - fr.z;
        }
        const v4u a0 = loop_terms(dx), a1 = loop_terms(dy), a2 = loop_terms(dz);
        unsigned h, m, l;
        split_bf16x3(fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, 1.0f))), h, m, l);
        v4u a3;
        a3[0] = pack_bf16(h, m);
        a3[1] = l >> 16;
        a3[2] = 0u;
        a3[3] = 0u;
        // the chunk's split right-hand sides: kMfmChunk / 4 quads x kBlkRhs
        // (a quad past j1 lies past n, where Vh holds zeros, or in the next
        // slice, which starts at a multiple of kMfmChunk: none is read)
        uint4 vq[4];
#pragma unroll
        for (int m4 = 0; m4 < 4; ++m4) {
            const int i = threadIdx.x + m4 * kBlock;
            const int64_t node = t0 + 4 * (i / kBlkRhs);
            vq[m4] = node < j1 ? Vh[((t0 >> 2) + i / kBlkRhs) * kBlkRhs + (i % kBlkRhs)] : make_uint4(0u, 0u, 0u, 0u);
        }
        __syncthreads();  // the previous chunk has been consumed
        lds_a[threadIdx.x * 4 + 0] = a0;
        lds_a[threadIdx.x * 4 + 1] = a1;
        lds_a[threadIdx.x * 4 + 2] = a2;
        lds_a[threadIdx.x * 4 + 3] = a3;
#pragma unroll
        for (int m4 = 0; m4 < 4; ++m4) lds_v[threadIdx.x + m4 * kBlock] = vq[m4];
        __syncthreads();
        const int64_t cend = t0 + kMfmChunk < j1 ? t0 + kMfmChunk : j1;
        if (ROWS ? fint : cend <= n_int)
            mfh_chunk<1, FT>(lds_a, lds_v, t0, n_int, c, bf, Cf, acc);
        else if (ROWS || t0 >= n_int)
            mfh_chunk<0, FT>(lds_a, lds_v, t0, n_int, c, bf, Cf, acc);
        else
            mfh_chunk<2, FT>(lds_a, lds_v, t0, n_int, c, bf, Cf, acc);
    }
}

template <bool ROWS, int FT>
__global__ __launch_bounds__(kBlock) void k_mfh_block(const float4* __restrict__ XS, const uint4* __restrict__ Vh,
                                                      const float4* __restrict__ frames, int64_t n, int64_t n_int,
                                                      int64_t nb_int, int64_t slice_len,
                                                      const float* __restrict__ vsc, double* __restrict__ P,
                                                      int64_t ldp, BlockEntry c) {
    __shared__ v4u lds_a[4 * kMfmChunk];
    __shared__ uint4 lds_v[(kMfmChunk / 4) * kBlkRhs];
    // blocks of kFix = 64 FT fixed nodes per class; the frame is that of the
    // kMfmFixed-node block holding the first of them
    constexpr int kFix = (kBlock / kWave) * FT * 16;
    const int64_t b = blockIdx.x;
    const bool fint = b < nb_int;
    const int64_t fb0 = fint ? b * kFix : n_int + (b - nb_int) * kFix;
    const int64_t fend = fint ? n_int : n;
    const int64_t fb1 = fb0 + kFix < fend ? fb0 + kFix : fend;
    const int64_t nbf_int = (n_int + kMfmFixed - 1) / kMfmFixed;
    const float4 fr = frames[fint ? (b * kFix) / kMfmFixed : nbf_int + ((b - nb_int) * kFix) / kMfmFixed];
    const int lane = threadIdx.x & (kWave - 1), g = lane >> 4, jj = lane & 15, wv = threadIdx.x / kWave;
    v4u bf[FT];
    v4f Cf[FT];
    double acc[FT][4];
#pragma unroll
    for (int f = 0; f < FT; ++f) {
        const int64_t i = fb0 + (int64_t)(wv * FT + f) * 16 + jj;
        float d[3] = {0.f, 0.f, 0.f};
        if (i < fb1) {
            const float4 q = XS[i];
            d[0] = q.x - fr.x;
            d[1] = q.y - fr.y;
            d[2] = q.z - fr.z;
        }
        if (g < 3) {
            bf[f] = fixed_terms(-2.0f * d[g]);
        } else {
            const unsigned one = 0x3F80u;  // bf16 1.0
            bf[f][0] = one | (one << 16);
            bf[f][1] = one;
            bf[f][2] = 0u;
            bf[f][3] = 0u;
        }
        const float d2 = fmaf(d[2], d[2], fmaf(d[1], d[1], d[0] * d[0]));
        Cf[f] = v4f{d2, d2, d2, d2};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[f][r] = 0.0;
    }
    const int64_t j0 = (int64_t)blockIdx.y * slice_len;
    const int64_t j1 = j0 + slice_len < n ? j0 + slice_len : n;
    // the entry constants in vector registers: an FP32 instruction with a
    // scalar operand does not pair with another in one issue cycle
    BlockEntry cv = c;
    asm volatile("" : "+v"(cv.k2), "+v"(cv.e2x2), "+v"(cv.e2), "+v"(cv.bsc));
    mfh_span<ROWS, FT>(XS, Vh, j0, j1, n_int, fint, fr, cv, bf, Cf, acc, lds_a, lds_v);
    // the scales out: 2^-se of the entries and the column's own
    const double un = c.unscale / (double)vsc[jj];
#pragma unroll
    for (int f = 0; f < FT; ++f) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t i = fb0 + (int64_t)(wv * FT + f) * 16 + 4 * g + r;
            if (i < fb1) P[((int64_t)blockIdx.y * kBlkRhs + jj) * ldp + i] = acc[f][r] * un;
        }
    }
}

// Vh[q][k] = the split of the scaled values vsc[k] Vg[4q + r][k], r = 0..3
// (zeros past n): (H01, H23, L01, L23), fp16 pairs as in split_f16x2.
// Values beyond the scaled range are clamped to it (NaN stays NaN); the
// block products only receive such values from steps whose results are
// discarded (after a breakdown), the unit-norm operands of the Golub-Kahan
// runs stay within it by construction.
__global__ __launch_bounds__(kBlock) void k_split_block(const float* __restrict__ Vg, int64_t n,
                                                        const float* __restrict__ vsc, uint4* __restrict__ Vh) {
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t nq = (n + 3) / 4;
    if (e >= nq * kBlkRhs) return;
    const int64_t q = e / kBlkRhs;
    const int k = (int)(e % kBlkRhs);
    float sc = vsc[k];
    float v[4];  // all loads in flight together
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = Vg[(4 * q + r < n ? 4 * q + r : 4 * q) * kBlkRhs + k];
    arrived(sc);
#pragma unroll
    for (int r = 0; r < 4; ++r) arrived(v[r]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float x = 4 * q + r < n ? v[r] * sc : 0.f;
        if (__builtin_isfinite(x) && fabsf(x) > kBlkRange) x = copysignf(kBlkRange, x);
        v[r] = x;
    }
    uint4 o;
    split_f16x2(v[0], v[1], o.x, o.z);
    split_f16x2(v[2], v[3], o.y, o.w);
    Vh[e] = o;
}

// vsc[k] = 2^(14 - e_k) with max_j |Vg[j][k]| < 2^e_k (1 for a zero column):
// column k scaled below kBlkRange.  One workgroup per column.
__global__ __launch_bounds__(kBlock) void k_block_vscale(const float* __restrict__ Vg, int64_t n,
                                                         float* __restrict__ vsc) {
    __shared__ float red[kBlock / kWave];
    const int k = blockIdx.x;
    float m = 0.f;
    for (int64_t j = threadIdx.x; j < n; j += kBlock) m = fmaxf(m, fabsf(Vg[j * kBlkRhs + k]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, kWave));
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        float mm = 0.f;
        for (int w = 0; w < kBlock / kWave; ++w) mm = fmaxf(mm, red[w]);
        float s = 1.f;
        if (mm > 0.f) {
            int ex;
            (void)frexpf(mm, &ex);
            int p = 14 - ex;
            p = p > 126 ? 126 : (p < -126 ? -126 : p);
            s = ldexpf(1.f, p);
        }
        vsc[k] = s;
    }
}

// Vg[q][k] = x_k[perm[q]] in FP32 for k < s (zero for s <= k < kBlkRhs and
// for stopped runs); x_k = X + k * ldx.
__global__ __launch_bounds__(kBlock) void k_gather_block(const double* __restrict__ X, int64_t ldx, int s,
                                                         const int32_t* __restrict__ perm, int64_t n,
                                                         const GkbState* __restrict__ st, float* __restrict__ Vg) {
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= n * kBlkRhs) return;
    const int64_t q = e / kBlkRhs;
    const int k = (int)(e % kBlkRhs);
    const bool live = k < s && (st == nullptr || !st[k].stopped);
    Vg[e] = live ? (float)X[k * ldx + perm[q]] : 0.f;
}

// Vg[e] = a fixed pseudo-random value in [-0.5, 0.5) (an operand for timing
// runs: finite, with the spread of real data).
__global__ __launch_bounds__(kBlock) void k_fill_hash(float* __restrict__ Vg, int64_t count) {
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= count) return;
    uint32_t h = (uint32_t)e * 0x9E3779B1u;
    h ^= h >> 15;
    h *= 0x85EBCA77u;
    h ^= h >> 13;
    Vg[e] = (float)(h >> 8) * (1.0f / 16777216.0f) - 0.5f;
}

// y_k[perm[i]] = sum_slices P[slice][k][i] - shift_k z_k[perm[i]] for right-hand
// side k = blockIdx.y (shift_k = shift[k * sstride], z_k = z + k * ldz,
// y_k = y + k * ldy); skipped when state k has stopped.
__global__ __launch_bounds__(kBlock) void k_reduce_block(const double* __restrict__ P,
                                                         const GkbState* __restrict__ st,
                                                         const int32_t* __restrict__ perm, int64_t ldp, int64_t n,
                                                         int S, const double* __restrict__ shift, int64_t sstride,
                                                         const double* __restrict__ z, int64_t ldz,
                                                         double* __restrict__ y, int64_t ldy) {
    const int k = blockIdx.y;
    if (st != nullptr && st[k].stopped) return;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    // eight slices in flight, added evens and odds apart
    const double* Pk = P + (int64_t)k * ldp + i;
    const int64_t ss = (int64_t)kBlkRhs * ldp;
    double a0 = 0.0, a1 = 0.0;
    int sl = 0;
    for (; sl + 8 <= S; sl += 8) {
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = Pk[(sl + q) * ss];
#pragma unroll
        for (int q = 0; q < 8; q += 2) {
            a0 += v[q];
            a1 += v[q + 1];
        }
    }
    for (; sl + 1 < S; sl += 2) {
        a0 += Pk[sl * ss];
        a1 += Pk[(sl + 1) * ss];
    }
    if (sl < S) a0 += Pk[sl * ss];
    double v = a0 + a1;
    const int64_t o = perm[i];
    if (z != nullptr) v -= shift[k * sstride] * z[k * ldz + o];
    y[k * ldy + o] = v;
}

// ---------------------------------------------------------------------------
// Rows of A as a product sees them (entry checks).
// ---------------------------------------------------------------------------

template <typename R>
__global__ __launch_bounds__(kBlock) void k_gen_rows(const typename NodeOf<R>::type* __restrict__ X, int64_t n,
                                                     int64_t n_int, int64_t row0, EntryConst c,
                                                     double* __restrict__ out) {
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t i = row0 + blockIdx.y;
    if (j >= n) return;
    const auto p = X[i];
    const auto q = X[j];
    const R t = t_of(p.x, p.y, p.z, q.x, q.y, q.z);
    const R e = i < n_int ? entry_interior(t, c) : entry_boundary(t, c);
    out[(int64_t)blockIdx.y * n + j] = (double)e;
}

// ---------------------------------------------------------------------------
// Evaluation u(P_e) = sum_j coef_j phi(|P_e - X_j|), FP64.  A wave takes 64 points
// against a slice of the centres; the centre index is wave-uniform, so records and
// coefficients are scalar loads.  The kEvalWaves slices of a workgroup are added in
// LDS in wave order, the workgroups' sums by k_eval_reduce.  Bound by the FP64 units:
// six operations for the squared distance, the estimate of the root, five to
// refine it and one for the sum, by their measured issue times (5.2 cycles, 17 for the
// estimate) 79 cycles a term and wave, 605 us at 2.4 GHz for 20 000 points and 60 000
// centres; the call takes 598 (842 with slices of a workgroup's width, six
// refining operations and 256 partial sums a point).
// ---------------------------------------------------------------------------

// Points as records (centred, times eps); a point that is not finite leaves the
// call's number in *flag.
__global__ __launch_bounds__(kBlock) void k_eval_records(const double* __restrict__ xyz, int64_t m, double eps,
                                                         double3 center, int32_t call, double4* __restrict__ E,
                                                         int32_t* __restrict__ flag) {
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= m) return;
    const double a = xyz[3 * e], b = xyz[3 * e + 1], d = xyz[3 * e + 2];
    if (!(isfinite(a) && isfinite(b) && isfinite(d))) *flag = call;
    E[e] = make_double4(eps * (a - center.x), eps * (b - center.y), eps * (d - center.z), 0.0);
}

// sqrt(t) for t >= 1: with s the estimate of 1/sqrt(t), h = fl(t s) and r = 1 -
// h s, sqrt(t) = h (1 + r/2 + 3 r^2/8 + ..) up to half of h's rounding.
__device__ __forceinline__ double sqrt_f64(double t) {
    const double s = __builtin_amdgcn_rsq(t);
    const double h = t * s;
    const double r = fma(-h, s, 1.0);
    const double p = fma(0.375, r, 0.5);
    return fma(h * r, p, h);
}

__global__ __launch_bounds__(kEvalWaves* kWave) void k_eval_partial(const double4* __restrict__ X,
                                                                    const double* __restrict__ coef, int64_t n,
                                                                    const double4* __restrict__ E, int64_t m,
                                                                    int64_t slice_len, double* __restrict__ P,
                                                                    int64_t ldp) {
    __shared__ double part[kEvalWaves][kWave];
    const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int64_t e = (int64_t)blockIdx.x * kWave + lane;
    const double4 p = E[e < m ? e : 0];
    const int64_t j0 = ((int64_t)blockIdx.y * kEvalWaves + wv) * slice_len;
    const int64_t j1 = j0 + slice_len < n ? j0 + slice_len : n;
    double a = 0.0;
#pragma unroll 4
    for (int64_t j = j0; j < j1; ++j) {
        const double4 q = X[j];
        a = fma(sqrt_f64(t_of(p.x, p.y, p.z, q.x, q.y, q.z)), coef[j], a);
    }
    part[wv][lane] = a;
    __syncthreads();
    if (wv == 0 && e < m) {
#pragma unroll
        for (int g = 1; g < kEvalWaves; ++g) a += part[g][lane];
        P[(int64_t)blockIdx.y * ldp + e] = a;
    }
}

// u_e = sum over the S slices, four interleaved groups combined in a fixed order;
// nothing is written when the points' flag bears the call's number, which goes to
// the host (pinned memory) with it.
__global__ __launch_bounds__(kWave) void k_eval_reduce(const double* __restrict__ P, int64_t ldp, int S, int64_t m,
                                                       int32_t call, const int32_t* __restrict__ flag,
                                                       double* __restrict__ u, int32_t* __restrict__ hflag) {
    const bool bad = *flag == call;
    if (blockIdx.x == 0 && threadIdx.x == 0) *hflag = bad ? call : 0;
    const int64_t i = (int64_t)blockIdx.x * kWave + threadIdx.x;
    if (bad || i >= m) return;
    double a[4] = {};
    int k = 0;
    for (; k + 3 < S; k += 4) {
#pragma unroll
        for (int g = 0; g < 4; ++g) a[g] += P[(int64_t)(k + g) * ldp + i];
    }
    for (; k < S; ++k) a[0] += P[(int64_t)k * ldp + i];
    u[i] = (a[0] + a[1]) + (a[2] + a[3]);
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------

int64_t mfm_blocks(int64_t n, int64_t n_int) {
    return (n_int + kMfmFixed - 1) / kMfmFixed + (n - n_int + kMfmFixed - 1) / kMfmFixed;
}

void launch_gather_w32(const double* x, const int32_t* perm, int64_t n, float4* XS, const GkbState* st,
                       hipStream_t s) {
    k_gather_w32<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(x, perm, n, XS, st);
}

void launch_mfs_product(int trans, const float4* XS, const float4* frames, const SymLayout& L, const EntryConst& c,
                        double* RowP, double* ColP, const GkbState* st, hipStream_t s) {
    if (L.nitems <= 0) return;
    if (trans)
        k_mfs<true><<<(unsigned)L.nitems, kBlock, 0, s>>>(L.items, st, XS, frames, RowP, ColP, L, c);
    else
        k_mfs<false><<<(unsigned)L.nitems, kBlock, 0, s>>>(L.items, st, XS, frames, RowP, ColP, L, c);
}

void launch_gather_w64(const double* x, const int32_t* perm, int64_t n, double4* XS64, const GkbState* st,
                       hipStream_t s) {
    k_gather_w64<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(x, perm, n, XS64, st);
}

void launch_mfs64_product(int trans, const double4* XS64, const SymLayout& L, const EntryConst& c, double* RowP,
                          double* ColP, const GkbState* st, hipStream_t s) {
    if (L.nitems <= 0) return;
    const unsigned g = (unsigned)L.nitems;
    if (L.blk == 64) {
        if (trans)
            k_mfs64<true, 1><<<g, kBlock, 0, s>>>(L.items, st, XS64, RowP, ColP, L, c);
        else
            k_mfs64<false, 1><<<g, kBlock, 0, s>>>(L.items, st, XS64, RowP, ColP, L, c);
    } else {
        if (trans)
            k_mfs64<true, 2><<<g, kBlock, 0, s>>>(L.items, st, XS64, RowP, ColP, L, c);
        else
            k_mfs64<false, 2><<<g, kBlock, 0, s>>>(L.items, st, XS64, RowP, ColP, L, c);
    }
}

void launch_mfs_reduce(const SymLayout& L, const double* RowP, const double* ColP, const int32_t* perm,
                       const double* shift_ptr, double shift_val, const double* z, double* y, const GkbState* st,
                       hipStream_t s) {
    if (L.nb <= 0) return;
    if (L.blk == 64)
        k_mfs_reduce<64><<<(unsigned)L.nb, kSymRedThreads, 0, s>>>(L.item_first, st, RowP, ColP, perm, L.F, L,
                                                                 shift_ptr, shift_val, z, y);
    else
        k_mfs_reduce<128><<<(unsigned)L.nb, kSymRedThreads, 0, s>>>(L.item_first, st, RowP, ColP, perm, L.F, L,
                                                                  shift_ptr, shift_val, z, y);
}

int64_t mfh_block_blocks(int64_t n, int64_t n_int, int ft) {
    const int64_t fix = (kBlock / kWave) * ft * 16;
    return (n_int + fix - 1) / fix + (n - n_int + fix - 1) / fix;
}

BlockEntry block_entry(const EntryConst& c, double tmax) {
    // every term of the interior entry (kappa^2 t + 2 eps^2 + eps^2 s^2) s is
    // positive and at most kappa^2 sqrt(tmax), 2 eps^2, eps^2 (s <= 1); the
    // boundary entry sqrt(t) is at most sqrt(tmax)
    const double st = sqrt(tmax > 1.0 ? tmax : 1.0);
    double bound = fabs((double)c.k2f) * st + fabs((double)c.e2x2f) + fabs((double)c.e2f);
    if (st > bound) bound = st;
    int ex = 0;
    (void)frexp(bound, &ex);  // bound < 2^ex
    int se = 14 - ex;
    se = se > 60 ? 60 : (se < -60 ? -60 : se);
    BlockEntry b{};
    b.k2 = ldexpf(c.k2f, se);
    b.e2x2 = ldexpf(c.e2x2f, se);
    b.e2 = ldexpf(c.e2f, se);
    b.bsc = ldexpf(1.0f, se);
    b.unscale = ldexp(1.0, -se);
    return b;
}

void launch_mfh_block(int trans, int ft, const float4* XS, const float4* frames, const uint4* Vh, const float* vsc,
                      int64_t n, int64_t n_int, int S, int64_t slice_len, const BlockEntry& c, double* P,
                      int64_t ldp, hipStream_t s) {
    const int64_t fix = (kBlock / kWave) * ft * 16;
    const int64_t nb_int = (n_int + fix - 1) / fix;
    dim3 grid((unsigned)mfh_block_blocks(n, n_int, ft), (unsigned)S);
    if (ft == 1) {
        if (trans)
            k_mfh_block<false, 1><<<grid, kBlock, 0, s>>>(XS, Vh, frames, n, n_int, nb_int, slice_len, vsc, P, ldp, c);
        else
            k_mfh_block<true, 1><<<grid, kBlock, 0, s>>>(XS, Vh, frames, n, n_int, nb_int, slice_len, vsc, P, ldp, c);
    } else {
        if (trans)
            k_mfh_block<false, 2><<<grid, kBlock, 0, s>>>(XS, Vh, frames, n, n_int, nb_int, slice_len, vsc, P, ldp, c);
        else
            k_mfh_block<true, 2><<<grid, kBlock, 0, s>>>(XS, Vh, frames, n, n_int, nb_int, slice_len, vsc, P, ldp, c);
    }
}

void launch_split_block(const float* Vg, int64_t n, const float* vsc, uint4* Vh, hipStream_t s) {
    const int64_t cnt = (n + 3) / 4 * kBlkRhs;
    if (cnt <= 0) return;
    k_split_block<<<(unsigned)((cnt + kBlock - 1) / kBlock), kBlock, 0, s>>>(Vg, n, vsc, Vh);
}

void launch_block_vscale(const float* Vg, int64_t n, float* vsc, hipStream_t s) {
    k_block_vscale<<<kBlkRhs, kBlock, 0, s>>>(Vg, n, vsc);
}

void launch_fill_hash(float* Vg, int64_t count, hipStream_t s) {
    if (count <= 0) return;
    k_fill_hash<<<(unsigned)((count + kBlock - 1) / kBlock), kBlock, 0, s>>>(Vg, count);
}

void launch_gather_block(const double* X, int64_t ldx, int nrhs, const int32_t* perm, int64_t n,
                         const GkbState* st, float* Vg, hipStream_t s) {
    k_gather_block<<<(unsigned)((n * kBlkRhs + kBlock - 1) / kBlock), kBlock, 0, s>>>(X, ldx, nrhs, perm, n, st, Vg);
}

void launch_reduce_block(const double* P, int64_t ldp, int S, int64_t n, int nrhs, const int32_t* perm,
                         const double* shift, int64_t sstride, const double* z, int64_t ldz, double* y, int64_t ldy,
                         const GkbState* st, hipStream_t s) {
    k_reduce_block<<<dim3((unsigned)((n + kBlock - 1) / kBlock), nrhs), kBlock, 0, s>>>(P, st, perm, ldp, n, S,
                                                                                       shift, sstride, z, ldz, y, ldy);
}

void launch_gen_rows(int prec, const void* X, int64_t n, int64_t n_int, int64_t row0, int64_t count,
                     const EntryConst& c, double* out, hipStream_t s) {
    dim3 grid((unsigned)((n + kBlock - 1) / kBlock), (unsigned)count);
    if (prec == 64)
        k_gen_rows<double><<<grid, kBlock, 0, s>>>((const double4*)X, n, n_int, row0, c, out);
    else
        k_gen_rows<float><<<grid, kBlock, 0, s>>>((const float4*)X, n, n_int, row0, c, out);
}

void launch_eval_records(const double* xyz, int64_t m, double eps, const double* center, int32_t call, double4* E,
                         int32_t* flag, hipStream_t s) {
    k_eval_records<<<(unsigned)((m + kBlock - 1) / kBlock), kBlock, 0, s>>>(
        xyz, m, eps, make_double3(center[0], center[1], center[2]), call, E, flag);
}

EvalShape eval_shape(int64_t n, int64_t m) {
    EvalShape g;
    g.blocks = (m + kWave - 1) / kWave;
    const int64_t waves = (kEvalTarget + g.blocks - 1) / g.blocks;
    g.len = (n + waves - 1) / waves;
    g.len = g.len < kEvalMinLen ? kEvalMinLen : g.len;
    g.S = (int)((n + g.len * kEvalWaves - 1) / (g.len * kEvalWaves));
    return g;
}

void launch_eval(const double4* X, const double* coef, int64_t n, const double4* E, int64_t m, const EvalShape& g,
                 double* P, int64_t ldp, int32_t call, const int32_t* flag, double* u, int32_t* hflag,
                 hipStream_t s) {
    const dim3 grid((unsigned)g.blocks, (unsigned)g.S);
    k_eval_partial<<<grid, kEvalWaves * kWave, 0, s>>>(X, coef, n, E, m, g.len, P, ldp);
    k_eval_reduce<<<(unsigned)((m + kWave - 1) / kWave), kWave, 0, s>>>(P, ldp, g.S, m, call, flag, u, hflag);
}

}  // namespace mqh
