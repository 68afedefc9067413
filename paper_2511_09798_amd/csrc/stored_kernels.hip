// stored_kernels.hip -- the stored FP64 Kansa matrix on gfx950: assembly
// (tiled, and dense row-major for the full-SVD reference), the products
// A x and A^T x on the tiles with their fixed-order reduction, and rows of A.
//
// Vectors have a leading dimension ldn (multiple of 64, >= n) and are zero
// past n; nodes are double4 records (centred, scaled by eps).
#include "kernels.hpp"

namespace mqh {

// ---------------------------------------------------------------------------
// Stored FP64 operator: one value per unordered pair of nodes, in tiles.
//
// A_ij and A_ji are functions of the same distance |X_i - X_j|, so one stored
// value serves both.  Node indices are cut into tiles of kTile per class
// (interior tiles 0 .. nti-1, boundary tiles nti .. nt-1, each class padded to
// whole tiles), and the tiles (R, C) with C >= R are stored, kTile x kTile,
// row-major inside a tile, tile row after tile row:
//   both interior:  L phi (= A_ij = A_ji);
//   both boundary:  phi   (= A_ij = A_ji);
//   mixed (R interior, C boundary): t = 1 + |X_i - X_j|^2, from which the product
//                   forms A_ij = L phi and A_ji = phi as the assembly does
//                   for the other tiles, so that every entry is rounded alike.
// A product visits every stored tile once, as T x_C for y_R (row use) and, off
// the diagonal, as T^T x_R for y_C (column use).  On a mixed tile A x takes L phi
// for the rows and phi for the columns, A^T x the other way round.
// The product is bound by HBM, and the mixed blocks' second copy was a
// quarter of its bytes at 20% boundary nodes: 100 000 nodes 53.0 -> 40.1 GB,
// A^T x 8.60 -> 6.46 ms (6.2 TB/s either way); 20 000 nodes 2.27 -> 1.63 GB,
// 375 -> 268 us.  Forming the two entries costs 9 FP64 instructions and one v_rsq_f64
// per mixed value, under the streaming time (about 49 FP64 issue slots per value).
// ---------------------------------------------------------------------------

// Dense row-major A (n rows, leading dimension lda, zero columns past n), for
// the full-SVD reference's work matrix: one block = RB rows x 512 columns
// (two columns per lane, 16-byte non-temporal stores); the column records stay
// in registers across rows.
template <int RB>
__global__ __launch_bounds__(kBlock) void k_assemble(const double4* __restrict__ X, int64_t n, int64_t n_int,
                                                     int64_t lda, EntryConst c, double* __restrict__ A) {
    const int64_t c0 = (int64_t)blockIdx.x * (2 * kBlock) + 2 * threadIdx.x;
    if (c0 >= lda) return;  // no barriers below
    const bool va = c0 < n, vb = c0 + 1 < n;
    const double4 qa = X[va ? c0 : 0];
    const double4 qb = X[vb ? c0 + 1 : 0];
    const int64_t r0 = (int64_t)blockIdx.y * RB;
    const int64_t r1 = r0 + RB < n ? r0 + RB : n;
    for (int64_t i = r0; i < r1; ++i) {
        const double4 p = X[i];
        const double ta = t_of(p.x, p.y, p.z, qa.x, qa.y, qa.z);
        const double tb = t_of(p.x, p.y, p.z, qb.x, qb.y, qb.z);
        double ea, eb;
        if (i < n_int) {
            ea = entry_interior(ta, c);
            eb = entry_interior(tb, c);
        } else {
            ea = entry_boundary(ta, c);
            eb = entry_boundary(tb, c);
        }
        v2d v;
        v.x = va ? ea : 0.0;
        v.y = vb ? eb : 0.0;
        store_nt(A + i * lda + c0, v);
    }
}

__device__ __forceinline__ int64_t pk_start(const PackedLayout& L, int T) {
    return T < L.nti ? (int64_t)T * kTile : L.n_int + (int64_t)(T - L.nti) * kTile;
}
__device__ __forceinline__ int64_t pk_end(const PackedLayout& L, int T) { return T < L.nti ? L.n_int : L.n; }
// index of stored tile (R, C), C >= R
__device__ __forceinline__ int64_t pk_tile(const PackedLayout& L, int R, int C) {
    return (int64_t)R * L.nt - (int64_t)R * (R - 1) / 2 + (C - R);
}

// The stored value of pair (node R_i, node C_j) in tile (blockIdx.y = R, C = R +
// blockIdx.x): one workgroup per stored tile, four rows at a time, two columns
// per lane, 16-byte non-temporal stores.  Padding rows and columns hold zero,
// in mixed tiles one (they multiply zeros of x, and the entries formed of them are finite).
__global__ __launch_bounds__(kBlock) void k_assemble_packed(const double4* __restrict__ X, PackedLayout L,
                                                            EntryConst c, double* __restrict__ A) {
    const int R = blockIdx.y, C = R + (int)blockIdx.x;
    if (C >= L.nt) return;  // whole workgroup; no barriers in this kernel
    const int64_t r0 = pk_start(L, R), rend = pk_end(L, R);
    const int64_t c0 = pk_start(L, C), cend = pk_end(L, C);
    const bool lphi = C < L.nti, mixed = R < L.nti && !lphi;
    const double pad = mixed ? 1.0 : 0.0;
    const int lane2 = 2 * (threadIdx.x & (kWave - 1));
    const int64_t ja = c0 + lane2, jb = ja + 1;
    const bool va = ja < cend, vb = jb < cend;
    const double4 qa = X[va ? ja : 0];
    const double4 qb = X[vb ? jb : 0];
    double* T = A + pk_tile(L, R, C) * kTileElems + lane2;
    for (int i = threadIdx.x / kWave; i < kTile; i += kBlock / kWave) {
        const int64_t g = r0 + i;
        v2d v;
        v.x = pad;
        v.y = pad;
        if (g < rend) {
            const double4 q = X[g];
            const double ta = t_of(q.x, q.y, q.z, qa.x, qa.y, qa.z);
            const double tb = t_of(q.x, q.y, q.z, qb.x, qb.y, qb.z);
            const double ea = mixed ? ta : (lphi ? entry_interior(ta, c) : entry_boundary(ta, c));
            const double eb = mixed ? tb : (lphi ? entry_interior(tb, c) : entry_boundary(tb, c));
            v.x = va ? ea : pad;
            v.y = vb ? eb : pad;
        }
        store_nt(T + (int64_t)i * kTile, v);
    }
}

// One work item = consecutive tiles of one tile row R, all four waves on the
// same tile at once (wave w: rows 32 w .. 32 w + 31, lane l: columns 2l, 2l+1,
// 1 KB per wave load, so a workgroup reads 32 KB runs), the next 8-row group's
// loads always in flight.  Column use: per-lane sums over the wave's rows, added
// over the waves through LDS, one partial per tile, PC[tile index][0 .. kTile).
// Row use: the per-lane products of 8 rows go through LDS and are summed by
// groups of 8 lanes (no per-row wave reduction); one partial per item,
// PR[item][0 .. kTile).
template <int TRANS>
__global__ __launch_bounds__(kBlock) void k_packed_product(const double* __restrict__ A, PackedLayout L,
                                                           EntryConst ec, const double* __restrict__ x,
                                                           double* __restrict__ PR, double* __restrict__ PC,
                                                           const GkbState* __restrict__ st) {
    int stop = st != nullptr ? st->stopped : 0;
    constexpr int GR = 8;
    constexpr int kWaves = kBlock / kWave;
    constexpr int kRows = kTile / kWaves;   // rows of a tile per wave (32)
    constexpr int kGpw = kRows / GR;        // groups per wave and tile (4)
    constexpr int kRed = GR * (kWave + 1);
    constexpr int kLpr = kWave / GR;
    __shared__ double xr[kTile];
    __shared__ double rsum[kTile];
    __shared__ double red[kWaves][kRed];
    __shared__ double csum[2][kWaves][kTile];  // double-buffered: one barrier per tile
    int4 it = L.items[blockIdx.x];
    arrived_uniform(it.x);
    arrived_uniform(stop);
    if (stop) return;  // uniform over the grid
    const int R = it.x, C0 = it.y, cnt = it.z;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int total = cnt * kGpw;
    const int64_t tile0 = pk_tile(L, R, C0);
    const double* A0 = A + tile0 * kTileElems + (int64_t)(w * kRows) * kTile + 2 * lane;
    auto gptr = [&](int G) { return A0 + (G / kGpw) * kTileElems + (int64_t)(GR * (G % kGpw)) * kTile; };
    v2d a0[GR], a1[GR];
    {
        const double* T = gptr(0);
#pragma unroll
        for (int r = 0; r < GR; ++r) a0[r] = load_nt(T + (int64_t)r * kTile);
    }
    const int64_t r0 = pk_start(L, R), rend = pk_end(L, R);
    if (tid < kTile) {
        xr[tid] = r0 + tid < rend ? x[r0 + tid] : 0.0;
        rsum[tid] = 0.0;
    }
    __syncthreads();
    double* buf = red[w];
    const int rq = lane / kLpr, qq = lane % kLpr;
    bool use_col = false, mixed = false;
    double xc0 = 0.0, xc1 = 0.0, cs0 = 0.0, cs1 = 0.0;
    auto setup = [&](int q) {
        const int C = C0 + q;
        use_col = C != R;
        mixed = R < L.nti && C >= L.nti;
        const int64_t c0 = pk_start(L, C), cend = pk_end(L, C);
        const int64_t ca = c0 + 2 * lane, cb = ca + 1;
        xc0 = ca < cend ? x[ca] : 0.0;
        xc1 = cb < cend ? x[cb] : 0.0;
        cs0 = 0.0;
        cs1 = 0.0;
    };
    // all waves reach finish (uniform trip count); tile q uses buffer q % 2,
    // whose previous readers (tile q - 2) finished before the barrier of
    // tile q - 1
    auto finish = [&](int q) {
        double* cb = &csum[q & 1][0][0];
        if (use_col) {
            cb[w * kTile + 2 * lane] = cs0;
            cb[w * kTile + 2 * lane + 1] = cs1;
        }
        __syncthreads();
        if (use_col && tid < kTile) {
            double sm = cb[tid];
#pragma unroll
            for (int v = 1; v < kWaves; ++v) sm += cb[v * kTile + tid];
            PC[(tile0 + q) * kTile + tid] = sm;
        }
    };
    auto group = [&](int g, const v2d* a) {  // g: group of this wave within the tile
        const int rbase = w * kRows + GR * g;
        double rp[GR];
        if (mixed) {
#pragma unroll
            for (int r = 0; r < GR; ++r) {
                const double l0 = entry_interior(a[r].x, ec), l1 = entry_interior(a[r].y, ec);
                const double f0 = entry_boundary(a[r].x, ec), f1 = entry_boundary(a[r].y, ec);
                const double xi = xr[rbase + r];
                cs0 = fma(TRANS ? l0 : f0, xi, cs0);
                cs1 = fma(TRANS ? l1 : f1, xi, cs1);
                rp[r] = TRANS ? fma(f1, xc1, f0 * xc0) : fma(l1, xc1, l0 * xc0);
            }
        } else {
#pragma unroll
            for (int r = 0; r < GR; ++r) {
                if (use_col) {
                    const double xi = xr[rbase + r];
                    cs0 = fma(a[r].x, xi, cs0);
                    cs1 = fma(a[r].y, xi, cs1);
                }
                rp[r] = fma(a[r].y, xc1, a[r].x * xc0);
            }
        }
#pragma unroll
        for (int r = 0; r < GR; ++r) buf[r * (kWave + 1) + lane] = rp[r];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
        double sm = 0.0;
#pragma unroll
        for (int k = 0; k < GR; ++k) sm += buf[rq * (kWave + 1) + qq * GR + k];
#pragma unroll
        for (int o = 1; o < kLpr; o <<= 1) sm += __shfl_xor(sm, o, kWave);
        if (qq == 0) rsum[rbase + rq] += sm;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    };
    for (int G = 0; G < total; G += 2) {  // kGpw is even: G and G + 1 in the same tile
        {
            const double* T = gptr(G + 1);
#pragma unroll
            for (int r = 0; r < GR; ++r) a1[r] = load_nt(T + (int64_t)r * kTile);
        }
        if (G % kGpw == 0) setup(G / kGpw);
        group(G % kGpw, a0);
        if (G + 2 < total) {
            const double* T = gptr(G + 2);
#pragma unroll
            for (int r = 0; r < GR; ++r) a0[r] = load_nt(T + (int64_t)r * kTile);
        }
        group((G + 1) % kGpw, a1);
        if ((G + 2) % kGpw == 0) finish(G / kGpw);
    }
    __syncthreads();
    if (tid < kTile) PR[(int64_t)blockIdx.x * kTile + tid] = rsum[tid];
}

// y_X = sum over the items of tile row X (row use, item order) + sum over the
// tiles (R, X), R < X (column use, R ascending) - shift z; one workgroup per
// output tile X, kRedGroups groups of kTile threads taking every
// kRedGroups-th source, combined in group order.  Bound by the latency of the
// strided 1 KB reads: eight groups with eight loads in flight each instead of
// four with four (20 000 nodes 20 -> 7.6 us, 100 000 nodes 157 -> 80 us).
constexpr int kRedGroups = 8;

__global__ __launch_bounds__(kRedGroups * kTile) void k_packed_reduce(PackedLayout L, const double* __restrict__ PR,
                                                                      const double* __restrict__ PC,
                                                                      const double* __restrict__ shift_ptr,
                                                                      double shift_val, const double* __restrict__ z,
                                                                      double* __restrict__ y,
                                                                      const GkbState* __restrict__ st) {
    __shared__ double part[kRedGroups][kTile];
    int stop = st != nullptr ? st->stopped : 0;
    const int X = blockIdx.x;
    const int t = threadIdx.x & (kTile - 1), grp = threadIdx.x / kTile;
    int i0 = L.item_first[X], i1 = L.item_first[X + 1];
    arrived_uniform(i0);
    arrived_uniform(i1);
    arrived_uniform(stop);
    if (stop) return;
    const int nrow = i1 - i0, total = nrow + X;
    const int64_t o = pk_start(L, X) + t;
    double s = 0.0, zo = 0.0, sh = 0.0;
    if (grp == 0 && z != nullptr && o < pk_end(L, X)) {  // the shift term, while the partials are on their way
        zo = z[o];
        sh = shift_ptr != nullptr ? *shift_ptr : shift_val;
    }
#pragma unroll 8
    for (int k = grp; k < total; k += kRedGroups) {
        const double* src = k < nrow ? PR + (int64_t)(i0 + k) * kTile : PC + pk_tile(L, k - nrow, X) * kTile;
        s += src[t];
    }
    part[grp][t] = s;
    __syncthreads();
    if (grp == 0) {
        s = ((part[0][t] + part[1][t]) + (part[2][t] + part[3][t])) +
            ((part[4][t] + part[5][t]) + (part[6][t] + part[7][t]));
        if (o < pk_end(L, X)) {
            if (z != nullptr) s -= sh * zo;
            y[o] = s;
        }
    }
}

// Rows [row0, row0 + gridDim.y) of the stored tiled matrix, row-major with
// leading dimension n (an entry below the diagonal is read from the transposed
// stored tile; an entry of a mixed tile is formed as the products do).
__global__ __launch_bounds__(kBlock) void k_packed_rows(const double* __restrict__ A, PackedLayout L, EntryConst ec,
                                                        int64_t row0, double* __restrict__ out) {
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t i = row0 + blockIdx.y;
    if (j >= L.n) return;
    const int R = i < L.n_int ? (int)(i / kTile) : L.nti + (int)((i - L.n_int) / kTile);
    const int ir = (int)(i - pk_start(L, R));
    const int C = j < L.n_int ? (int)(j / kTile) : L.nti + (int)((j - L.n_int) / kTile);
    const int jc = (int)(j - pk_start(L, C));
    double v = C < R ? A[pk_tile(L, C, R) * kTileElems + (int64_t)jc * kTile + ir]
                     : A[pk_tile(L, R, C) * kTileElems + (int64_t)ir * kTile + jc];
    if ((R < L.nti) != (C < L.nti)) v = R < L.nti ? entry_interior(v, ec) : entry_boundary(v, ec);
    out[(int64_t)blockIdx.y * L.n + j] = v;
}

void launch_assemble(const double4* X, int64_t n, int64_t n_int, int64_t lda, const EntryConst& c, double* A,
                     hipStream_t s) {
    constexpr int RB = 64;
    dim3 grid((unsigned)((lda + 2 * kBlock - 1) / (2 * kBlock)), (unsigned)((n + RB - 1) / RB));
    k_assemble<RB><<<grid, kBlock, 0, s>>>(X, n, n_int, lda, c, A);
}

void launch_assemble_packed(const double4* X, const PackedLayout& L, const EntryConst& c, double* A, hipStream_t s) {
    k_assemble_packed<<<dim3((unsigned)L.nt, (unsigned)L.nt), kBlock, 0, s>>>(X, L, c, A);
}

void launch_packed_product(int trans, const double* A, const PackedLayout& L, const EntryConst& c, const double* x,
                           double* PR, double* PC, const GkbState* st, hipStream_t s) {
    if (trans)
        k_packed_product<1><<<(unsigned)L.nitems, kBlock, 0, s>>>(A, L, c, x, PR, PC, st);
    else
        k_packed_product<0><<<(unsigned)L.nitems, kBlock, 0, s>>>(A, L, c, x, PR, PC, st);
}

void launch_packed_reduce(const PackedLayout& L, const double* PR, const double* PC, const double* shift_ptr,
                          double shift_val, const double* z, double* y, const GkbState* st, hipStream_t s) {
    k_packed_reduce<<<(unsigned)L.nt, kRedGroups * kTile, 0, s>>>(L, PR, PC, shift_ptr, shift_val, z, y, st);
}

void launch_packed_rows(const double* A, const PackedLayout& L, const EntryConst& c, int64_t row0, int64_t count,
                        double* out, hipStream_t s) {
    dim3 grid((unsigned)((L.n + kBlock - 1) / kBlock), (unsigned)count);
    k_packed_rows<<<grid, kBlock, 0, s>>>(A, L, c, row0, out);
}

}  // namespace mqh
