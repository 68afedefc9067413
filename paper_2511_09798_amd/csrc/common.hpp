// common.hpp -- device helpers shared by the gfx950 kernels of the MQ-RBF
// Golub-Kahan solver: launch constants, deterministic wave/block reductions,
// the Golub-Kahan device state and the multiquadric entry generators.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mqh {

constexpr int kBlock = 256;  // threads per workgroup for the streaming kernels
constexpr int kWave = 64;    // CDNA wavefront

// Device-resident state of one Golub-Kahan run.  Every kernel of the loop
// reads `stopped` first and returns at once after a breakdown, so the host
// can enqueue all ell steps without synchronising.
struct GkbState {
    int32_t stopped;   // 1 after a breakdown
    int32_t ell_done;  // steps kept (initialised to ell)
    int32_t flag;      // 0, 1 = alpha breakdown, 2 = beta breakdown
    int32_t pad;
    double scale;      // running max of alpha_j, beta_{j+1}: the operator scale
    // copies of stopped and scale taken by the kernel that produces a norm's
    // partial sums; the normalisation kernel decides from these while its
    // block 0 updates stopped and scale
    int32_t snap_stopped;
    int32_t pad2;
    double snap_scale;
};

// Per-batch-slice strides of a kernel's pointer arguments (in elements):
// slice z of a batched launch uses pointer + z * stride; which argument
// takes which stride is stated at each kernel.  Zero strides with one slice
// are the unbatched call.  Problem 0 does not read the strides: they lie past the
// arguments a wave starts with.
struct Bz {
    int64_t a = 0, b = 0, c = 0, d = 0;
};

// Per-problem strides (in elements) of a batched launch of the projected-
// problem kernels, one workgroup (row of workgroups) per problem z:
// vec for alpha, beta, sv, ftil, y, rho, eta; mat for Vw and V; lstr for
// the step-count pointer (int32 elements); curve for the criterion curve;
// ParamOut and the status word advance by one per problem; ws for the
// projected SVD's workspace (svd_ws_doubles of the allocation's l).
struct ProjBatch {
    int64_t vec = 0, mat = 0, lstr = 0, curve = 0, ws = 0;
};

// Native 2 x FP64 vector for 16-byte (non-temporal) loads and stores.
typedef double v2d __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v2d load_nt(const double* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const v2d*>(p));
}
__device__ __forceinline__ void store_nt(double* p, v2d v) {
    __builtin_nontemporal_store(v, reinterpret_cast<v2d*>(p));
}
__device__ __forceinline__ v2d load2(const double* p) { return *reinterpret_cast<const v2d*>(p); }

// A value that later code needs from a load: waits for it where this stands.  The
// kernels of a run load what they need together with the run's state and branch on
// the state behind it, so that one memory latency covers both; without this
// the compiler moves such loads behind the branch.
__device__ __forceinline__ void arrived(double& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void arrived(int& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void arrived(float& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void arrived(float4& v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }
__device__ __forceinline__ void arrived_uniform(int& v) { asm volatile("" : "+s"(v)); }

// v + p[first stride] + p[(first + step) stride] + .. below count, in that order, with U
// loads in flight throughout: the last batch repeats the last element and drops it
// when it adds.  (A loop over the remainder waits for each of its loads, and a choice
// the compiler sees beside a load becomes a branch around it.)  In the reductions of
// a Golub-Kahan step 2 % of a 20 000-node solve; with many short sums per
// workgroup (the stored products' reduction, the block QR) the plain loop is faster.
template <int U>
__device__ __forceinline__ double batched_sum(double v, const double* __restrict__ p, int first, int count, int step,
                                              int64_t stride) {
    for (int k0 = first; k0 < count; k0 += U * step) {
        double t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u * step;
            t[u] = p[(int64_t)(k < count ? k : count - 1) * stride];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) arrived(t[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) v += k0 + u * step < count ? t[u] : 0.0;
    }
    return v;
}

// Orders a wave's LDS accesses across its lanes: what one lane wrote before
// this point is seen by every lane's reads after it.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// Deterministic reductions (fixed butterfly / fixed order, no atomics)
// ---------------------------------------------------------------------------

template <int CTRL>
__device__ __forceinline__ double row_move(double v) {
    const int2 b = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_mov_dpp(b.x, CTRL, 0xF, 0xF, true),
                                                __builtin_amdgcn_mov_dpp(b.y, CTRL, 0xF, 0xF, true)));
}

// v + v of lane l ^ O, in registers: a lane exchange through LDS takes a latency of
// its own, six of them a sum over the wave (1 800-node solve 3497 -> 3398 us).
// O = 4: v is the same in lanes l and l ^ 8, as it is after O = 8.
template <int O>
__device__ __forceinline__ double add_xor(double v) {
    static_assert(O == 32 || O == 16 || O == 8 || O == 4 || O == 2 || O == 1, "a power of two below the wave");
    if constexpr (O >= 16) {
        const uint2 b = __builtin_bit_cast(uint2, v);
        unsigned x0, x1, y0, y1;
        if constexpr (O == 32) {  // each half of the wave beside the other
            const auto x = __builtin_amdgcn_permlane32_swap(b.x, b.x, false, false);
            const auto y = __builtin_amdgcn_permlane32_swap(b.y, b.y, false, false);
            x0 = x[0], x1 = x[1], y0 = y[0], y1 = y[1];
        } else {  // each even row of 16 beside the odd one after it
            const auto x = __builtin_amdgcn_permlane16_swap(b.x, b.x, false, false);
            const auto y = __builtin_amdgcn_permlane16_swap(b.y, b.y, false, false);
            x0 = x[0], x1 = x[1], y0 = y[0], y1 = y[1];
        }
        return __builtin_bit_cast(double, make_uint2(x0, y0)) + __builtin_bit_cast(double, make_uint2(x1, y1));
    }
    if constexpr (O == 8) return v + row_move<0x128>(v);  // row_ror:8
    if constexpr (O == 4) return v + row_move<0x124>(v);  // row_ror:4
    if constexpr (O == 2) return v + row_move<0x4E>(v);   // quad_perm 2 3 0 1
    return v + row_move<0xB1>(v);                         // quad_perm 1 0 3 2
}

__device__ __forceinline__ double wave_sum(double v) {
    v = add_xor<32>(v);
    v = add_xor<16>(v);
    v = add_xor<8>(v);
    v = add_xor<4>(v);
    v = add_xor<2>(v);
    return add_xor<1>(v);
}

// Sum over a whole block of NT threads; every thread gets the total.
// `lds` must hold NT/64 doubles.  Contains barriers: call from all threads.
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* lds) {
    v = wave_sum(v);
    const int w = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) lds[w] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < NT / kWave; ++i) s += lds[i];
    __syncthreads();
    return s;
}

// ---------------------------------------------------------------------------
// Multiquadric entries.  Nodes are stored centred on their bounding box and
// pre-multiplied by eps, so for two stored nodes P, Q
//     t = 1 + |P - Q|^2 = 1 + eps^2 r^2 .
// With s = t^{-1/2}:
//   boundary row (Dirichlet, eq. (3)):     phi      = sqrt(t)          = t s
//   interior row (eq. (8)):         L phi    = eps^2 (2t+1) t^{-3/2} + kappa^2 t^{1/2}
//                                                  = (kappa^2 t + 2 eps^2 + eps^2 s^2) s
// (the Laplacian of phi in 3-D is eps^2 (3 + 2 eps^2 r^2) / t^{3/2}, and
//  3 + 2 eps^2 r^2 = 2t + 1; all three terms are positive, so the form has
//  no cancellation).
// ---------------------------------------------------------------------------

struct EntryConst {
    double k2;    // kappa^2
    double e2;    // eps^2
    double e2x2;  // 2 eps^2
    float k2f, e2f, e2x2f, padf;
};

// 1/sqrt(t) for finite t > 0 in FP64 (the entries take t >= 1, the block QR's pivots and
// the band's reflectors any scale): the hardware estimate s refined by one
// third-order step.  With r = 1 - t s^2, 1/sqrt(t) = s (1 - r)^(-1/2) = s (1 + r/2 +
// 3 r^2/8 + 5 r^3/16 + ...); the dropped terms are below 2^-70 relative, so what is left
// is the final rounding and half of h's.  Measured over 4 million values in each of eight
// ranges from 2^-1060 to 2^1022: the estimate within 2^-24.1 of 1/sqrt(t), the
// result within 0.63 eps (1.00 ulp) in all of them, as two Newton steps, in five
// instructions instead of eight.
__device__ __forceinline__ double rsqrt_f64(double t) {
    const double s = __builtin_amdgcn_rsq(t);
    const double h = t * s;
    const double r = fma(-h, s, 1.0);
    const double p = fma(0.375, r, 0.5);
    return fma(s * r, p, s);
}

__device__ __forceinline__ double t_of(double px, double py, double pz, double qx, double qy, double qz) {
    const double dx = px - qx, dy = py - qy, dz = pz - qz;
    return fma(dz, dz, fma(dy, dy, fma(dx, dx, 1.0)));
}

__device__ __forceinline__ float t_of(float px, float py, float pz, float qx, float qy, float qz) {
    const float dx = px - qx, dy = py - qy, dz = pz - qz;
    return fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, 1.0f)));
}

__device__ __forceinline__ double entry_interior(double t, const EntryConst& c) {
    const double s = rsqrt_f64(t);
    return fma(c.e2, s * s, fma(c.k2, t, c.e2x2)) * s;
}

__device__ __forceinline__ double entry_boundary(double t, const EntryConst&) { return t * rsqrt_f64(t); }

// FP32 evaluation: one v_rsq_f32 / v_sqrt_f32 per entry (1 ulp), the rest in FP32.
__device__ __forceinline__ float entry_interior(float t, const EntryConst& c) {
    const float s = __builtin_amdgcn_rsqf(t);
    return fmaf(c.e2f, s * s, fmaf(c.k2f, t, c.e2x2f)) * s;
}

__device__ __forceinline__ float entry_boundary(float t, const EntryConst&) { return __builtin_amdgcn_sqrtf(t); }

// Node record types per evaluation precision.
template <typename R>
struct NodeOf;
template <>
struct NodeOf<double> {
    using type = double4;
};
template <>
struct NodeOf<float> {
    using type = float4;
};

}  // namespace mqh
