// FP32 pair arithmetic, precision-mode accumulators and output records shared
// by the direct-sum and tree-code force kernels (device code only).  See
// accel.hip for the instruction count and the precision modes.
#pragma once

#include "internal.h"

namespace nbi {
namespace {

enum { M_F32 = 1, M_KAHAN = 2, M_F64ACC = 3 };

template <int MODE>
struct Run;

template <>
struct Run<M_F32> {
    float s;
    __device__ void zero() { s = 0.0f; }
    __device__ void fold(float p) { s += p; }
    __device__ double get() const { return s; }
};

// Classic Kahan: y = p - c; t = s + y; c = (t - s) - y; s = t.  The reported
// value applies the final compensation, s - c, formed in FP64.
template <>
struct Run<M_KAHAN> {
    float s, c;
    __device__ void zero() { s = 0.0f; c = 0.0f; }
    __device__ void fold(float p)
    {
        const float y = p - c;
        const float t = s + y;
        c = (t - s) - y;
        s = t;
    }
    __device__ double get() const { return (double)s - (double)c; }
};

template <>
struct Run<M_F64ACC> {
    double s;
    __device__ void zero() { s = 0.0; }
    __device__ void fold(double p) { s += p; }
    __device__ double get() const { return s; }
};

template <typename T, int TPL>
struct Targets {
    T x[TPL], y[TPL], z[TPL];
    int i[TPL];
};

template <typename T, int TPL>
struct Sums {
    T ax[TPL], ay[TPL], az[TPL], ph[TPL];
    __device__ void zero()
    {
#pragma unroll
        for (int t = 0; t < TPL; ++t) ax[t] = ay[t] = az[t] = ph[t] = T(0);
    }
};

// ---- FP32 pair ---------------------------------------------------------------
// One source against the lane's TPL targets, in groups of G whose reciprocal
// square roots share one stretch at raised priority.  Nothing is reordered
// across a stretch, so with one for each target a wave that is alone on its SIMD
// waits for every result in turn (pinned shapes with 4 targets per lane, 700 to
// 10007 bodies: 0.85 to 0.98 of the rate without raised priority; in one group
// 0.95 to 1.12).  The FMM's leaves, many waves of a few sources each, take the
// targets one by one (in groups 1 to 3% slower at 2^20 bodies).
template <int TPL, bool MASK, int G = TPL>
__device__ __forceinline__ void pair_f32(const float4 b, const int j, const Targets<float, TPL> &T,
                                         const float eps2, Sums<float, TPL> &S)
{
    static_assert(TPL % G == 0, "whole groups");
#pragma unroll
    for (int t0 = 0; t0 < TPL; t0 += G) {
        float dx[G], dy[G], dz[G], rho[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            dx[g] = b.x - T.x[t0 + g];
            dy[g] = b.y - T.y[t0 + g];
            dz[g] = b.z - T.z[t0 + g];
            rho[g] = __builtin_fmaf(dz[g], dz[g], __builtin_fmaf(dy[g], dy[g], __builtin_fmaf(dx[g], dx[g], eps2)));
        }
        rsq_prio(rho);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int t = t0 + g;
            if (MASK) rho[g] = (j == T.i[t]) ? 0.0f : rho[g];
            const float mr = b.w * rho[g];
            const float s = mr * (rho[g] * rho[g]);
            S.ph[t] = __builtin_fmaf(b.w, rho[g], S.ph[t]);
            S.ax[t] = __builtin_fmaf(s, dx[g], S.ax[t]);
            S.ay[t] = __builtin_fmaf(s, dy[g], S.ay[t]);
            S.az[t] = __builtin_fmaf(s, dz[g], S.az[t]);
        }
    }
}

// SEQ: a scheduling barrier after each source keeps the per-source chain
// that the compiler otherwise chooses (it sometimes interleaves the sources
// of an unrolled step over twice the registers instead, which measured about
// 18% slower).  U: sources per unrolled step; steps of kUnroll and single
// sources take what is left.  Long ranges use 16 (all targets of 16384 to
// 200000 sources: 2% faster than 8), the tree code's short ones 8.
template <int TPL, bool MASK, bool SEQ, int U>
__device__ __forceinline__ void sweep_steps(const float4 *__restrict__ src, int &j, int j1,
                                            const Targets<float, TPL> &T, float eps2, Sums<float, TPL> &S)
{
    for (; j + U <= j1; j += U) {
        float4 b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) b[u] = src[j + u];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pair_f32<TPL, MASK>(b[u], j + u, T, eps2, S);
            if constexpr (SEQ) __builtin_amdgcn_sched_barrier(0);
        }
    }
}

template <int TPL, bool MASK, bool SEQ = false, int U = kUnroll>
__device__ __forceinline__ void sweep_f32(const float4 *__restrict__ src, int j0, int j1,
                                          const Targets<float, TPL> &T, float eps2,
                                          Sums<float, TPL> &S)
{
    int j = j0;
    if constexpr (U > kUnroll) sweep_steps<TPL, MASK, SEQ, U>(src, j, j1, T, eps2, S);
    sweep_steps<TPL, MASK, SEQ, kUnroll>(src, j, j1, T, eps2, S);
    for (; j < j1; ++j) pair_f32<TPL, MASK>(src[j], j, T, eps2, S);
}

// Sources [j0, j1) against the wave's targets [d0, d1): only the overlap runs
// the masked variant.
template <int TPL, bool SEQ = false, int U = kUnroll>
__device__ __forceinline__ void range_f32(const float4 *__restrict__ src, int j0, int j1, int d0,
                                          int d1, const Targets<float, TPL> &T, float eps2,
                                          Sums<float, TPL> &S)
{
    const int lo = min(max(d0, j0), j1);
    const int hi = min(max(d1, j0), j1);
    sweep_f32<TPL, false, SEQ, U>(src, j0, lo, T, eps2, S);
    sweep_f32<TPL, true, SEQ>(src, lo, hi, T, eps2, S);
    sweep_f32<TPL, false, SEQ, U>(src, hi, j1, T, eps2, S);
}

// ---- output records ------------------------------------------------------------
__device__ __forceinline__ void put(float4 *out, long k, const double (&r)[4], double G)
{
    out[k] = make_float4((float)(G * r[0]), (float)(G * r[1]), (float)(G * r[2]), (float)(-G * r[3]));
}
__device__ __forceinline__ void put(double4 *out, long k, const double (&r)[4], double G)
{
    out[k] = make_double4(G * r[0], G * r[1], G * r[2], -G * r[3]);
}
// Pure FP32 mode scales in FP32.
__device__ __forceinline__ void put_f32(float4 *out, long k, const double (&r)[4], float G)
{
    out[k] = make_float4(G * (float)r[0], G * (float)r[1], G * (float)r[2], -G * (float)r[3]);
}

// ---- leapfrog step of one body -----------------------------------------------------
// close: v += h a;  energies (1/2 m |v|^2, 1/2 m phi) in FP64;
// open: v += h a; x += dt v.
template <typename V, typename S>
__device__ __forceinline__ void step_body(V &x, V &vel, const V a, S h, S dt, int close, int open, bool energy,
                                          double &ek, double &eu)
{
    V v = vel;
    if (close) {
        v.x = v.x + h * a.x;
        v.y = v.y + h * a.y;
        v.z = v.z + h * a.z;
    }
    if (energy) {
        const double vx = v.x, vy = v.y, vz = v.z, m = x.w;
        ek = 0.5 * m * ((vx * vx + vy * vy) + vz * vz);
        eu = 0.5 * m * (double)a.w;
    }
    if (open) {
        v.x = v.x + h * a.x;
        v.y = v.y + h * a.y;
        v.z = v.z + h * a.z;
        x.x = x.x + dt * v.x;
        x.y = x.y + dt * v.y;
        x.z = x.z + dt * v.z;
    }
    if (close || open) vel = v;
}

}  // namespace
}  // namespace nbi
