// Direct-sum force and potential kernels for gfx950.
//
// Computes, for each target i, the paper's force calculation (Section IV.B,
// Calculate_forces) with every other body on the interaction list, i.e. the
// exact softened pair sum
//     a_i   =  G sum_{j != i} m_j d_ij (|d_ij|^2 + eps^2)^(-3/2),  d_ij = x_j - x_i
//     phi_i = -G sum_{j != i} m_j (|d_ij|^2 + eps^2)^(-1/2)
//
// Design (CDNA4, wave64):
// * A wave owns 64*TPL targets held in VGPRs.  Sources are streamed with
//   wave-uniform addresses, so every source record arrives through a scalar
//   load into SGPRs and feeds the VALU directly as the one scalar operand an
//   instruction may take: no LDS staging, no barriers, and the 16-byte source
//   record is fetched once per wave for 64*TPL interactions.
// * Pair arithmetic (FP32 modes): 3 sub, 3 FMA, 1 v_rsq_f32, 2 mul, 1 mul,
//   1 FMA (potential), 3 FMA = 14 VALU instructions = 20 flop by the usual
//   count.  The library is built with contraction off and every fused
//   multiply-add is written out, so the same arithmetic is emitted in every
//   kernel that shares these routines (batched results equal standalone ones
//   of the sweep in the same shape bit for bit).
// * Sources are processed in tiles of `jtile`; the FP32 partial sum of a tile
//   is folded into the running per-target sum by the precision mode (plain
//   FP32, Kahan-compensated FP32, or FP64).
// * The self pair is removed exactly: only the sub-range of sources that
//   overlaps the wave's own targets runs the masked variant (one compare and
//   one select per pair); every other source range runs unmasked.
// * Where the targets alone are too few waves to fill the chip, the source
//   range is split over gridDim.y workgroup rows; the per-split records go to
//   scratch and are reduced in split order by a second kernel, so the result
//   never depends on scheduling.
// * Unless a shape is pinned, small problems run k_accel_slice instead (one
//   launch, no scratch), and the force on all of many bodies the kernels of
//   sym.hip.
#include <mutex>

#include "internal.h"
#include "pair.h"

namespace nbi {
namespace {

// Sums over sources [jb, je) of one system (records src[0..n)) for the wave
// whose first target is t0; returns the unscaled sums per target and
// component (ax, ay, az, sum m rho) through `res`.
template <int TPL, int MODE>
__device__ __forceinline__ void wave_f32(const float4 *__restrict__ src, int n, int t0, int jb,
                                         int je, int jtile, float eps2_in, double (&res)[TPL][4])
{
    const int lane = threadIdx.x & 63;
    const float eps2 = lane_copy(eps2_in);
    Targets<float, TPL> T;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const int i = t0 + t * 64 + lane;
        T.i[t] = i;
        const float4 p = src[min(i, n - 1)];
        T.x[t] = p.x;
        T.y[t] = p.y;
        T.z[t] = p.z;
    }
    const int d0 = t0, d1 = t0 + 64 * TPL;
    Sums<float, TPL> S;
    Run<MODE> R[TPL][4];
#pragma unroll
    for (int t = 0; t < TPL; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) R[t][c].zero();
    for (int jc = jb, ce; jc < je; jc = ce) {
        ce = je - jc > jtile ? jc + jtile : je;  // no jc + jtile past je (int range)
        S.zero();
        // pure FP32 pins the per-source schedule (see sweep_f32)
        range_f32<TPL, MODE == M_F32, 2 * kUnroll>(src, jc, ce, d0, d1, T, eps2, S);
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            R[t][0].fold(S.ax[t]);
            R[t][1].fold(S.ay[t]);
            R[t][2].fold(S.az[t]);
            R[t][3].fold(S.ph[t]);
        }
    }
#pragma unroll
    for (int t = 0; t < TPL; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) res[t][c] = R[t][c].get();
}

// ---- FP64 pair ---------------------------------------------------------------
template <int TPL, bool MASK>
__device__ __forceinline__ void pair_f64(const double4 b, const int j, const Targets<double, TPL> &T,
                                         const double eps2, Sums<double, TPL> &S)
{
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const double dx = b.x - T.x[t];
        const double dy = b.y - T.y[t];
        const double dz = b.z - T.z[t];
        const double r2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, __builtin_fma(dx, dx, eps2)));
        double rho = rsq_f64(r2);
        if (MASK) rho = (j == T.i[t]) ? 0.0 : rho;
        const double mr = b.w * rho;
        const double s = mr * (rho * rho);
        S.ph[t] = __builtin_fma(b.w, rho, S.ph[t]);
        S.ax[t] = __builtin_fma(s, dx, S.ax[t]);
        S.ay[t] = __builtin_fma(s, dy, S.ay[t]);
        S.az[t] = __builtin_fma(s, dz, S.az[t]);
    }
}

template <int TPL, bool MASK>
__device__ __forceinline__ void sweep_f64(const double4 *__restrict__ src, int j0, int j1,
                                          const Targets<double, TPL> &T, double eps2,
                                          Sums<double, TPL> &S)
{
    int j = j0;
    for (; j + kUnroll <= j1; j += kUnroll) {
        double4 b[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) b[u] = src[j + u];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) pair_f64<TPL, MASK>(b[u], j + u, T, eps2, S);
    }
    for (; j < j1; ++j) pair_f64<TPL, MASK>(src[j], j, T, eps2, S);
}

template <int TPL>
__device__ __forceinline__ void wave_f64(const double4 *__restrict__ src, int n, int t0, int jb,
                                         int je, int jtile, double eps2, double (&res)[TPL][4])
{
    const int lane = threadIdx.x & 63;
    Targets<double, TPL> T;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const int i = t0 + t * 64 + lane;
        T.i[t] = i;
        const double4 p = src[min(i, n - 1)];
        T.x[t] = p.x;
        T.y[t] = p.y;
        T.z[t] = p.z;
    }
    const int d0 = t0, d1 = t0 + 64 * TPL;
    double R[TPL][4];
#pragma unroll
    for (int t = 0; t < TPL; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) R[t][c] = 0.0;
    Sums<double, TPL> S;
    for (int jc = jb, ce; jc < je; jc = ce) {
        ce = je - jc > jtile ? jc + jtile : je;  // no jc + jtile past je (int range)
        S.zero();
        const int lo = min(max(d0, jc), ce);
        const int hi = min(max(d1, jc), ce);
        sweep_f64<TPL, false>(src, jc, lo, T, eps2, S);
        sweep_f64<TPL, true>(src, lo, hi, T, eps2, S);
        sweep_f64<TPL, false>(src, hi, ce, T, eps2, S);
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            R[t][0] += S.ax[t];
            R[t][1] += S.ay[t];
            R[t][2] += S.az[t];
            R[t][3] += S.ph[t];
        }
    }
#pragma unroll
    for (int t = 0; t < TPL; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) res[t][c] = R[t][c];
}

// ---- FP32 sweep with sources staged in LDS ----------------------------------
// Same pair arithmetic and the same order of every sum as the scalar-load
// sweep (identical results), but each source record reaches the VALU as a
// VGPR from a broadcast LDS read instead of as an SGPR: on gfx950 VALU
// instructions whose operands are all VGPRs can issue about twice per clock
// per CU, while those that read an SGPR stay near one.
constexpr int kLdsTile = 256;  // sources per LDS buffer (one per thread)

template <int TPL, bool MASK>
__device__ __forceinline__ void sweep_lds(const float4 *tl, int jbase, int u0, int u1,
                                          const Targets<float, TPL> &T, float eps2,
                                          Sums<float, TPL> &S)
{
    int u = u0;
    for (; u + kUnroll <= u1; u += kUnroll) {
        float4 b[kUnroll];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) b[k] = tl[u + k];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) pair_f32<TPL, MASK>(b[k], jbase + u + k, T, eps2, S);
    }
    for (; u < u1; ++u) pair_f32<TPL, MASK>(tl[u], jbase + u, T, eps2, S);
}

// Whole workgroup: all four waves sweep the same source range [jb, je); the
// tiles are double-buffered through LDS with a register prefetch.  jtile is
// a multiple of kLdsTile, so the partial sums fold at the same source
// indices as in the scalar-load sweep.
template <int TPL, int MODE>
__device__ __forceinline__ void block_lds_f32(const float4 *__restrict__ src, int n, int t0, int jb,
                                              int je, int jtile, float eps2_in,
                                              float4 (*tile)[kLdsTile], double (&res)[TPL][4])
{
    const int lane = threadIdx.x & 63;
    const float eps2 = lane_copy(eps2_in);
    Targets<float, TPL> T;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const int i = t0 + t * 64 + lane;
        T.i[t] = i;
        const float4 p = src[min(i, n - 1)];
        T.x[t] = p.x;
        T.y[t] = p.y;
        T.z[t] = p.z;
    }
    const int d0 = t0, d1 = t0 + 64 * TPL;
    Sums<float, TPL> S;
    S.zero();
    Run<MODE> R[TPL][4];
#pragma unroll
    for (int t = 0; t < TPL; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) R[t][c].zero();
    float4 pre = make_float4(0.f, 0.f, 0.f, 0.f);
    if (jb + (int)threadIdx.x < je) pre = src[jb + threadIdx.x];
    tile[0][threadIdx.x] = pre;
    __syncthreads();
    int buf = 0, since = 0;
    for (int j0 = jb; j0 < je; j0 += kLdsTile) {
        const int cnt = min(kLdsTile, je - j0);
        const int jn = j0 + kLdsTile;
        if (jn + (int)threadIdx.x < je) pre = src[jn + threadIdx.x];
        const int lo = min(max(d0, j0), j0 + cnt) - j0;
        const int hi = min(max(d1, j0), j0 + cnt) - j0;
        sweep_lds<TPL, false>(tile[buf], j0, 0, lo, T, eps2, S);
        sweep_lds<TPL, true>(tile[buf], j0, lo, hi, T, eps2, S);
        sweep_lds<TPL, false>(tile[buf], j0, hi, cnt, T, eps2, S);
        since += cnt;
        if (since >= jtile || jn >= je) {
#pragma unroll
            for (int t = 0; t < TPL; ++t) {
                R[t][0].fold(S.ax[t]);
                R[t][1].fold(S.ay[t]);
                R[t][2].fold(S.az[t]);
                R[t][3].fold(S.ph[t]);
            }
            S.zero();
            since = 0;
        }
        if (jn < je) tile[buf ^ 1][threadIdx.x] = pre;
        __syncthreads();
        buf ^= 1;
    }
#pragma unroll
    for (int t = 0; t < TPL; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) res[t][c] = R[t][c].get();
}

// ---- kernels -------------------------------------------------------------------
// The chip hands workgroups to its 8 XCDs in turn (linear workgroup id modulo
// 8), and each XCD has its own L2.  When the source range is split in a
// multiple of 8, workgroup (bx, by) = (target block, source split) is taken
// from the linear id so that XCD x runs only the splits x J/8 .. (x + 1) J/8
// - 1, one after the other with the target blocks fastest: the waves on an
// XCD then stream one source segment at a time, which stays in that L2, and
// each segment is fetched from memory about once instead of once per pass of
// the resident waves.  Any other split count, or sources that fit in one
// XCD's L2 anyway (there the new order measured up to 18% slower, at 2^12),
// keeps the plain mapping.  Either way every (bx, by) is run exactly once, so
// results do not depend on it.
constexpr int kXcds = 8;
constexpr long kXcdL2Bytes = 4l << 20;

__device__ __forceinline__ void xcd_block(long src_bytes, int &bx, int &by)
{
    const int gx = gridDim.x, J = gridDim.y;
    if (J % kXcds || src_bytes <= kXcdL2Bytes) {
        bx = blockIdx.x;
        by = blockIdx.y;
        return;
    }
    const long L = (long)blockIdx.y * gx + blockIdx.x;
    const long i = L / kXcds;  // this workgroup's place in its XCD's sequence
    by = (int)(L % kXcds) * (J / kXcds) + (int)(i / gx);
    bx = (int)(i % gx);
}

// Source range of split `split` out of `js` over n sources.
__device__ __forceinline__ void split_range(int n, int js, int split, int &jb, int &je)
{
    const long per = ((long)n + js - 1) / js;
    jb = (int)min((long)n, (long)split * per);
    je = (int)min((long)n, (long)jb + per);
}

template <int TPL, int MODE>
__global__ __launch_bounds__(kBlock) void k_accel_f32(const float4 *__restrict__ src, int n,
                                                      float eps2, double G, int tbeg, int tcount,
                                                      int jtile, float4 *__restrict__ out,
                                                      void *__restrict__ partial)
{
    constexpr int WT = 64 * TPL;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int bx, by;
    xcd_block((long)n * sizeof(float4), bx, by);
    const int t0 = tbeg + (bx * (kBlock / 64) + wave) * WT;
    const int tend = tbeg + tcount;
    if (t0 >= tend) return;
    int jb, je;
    split_range(n, gridDim.y, by, jb, je);
    double res[TPL][4];
    wave_f32<TPL, MODE>(src, n, t0, jb, je, jtile, eps2, res);
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const int i = t0 + t * 64 + lane;
        if (i >= tend) continue;
        const long k = i - tbeg;
        if (gridDim.y == 1) {
            if constexpr (MODE == M_F32)
                put_f32(out, k, res[t], (float)G);
            else
                put(out, k, res[t], G);
        } else if constexpr (MODE == M_F32) {
            reinterpret_cast<float4 *>(partial)[split_at(k, by, gridDim.y, tcount)] =
                make_float4((float)res[t][0], (float)res[t][1], (float)res[t][2], (float)res[t][3]);
        } else {
            reinterpret_cast<double4 *>(partial)[split_at(k, by, gridDim.y, tcount)] =
                make_double4(res[t][0], res[t][1], res[t][2], res[t][3]);
        }
    }
}

template <int TPL, int MODE>
__global__ __launch_bounds__(kBlock) void k_accel_lds_f32(const float4 *__restrict__ src, int n,
                                                          float eps2, double G, int tbeg, int tcount,
                                                          int jtile, float4 *__restrict__ out,
                                                          void *__restrict__ partial)
{
    __shared__ float4 tile[2][kLdsTile];
    constexpr int WT = 64 * TPL;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tend = tbeg + tcount;
    // waves past the last target still take part in the shared tile loop
    // (on a valid target range) but store nothing
    int bx, by;
    xcd_block((long)n * sizeof(float4), bx, by);
    const long t0l = (long)tbeg + ((long)bx * (kBlock / 64) + wave) * WT;
    const bool active = t0l < tend;
    const int t0 = active ? (int)t0l : tbeg;
    int jb, je;
    split_range(n, gridDim.y, by, jb, je);
    double res[TPL][4];
    block_lds_f32<TPL, MODE>(src, n, t0, jb, je, jtile, eps2, tile, res);
    if (!active) return;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const int i = t0 + t * 64 + lane;
        if (i >= tend) continue;
        const long k = i - tbeg;
        if (gridDim.y == 1) {
            if constexpr (MODE == M_F32)
                put_f32(out, k, res[t], (float)G);
            else
                put(out, k, res[t], G);
        } else if constexpr (MODE == M_F32) {
            reinterpret_cast<float4 *>(partial)[split_at(k, by, gridDim.y, tcount)] =
                make_float4((float)res[t][0], (float)res[t][1], (float)res[t][2], (float)res[t][3]);
        } else {
            reinterpret_cast<double4 *>(partial)[split_at(k, by, gridDim.y, tcount)] =
                make_double4(res[t][0], res[t][1], res[t][2], res[t][3]);
        }
    }
}

template <int TPL>
__global__ __launch_bounds__(kBlock) void k_accel_f64(const double4 *__restrict__ src, int n,
                                                      double eps2, double G, int tbeg, int tcount,
                                                      int jtile, double4 *__restrict__ out,
                                                      double4 *__restrict__ partial)
{
    constexpr int WT = 64 * TPL;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int bx, by;
    xcd_block((long)n * sizeof(double4), bx, by);
    const int t0 = tbeg + (bx * (kBlock / 64) + wave) * WT;
    const int tend = tbeg + tcount;
    if (t0 >= tend) return;
    int jb, je;
    split_range(n, gridDim.y, by, jb, je);
    double res[TPL][4];
    wave_f64<TPL>(src, n, t0, jb, je, jtile, eps2, res);
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const int i = t0 + t * 64 + lane;
        if (i >= tend) continue;
        const long k = i - tbeg;
        if (gridDim.y == 1)
            put(out, k, res[t], G);
        else
            partial[split_at(k, by, gridDim.y, tcount)] = make_double4(res[t][0], res[t][1], res[t][2], res[t][3]);
    }
}

// ---- small problems: sources over the lanes and waves of one workgroup ---------
// A few thousand bodies are too few targets for 64 per wave to reach all 256
// CUs, and a source split costs a second launch.  Here a workgroup of 1024
// threads takes kSliceT targets and kSlices slices of the sources (slice s
// takes sources s, s + kSlices, ...), which it stages in LDS in chunks; a wave
// holds 64 / kSliceT slices, whose lanes read neighbouring records.  The
// slices' sums meet in LDS in a fixed order, so an evaluation is one launch:
// at 4096 FP64 bodies 256 workgroups, one per CU.  Only the steps that meet
// the workgroup's own targets run the masked pair.  FP32 partial sums hold at
// most 32 sources and are added in FP64 in every mode.  What bounds it: up to
// about 4000 FP32 bodies the call itself (12.5 us from Python); above, the
// pair arithmetic at 4 to 8 waves per SIMD.
constexpr int kSliceThreads = 1024;
constexpr int kSliceT = 16;
constexpr int kSlices = kSliceThreads / kSliceT;

template <typename T>
struct SliceRec;
template <>
struct SliceRec<float> {
    using V = float4;
    static constexpr int kChunk = 2048;
};
template <>
struct SliceRec<double> {
    using V = double4;
    static constexpr int kChunk = 1024;
};

template <bool MASK>
__device__ __forceinline__ void slice_pair(const float4 b, int j, const Targets<float, 1> &T, float eps2,
                                           Sums<float, 1> &S)
{
    pair_f32<1, MASK>(b, j, T, eps2, S);
}
template <bool MASK>
__device__ __forceinline__ void slice_pair(const double4 b, int j, const Targets<double, 1> &T, double eps2,
                                           Sums<double, 1> &S)
{
    pair_f64<1, MASK>(b, j, T, eps2, S);
}

// Steps [k0, k1) of slice sl over the chunk that starts at source c0.
template <bool MASK, typename T, typename V>
__device__ __forceinline__ void slice_sweep(const V *buf, int c0, int sl, int k0, int k1, const Targets<T, 1> &TT,
                                            T eps2, Sums<T, 1> &S)
{
    constexpr int U = 4;
    int k = k0;
    for (; k + U <= k1; k += U) {
        V b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) b[u] = buf[kSlices * (k + u) + sl];
#pragma unroll
        for (int u = 0; u < U; ++u) slice_pair<MASK>(b[u], c0 + kSlices * (k + u) + sl, TT, eps2, S);
    }
    for (; k < k1; ++k) slice_pair<MASK>(buf[kSlices * k + sl], c0 + kSlices * k + sl, TT, eps2, S);
}

// The leapfrog step that follows the force (STEP): each body's kick and drift by
// the lane that has its sum, the drifted positions to `to`, since other
// workgroups still read the old ones; without a drift `to` is null or takes a copy.
// The step's own launch took 4.5 us of 24 at 4096 FP64 bodies: ten steps with
// energies 225 -> 199 us, of 1000 FP32 bodies without 88 -> 59 us.
template <typename T>
struct SliceStep {
    typename SliceRec<T>::V *vel, *to;
    T h, dt;
    int close, open;
    double *epart;  // FP64: per workgroup, kinetic and potential energy, or null (FP32 runs with energies take the sweep)
};

template <typename T, int MODE, bool STEP>
__global__ __launch_bounds__(kSliceThreads) void k_accel_slice(const typename SliceRec<T>::V *__restrict__ src, int n,
                                                              T eps2_in, double G, int tbeg, int tcount,
                                                              typename SliceRec<T>::V *__restrict__ out,
                                                              SliceStep<T> step)
{
    using V = typename SliceRec<T>::V;
    constexpr int C = SliceRec<T>::kChunk;
    static_assert(C % kSlices == 0 && sizeof(V) * C >= sizeof(double) * 4 * kSliceThreads, "the sums reuse the chunk");
    constexpr bool ENERGY = STEP && sizeof(T) == 8;
    __shared__ V buf[C];
    const int tid = threadIdx.x, tg = tid % kSliceT, sl = tid / kSliceT;
    const int t0 = tbeg + blockIdx.x * kSliceT, i = t0 + tg;
    T eps2;
    if constexpr (sizeof(T) == 4)
        eps2 = lane_copy(eps2_in);
    else
        eps2 = eps2_in;
    Targets<T, 1> TT;
    {
        const V p = src[min(i, n - 1)];
        TT.x[0] = p.x;
        TT.y[0] = p.y;
        TT.z[0] = p.z;
        TT.i[0] = i;
    }
    double R[4] = {0.0, 0.0, 0.0, 0.0};
    for (int c0 = 0; c0 < n; c0 += C) {
        const int cnt = min(C, n - c0);
        __syncthreads();
        for (int k = tid; k < cnt; k += kSliceThreads) buf[k] = src[c0 + k];
        __syncthreads();
        Sums<T, 1> S;
        S.zero();
        const int kf = cnt / kSlices;  // steps that every slice has
        // steps that meet targets [t0, t0 + kSliceT)
        const int lo = min(max(t0 - c0, 0) / kSlices, kf);
        const int hi = min((max(t0 + kSliceT - c0, 0) + kSlices - 1) / kSlices, kf);
        slice_sweep<false>(buf, c0, sl, 0, lo, TT, eps2, S);
        slice_sweep<true>(buf, c0, sl, lo, hi, TT, eps2, S);
        slice_sweep<false>(buf, c0, sl, hi, kf, TT, eps2, S);
        if (kSlices * kf + sl < cnt) slice_sweep<true>(buf, c0, sl, kf, kf + 1, TT, eps2, S);
        R[0] += S.ax[0];
        R[1] += S.ay[0];
        R[2] += S.az[0];
        R[3] += S.ph[0];
    }
    // Sum over the slices: red[slice][4][target], one (component, target) and
    // kPart slices per thread, then the parts in order.
    constexpr int kOut = 4 * kSliceT, kParts = kSliceThreads / kOut, kPart = kSlices / kParts;
    double *red = reinterpret_cast<double *>(buf);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c) red[(sl * 4 + c) * kSliceT + tg] = R[c];
    __syncthreads();
    const int o = tid % kOut, part = tid / kOut;
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < kPart; ++q) v += red[(part * kPart + q) * kOut + o];
    __syncthreads();
    red[part * kOut + o] = v;
    __syncthreads();
    if (tid >= kSliceT) return;
    double ek = 0.0, eu = 0.0;
    if (i < tbeg + tcount) {
        double r[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double w = 0.0;
#pragma unroll
            for (int q = 0; q < kParts; ++q) w += red[q * kOut + c * kSliceT + tg];
            r[c] = w;
        }
        if constexpr (MODE == M_F32)
            put_f32(out, i - tbeg, r, (float)G);
        else
            put(out, i - tbeg, r, G);
        if constexpr (STEP) {
            V x = src[i];
            step_body<V, T>(x, step.vel[i], out[i], step.h, step.dt, step.close, step.open,
                            ENERGY && step.epart != nullptr, ek, eu);
            if (step.to) step.to[i] = x;
        }
    }
    if constexpr (ENERGY) {
        if (!step.epart) return;
        static_assert(kSliceT == kEnergyRow, "the workgroup's bodies are a row");
#pragma unroll
        for (int o = kEnergyRow / 2; o >= 1; o >>= 1) {
            ek += __shfl_xor(ek, o);
            eu += __shfl_xor(eu, o);
        }
        if (tid == 0) {
            step.epart[2 * blockIdx.x] = ek;
            step.epart[2 * blockIdx.x + 1] = eu;
        }
    }
}

// Fixed-order reduction of the per-split records.
template <typename OUT, typename E = double>
__global__ __launch_bounds__(kBlock) void k_split_reduce(const void *__restrict__ partial,
                                                         int js, int tcount, double G,
                                                         OUT *__restrict__ out)
{
    const long k = ((long)blockIdx.x * kBlock + threadIdx.x) / kSumLanes;
    double r[4];
    split_sum<kSumLanes>(reinterpret_cast<const E *>(partial), js, tcount, min(k, (long)tcount - 1), r);
    if (threadIdx.x % kSumLanes == 0 && k < tcount) put(out, k, r, G);
}

__global__ __launch_bounds__(kBlock) void k_split_reduce_f32(const float4 *__restrict__ partial,
                                                             int js, int tcount, float G,
                                                             float4 *__restrict__ out)
{
    const long k = ((long)blockIdx.x * kBlock + threadIdx.x) / kSumLanes;
    float r[4];
    split_sum<kSumLanes>(reinterpret_cast<const float *>(partial), js, tcount, min(k, (long)tcount - 1), r);
    if (threadIdx.x % kSumLanes == 0 && k < tcount) out[k] = make_float4(G * r[0], G * r[1], G * r[2], -G * r[3]);
}

// ---- batched persistent kernel -------------------------------------------------
// Workgroups of 4 waves take units from a longest-first list, the first by
// their own number and the others with one integer atomic.  A unit is 256 TPL / q targets of one system, q waves to each 64
// TPL targets: the q waves take the source tiles in turn, leave their FP32 (or
// FP64) tile sums in LDS, and fold them in tile order into running sums kept
// one component per wave.  The sums are those of k_accel_f32 with one split
// over the same tiles, folded in the same order, so each system's result
// equals bit for bit its standalone evaluation with this shape pinned; but the
// longest system no longer takes one wave's time for all its sources, which
// had bound batches whose units all fit the chip at once: 128 systems of 256
// to 8192 bodies ran 655 us with one wave per 64 targets, 361 us now (the
// pairs alone need about 290 at the force kernel's rate).  The workgroup that
// finishes last returns both counters to zero, which keeps repeated launches
// and graph replays self-contained.
template <int TPL, bool SEQ>
__device__ __forceinline__ void tile_sums(const float4 *__restrict__ src, int jc, int ce, int d0, int d1,
                                          const Targets<float, TPL> &T, float eps2, Sums<float, TPL> &S)
{
    range_f32<TPL, SEQ>(src, jc, ce, d0, d1, T, eps2, S);
}
template <int TPL, bool SEQ>
__device__ __forceinline__ void tile_sums(const double4 *__restrict__ src, int jc, int ce, int d0, int d1,
                                          const Targets<double, TPL> &T, double eps2, Sums<double, TPL> &S)
{
    const int lo = min(max(d0, jc), ce);
    const int hi = min(max(d1, jc), ce);
    sweep_f64<TPL, false>(src, jc, lo, T, eps2, S);
    sweep_f64<TPL, true>(src, lo, hi, T, eps2, S);
    sweep_f64<TPL, false>(src, hi, ce, T, eps2, S);
}

template <typename T, int TPL, int MODE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 8 : 4))) void k_batched(
    const typename SliceRec<T>::V *__restrict__ pm, const int64_t *__restrict__ offsets,
    const int2 *__restrict__ units, int nunits, const float *__restrict__ eps_sys, T eps2_all, double G, int jtile,
    typename SliceRec<T>::V *__restrict__ out, unsigned *__restrict__ counter)
{
    using V = typename SliceRec<T>::V;
    constexpr int K = 4 * TPL;  // sums per lane
    constexpr int kWaves = kBlock / 64;
    __shared__ T part[2][kWaves][K][64];
    __shared__ unsigned next;
    static_assert(sizeof(part) >= sizeof(double) * (kWaves / 2) * K * 64, "the results reuse the tile sums");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // With no more units than workgroups nothing is popped at all (two atomics
    // and their hand-over through LDS were 1.4 of the 6.7 us of one system of 64
    // bodies; a wave by itself, without the hand-over, had taken 5.5).
    const bool more = (unsigned)nunits > gridDim.x;
    auto pop = [&]() -> unsigned {
        if (!more) return (unsigned)nunits;
        __syncthreads();  // the unit's results have been read
        if (threadIdx.x == 0) next = gridDim.x + atomicAdd(&counter[0], 1u);
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(next);
    };
    for (unsigned u = blockIdx.x; u < (unsigned)nunits; u = pop()) {
        const int2 un = units[u];
        const int64_t base = offsets[un.x];
        const int n = (int)(offsets[un.x + 1] - base);
        const V *src = pm + base;
        T eps2 = eps2_all;
        if (eps_sys) {
            const double e = eps_sys[un.x];
            eps2 = (T)(e * e);
        }
        if constexpr (sizeof(T) == 4) eps2 = lane_copy(eps2);
        const int q = batch_split(n, jtile);
        const int sub = wave & (q - 1), grp = wave / q;
        const int nt = (int)(((long)n + jtile - 1) / jtile);
        const int t0 = un.y + grp * 64 * TPL;
        Targets<T, TPL> TT;
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            const int i = t0 + t * 64 + lane;
            TT.i[t] = i;
            const V p = src[min(i, n - 1)];
            TT.x[t] = p.x;
            TT.y[t] = p.y;
            TT.z[t] = p.z;
        }
        Run<MODE> R[K];  // of the components this wave folds: k mod q == sub
#pragma unroll
        for (int k = 0; k < K; ++k) R[k].zero();
        int buf = 0;
        for (int k0 = 0; k0 < nt; k0 += q) {
            Sums<T, TPL> S;
            S.zero();
            if (k0 + sub < nt && t0 < n) {
                const int jc = (k0 + sub) * jtile;
                tile_sums<TPL, MODE == M_F32>(src, jc, n - jc > jtile ? jc + jtile : n, t0, t0 + 64 * TPL, TT, eps2, S);
            }
            if (q == 1) {
#pragma unroll
                for (int t = 0; t < TPL; ++t) {
                    R[4 * t].fold(S.ax[t]);
                    R[4 * t + 1].fold(S.ay[t]);
                    R[4 * t + 2].fold(S.az[t]);
                    R[4 * t + 3].fold(S.ph[t]);
                }
                continue;
            }
#pragma unroll
            for (int t = 0; t < TPL; ++t) {
                part[buf][wave][4 * t][lane] = S.ax[t];
                part[buf][wave][4 * t + 1][lane] = S.ay[t];
                part[buf][wave][4 * t + 2][lane] = S.az[t];
                part[buf][wave][4 * t + 3][lane] = S.ph[t];
            }
            __syncthreads();
            const int m = min(q, nt - k0);
#pragma unroll
            for (int k = 0; k < K; ++k)
                if ((k & (q - 1)) == sub)
                    for (int r = 0; r < m; ++r) R[k].fold(part[buf][grp * q + r][k][lane]);
            buf ^= 1;  // the other buffer's sums were read before this round's barrier
        }
        double *fin = reinterpret_cast<double *>(part);  // [group][K][64]
        if (q > 1) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < K; ++k)
                if ((k & (q - 1)) == sub) fin[(grp * K + k) * 64 + lane] = R[k].get();
            __syncthreads();
            if (sub > 0) continue;
        }
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
            const int i = t0 + t * 64 + lane;
            if (i >= n) continue;
            double r[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) r[c] = q > 1 ? fin[(grp * K + 4 * t + c) * 64 + lane] : R[4 * t + c].get();
            if constexpr (MODE == M_F32)
                put_f32(out + base, i, r, (float)G);
            else
                put(out + base, i, r, G);
        }
    }
    if (more && threadIdx.x == 0) {
        const unsigned done = atomicAdd(&counter[1], 1u);
        if (done == gridDim.x - 1) {
            atomicExch(&counter[0], 0u);
            atomicExch(&counter[1], 0u);
        }
    }
}

unsigned split_reduce_blocks(int tcount)
{
    return (unsigned)(((long)tcount * kSumLanes + kBlock - 1) / kBlock);
}

template <int TPL, int MODE>
hipError_t go_f32(const float4 *pm, int n, float eps2, double G, float4 *out, int tbeg, int tcount,
                  const Tune &t, void *partial, bool reduce, hipStream_t s)
{
    const int per_block = (kBlock / 64) * 64 * TPL;
    dim3 grid((tcount + per_block - 1) / per_block, t.jsplit);
    if (t.variant == 1)
        hipLaunchKernelGGL((k_accel_lds_f32<TPL, MODE>), grid, dim3(kBlock), 0, s, pm, n, eps2, G,
                           tbeg, tcount, t.jtile, out, partial);
    else
        hipLaunchKernelGGL((k_accel_f32<TPL, MODE>), grid, dim3(kBlock), 0, s, pm, n, eps2, G, tbeg,
                           tcount, t.jtile, out, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || t.jsplit == 1 || !reduce) return e;
    const unsigned rb = split_reduce_blocks(tcount);
    if constexpr (MODE == M_F32)
        hipLaunchKernelGGL(k_split_reduce_f32, dim3(rb), dim3(kBlock), 0, s,
                           (const float4 *)partial, t.jsplit, tcount, (float)G, out);
    else
        hipLaunchKernelGGL((k_split_reduce<float4, double>), dim3(rb), dim3(kBlock), 0, s,
                           partial, t.jsplit, tcount, G, out);
    return hipGetLastError();
}

template <int TPL>
hipError_t go_f64(const double4 *pm, int n, double eps2, double G, double4 *out, int tbeg,
                  int tcount, const Tune &t, void *partial, bool reduce, hipStream_t s)
{
    const int per_block = (kBlock / 64) * 64 * TPL;
    dim3 grid((tcount + per_block - 1) / per_block, t.jsplit);
    hipLaunchKernelGGL((k_accel_f64<TPL>), grid, dim3(kBlock), 0, s, pm, n, eps2, G, tbeg, tcount,
                       t.jtile, out, (double4 *)partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || t.jsplit == 1 || !reduce) return e;
    const unsigned rb = split_reduce_blocks(tcount);
    hipLaunchKernelGGL((k_split_reduce<double4, double>), dim3(rb), dim3(kBlock), 0, s,
                       partial, t.jsplit, tcount, G, out);
    return hipGetLastError();
}

template <int MODE>
hipError_t by_tpl_f32(const float4 *pm, int n, float eps2, double G, float4 *out, int tbeg,
                      int tcount, const Tune &t, void *partial, bool reduce, hipStream_t s)
{
    switch (t.tpl) {
    case 1: return go_f32<1, MODE>(pm, n, eps2, G, out, tbeg, tcount, t, partial, reduce, s);
    case 2: return go_f32<2, MODE>(pm, n, eps2, G, out, tbeg, tcount, t, partial, reduce, s);
    default: return go_f32<4, MODE>(pm, n, eps2, G, out, tbeg, tcount, t, partial, reduce, s);
    }
}

template <int TPL, int MODE>
hipError_t go_batched_f32(const float4 *pm, const int64_t *off, const int2 *units, int nunits,
                          const float *eps_sys, float eps2, double G, float4 *out, const Tune &t,
                          unsigned *counter, int grid, hipStream_t s)
{
    hipLaunchKernelGGL((k_batched<float, TPL, MODE>), dim3(grid), dim3(kBlock), 0, s, pm, off, units,
                       nunits, eps_sys, eps2, G, t.jtile, out, counter);
    return hipGetLastError();
}

template <int MODE>
hipError_t batched_by_tpl(const float4 *pm, const int64_t *off, const int2 *units, int nunits,
                          const float *eps_sys, float eps2, double G, float4 *out, const Tune &t,
                          unsigned *counter, int grid, hipStream_t s)
{
    switch (t.tpl) {
    case 1: return go_batched_f32<1, MODE>(pm, off, units, nunits, eps_sys, eps2, G, out, t, counter, grid, s);
    case 2: return go_batched_f32<2, MODE>(pm, off, units, nunits, eps_sys, eps2, G, out, t, counter, grid, s);
    default: return go_batched_f32<4, MODE>(pm, off, units, nunits, eps_sys, eps2, G, out, t, counter, grid, s);
    }
}

}  // namespace

bool tune_valid(const Tune &t)
{
    return (t.tpl == 1 || t.tpl == 2 || t.tpl == 4) && t.jsplit >= 1 && t.jsplit <= 32 &&
           t.jtile >= 8 && t.jtile % kUnroll == 0 && t.jtile <= (1 << 24) &&
           (t.variant == 0 || (t.variant == 1 && t.jtile % kLdsTile == 0));
}

int accel_partial_records(int tcount, const Tune &t)
{
    if (t.path == kPathSlice) return 0;
    if (t.path == kPathSym) return sym_plan(tcount).slots();
    return t.jsplit > 1 ? t.jsplit : 0;
}

RecordKind accel_record_kind(int prec, int tcount, const Tune &t)
{
    if (t.path == kPathSym) return sym_plan(tcount).tpl == 2 ? kRecTile : kRecF64;
    return prec == NBODY_F32 ? kRecF32 : kRecF64;
}

size_t accel_partial_bytes(int prec, int tcount, const Tune &t)
{
    const size_t rec = accel_record_kind(prec, tcount, t) == kRecF64 ? sizeof(double4) : sizeof(float4);
    return rec * (size_t)accel_partial_records(tcount, t) * (size_t)tcount;
}

static float eps2_f32(double eps) { return (float)((double)eps * (double)eps); }

namespace {
template <typename T, int MODE, bool STEP>
hipError_t go_slice_t(const void *pm, int n, double G, double eps, void *out, int tbeg, int tcount, SliceStep<T> step,
                      hipStream_t s)
{
    using V = typename SliceRec<T>::V;
    T eps2;
    if constexpr (sizeof(T) == 4)
        eps2 = eps2_f32(eps);
    else
        eps2 = eps * eps;
    hipLaunchKernelGGL((k_accel_slice<T, MODE, STEP>), dim3((tcount + kSliceT - 1) / kSliceT), dim3(kSliceThreads), 0, s,
                       (const V *)pm, n, eps2, G, tbeg, tcount, (V *)out, step);
    return hipGetLastError();
}

template <bool STEP>
hipError_t go_slice(int prec, const void *pm, int n, double G, double eps, void *out, int tbeg, int tcount, void *vel,
                    void *to, double h, double dt, bool close, bool open, double *epart, hipStream_t s)
{
    const SliceStep<double> d{(double4 *)vel, (double4 *)to, h, dt, close, open, epart};
    const SliceStep<float> f{(float4 *)vel, (float4 *)to, (float)h, (float)dt, close, open, epart};
    if (prec == NBODY_F64) return go_slice_t<double, M_F64ACC, STEP>(pm, n, G, eps, out, tbeg, tcount, d, s);
    if (prec == NBODY_F32) return go_slice_t<float, M_F32, STEP>(pm, n, G, eps, out, tbeg, tcount, f, s);
    return go_slice_t<float, M_F64ACC, STEP>(pm, n, G, eps, out, tbeg, tcount, f, s);
}
}  // namespace

int slice_blocks(int n) { return (n + kSliceT - 1) / kSliceT; }

hipError_t launch_slice_step(int prec, const void *pm, int n, double G, double eps, void *acc, void *vel, void *to,
                             double h, double dt, bool close, bool open, double *epart, hipStream_t s)
{
    return go_slice<true>(prec, pm, n, G, eps, acc, 0, n, vel, to, h, dt, close, open, epart, s);
}

hipError_t launch_accel(int prec, const void *pm, int n, double G, double eps, void *out, int tbeg,
                        int tcount, const Tune &t, void *partial, hipStream_t s, bool reduce)
{
    if (t.path == kPathSlice)
        return go_slice<false>(prec, pm, n, G, eps, out, tbeg, tcount, nullptr, nullptr, 0.0, 0.0, false, false, nullptr,
                               s);
    if (t.path == kPathSym) {  // all bodies
        const hipError_t e = launch_sym(pm, n, eps, partial, s);
        if (e != hipSuccess || !reduce) return e;
        const auto kernel = accel_record_kind(prec, n, t) == kRecTile ? k_split_reduce<float4, float>
                                                                      : k_split_reduce<float4, double>;
        hipLaunchKernelGGL(kernel, dim3(split_reduce_blocks(n)), dim3(kBlock), 0, s, (const void *)partial,
                           accel_partial_records(n, t), n, G, (float4 *)out);
        return hipGetLastError();
    }
    if (prec == NBODY_F64) {
        const double4 *p = (const double4 *)pm;
        double4 *o = (double4 *)out;
        const double e2 = eps * eps;
        switch (t.tpl) {
        case 1: return go_f64<1>(p, n, e2, G, o, tbeg, tcount, t, partial, reduce, s);
        default: return go_f64<2>(p, n, e2, G, o, tbeg, tcount, t, partial, reduce, s);
        }
    }
    const float4 *p = (const float4 *)pm;
    float4 *o = (float4 *)out;
    const float e2 = eps2_f32(eps);
    switch (prec) {
    case NBODY_F32: return by_tpl_f32<M_F32>(p, n, e2, G, o, tbeg, tcount, t, partial, reduce, s);
    case NBODY_F32_KAHAN: return by_tpl_f32<M_KAHAN>(p, n, e2, G, o, tbeg, tcount, t, partial, reduce, s);
    default: return by_tpl_f32<M_F64ACC>(p, n, e2, G, o, tbeg, tcount, t, partial, reduce, s);
    }
}

hipError_t launch_batched(int prec, const void *pm, const int64_t *offsets, const int2 *units,
                          int nunits, double G, const float *eps_sys, double eps, void *out,
                          const Tune &t, unsigned *counter, int grid, hipStream_t s)
{
    if (prec == NBODY_F64) {
        const double4 *p = (const double4 *)pm;
        double4 *o = (double4 *)out;
        if (t.tpl == 1)
            hipLaunchKernelGGL((k_batched<double, 1, M_F64ACC>), dim3(grid), dim3(kBlock), 0, s, p, offsets, units,
                               nunits, eps_sys, eps * eps, G, t.jtile, o, counter);
        else
            hipLaunchKernelGGL((k_batched<double, 2, M_F64ACC>), dim3(grid), dim3(kBlock), 0, s, p, offsets, units,
                               nunits, eps_sys, eps * eps, G, t.jtile, o, counter);
        return hipGetLastError();
    }
    const float4 *p = (const float4 *)pm;
    float4 *o = (float4 *)out;
    const float e2 = eps2_f32(eps);
    switch (prec) {
    case NBODY_F32: return batched_by_tpl<M_F32>(p, offsets, units, nunits, eps_sys, e2, G, o, t, counter, grid, s);
    case NBODY_F32_KAHAN: return batched_by_tpl<M_KAHAN>(p, offsets, units, nunits, eps_sys, e2, G, o, t, counter, grid, s);
    default: return batched_by_tpl<M_F64ACC>(p, offsets, units, nunits, eps_sys, e2, G, o, t, counter, grid, s);
    }
}

// ---- static split scratch (nbody_accel_noalloc) -------------------------------
// The split partials of the entry point that allocates nothing live in this
// file-scope device array; every GPU the library runs on holds its own copy
// for the life of the process.  Host code never passes the array's name to a
// kernel: its device address is looked up once per device with
// hipGetSymbolAddress and that address is what the kernels receive.
__device__ __align__(256) static unsigned char g_split_scratch[kStaticScratchBytes];

void *static_split_scratch()
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        set_error("hipGetDevice: %s", hipGetErrorString(e));
        return nullptr;
    }
    if (dev < 0 || dev >= kMaxDevices) {
        set_error("device %d beyond the %d devices the static scratch table covers", dev, kMaxDevices);
        return nullptr;
    }
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_split_scratch));
        if (e != hipSuccess || !p) {
            set_error("hipGetSymbolAddress(static split scratch): %s", hipGetErrorString(e));
            return nullptr;
        }
        addr[dev] = p;
    }
    return addr[dev];
}

}  // namespace nbi
