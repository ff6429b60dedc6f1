// Elementwise kernels around the force evaluation: the leapfrog kicks and
// drift (the paper's Move_bodies, Section IV.B pseudo-code, read as
// kick-drift-kick with one force evaluation per step), the FP64 energy
// diagnostics, and record permutations for the ORB order.
//
// All are HBM-bound streams over 16- or 32-byte records: one record per lane,
// coalesced 16-byte vector loads and stores, workgroups of 256 lanes.
#include <type_traits>

#include "internal.h"
#include "pair.h"

namespace nbi {
namespace {

// Fixed-order sum over kBlock slots of two doubles, slot k set by one thread
// of the workgroup (owner); thread 0 holds the result.
__device__ __forceinline__ void block_sum2(double &a, double &b, int slot, bool owner)
{
    __shared__ double sa[kBlock], sb[kBlock];
    if (owner) {
        sa[slot] = a;
        sb[slot] = b;
    }
    __syncthreads();
    // rows of kEnergyRow first, then the rows: the fused small-problem step
    // leaves its rows' sums, and both give the same bits
    const int t = threadIdx.x, row = t % kEnergyRow;
#pragma unroll
    for (int w = kEnergyRow / 2; w > 0; w >>= 1) {
        if (t < kBlock && row < w) {
            sa[t] += sa[t + w];
            sb[t] += sb[t + w];
        }
        __syncthreads();
    }
    for (int w = kBlock / 2; w >= kEnergyRow; w >>= 1) {
        if (t < w && row == 0) {
            sa[t] += sa[t + w];
            sb[t] += sb[t + w];
        }
        __syncthreads();
    }
    a = sa[0];
    b = sb[0];
}

template <typename V, typename S>
__device__ __forceinline__ void step_one(V *__restrict__ pm, V *__restrict__ vel, int i, const V a,
                                         S h, S dt, int close, int open, bool energy, double &ek,
                                         double &eu)
{
    V x = pm[i];
    step_body(x, vel[i], a, h, dt, close, open, energy, ek, eu);
    if (open) pm[i] = x;
}

template <typename V, typename S>
__global__ __launch_bounds__(kBlock) void k_step(V *__restrict__ pm, V *__restrict__ vel,
                                                 const V *__restrict__ acc, int n, S h, S dt,
                                                 int close, int open, double *__restrict__ epart)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    double ek = 0.0, eu = 0.0;
    if (i < n) step_one(pm, vel, i, acc[i], h, dt, close, open, epart != nullptr, ek, eu);
    if (epart) {
        block_sum2(ek, eu, threadIdx.x, true);
        if (threadIdx.x == 0) {
            epart[2 * blockIdx.x] = ek;
            epart[2 * blockIdx.x + 1] = eu;
        }
    }
}

// The force kernel's source-split reduction and the step in one pass: the
// js partial records of body i are summed in split order (4 lanes per body, see
// split_sum) and scaled exactly as the stand-alone reduction does (R = the type
// of the sums, GT = the type G is applied in); the first of the 4 lanes stores
// the record to acc and applies the kick, drift and energy partials to the same
// value.  Results equal reduce-then-step bit for bit; one launch and one pass
// over acc fewer.  A workgroup holds kBlock bodies, as k_step's.
constexpr int kReduceThreads = kBlock * kSumLanes;
template <typename V, typename S, typename P, typename R, typename GT>
__global__ __launch_bounds__(kReduceThreads) void k_reduce_step(const P *__restrict__ partial, int js, GT G,
                                                                V *__restrict__ pm, V *__restrict__ vel,
                                                                V *__restrict__ acc, int n, S h, S dt, int close,
                                                                int open, double *__restrict__ epart)
{
    using E = typename std::conditional<sizeof(V) == 16, float, double>::type;
    using PE = typename std::conditional<sizeof(P) == 16, float, double>::type;
    const int slot = threadIdx.x / kSumLanes;
    const int i = blockIdx.x * kBlock + slot;
    const bool owner = threadIdx.x % kSumLanes == 0;
    double ek = 0.0, eu = 0.0;
    R r[4];
    split_sum<kSumLanes>(reinterpret_cast<const PE *>(partial), js, n, min(i, n - 1), r);
    if (owner && i < n) {
        V a;
        a.x = (E)(G * r[0]);
        a.y = (E)(G * r[1]);
        a.z = (E)(G * r[2]);
        a.w = (E)(-G * r[3]);
        acc[i] = a;
        step_one(pm, vel, i, a, h, dt, close, open, epart != nullptr, ek, eu);
    }
    if (epart) {
        block_sum2(ek, eu, slot, owner);
        if (threadIdx.x == 0) {
            epart[2 * blockIdx.x] = ek;
            epart[2 * blockIdx.x + 1] = eu;
        }
    }
}

// One workgroup per state: each lane sums a strided subset of the block
// partials in order, then a fixed-order tree.  With ROWS a state's `parts` are
// row sums, of which a block has kBlock / kEnergyRow.
template <bool ROWS>
__global__ __launch_bounds__(kBlock) void k_energy_final(const double *__restrict__ epart,
                                                         int parts, double *__restrict__ out)
{
    double a = 0.0, b = 0.0;
    epart += 2 * (size_t)parts * blockIdx.x;
    out += 2 * blockIdx.x;
    constexpr int R = ROWS ? kBlock / kEnergyRow : 1;
    for (int k = threadIdx.x; k * R < parts; k += kBlock) {
        double x[R], y[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int p = k * R + j;
            x[j] = p < parts ? epart[2 * p] : 0.0;
            y[j] = p < parts ? epart[2 * p + 1] : 0.0;
        }
#pragma unroll
        for (int w = R / 2; w > 0; w >>= 1)
#pragma unroll
            for (int j = 0; j < R; ++j)
                if (j < w) {
                    x[j] += x[j + w];
                    y[j] += y[j + w];
                }
        a += x[0];
        b += y[0];
    }
    block_sum2(a, b, threadIdx.x, true);
    if (threadIdx.x == 0) {
        out[0] = a;
        out[1] = b;
    }
}

template <typename R>
__global__ __launch_bounds__(kBlock) void k_permute(const R *__restrict__ src, R *__restrict__ dst,
                                                    const int32_t *__restrict__ perm, int n,
                                                    int inverse)
{
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p >= n) return;
    const int q = perm[p];
    if ((unsigned)q >= (unsigned)n) return;  // not a permutation entry: no access
    if (inverse)
        dst[q] = src[p];
    else
        dst[p] = src[q];
}

__global__ __launch_bounds__(kBlock) void k_copy16(const float4 *__restrict__ src,
                                                   float4 *__restrict__ dst, size_t nrec)
{
    const size_t k = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (k < nrec) dst[k] = src[k];
}

__global__ __launch_bounds__(kBlock) void k_zero4(uint32_t *__restrict__ p, size_t nwords)
{
    const size_t k = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (k < nwords) p[k] = 0u;
}

}  // namespace

// Zero fill as a kernel (no memset node in captured graphs); bytes must be a
// multiple of 4.
hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s)
{
    const size_t nw = bytes / 4;
    const size_t nb = (nw + kBlock - 1) / kBlock;
    if (nw) hipLaunchKernelGGL(k_zero4, dim3((unsigned)nb), dim3(kBlock), 0, s, (uint32_t *)p, nw);
    return hipGetLastError();
}

int step_blocks(int n) { return (n + kBlock - 1) / kBlock; }

hipError_t launch_step(int prec, void *pm, void *vel, const void *acc, int n, double h, double dt,
                       bool close, bool open, double *epart, int *eblocks, hipStream_t s)
{
    const int nb = step_blocks(n);
    if (eblocks) *eblocks = nb;
    if (prec == NBODY_F64)
        hipLaunchKernelGGL((k_step<double4, double>), dim3(nb), dim3(kBlock), 0, s, (double4 *)pm,
                           (double4 *)vel, (const double4 *)acc, n, h, dt, (int)close, (int)open,
                           epart);
    else
        hipLaunchKernelGGL((k_step<float4, float>), dim3(nb), dim3(kBlock), 0, s, (float4 *)pm,
                           (float4 *)vel, (const float4 *)acc, n, (float)h, (float)dt, (int)close,
                           (int)open, epart);
    return hipGetLastError();
}

hipError_t launch_reduce_step(int prec, RecordKind kind, const void *partial, int js, double G, void *pm, void *vel,
                              void *acc, int n, double h, double dt, bool close, bool open,
                              double *epart, int *eblocks, hipStream_t s)
{
    const int nb = step_blocks(n);
    if (eblocks) *eblocks = nb;
    if (prec == NBODY_F64)
        hipLaunchKernelGGL((k_reduce_step<double4, double, double4, double, double>), dim3(nb),
                           dim3(kReduceThreads), 0, s, (const double4 *)partial, js, G, (double4 *)pm,
                           (double4 *)vel, (double4 *)acc, n, h, dt, (int)close, (int)open, epart);
    else if (kind == kRecTile)
        hipLaunchKernelGGL((k_reduce_step<float4, float, float4, double, double>), dim3(nb),
                           dim3(kReduceThreads), 0, s, (const float4 *)partial, js, G, (float4 *)pm,
                           (float4 *)vel, (float4 *)acc, n, (float)h, (float)dt, (int)close,
                           (int)open, epart);
    else if (kind == kRecF32)
        hipLaunchKernelGGL((k_reduce_step<float4, float, float4, float, float>), dim3(nb),
                           dim3(kReduceThreads), 0, s, (const float4 *)partial, js, (float)G, (float4 *)pm,
                           (float4 *)vel, (float4 *)acc, n, (float)h, (float)dt, (int)close,
                           (int)open, epart);
    else
        hipLaunchKernelGGL((k_reduce_step<float4, float, double4, double, double>), dim3(nb),
                           dim3(kReduceThreads), 0, s, (const double4 *)partial, js, G, (float4 *)pm,
                           (float4 *)vel, (float4 *)acc, n, (float)h, (float)dt, (int)close,
                           (int)open, epart);
    return hipGetLastError();
}

hipError_t launch_energy_final(const double *epart, int parts, bool rows, int states, double *out, hipStream_t s)
{
    if (rows)
        hipLaunchKernelGGL(k_energy_final<true>, dim3(states), dim3(kBlock), 0, s, epart, parts, out);
    else
        hipLaunchKernelGGL(k_energy_final<false>, dim3(states), dim3(kBlock), 0, s, epart, parts, out);
    return hipGetLastError();
}

hipError_t launch_permute(const void *src, void *dst, const int32_t *perm, int n, int rec_bytes,
                          bool inverse, hipStream_t s)
{
    const int nb = (n + kBlock - 1) / kBlock;
    if (rec_bytes == 16)
        hipLaunchKernelGGL((k_permute<float4>), dim3(nb), dim3(kBlock), 0, s, (const float4 *)src,
                           (float4 *)dst, perm, n, (int)inverse);
    else
        hipLaunchKernelGGL((k_permute<double4>), dim3(nb), dim3(kBlock), 0, s,
                           (const double4 *)src, (double4 *)dst, perm, n, (int)inverse);
    return hipGetLastError();
}

// Device-to-device copy as a kernel (16-byte records), so that it can sit in
// captured graphs without a memcpy node.
hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s)
{
    const size_t nrec = bytes / 16;
    const size_t nb = (nrec + kBlock - 1) / kBlock;
    if (nrec) hipLaunchKernelGGL(k_copy16, dim3((unsigned)nb), dim3(kBlock), 0, s, (const float4 *)src, (float4 *)dst, nrec);
    return hipGetLastError();
}

}  // namespace nbi
