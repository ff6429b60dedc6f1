// Direct-sum force over all bodies, every unordered pair evaluated once
// (gfx950, FP32 pair arithmetic).
//
// The law is the force kernel's (accel.hip).  A pair's separation, its
// reciprocal square root and rho^2 serve both bodies: 19 FP32 instructions
// and one v_rsq_f32 for two interactions, against 2 x (13 + 1).
//
// * The bodies form M blocks of B = 256 TPL (the last one may be short).
//   Every pair of blocks (I, J = I + d mod M), d = 0 .. M/2, is one tile (for
//   even M and d = M/2 only the first half of the I).  A workgroup of 4 waves
//   takes block I and a run of consecutive d.
// * In a tile each wave holds 64 TPL targets of I in registers and meets the
//   4 sub-blocks of J one per phase, in rotated order, so that two waves never
//   work on the same sources; a barrier ends the phase.
// * Within a sub-block, 64 sources at a time: at step k lane l meets source
//   (l + k) mod 64, whose record it reads from the wave's own LDS copy
//   (stored twice, so the address is the lane's plus a constant).  The
//   source's sums follow it from lane to lane with one DPP wave rotation per
//   step and component, and are added to the workgroup's FP64 sums of J in LDS
//   after the 64 steps (64 TPL FP32 terms per partial sum).  The targets'
//   FP32 partials (64 TPL sources) are folded into FP64 at the end of a phase.
// * The diagonal tile (d = 0) takes phase 0 (a wave's own targets) one-sided
//   with the self pair masked, and of the others each pair of sub-blocks once.
// * A tile's sums of J go to slot (d - first d of the launch), a run's sums of
//   I to a slot of its run: within a launch every slot of a body is written by
//   exactly one workgroup, and later launches add to it in launch order.  The
//   split reduction (accel.hip, step.hip) then adds a body's slots in order,
//   so results do not depend on scheduling.
//
// What bounds it: FP32 instruction issue.  A step of 4 targets is 80
// instructions, 4 of them v_rsq_f32, plus 4 DPP moves and one LDS read, which
// at the rates measured in isolation (1.75 instructions per clock and CU, 2.1
// clocks per v_rsq_f32, 1.1 per DPP move) take 56 clocks for 512 interactions
// of a wave; it runs at 60 (1.41 instructions per clock, 2.36 GHz).  A step of
// 2^20 bodies takes 212.8 ms, 5.17e12 interactions per second, against 256.6
// for the one-sided sweep with 8 source splits.  The reciprocal square roots and the DPP
// moves, which issue alone, stand together at raised wave priority (see
// rsq_prio).  TPL = 4 and 4 waves per SIMD (99 VGPRs, 40 KB of LDS) measured
// best: with 2 targets per lane the rotation costs twice as much per pair.
#include <algorithm>
#include <cfloat>

#include "internal.h"

namespace nbi {
namespace {

constexpr int kSymWaves = 4;
constexpr int kSymThreads = 64 * kSymWaves;

// Value of the next lane (lane 63: of lane 0).
__device__ __forceinline__ float next_lane(float x)
{
    constexpr int kWaveRol1 = 0x134;
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), kWaveRol1, 0xf, 0xf, false));
}

template <int TPL>
struct SymTargets {
    float x[TPL], y[TPL], z[TPL], m[TPL];
    float ax[TPL], ay[TPL], az[TPL], ph[TPL];
    int i0;  // target t of a lane is body i0 + 64 t + lane
};

// Record of body i.  The places past n in the last block hold massless bodies
// far away: with eps2 > 0 (a normal number) every pair with one adds exactly
// zero to the other body.  A smaller eps2 masks them instead, since a body
// exactly there would meet an infinite rho.
__device__ __forceinline__ float4 sym_record(const float4 *__restrict__ src, int i, int n)
{
    const float4 p = src[min(i, n - 1)];
    return i < n ? p : make_float4(1e18f, 1e18f, 1e18f, 0.0f);
}

// 64 sources [j0, j0 + 64) (records in jp, twice) against the wave's targets.
// BOTH: also the sources' sums s (ax, ay, az, sum m rho of source j0 + lane);
// else the sources are the wave's own targets number `self` of each lane, and
// the self pairs, all in step 0 of that target, count nothing.
// MASK: nor do pairs with a body past n.
template <int TPL, bool MASK, bool BOTH>
__device__ __forceinline__ void sym_chunk(const float4 *jp, int j0, int n, int self, SymTargets<TPL> &T, float eps2,
                                          float (&s)[4])
{
    constexpr int kUnr = MASK ? 2 : 8;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int c = 0; c < 4; ++c) s[c] = 0.0f;
#pragma unroll 1
    for (int k0 = 0; k0 < 64; k0 += kUnr) {
#pragma unroll
        for (int u = 0; u < kUnr; ++u) {
            const float4 q = jp[lane + k0 + u];
            float dx[TPL], dy[TPL], dz[TPL], rho[TPL];
#pragma unroll
            for (int t = 0; t < TPL; ++t) {
                dx[t] = q.x - T.x[t];
                dy[t] = q.y - T.y[t];
                dz[t] = q.z - T.z[t];
                rho[t] = __builtin_fmaf(dz[t], dz[t], __builtin_fmaf(dy[t], dy[t], __builtin_fmaf(dx[t], dx[t], eps2)));
            }
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int t = 0; t < TPL; ++t) rho[t] = __builtin_amdgcn_rsqf(rho[t]);
            if constexpr (BOTH) {
#pragma unroll
                for (int c = 0; c < 4; ++c) s[c] = next_lane(s[c]);
            }
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (MASK) {
                const int j = j0 + ((lane + k0 + u) & 63);
#pragma unroll
                for (int t = 0; t < TPL; ++t)
                    if (j >= n || T.i0 + 64 * t + lane >= n) rho[t] = 0.0f;
            }
            if constexpr (!BOTH) {
                if (u == 0 && k0 == 0) {
#pragma unroll
                    for (int t = 0; t < TPL; ++t)
                        if (t == self) rho[t] = 0.0f;
                }
            }
#pragma unroll
            for (int t = 0; t < TPL; ++t) {
                const float r2 = rho[t] * rho[t];
                const float mj = q.w * rho[t];
                const float si = mj * r2;
                T.ph[t] += mj;
                T.ax[t] = __builtin_fmaf(si, dx[t], T.ax[t]);
                T.ay[t] = __builtin_fmaf(si, dy[t], T.ay[t]);
                T.az[t] = __builtin_fmaf(si, dz[t], T.az[t]);
                if constexpr (BOTH) {
                    const float mi = T.m[t] * rho[t];
                    const float sj = mi * r2;
                    s[3] += mi;
                    s[0] = __builtin_fmaf(-sj, dx[t], s[0]);
                    s[1] = __builtin_fmaf(-sj, dy[t], s[1]);
                    s[2] = __builtin_fmaf(-sj, dz[t], s[2]);
                }
            }
        }
    }
    if constexpr (BOTH) {  // after 64 steps lane l holds source l - 1: one more rotation
#pragma unroll
        for (int c = 0; c < 4; ++c) s[c] = next_lane(s[c]);
    }
}

// The unmasked two-sided 64 steps of 4 targets, with the registers laid out
// by hand: an FMA whose accumulator lies in the register bank (number mod 4)
// of a multiplicand issues at half the rate, so dx, dy, dz sit in banks 0, 1,
// 2, the weights and eps2 in bank 3, and the x, y, z sums in banks 1, 2, 0
// (the compiler's own allocation put a third of the FMAs in conflict: 215.4 ms
// per step of 2^20 bodies against 213.7).  Each step reads the next step's
// record before it uses its own; the DPP moves and the reciprocal square roots,
// which issue alone, stand together at raised priority.
//   v16-31 targets (x, y, z, m) x 4     v32-47 their sums (az, ax, ay, ph) x 4
//   v48-51 sources' sums (az, ax, ay, ph)      v55 eps2
//   v56-59, v60-63 source records       v64-95 temporaries, 8 per target
#define NB_SYM_STEP(NEXT, OFF, QX, QY, QZ, QM) \
    "s_waitcnt lgkmcnt(0)\n" \
    "ds_read_b128 v[" NEXT "], %[addr] offset:" OFF "\n" \
    "v_sub_f32 v64, v" QX ", v16\n" \
    "v_sub_f32 v72, v" QX ", v20\n" \
    "v_sub_f32 v80, v" QX ", v24\n" \
    "v_sub_f32 v88, v" QX ", v28\n" \
    "v_sub_f32 v65, v" QY ", v17\n" \
    "v_sub_f32 v73, v" QY ", v21\n" \
    "v_sub_f32 v81, v" QY ", v25\n" \
    "v_sub_f32 v89, v" QY ", v29\n" \
    "v_sub_f32 v66, v" QZ ", v18\n" \
    "v_sub_f32 v74, v" QZ ", v22\n" \
    "v_sub_f32 v82, v" QZ ", v26\n" \
    "v_sub_f32 v90, v" QZ ", v30\n" \
    "v_fma_f32 v67, v64, v64, v55\n" \
    "v_fma_f32 v75, v72, v72, v55\n" \
    "v_fma_f32 v83, v80, v80, v55\n" \
    "v_fma_f32 v91, v88, v88, v55\n" \
    "v_fmac_f32 v67, v65, v65\n" \
    "v_fmac_f32 v75, v73, v73\n" \
    "v_fmac_f32 v83, v81, v81\n" \
    "v_fmac_f32 v91, v89, v89\n" \
    "v_fmac_f32 v67, v66, v66\n" \
    "v_fmac_f32 v75, v74, v74\n" \
    "v_fmac_f32 v83, v82, v82\n" \
    "v_fmac_f32 v91, v90, v90\n" \
    "s_setprio 1\n" \
    "v_mov_b32_dpp v49, v49 wave_rol:1 row_mask:0xf bank_mask:0xf\n" \
    "v_mov_b32_dpp v50, v50 wave_rol:1 row_mask:0xf bank_mask:0xf\n" \
    "v_mov_b32_dpp v48, v48 wave_rol:1 row_mask:0xf bank_mask:0xf\n" \
    "v_rsq_f32 v67, v67\n" \
    "v_rsq_f32 v75, v75\n" \
    "v_rsq_f32 v83, v83\n" \
    "v_rsq_f32 v91, v91\n" \
    "s_setprio 0\n" \
    "v_mul_f32 v68, v67, v67\n" \
    "v_mul_f32 v76, v75, v75\n" \
    "v_mul_f32 v84, v83, v83\n" \
    "v_mul_f32 v92, v91, v91\n" \
    "v_mul_f32 v69, v" QM ", v67\n" \
    "v_mul_f32 v77, v" QM ", v75\n" \
    "v_mul_f32 v85, v" QM ", v83\n" \
    "v_mul_f32 v93, v" QM ", v91\n" \
    "v_mul_f32 v70, v19, v67\n" \
    "v_mul_f32 v78, v23, v75\n" \
    "v_mul_f32 v86, v27, v83\n" \
    "v_mul_f32 v94, v31, v91\n" \
    "v_mul_f32 v67, v69, v68\n" \
    "v_mul_f32 v75, v77, v76\n" \
    "v_mul_f32 v83, v85, v84\n" \
    "v_mul_f32 v91, v93, v92\n" \
    "v_mul_f32 v71, -v70, v68\n" \
    "v_mul_f32 v79, -v78, v76\n" \
    "v_mul_f32 v87, -v86, v84\n" \
    "v_mul_f32 v95, -v94, v92\n" \
    "v_add_f32_dpp v51, v51, v70 wave_rol:1 row_mask:0xf bank_mask:0xf\n" \
    "v_add_f32 v35, v35, v69\n" \
    "v_fmac_f32 v33, v67, v64\n" \
    "v_fmac_f32 v34, v67, v65\n" \
    "v_fmac_f32 v32, v67, v66\n" \
    "v_fmac_f32 v49, v71, v64\n" \
    "v_fmac_f32 v50, v71, v65\n" \
    "v_fmac_f32 v48, v71, v66\n" \
    "v_add_f32 v51, v51, v78\n" \
    "v_add_f32 v39, v39, v77\n" \
    "v_fmac_f32 v37, v75, v72\n" \
    "v_fmac_f32 v38, v75, v73\n" \
    "v_fmac_f32 v36, v75, v74\n" \
    "v_fmac_f32 v49, v79, v72\n" \
    "v_fmac_f32 v50, v79, v73\n" \
    "v_fmac_f32 v48, v79, v74\n" \
    "v_add_f32 v51, v51, v86\n" \
    "v_add_f32 v43, v43, v85\n" \
    "v_fmac_f32 v41, v83, v80\n" \
    "v_fmac_f32 v42, v83, v81\n" \
    "v_fmac_f32 v40, v83, v82\n" \
    "v_fmac_f32 v49, v87, v80\n" \
    "v_fmac_f32 v50, v87, v81\n" \
    "v_fmac_f32 v48, v87, v82\n" \
    "v_add_f32 v51, v51, v94\n" \
    "v_add_f32 v47, v47, v93\n" \
    "v_fmac_f32 v45, v91, v88\n" \
    "v_fmac_f32 v46, v91, v89\n" \
    "v_fmac_f32 v44, v91, v90\n" \
    "v_fmac_f32 v49, v95, v88\n" \
    "v_fmac_f32 v50, v95, v89\n" \
    "v_fmac_f32 v48, v95, v90\n"

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ void sym_chunk4(const float4 *jp, SymTargets<4> &T, float eps2,
                                           float (&s)[4])
{
    f32x16 tg, sum;
    f32x4 js = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        tg[4 * t] = T.x[t];
        tg[4 * t + 1] = T.y[t];
        tg[4 * t + 2] = T.z[t];
        tg[4 * t + 3] = T.m[t];
        sum[4 * t] = T.az[t];
        sum[4 * t + 1] = T.ax[t];
        sum[4 * t + 2] = T.ay[t];
        sum[4 * t + 3] = T.ph[t];
    }
    unsigned addr = (unsigned)(size_t)(__attribute__((address_space(3))) const float4 *)(jp + (threadIdx.x & 63));
    int cnt = 8;
    asm volatile("ds_read_b128 v[56:59], %[addr]\n"
                 ".Lsym%=:\n"
                 NB_SYM_STEP("60:63", "16", "56", "57", "58", "59")
                 NB_SYM_STEP("56:59", "32", "60", "61", "62", "63")
                 NB_SYM_STEP("60:63", "48", "56", "57", "58", "59")
                 NB_SYM_STEP("56:59", "64", "60", "61", "62", "63")
                 NB_SYM_STEP("60:63", "80", "56", "57", "58", "59")
                 NB_SYM_STEP("56:59", "96", "60", "61", "62", "63")
                 NB_SYM_STEP("60:63", "112", "56", "57", "58", "59")
                 NB_SYM_STEP("56:59", "128", "60", "61", "62", "63")
                 "v_add_u32 %[addr], 0x80, %[addr]\n"
                 "s_sub_i32 %[cnt], %[cnt], 1\n"
                 "s_cmp_lg_u32 %[cnt], 0\n"
                 "s_cbranch_scc1 .Lsym%=\n"
                 "s_waitcnt lgkmcnt(0)\n"
                 "s_nop 1\n"
                 : "+{v[32:47]}"(sum), "+{v[48:51]}"(js), [addr] "+v"(addr), [cnt] "+s"(cnt)
                 : "{v[16:31]}"(tg), "{v55}"(eps2)
                 : "v56", "v57", "v58", "v59", "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69",
                   "v70", "v71", "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", "v80", "v81", "v82", "v83",
                   "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95", "scc", "memory");
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        T.az[t] = sum[4 * t];
        T.ax[t] = sum[4 * t + 1];
        T.ay[t] = sum[4 * t + 2];
        T.ph[t] = sum[4 * t + 3];
    }
    s[0] = next_lane(js[1]);
    s[1] = next_lane(js[2]);
    s[2] = next_lane(js[0]);
    s[3] = next_lane(js[3]);
}

// One wave's phase: its targets against the sub-block of 64 TPL sources from
// j0; the sources' sums are added to jacc (their entries of the block).  q
// holds the record of source j0 + lane and is left with that of jnext + lane,
// read a chunk ahead.
template <int TPL, bool MASK, bool BOTH>
__device__ __forceinline__ void sym_phase(const float4 *__restrict__ src, int n, int j0, int jnext, float4 &q,
                                          float4 *jp, SymTargets<TPL> &T, float eps2, double4 *jacc,
                                          double (&R)[TPL][4])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int t = 0; t < TPL; ++t) T.ax[t] = T.ay[t] = T.az[t] = T.ph[t] = 0.0f;
    for (int c = 0; c < TPL; ++c) {
        const int jc = j0 + 64 * c;
        jp[lane] = q;
        jp[lane + 64] = q;
        q = sym_record(src, (c + 1 < TPL ? jc + 64 : jnext) + lane, n);
        __builtin_amdgcn_wave_barrier();
        float s[4];
        if constexpr (TPL == 4 && !MASK && BOTH)
            sym_chunk4(jp, T, eps2, s);
        else
            sym_chunk<TPL, MASK, BOTH>(jp, jc, n, c, T, eps2, s);
        __builtin_amdgcn_wave_barrier();
        if constexpr (BOTH) {
            double4 o = jacc[64 * c + lane];
            o.x += s[0];
            o.y += s[1];
            o.z += s[2];
            o.w += s[3];
            jacc[64 * c + lane] = o;
        }
    }
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        R[t][0] += T.ax[t];
        R[t][1] += T.ay[t];
        R[t][2] += T.az[t];
        R[t][3] += T.ph[t];
    }
}

__device__ __forceinline__ void sym_store(double4 *p, double4 v, int add)
{
    if (add) {
        const double4 o = *p;
        v.x += o.x;
        v.y += o.y;
        v.z += o.z;
        v.w += o.w;
    }
    *p = v;
}

// grid.x = M * runs: workgroup (run, I) takes d = d0 + run * len .. + len - 1.
// slots: runs (1 + len) records per body, placed as split records (split_at):
// first the runs' sums of I, then the sums of J per d of the launch.
template <int TPL>
__global__ __launch_bounds__(kSymThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_sym(
    const float4 *__restrict__ src, int n, int M, int d0, int len, int runs, float eps2_in, int add,
    double4 *__restrict__ slots)
{
    constexpr int W = 64 * TPL, B = kSymWaves * W;
    __shared__ double4 jacc[B];
    __shared__ float4 jp[kSymWaves][128];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int run = blockIdx.x / M, I = blockIdx.x % M;
    const int total = runs * (1 + len);  // slots per body
    const float eps2 = lane_copy(eps2_in);
    SymTargets<TPL> T;
    double R[TPL][4];
    T.i0 = I * B + w * W;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const float4 p = sym_record(src, T.i0 + 64 * t + lane, n);
        T.x[t] = p.x;
        T.y[t] = p.y;
        T.z[t] = p.z;
        T.m[t] = p.w;
#pragma unroll
        for (int c = 0; c < 4; ++c) R[t][c] = 0.0;
    }
    for (int e = run * len; e < (run + 1) * len; ++e) {
        const int d = d0 + e;
        // past the last distance, or the second half of the opposite one: nothing to add, but a first launch
        // has to set its slots
        const bool none = 2 * d > M || (2 * d == M && d > 0 && I >= M / 2);
        if (none && add) continue;
        const int J = (I + d) % M;
        for (int k = threadIdx.x; k < B; k += kSymThreads) jacc[k] = make_double4(0.0, 0.0, 0.0, 0.0);
        __syncthreads();
        if (!none) {
            const bool mask = eps2_in < FLT_MIN && (max(I, J) + 1L) * B > n;
            // the diagonal tile ends with the phase that meets the opposite sub-block, from one side
            const int phases = d == 0 ? kSymWaves / 2 + 1 : kSymWaves;
            float4 q = sym_record(src, J * B + w * W + lane, n);
            for (int p = 0; p < phases; ++p) {
                const int sb = (w + p) % kSymWaves;
                const int j0 = J * B + sb * W, jn = J * B + (w + p + 1) % kSymWaves * W;
                double4 *ja = jacc + sb * W;
                if (d == 0 && p == 0) {
                    if (mask)
                        sym_phase<TPL, true, false>(src, n, j0, jn, q, jp[w], T, eps2, ja, R);
                    else
                        sym_phase<TPL, false, false>(src, n, j0, jn, q, jp[w], T, eps2, ja, R);
                } else if (d > 0 || p < kSymWaves / 2 || w < kSymWaves / 2) {
                    if (mask)
                        sym_phase<TPL, true, true>(src, n, j0, jn, q, jp[w], T, eps2, ja, R);
                    else
                        sym_phase<TPL, false, true>(src, n, j0, jn, q, jp[w], T, eps2, ja, R);
                }
                __syncthreads();
            }
        }
        for (int k = threadIdx.x; k < B; k += kSymThreads) {
            const long j = (long)J * B + k;
            if (j < n) sym_store(slots + split_at(j, runs + e, total, n), jacc[k], add);
        }
        __syncthreads();  // jacc is cleared for the next tile
    }
#pragma unroll
    for (int t = 0; t < TPL; ++t)
        if (const int i = T.i0 + 64 * t + lane; i < n)
            sym_store(slots + split_at(i, run, total, n), make_double4(R[t][0], R[t][1], R[t][2], R[t][3]), add);
}

}  // namespace

SymPlan sym_plan(int n)
{
    SymPlan p;
    p.blocks = (int)(((long)n + kSymBlock - 1) / kSymBlock);
    const int dist = p.blocks / 2 + 1;  // distances 0 .. M/2
    const long room = std::max(2L, (long)(kSymScratch / sizeof(double4) / n));  // slots that fit
    // runs of up to 8 tiles: fewer sums of I to store; shorter ones while the
    // tiles are few, so that the launch still fills the chip evenly
    p.len = (int)std::min(std::min(8L, room - 1), std::max(1L, (long)p.blocks / 64));
    const int all = (dist + p.len - 1) / p.len;
    p.runs = (int)std::min((long)all, std::max(1L, room / (p.len + 1)));
    p.launches = (all + p.runs - 1) / p.runs;
    return p;
}

hipError_t launch_sym(const void *pm, int n, double eps, void *slots, hipStream_t s)
{
    const SymPlan p = sym_plan(n);
    const float e2 = (float)(eps * eps);
    hipError_t e = hipSuccess;
    for (int l = 0; l < p.launches && e == hipSuccess; ++l) {
        hipLaunchKernelGGL(k_sym<kSymBlock / kSymThreads>, dim3((unsigned)p.blocks * p.runs), dim3(kSymThreads), 0, s,
                           (const float4 *)pm, n, p.blocks, l * p.runs * p.len, p.len, p.runs, e2, l > 0 ? 1 : 0,
                           (double4 *)slots);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace nbi
