// Direct-sum force over all bodies, every unordered pair evaluated once
// (gfx950, FP32 pair arithmetic).
//
// The law is the force kernel's (accel.hip).  A pair's separation, its
// reciprocal square root and rho^2 serve both bodies: 19 FP32 instructions
// and one v_rsq_f32 for two interactions, against 2 x (13 + 1).
//
// * The bodies form M blocks of B = 256 TPL, TPL 2 or 4 (the last one may be
//   short).
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
// of a wave.  By the counters it issues 1.45 instructions per clock and CU at
// 2.25 GHz.  The force on 2^20 bodies takes 207 to 235 ms, which differs by the
// GPU, 4.7 to 5.3e12 interactions per second; where it takes 213 the one-sided
// sweep with 8 source splits takes 263.  The reciprocal square roots
// and the DPP moves, which issue alone, stand together at raised wave priority
// (see rsq_prio).  4 targets per lane and 4 waves per SIMD (128 VGPRs, 40 KB of
// LDS) measured best for many tiles, 2 targets and 6 waves for few (kSymWide).
#include <algorithm>
#include <cfloat>
#include <type_traits>

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

// The unmasked two-sided 64 steps, with the registers laid out by hand: an FMA
// whose accumulator lies in the register bank (number mod 4) of a multiplicand
// issues at half the rate, so a pair's dx, dy, dz sit in banks 0, 1, 2, the
// weights and eps2 in bank 3, and the x, y, z sums in banks 1, 2, 0 (the
// compiler's own allocation put a third of the FMAs in conflict: 215.4 ms per
// step of 2^20 bodies against 213.7).  Each step reads the next step's record
// before it uses its own; the DPP moves and the reciprocal square roots, which
// issue alone, stand together at raised priority.  Base registers (multiples
// of 4): T targets (x, y, z, m), S their sums (az, ax, ay, ph), J the sources'
// sums (az, ax, ay, ph), E + 3 eps2, Q the step's record, D temporaries, 8 per
// target: dx, dy, dz, r2 then rho then the weight of the target's sums, rho^2,
// m_j rho, m_i rho, minus the weight of the sources' sums.
#define NB_EACH(LIST, INS) ".irp t," LIST "\n" INS "\n.endr\n"
#define NB_SYM_ADD(S, J, D)                                                                                       \
    "v_add_f32 v[" S "+4*\\t+3], v[" S "+4*\\t+3], v[" D "+8*\\t+5]\n"                                            \
    "v_fmac_f32 v[" S "+4*\\t+1], v[" D "+8*\\t+3], v[" D "+8*\\t]\n"                                             \
    "v_fmac_f32 v[" S "+4*\\t+2], v[" D "+8*\\t+3], v[" D "+8*\\t+1]\n"                                           \
    "v_fmac_f32 v[" S "+4*\\t], v[" D "+8*\\t+3], v[" D "+8*\\t+2]\n"                                             \
    "v_fmac_f32 v[" J "+1], v[" D "+8*\\t+7], v[" D "+8*\\t]\n"                                                    \
    "v_fmac_f32 v[" J "+2], v[" D "+8*\\t+7], v[" D "+8*\\t+1]\n"                                                  \
    "v_fmac_f32 v[" J "], v[" D "+8*\\t+7], v[" D "+8*\\t+2]"
#define NB_SYM_STEP(LIST, LIST1, T, S, J, E, Q, NEXT, D, OFF)                                                     \
    "s_waitcnt lgkmcnt(0)\n"                                                                                      \
    "ds_read_b128 v[" NEXT ":" NEXT "+3], %[addr] offset:" OFF "\n"                                               \
    NB_EACH(LIST, "v_sub_f32 v[" D "+8*\\t], v[" Q "], v[" T "+4*\\t]")                                           \
    NB_EACH(LIST, "v_sub_f32 v[" D "+8*\\t+1], v[" Q "+1], v[" T "+4*\\t+1]")                                     \
    NB_EACH(LIST, "v_sub_f32 v[" D "+8*\\t+2], v[" Q "+2], v[" T "+4*\\t+2]")                                     \
    NB_EACH(LIST, "v_fma_f32 v[" D "+8*\\t+3], v[" D "+8*\\t], v[" D "+8*\\t], v[" E "+3]")                      \
    NB_EACH(LIST, "v_fmac_f32 v[" D "+8*\\t+3], v[" D "+8*\\t+1], v[" D "+8*\\t+1]")                             \
    NB_EACH(LIST, "v_fmac_f32 v[" D "+8*\\t+3], v[" D "+8*\\t+2], v[" D "+8*\\t+2]")                             \
    "s_setprio 1\n"                                                                                               \
    "v_mov_b32_dpp v[" J "+1], v[" J "+1] wave_rol:1 row_mask:0xf bank_mask:0xf\n"                                \
    "v_mov_b32_dpp v[" J "+2], v[" J "+2] wave_rol:1 row_mask:0xf bank_mask:0xf\n"                                \
    "v_mov_b32_dpp v[" J "], v[" J "] wave_rol:1 row_mask:0xf bank_mask:0xf\n"                                    \
    NB_EACH(LIST, "v_rsq_f32 v[" D "+8*\\t+3], v[" D "+8*\\t+3]")                                                 \
    "s_setprio 0\n"                                                                                               \
    NB_EACH(LIST, "v_mul_f32 v[" D "+8*\\t+4], v[" D "+8*\\t+3], v[" D "+8*\\t+3]")                              \
    NB_EACH(LIST, "v_mul_f32 v[" D "+8*\\t+5], v[" Q "+3], v[" D "+8*\\t+3]")                                     \
    NB_EACH(LIST, "v_mul_f32 v[" D "+8*\\t+6], v[" T "+4*\\t+3], v[" D "+8*\\t+3]")                              \
    NB_EACH(LIST, "v_mul_f32 v[" D "+8*\\t+3], v[" D "+8*\\t+5], v[" D "+8*\\t+4]")                              \
    NB_EACH(LIST, "v_mul_f32 v[" D "+8*\\t+7], -v[" D "+8*\\t+6], v[" D "+8*\\t+4]")                             \
    "v_add_f32_dpp v[" J "+3], v[" J "+3], v[" D "+6] wave_rol:1 row_mask:0xf bank_mask:0xf\n"                    \
    NB_EACH("0", NB_SYM_ADD(S, J, D))                                                                             \
    NB_EACH(LIST1, "v_add_f32 v[" J "+3], v[" J "+3], v[" D "+8*\\t+6]\n" NB_SYM_ADD(S, J, D))
// 64 steps, 8 per turn of the loop, the records alternating between Q and P.
#define NB_SYM_LOOP(LIST, LIST1, T, S, J, E, Q, P, D)                                                             \
    "ds_read_b128 v[" Q ":" Q "+3], %[addr]\n"                                                                    \
    ".Lsym%=:\n"                                                                                                  \
    NB_SYM_STEP(LIST, LIST1, T, S, J, E, Q, P, D, "16") NB_SYM_STEP(LIST, LIST1, T, S, J, E, P, Q, D, "32")       \
    NB_SYM_STEP(LIST, LIST1, T, S, J, E, Q, P, D, "48") NB_SYM_STEP(LIST, LIST1, T, S, J, E, P, Q, D, "64")       \
    NB_SYM_STEP(LIST, LIST1, T, S, J, E, Q, P, D, "80") NB_SYM_STEP(LIST, LIST1, T, S, J, E, P, Q, D, "96")       \
    NB_SYM_STEP(LIST, LIST1, T, S, J, E, Q, P, D, "112") NB_SYM_STEP(LIST, LIST1, T, S, J, E, P, Q, D, "128")     \
    "v_add_u32 %[addr], 0x80, %[addr]\n"                                                                          \
    "s_sub_i32 %[cnt], %[cnt], 1\n"                                                                               \
    "s_cmp_lg_u32 %[cnt], 0\n"                                                                                    \
    "s_cbranch_scc1 .Lsym%=\n"                                                                                    \
    "s_waitcnt lgkmcnt(0)\n"                                                                                      \
    "s_nop 1\n"

template <int TPL>
__device__ __forceinline__ void sym_chunk_asm(const float4 *jp, SymTargets<TPL> &T, float eps2, float (&s)[4])
{
    typename std::conditional<TPL == 4, f32x16, f32x8>::type tg, sum;
    f32x4 js = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
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
    if constexpr (TPL == 4)
        asm volatile(NB_SYM_LOOP("0,1,2,3", "1,2,3", "16", "32", "48", "52", "56", "60", "64")
                     : "+{v[32:47]}"(sum), "+{v[48:51]}"(js), [addr] "+&v"(addr), [cnt] "+&s"(cnt)
                     : "{v[16:31]}"(tg), "{v55}"(eps2)
                     : "v56", "v57", "v58", "v59", "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68",
                       "v69", "v70", "v71", "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", "v80", "v81",
                       "v82", "v83", "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91", "v92", "v93", "v94",
                       "v95", "scc", "memory");
    else
        asm volatile(NB_SYM_LOOP("0,1", "1", "16", "24", "32", "36", "40", "44", "48")
                     : "+{v[24:31]}"(sum), "+{v[32:35]}"(js), [addr] "+&v"(addr), [cnt] "+&s"(cnt)
                     : "{v[16:23]}"(tg), "{v39}"(eps2)
                     : "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47", "v48", "v49", "v50", "v51", "v52",
                       "v53", "v54", "v55", "v56", "v57", "v58", "v59", "v60", "v61", "v62", "v63", "scc", "memory");
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
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
        if constexpr (!MASK && BOTH)
            sym_chunk_asm<TPL>(jp, T, eps2, s);
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
__device__ __forceinline__ void sym_store(float4 *p, double4 v, int)
{
    *p = make_float4((float)v.x, (float)v.y, (float)v.z, (float)v.w);
}

// grid.x = M * runs: workgroup (run, I) takes d = d0 + run * len .. + len - 1.
// slots: runs (1 + len) records per body, placed as split records (split_at):
// first the runs' sums of I, then the sums of J per d of the launch.
// REC float4: one launch and runs of one tile, so that no record is added to.
template <int TPL, typename REC>
__global__ __launch_bounds__(kSymThreads) __attribute__((amdgpu_waves_per_eu(TPL == 4 ? 4 : 6))) void k_sym(
    const float4 *__restrict__ src, int n, int M, int d0, int len, int runs, float eps2_in, int add,
    REC *__restrict__ slots)
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
    p.tpl = n < kSymWide ? 2 : 4;
    p.blocks = (int)(((long)n + kSymThreads * p.tpl - 1) / (kSymThreads * p.tpl));
    const int dist = p.blocks / 2 + 1;  // distances 0 .. M/2
    const long room = std::max(2L, (long)(kSymScratch / p.record() / n));  // slots that fit
    // runs of up to 8 tiles: fewer sums of I to store; shorter ones while the
    // tiles are few, so that the launch still fills the chip evenly
    p.len = p.tpl == 2 ? 1 : (int)std::min(std::min(8L, room - 1), std::max(1L, (long)p.blocks / 64));
    const int all = (dist + p.len - 1) / p.len;
    p.runs = (int)std::min((long)all, std::max(1L, room / (p.len + 1)));
    p.launches = (all + p.runs - 1) / p.runs;
    return p;
}

hipError_t launch_sym(const void *pm, int n, double eps, void *slots, hipStream_t s)
{
    const SymPlan p = sym_plan(n);
    const float e2 = (float)(eps * eps);
    if (p.tpl == 2) {
        hipLaunchKernelGGL((k_sym<2, float4>), dim3((unsigned)p.blocks * p.runs), dim3(kSymThreads), 0, s,
                           (const float4 *)pm, n, p.blocks, 0, 1, p.runs, e2, 0, (float4 *)slots);
        return hipGetLastError();
    }
    hipError_t e = hipSuccess;
    for (int l = 0; l < p.launches && e == hipSuccess; ++l) {
        hipLaunchKernelGGL((k_sym<4, double4>), dim3((unsigned)p.blocks * p.runs), dim3(kSymThreads), 0, s,
                           (const float4 *)pm, n, p.blocks, l * p.runs * p.len, p.len, p.runs, e2, l > 0 ? 1 : 0,
                           (double4 *)slots);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace nbi
