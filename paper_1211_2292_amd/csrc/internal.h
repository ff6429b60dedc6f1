// Internal declarations of the gfx950 n-body library (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "nbody.h"

namespace nbi {

// Kernel shape of the force sweep.
//   tpl    targets held per lane (1, 2 or 4): a wave owns 64*tpl targets
//   jsplit number of independent source ranges per target (pinned and tuned
//          shapes 1..32, the library's own up to 256); each range is a
//          separate workgroup row, reduced in fixed order after
//   jtile  sources per partial sum (multiple of 8); the partials are folded
//          into the running sum by the precision mode
//   variant 0: sources through scalar loads (SGPR operands);
//           1: sources staged in LDS (VGPR operands; FP32 force kernel only,
//              jtile a multiple of 256).  Both give identical results.
struct Tune {
    int tpl = 2;
    int jsplit = 1;
    int jtile = 512;
    int variant = 0;
    // Which force kernels run the shape: the sweep above (every pinned or
    // measured shape), or one of the library's own choices for a whole call.
    int path = 0;
};
enum { kPathSweep = 0, kPathSlice = 1, kPathSym = 2 };

constexpr int kBlock = 256;  // threads per workgroup: four independent waves
constexpr int kUnroll = 8;   // sources per unrolled step of the sweep

// Returns x in a vector register that the compiler treats as per-lane, so a
// loop invariant such as eps^2 is not kept as a scalar operand of the pair
// arithmetic: on gfx950 an FP32 VALU instruction that reads a scalar register
// issues at roughly half the rate of its all-vector-register form.
__device__ __forceinline__ float lane_copy(float x)
{
    float r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// Reciprocal square root estimate (v_rsq_f32) issued at raised wave priority.
// FP32 VALU instructions of two waves of a SIMD issue together as long as
// those waves run in step; a v_rsq_f32 (8 cycles, issued alone) puts them out
// of step, and what follows then issues at half the rate until something
// aligns them again.  Raising the wave's priority for this one instruction
// lets it go at once and keeps the pairing.  Measured in isolation (20 VALU
// and 1 v_rsq_f32 per step, 4 waves per SIMD): 20.9 CU clocks per step
// without, 13.2 with; in the force kernel at 2^20 bodies 301 against 256 ms.
// Kernels bound by the latency of their loads (the tree walk's quadrupole
// sweep) lose a few percent by it and use the plain instruction.
template <int N>
__device__ __forceinline__ void rsq_prio(float (&q)[N])
{
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int k = 0; k < N; ++k) q[k] = __builtin_amdgcn_rsqf(q[k]);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ float rsq_prio(float q)
{
    float one[1] = {q};
    rsq_prio(one);
    return one[0];
}

// 1/sqrt(q) in FP64 from the hardware estimate (relative error 2^-24) and one
// third-order step y + y e (1/2 + 3/8 e), e = 1 - q y^2, whose own error is 5/16
// e^3, below 2^-68.  FP64 instructions issue at 0.85 per clock and CU and
// v_rsq_f64 at a quarter of that, so the three instructions fewer than two
// Newton steps are a tenth of a pair (20001 FP64 bodies:
// 311 against 275 us).
__device__ __forceinline__ double rsq_f64(double q)
{
    const double y = __builtin_amdgcn_rsq(q);
    const double e = __builtin_fma(-q, y * y, 1.0);
    return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// Orders the wave's LDS accesses around this point (the lanes of a wave run
// together, so a barrier is not needed between them).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Register tuples of the hand-scheduled loops.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

bool tune_valid(const Tune &t);

// Place of target k's record of split s among js splits of tcount targets:
// 64 targets' records of one split side by side, the splits of those targets
// after one another.  (With all records of a split side by side, a power of two
// of targets puts every split of a target on the same memory channels.)
__device__ __forceinline__ long split_at(long k, int s, int js, long tcount)
{
    const long g = k & ~63L;
    return g * js + s * min(64L, tcount - g) + (k - g);
}

// Fixed-order sum of the js split records (L values of type E each) of target
// k by L neighbouring lanes, one value each with 8 splits in flight; every lane
// of the L receives all sums.  (One lane per target was bound by the latency
// of its loads: 23457 bodies and 32 splits 10.6 us, 4.9 now; with the order of
// split_at, pairwise sums of 65536 bodies 926 against 897 us per force.)
constexpr int kSumLanes = 4;
template <int L, typename E, typename R>
__device__ __forceinline__ void split_sum(const E *__restrict__ partial, int js, long tcount, long k, R (&r)[L])
{
    const int c = threadIdx.x % L;
    const E *src = partial + L * split_at(k, 0, js, tcount) + c;
    const long stride = L * min(64L, tcount - (k & ~63L));
    R v = R(0);
    int s = 0;
    for (; s + 8 <= js; s += 8) {
        E a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = src[(s + u) * stride];
#pragma unroll
        for (int u = 0; u < 8; ++u) v += a[u];
    }
    for (; s < js; ++s) v += src[s * stride];
    const int first = (threadIdx.x & 63) - c;
#pragma unroll
    for (int q = 0; q < L; ++q) r[q] = __shfl(v, first + q);
}

// ---- force (accel.hip) -----------------------------------------------------
// pm: float4/double4 records; out: target_count records; partial: scratch of
// jsplit * target_count double4 (F32 mode: float4) records when jsplit > 1.
// reduce = false leaves a split result in `partial` (out untouched) for a
// consumer that reduces it itself (launch_reduce_step).
hipError_t launch_accel(int prec, const void *pm, int n, double G, double eps, void *out,
                        int tbeg, int tcount, const Tune &t, void *partial, hipStream_t s,
                        bool reduce = true);
size_t accel_partial_bytes(int prec, int tcount, const Tune &t);
int accel_partial_records(int tcount, const Tune &t);
// What those records hold: FP64 sums, FP32 sums to be added in FP32, or FP32
// tile sums to be added in FP64.
enum RecordKind { kRecF64 = 0, kRecF32 = 1, kRecTile = 2 };
RecordKind accel_record_kind(int prec, int tcount, const Tune &t);

// ---- force on all bodies, each unordered pair once (sym.hip) -----------------
// M blocks of 256 tpl bodies; each launch takes `runs` runs of `len` block
// distances.  The sums meet in `slots` = runs (1 + len) records per body,
// kSymScratch bytes at most (two records per body if that is more), to be added
// per body in slot order in FP64.  With blocks of 512 bodies every record is one
// tile's partial sum, in FP32 as the modes define it (len is 1 then): formed in
// FP64 from sums of 128 terms and rounded once, against FP64 records of 512-term
// FP32 sums in the sweep.  RMS errors of accelerations and potentials against
// FP64 are 0.56 to 0.78 of the sweep's in the compensated modes (22528 to 73727
// bodies; Plummer sphere, pair, ball; eps 0.005 and 0.02).
// kSymScratch: half of it makes more launches and costs up to 7% (400001 bodies
// 32.1 / 34.3 ms, 2^20 219 / 228), a quarter up to 35% (43.3 ms).
// Blocks of 512 bodies (2 targets per lane) below kSymWide: there the tiles of
// 1024 x 1024 are too few to fill 256 CUs evenly (40001 bodies 356 / 458 us,
// 65536 885 / 904); above, 4 targets per lane need half the rotations per pair
// (100000 bodies 2081 / 1954 us).
constexpr int kSymWide = 72 * 1024;
constexpr size_t kSymScratch = size_t(1) << 30;
struct SymPlan {
    int tpl = 0, blocks = 0, len = 0, runs = 0, launches = 0;
    int slots() const { return runs * (1 + len); }
    size_t record() const { return tpl == 2 ? sizeof(float4) : sizeof(double4); }
};
SymPlan sym_plan(int n);
hipError_t launch_sym(const void *pm, int n, double eps, void *slots, hipStream_t s);

// Split partials of nbody_accel_noalloc: a file-scope device array in
// accel.hip of kStaticScratchBytes.  static_split_scratch() returns its
// address on the current device (looked up once per device), or nullptr with
// the error set.
constexpr size_t kStaticScratchBytes = NBODY_NOALLOC_SCRATCH;
void *static_split_scratch();

// Waves of a batched unit that share each 64 tpl targets of a system of n
// bodies: 4, or as many as it has source tiles (a power of two); a unit of 4
// waves then holds 256 tpl / batch_split targets.
__host__ __device__ inline int batch_split(int64_t n, int jtile) { return n > 3 * (int64_t)jtile ? 4 : (n > jtile ? 2 : 1); }
// Batched force over a work list of (system, first target) units sorted
// longest first.  units: int2[nunits] = (system, target offset within the
// system); offsets: int64 device copy [nsys+1]; counter: one zeroed uint32
// pair, left zeroed again by the kernel on exit.
hipError_t launch_batched(int prec, const void *pm, const int64_t *offsets, const int2 *units,
                          int nunits, double G, const float *eps_sys, double eps, void *out,
                          const Tune &t, unsigned *counter, int grid, hipStream_t s);

// ---- fused force + VJP (vjp.hip) -------------------------------------------
// partial: scratch of vjp_partial_bytes(n, t) when t.jsplit > 1.
hipError_t launch_vjp(int prec, const void *pm, const void *cot, int n, double G, double eps,
                      void *pos_cot, void *mass_cot, void *acc_out, const Tune &t, void *partial,
                      hipStream_t s);
// scale multiplies the cotangent; accumulate adds into pos_cot/mass_cot;
// phi = false ignores the phibar component of the cotangent records.
hipError_t launch_vjp_ex(int prec, const void *pm, const void *cot, int n, double G, double eps,
                         bool phi, double scale, bool accumulate, void *pos_cot, void *mass_cot,
                         void *acc_out, const Tune &t, void *partial, hipStream_t s);
size_t vjp_partial_bytes(int n, const Tune &t);
hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s);

// ---- elementwise steps (step.hip) ------------------------------------------
// The small-problem force of all bodies (accel.hip) fused with the step below:
// acc receives the force, then the kick and drift; the positions go to `to`
// (drifted or, without a drift, copied; null: nowhere).  epart (FP64 only): two
// sums per workgroup, slice_blocks(n) of them.
constexpr int kEnergyRow = 16;  // bodies of a workgroup of it
int slice_blocks(int n);
hipError_t launch_slice_step(int prec, const void *pm, int n, double G, double eps, void *acc, void *vel, void *to,
                             double h, double dt, bool close, bool open, double *epart, hipStream_t s);
// One pass between two force evaluations:
//   close: v += h a          (closing kick of the previous step)
//   energy partials of (v, phi) after the closing kick, if epart != nullptr
//   open:  v += h a; x += dt v  (opening kick and drift of the next step)
hipError_t launch_step(int prec, void *pm, void *vel, const void *acc, int n, double h, double dt,
                       bool close, bool open, double *epart, int *eblocks, hipStream_t s);
int step_blocks(int n);
// Split reduction of the force (js partial records per body, as left by
// launch_accel(..., reduce = false) for all n targets) fused with the step:
// acc receives the reduced force, then the kick/drift of launch_step runs.
hipError_t launch_reduce_step(int prec, RecordKind kind, const void *partial, int js, double G, void *pm, void *vel,
                              void *acc, int n, double h, double dt, bool close, bool open,
                              double *epart, int *eblocks, hipStream_t s);
// Energies of `states` states whose partials follow one another.  parts: sums
// per state, of a step kernel's workgroups or (rows) of kEnergyRow bodies each.
hipError_t launch_energy_final(const double *epart, int parts, bool rows, int states, double *out, hipStream_t s);
hipError_t launch_permute(const void *src, void *dst, const int32_t *perm, int n, int rec_bytes,
                          bool inverse, hipStream_t s);
hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s);

// Reverse leapfrog step by time reversal plus vbar += dt xbar, refreshing the
// scaled cotangent vsc = vbar / m (vjp.hip).
hipError_t launch_reverse_step(int prec, void *x, void *vh, const void *acc, const void *xbar,
                               void *vbar, void *vsc, int n, double hk, double dt, hipStream_t s);
// y += a x and ysc = y / m (m from the records pm) (vjp.hip).
hipError_t launch_adj_axpy(int prec, void *y, const void *x, double a, const void *pm, void *ysc,
                           int n, hipStream_t s);
// sc = cot / m; *nonpos |= (some m <= 0).  *nonpos must be zero before.
// dst = (0, 0, 0, src.w) per record (the potential part of a cotangent).
hipError_t launch_phibar_only(int prec, const void *src, int n, void *dst, hipStream_t s);
hipError_t launch_prescale(int prec, const void *cot, const void *pm, int n, void *sc, int *nonpos,
                           hipStream_t s);
// Adjoint VJP (phibar = 0, accumulate): mass-scaled form on sc unless
// *nonpos, then the general form on raw.
hipError_t launch_vjp_adj(int prec, const void *pm, const void *raw, const void *sc,
                          const int *nonpos, int n, double G, double eps, double scale,
                          void *pos_cot, void *mass_cot, void *acc_out, const Tune &t, void *partial,
                          hipStream_t s);
// Adjoint VJP and the elementwise step after it in as few launches as the
// shape allows (post 1: vbar += dt xbar; post 2: time reversal of x, vh;
// post 3: as post 1, and the force to acc).  Uses tpl = 1 when the source
// range is split.
hipError_t launch_vjp_adj_step(int prec, int post, void *pm, void *raw, void *sc, const int *nonpos,
                               int n, double G, double eps, double scale, void *pos_cot,
                               void *mass_cot, void *acc, void *vh, double hk, double dt,
                               const Tune &t, void *partial, hipStream_t s);

// ---- ORB (orb.hip) -----------------------------------------------------------
int orb_order(const void *pm, int prec, int n, int leaf, int32_t *perm, hipStream_t s);
void orb_release();

// ---- tree code (tree.hip) ----------------------------------------------------
int tree_shape(int n, int leaf, int64_t *num_nodes, int64_t *num_groups, int32_t *nodes_out);
int tree_moments(const void *pm, int n, int leaf, double *mom, float *box, hipStream_t s);
int tree_lists(const void *pm, int n, int leaf, double theta, int max_far, int max_near, int32_t *far_cnt,
               int32_t *near_cnt, int32_t *far_ids, int32_t *near_ids, hipStream_t s);
int tree_accel(const void *pm, int n, int prec, double G, double eps, double theta, int leaf, int cells,
               void *out, hipStream_t s);
int tree_pseudo(const void *pm, int n, int leaf, void *out, hipStream_t s);
int tree_quad(const void *pm, int n, int leaf, void *out, hipStream_t s);
int tree_local_counts(const void *pm, int n, int leaf, double theta, int32_t *loc_cnt, int32_t *far_cnt,
                      int32_t *near_cnt, hipStream_t s);
int tree_leapfrog(void *pm, void *vel, void *acc, int32_t *order, int n, int prec, double G, double eps,
                  double theta, int leaf, double dt, int nsteps, int reorder_every, unsigned flags,
                  double *energy, hipStream_t s);
void tree_release();

// ---- multi-level FMM (fmm.hip) ------------------------------------------------
// pm: n float4 records in ORB order (leaf as given).  fmm_accel writes n
// records (ORB order); synchronises s once to check the list buffers.
int fmm_accel(const void *pm, int n, int prec, double G, double eps, double theta, int leaf, void *out,
              hipStream_t s);
// fmm_lists: per-node counts and concatenated source ids of the (M2L, M2P,
// P2P) lists, grouped by target node (device outputs; ids_out entries may be
// NULL to count only).
int fmm_lists(const void *pm, int n, int leaf, double theta, int32_t *const cnt_out[3], int32_t *const ids_out[3],
              const int64_t caps[3], hipStream_t s);
void fmm_release();

// ---- bit-reversible fixed-point leapfrog (janus.hip) ---------------------------
// state: 2n longlong4 (X then V); the force kernel and the fused VJP run with
// G = 1 and the shape of janus_tune so their forces agree bit for bit.
Tune janus_tune(const Tune &vjp_default);
int janus_forward(const void *pm, const void *vel, int n, double G, double eps, double dt, int nsteps, int sx,
                  int sv, const Tune &t, void *state, void *pm_out, void *vel_out, void *acc, void *partial,
                  hipStream_t s);
int janus_decode(const void *state, const void *pm, int n, int sx, void *dec, hipStream_t s);
int janus_unstep(void *state, const void *acc, int n, double G, double dt, int sx, int sv, int kicks, int drift,
                 void *dec, hipStream_t s);

// ---- runtime helpers (runtime.hip) -----------------------------------------
void set_error(const char *fmt, ...);
int hip_fail(hipError_t e, const char *what);
// Library scratch, one growable buffer per slot and device.
enum ScratchSlot { kSlotPartial = 0, kSlotEnergy, kSlotBatch, kSlotOrb0, kSlotOrb1, kSlotOrb2,
                   kSlotOrb3, kSlotOrb4, kSlotAdj0, kSlotAdj1, kSlotAdj2, kSlotAdj3, kSlotAdj4, kSlotTune,
                   kNumSlots };
void *scratch(int slot, size_t bytes);

}  // namespace nbi
