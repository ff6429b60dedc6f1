// Multi-level fast multipole method on the ORB nodes (gfx950).
//
// Section VI names the fast multipole method (its reference [20]) as the O(N)
// successor of the tree code.  Built here from the tree code's pieces: the
// ORB nodes with their FP64 moments, boxes and quadrupole records
// (tree.hip), the quadrupole cell's evaluation at a body and its M2L into a
// third-order local expansion (tree_shared.h), and the FP32 pair code of the
// direct sum (pair.h).  Definitions shared with the FP64 oracle (every node's
// lists are equal to the oracle's as sets):
// * MAC: target node A and source node B interact through M2L iff they share
//   no body and diag2_A + diag2_B < theta^2 |com_A - com_B|^2 (FP64).
// * Dual-tree traversal from (root, root): MAC -> B joins A's M2L list; A a
//   leaf and B accepted by the tree code's opening test against A's box
//   (diag2_B < theta^2 D2, D2 the squared distance from com_B to the box) ->
//   B joins A's M2P list; two leaves -> B joins A's P2P list; B a leaf, or A
//   an inner node with diag2_A >= diag2_B -> the pair passes to both
//   children of A; otherwise the pair is replaced by (A, B.left),
//   (A, B.right).
// * A node's total local expansion = its own M2L sum + its parent's total
//   re-expanded about its centre of mass (exact for a cubic); every body of
//   a leaf evaluates its leaf's expansion, its M2P cells as quadrupole cells
//   and its P2P source leaves body by body without the self pair.
//
// Device schedule:
// * Traversal, top-down by node depth.  For a target node A the pairs (A, .)
//   of the recursion are those inherited from its parent (the parent's
//   pass-down list) closed under source splits: the node's waves pop up to 64
//   pending sources each per step from an LDS stack, one per lane, and
//   classify them (ballot ranks give every output a fixed position); at the
//   deep depths one wave walks two sibling nodes, gathering each source once
//   for both.  Each depth runs one walk that writes every node's lists into slots of a
//   per-depth capacity; when that layout would take more than its memory
//   budget, each depth instead runs a count walk, a two-kernel scan (block
//   sums, then offsets) and a fill walk into compact lists.  Writes are
//   bounds-checked and an overflow flag makes the host resize (from the
//   exact counts) and run again.
// * M2L: one wave per node, one source cell per lane, the twenty
//   coefficients summed over the wave in a fixed butterfly (FP32).
// * L2L: one thread per node, depth by depth, in FP64, in two launches.
// * Leaves: one wave per leaf.  Each lane holds up to 8 of the leaf's
//   targets in registers and takes one source body (P2P) or cell (M2P) at a
//   time, so one load serves up to 8 pairs.  The lanes' FP32 partial sums are
//   folded by the precision mode in lane order through LDS, then each target
//   adds its leaf's expansion in FP64.
#include <algorithm>
#include <array>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

#include "internal.h"
#include "pair.h"
#include "tree_shared.h"

namespace nbi {
namespace {

#define NB_CHECK_RC(expr)                \
    do {                                 \
        const int rc_ = (expr);          \
        if (rc_ != NBODY_OK) return rc_; \
    } while (0)

constexpr int kFmmStack = 64;     // bound on the tree height the traversal admits
constexpr int kWalkStack = 2048;  // most LDS stack entries per walking wave (64 per source depth + refill)

// List kinds; per-node counts and offsets are stored [kind][nn].
constexpr int kM2L = 0, kP2P = 1, kM2P = 2, kPass = 3, kKinds = 4;
// tot: [0] the overflow flag; for the three interaction lists the running
// total before depth d at tot_at(kind, d); the pass-down total of depth d at
// tot_at(kPass, d).
constexpr int kRunStride = kFmmStack + 1;
constexpr int kTotWords = 1 + kKinds * kRunStride;
__host__ __device__ constexpr int tot_at(int kind, int d) { return 1 + kind * kRunStride + d; }

constexpr int kL2lRoots = 256;    // see k_fmm_l2l
constexpr int kScanBlock = 1024;  // positions per scan block (256 threads x 4)

struct FmmDev {
    const int4 *node;
    const NodeRec *nrec;
    const float4 *lo, *hi;
    const float4 *qr;
    const int *parent;
    int nn;
    int *cnt;   // [kKinds][nn] counts per node
    int *lcnt;  // [kKinds][nn] the same counts at each node's position in depth order
    int *off;   // [kKinds][nn] offsets (global; pass-down: in the depth's buffer)
    int *m2l;   // source node ids
    int *p2p;   // the first body of each source leaf
    int *m2p;   // source node ids
    int *pass0, *pass1;
    long cap_m2l, cap_p2p, cap_m2p, cap_pass;
    long *bsum;               // [blocks][kKinds] scan block sums
    unsigned long long *tot;  // see tot_at
    unsigned long long *flag; // host memory: the overflow flag as the evaluation found it
    float *own;               // [nn][20] own M2L sums
    double *loc;              // [nn][20] total expansions
};

__device__ __forceinline__ long cap_of(const FmmDev &F, int kind)
{
    return kind == kM2L ? F.cap_m2l : (kind == kP2P ? F.cap_p2p : (kind == kM2P ? F.cap_m2p : F.cap_pass));
}

__device__ __forceinline__ bool fmm_overlap(int4 a, int4 b) { return (a.x < b.y) & (b.x < a.y); }

__device__ __forceinline__ unsigned fmm_rank(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// One node's list as a walk writes it: where it begins and its room.  32-bit
// counts, so that an entry is stored at a scalar base and a 32-bit offset.
struct ListOut {
    int *at;
    int room;
};

// Bounds-checked store of one list entry: the entry's index in its list is
// done + its rank among the lanes of mask; returns false when it does not fit.
__device__ __forceinline__ bool put_entry(const ListOut &l, int done, unsigned long long mask, int value)
{
    const int q = done + (int)fmm_rank(mask);
    if (q >= l.room) return false;
    l.at[(unsigned)q] = value;
    return true;
}

// Walk passes.  kWalkCount counts every list of every node; kWalkFill writes
// them at the offsets the scan derived from the counts; kWalkSlot writes
// them, in one pass, into per-node slots of a per-depth capacity (and
// records the exact counts, so that slots too small can be resized).
enum { kWalkCount = 0, kWalkFill = 1, kWalkSlot = 2 };

// Slot layout of one depth: list kind k of the node at position t of the
// depth starts at base[k] + t * cap[k] (the pass-down list in the depth's
// ping-pong buffer); prev_pass is the previous depth's pass-down capacity.
struct SlotDepth {
    long base[kKinds];
    int cap[kKinds];
    int prev_pass;
};

// Where the lists of node A, the t-th of its depth, begin (o) and go: the slots
// of the one-pass layout, or the scanned offsets with the rest of the buffer
// as room (offsets are global).  A count pass stores nothing.
template <int WMODE>
__device__ __forceinline__ void list_outs(const FmmDev &F, int A, int t, int parity, const SlotDepth &sd,
                                          long (&o)[kKinds], ListOut (&out)[kKinds])
{
    int *const list[kKinds] = {F.m2l, F.p2p, F.m2p, parity ? F.pass1 : F.pass0};
#pragma unroll
    for (int q = 0; q < kKinds; ++q) {
        o[q] = WMODE == kWalkSlot ? sd.base[q] + (long)t * sd.cap[q] : WMODE == kWalkFill ? F.off[q * F.nn + A] : 0;
        const long room = WMODE == kWalkSlot ? sd.cap[q] : cap_of(F, q) - o[q];
        out[q].at = list[q] + o[q];
        out[q].room = (int)min(max(room, 0L), (long)INT32_MAX);
    }
}

// Places the wait for a loaded value here.
__device__ __forceinline__ void arrived(int &v) { asm volatile("" : "+v"(v)); }

// What becomes of source B (node record nb, centre and squared diagonal cb) at
// target A, by the definitions above.  Without branches on the lane, so that
// every value's one wait lies before the list stores.
struct Verdict {
    bool m2l, m2p, p2p, pass, split;
};

__device__ __forceinline__ Verdict classify(bool act, const int4 na, const double4 ca, bool aleaf, const float4 lo,
                                            const float4 hi, const int4 nb, const double4 cb, double theta2)
{
    Verdict v;
    const bool apart = act & !fmm_overlap(na, nb), bleaf = nb.z < 0;
    const double dx = ca.x - cb.x, dy = ca.y - cb.y, dz = ca.z - cb.z;
    const double dist2 = (dx * dx + dy * dy) + dz * dz;
    v.m2l = apart & (ca.w + cb.w < theta2 * dist2);
    v.m2p = false;
    if (aleaf) {
        const double gx = box_gap(cb.x, lo.x, hi.x);
        const double gy = box_gap(cb.y, lo.y, hi.y);
        const double gz = box_gap(cb.z, lo.z, hi.z);
        const double D2 = (gx * gx + gy * gy) + gz * gz;
        v.m2p = apart & !v.m2l & (cb.w < theta2 * D2);
    }
    const bool rest = act & !v.m2l & !v.m2p;
    v.p2p = rest & aleaf & bleaf;
    v.pass = rest & !aleaf & (bleaf | (ca.w >= cb.w));
    v.split = rest & !v.p2p & !v.pass;
    return v;
}

// The list that the children of node P inherit: P's pass-down list in the
// previous depth's buffer, cut where P's slot or its depth overflowed.  The
// root (P < 0) starts from itself, the one node of its depth.
template <int WMODE>
__device__ __forceinline__ const int *inherited(const FmmDev &F, const int *ids, int P, int parity,
                                                const SlotDepth &sd, int &nin)
{
    nin = 1;
    if (P < 0) return ids;
    nin = F.cnt[kPass * F.nn + P];
    const long base = F.off[kPass * F.nn + P];
    if (WMODE == kWalkSlot) nin = min(nin, sd.prev_pass);
    if (base + nin > F.cap_pass) nin = (int)max(0L, F.cap_pass - base);
    return (parity ? F.pass0 : F.pass1) + (nin > 0 ? base : 0L);
}

// W waves per target node of one depth: the walk of its inherited sources.
// The pending sources sit on an LDS stack; each step pops up to 64 W of them
// (one per thread) and classifies each: M2L, M2P, P2P, pass-down (to both
// children of A) or split (both children of B pushed).  Ballot ranks, and the
// counts of the waves before, keep every output in a fixed order, so every
// pass produces the same lists.
template <int WMODE, int W>
__global__ __launch_bounds__(64 * W) void k_fmm_walk(FmmDev F, const int *__restrict__ ids, int first, int parity,
                                                     double theta2, SlotDepth sd, int room)
{
    constexpr bool FILL = WMODE != kWalkCount;
    extern __shared__ int stk[];
    static_assert(W > 1, "one wave would need its own order of the stack's reads and writes");
    __shared__ int steps[W][kKinds + 1];  // this step's counts of each wave: the lists and the splits
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int t = blockIdx.x;
    const int A = ids[t];
    const int4 na = F.node[A];
    const double4 ca = F.nrec[A].cd;
    const bool aleaf = na.z < 0;
    const float4 blo = F.lo[A], bhi = F.hi[A];  // A's box (M2P test)
    const int nn = F.nn;
    int nin;
    const int *in = inherited<WMODE>(F, ids, A == 0 ? -1 : F.parent[A], parity, sd, nin);
    long o[kKinds];
    ListOut out[kKinds];
    list_outs<WMODE>(F, A, t, parity, sd, o, out);
    int cm = 0, cp = 0, cc = 0, cq = 0, top = 0, next = 0;
    bool bad = false;
    // Waits: the inherited entry that this thread pushes at the next refill is
    // loaded with the step's sources, and every lane loads (the idle ones the
    // root).  A load under a lane mask, or one that is used after the list stores, is
    // waited for together with those stores.
    int ahead = in[min(tid, max(nin - 1, 0))];
    for (;;) {
        if (top < 64 * W && next < nin) {  // refill from the inherited list
            const int k = min(64 * W, nin - next);
            if (tid < k) stk[top + tid] = ahead;
            top += k;
            next += k;
        }
        if (top == 0) break;
        const int k = min(64 * W, top);
        top -= k;
        __syncthreads();
        const bool act = tid < k;
        int B = act ? stk[top + tid] : 0;
        if ((unsigned)B >= (unsigned)nn) B = 0;  // only after an overflow upstream
        ahead = in[min(next + tid, max(nin - 1, 0))];
        const int4 nb = F.nrec[B].nd;
        const double4 cb = F.nrec[B].cd;
        const Verdict v = classify(act, na, ca, aleaf, blo, bhi, nb, cb, theta2);
        arrived(ahead);
        const bool m2l = v.m2l, m2p = v.m2p, p2p = v.p2p, pass = v.pass, split = v.split;
        const unsigned long long mm = __ballot(m2l), mc = __ballot(m2p), mp = __ballot(p2p), mq = __ballot(pass),
                                 ms = __ballot(split);
        // the step's counts, and how many of them lie in the waves before this one
        int sum[kKinds + 1] = {(int)__popcll(mm), (int)__popcll(mp), (int)__popcll(mc), (int)__popcll(mq), (int)__popcll(ms)};
        int before[kKinds + 1] = {0, 0, 0, 0, 0};
        if (lane == 0)
#pragma unroll
            for (int q = 0; q <= kKinds; ++q) steps[wave][q] = sum[q];
        __syncthreads();  // every wave has popped, too: the stack may be written
#pragma unroll
        for (int q = 0; q <= kKinds; ++q) {
            sum[q] = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                if (w == wave) before[q] = sum[q];
                sum[q] += steps[w][q];
            }
        }
        if (FILL) {
            if (m2l && !put_entry(out[kM2L], cm + before[kM2L], mm, B)) bad = true;
            if (m2p && !put_entry(out[kM2P], cc + before[kM2P], mc, B)) bad = true;
            if (p2p && !put_entry(out[kP2P], cp + before[kP2P], mp, nb.x)) bad = true;  // a leaf as its first body
            if (pass && !put_entry(out[kPass], cq + before[kPass], mq, B)) bad = true;
        }
        cm += sum[kM2L];
        cp += sum[kP2P];
        cc += sum[kM2P];
        cq += sum[kPass];
        const int ns = sum[kKinds];
        if (top + 2 * ns > room) {  // cannot happen for trees the host admits
            bad = true;
            break;
        }
        if (split) {
            const int q = top + 2 * (before[kKinds] + (int)fmm_rank(ms));
            stk[q] = nb.w;
            stk[q + 1] = nb.z;
        }
        top += 2 * ns;
        __syncthreads();
    }
    if (WMODE != kWalkFill && tid == 0) {
        const int c4[kKinds] = {cm, cp, cc, cq};
#pragma unroll
        for (int q = 0; q < kKinds; ++q) {
            F.cnt[q * nn + A] = c4[q];
            if (WMODE == kWalkCount)
                F.lcnt[q * nn + first + t] = c4[q];
            else
                F.off[q * nn + A] = (int)o[q];
        }
    }
    if (__ballot(bad) && lane == 0) atomicOr(&F.tot[0], 1ull);
}

// Two target nodes per wave: positions 2 b and 2 b + 1 of one depth.  Below the
// root every depth holds whole sibling pairs, adjacent in preorder, so these
// are the children of one parent and inherit the same list.  The stack holds
// the union of the targets' pending sources, each entry tagged with the
// targets that still need it (bit k for target k, in the four high bits of the
// entry; node ids stay below 2^28, which the host checks).  A popped source is
// gathered once and classified for each of its targets by the same tests as in
// the one-target walk; it is split (children pushed, tagged with the targets
// that split it) if any target splits it.  Each target's lists are written at
// ballot ranks in pop order, so every pass produces the same lists for a
// target: the same entries as the one-target walk's, in another order.
constexpr unsigned kTagShift = 28, kIdMask = (1u << kTagShift) - 1;

template <int WMODE>
__global__ __launch_bounds__(64) void k_fmm_walk_pair(FmmDev F, const int *__restrict__ ids, int first, int parity,
                                                      double theta2, SlotDepth sd, int room)
{
    constexpr int TPW = 2;
    constexpr bool FILL = WMODE != kWalkCount;
    extern __shared__ unsigned ustk[];
    unsigned *const stk = ustk;
    const int lane = threadIdx.x;
    const int nn = F.nn;
    int tpos[TPW], A[TPW];
    int4 na[TPW];
    double4 ca[TPW];
    bool aleaf[TPW];
    float4 blo[TPW], bhi[TPW];  // each target's box (M2P test)
    long o[TPW][kKinds];
    ListOut out[TPW][kKinds];
    int c[TPW][kKinds];
#pragma unroll
    for (int k = 0; k < TPW; ++k) {
        tpos[k] = TPW * blockIdx.x + k;
        A[k] = ids[tpos[k]];
        na[k] = F.node[A[k]];
        ca[k] = F.nrec[A[k]].cd;
        aleaf[k] = na[k].z < 0;
        blo[k] = F.lo[A[k]];
        bhi[k] = F.hi[A[k]];
        list_outs<WMODE>(F, A[k], tpos[k], parity, sd, o[k], out[k]);
#pragma unroll
        for (int q = 0; q < kKinds; ++q) c[k][q] = 0;
    }
    int nin;
    const int *in = inherited<WMODE>(F, ids, F.parent[A[0]], parity, sd, nin);
    int next = 0, top = 0;
    bool bad = false;
    int ahead = in[min(lane, max(nin - 1, 0))];  // loads and waits as in the one-target walk
    for (;;) {
        if (top < 64 && next < nin) {  // refill
            const int take = min(64, nin - next);
            if (lane < take) stk[top + lane] = (unsigned)ahead | (((1u << TPW) - 1) << kTagShift);
            top += take;
            next += take;
        }
        if (top == 0) break;
        const int kpop = min(64, top);
        top -= kpop;
        __syncthreads();
        const bool act = lane < kpop;
        const unsigned e = act ? stk[top + lane] : 0u;
        __syncthreads();
        int B = (int)(e & kIdMask);
        const unsigned tag = e >> kTagShift;
        if ((unsigned)B >= (unsigned)nn) B = 0;  // only after an overflow upstream
        ahead = in[min(next + lane, max(nin - 1, 0))];
        const int4 nb = F.nrec[B].nd;
        const double4 cb = F.nrec[B].cd;
        arrived(ahead);
        unsigned split_tag = 0;
#pragma unroll
        for (int k = 0; k < TPW; ++k) {
            const Verdict v = classify(act && (tag >> k & 1u), na[k], ca[k], aleaf[k], blo[k], bhi[k], nb, cb, theta2);
            const bool m2l = v.m2l, m2p = v.m2p, p2p = v.p2p, pass = v.pass, split = v.split;
            const unsigned long long mm = __ballot(m2l), mc = __ballot(m2p), mp = __ballot(p2p),
                                     mq = __ballot(pass);
            if (FILL) {
                if (m2l && !put_entry(out[k][kM2L], c[k][kM2L], mm, B)) bad = true;
                if (m2p && !put_entry(out[k][kM2P], c[k][kM2P], mc, B)) bad = true;
                if (p2p && !put_entry(out[k][kP2P], c[k][kP2P], mp, nb.x)) bad = true;
                if (pass && !put_entry(out[k][kPass], c[k][kPass], mq, B)) bad = true;
            }
            c[k][kM2L] += __popcll(mm);
            c[k][kM2P] += __popcll(mc);
            c[k][kP2P] += __popcll(mp);
            c[k][kPass] += __popcll(mq);
            if (split) split_tag |= 1u << k;
        }
        const unsigned long long ms = __ballot(split_tag != 0);
        const int ns = __popcll(ms);
        if (top + 2 * ns > room) {  // cannot happen for trees the host admits
            bad = true;
            break;
        }
        if (split_tag) {
            const int q = top + 2 * (int)fmm_rank(ms);
            stk[q] = (unsigned)nb.w | (split_tag << kTagShift);
            stk[q + 1] = (unsigned)nb.z | (split_tag << kTagShift);
        }
        top += 2 * ns;
        __syncthreads();
    }
    if (WMODE != kWalkFill && lane == 0) {
#pragma unroll
        for (int k = 0; k < TPW; ++k) {
#pragma unroll
            for (int q = 0; q < kKinds; ++q) {
                F.cnt[q * nn + A[k]] = c[k][q];
                if (WMODE == kWalkCount)
                    F.lcnt[q * nn + first + tpos[k]] = c[k][q];
                else
                    F.off[q * nn + A[k]] = (int)o[k][q];
            }
        }
    }
    if (__ballot(bad) && lane == 0) atomicOr(&F.tot[0], 1ull);
}

// How the nodes of one depth are walked.  The deep depths, with enough nodes to
// fill the chip more than once, walk 2 per wave (half the waves, each source
// gathered once for both).  Measured at 2^20 (leaf 8, theta 0.5) with the walks
// as they first were: the depths of 8192 to 131072 nodes took 239-1019 us
// against 311-1141 us with one target per wave, and 708-1299 us with 4 per wave
// from 32768 nodes on.  The depths above have fewer nodes than the chip has
// room for waves, and a depth lasts as long as its longest walk, a chain of
// steps: four waves per node take four steps' sources at once.  At 262144
// bodies (leaf 8, theta 0.5) an FMM force took 2131 us with one wave per node,
// 1952 us with four; eight gain 1% at up to 512 nodes and lose above.
constexpr int kPairNodes = 8192;
constexpr int kNodeWaves = 4;

template <int WMODE>
void launch_walk_depth(const FmmDev &F, const int *ids, int first, int count, int stack, int parity, double theta2,
                       const SlotDepth &sd, hipStream_t s)
{
    // (below the root a depth holds whole sibling pairs)
    if (count >= kPairNodes && count % 2 == 0 && F.nn <= (int)kIdMask)
        hipLaunchKernelGGL(k_fmm_walk_pair<WMODE>, dim3(count / 2), dim3(64), stack * sizeof(int), s, F, ids, first,
                           parity, theta2, sd, stack);
    else
        hipLaunchKernelGGL((k_fmm_walk<WMODE, kNodeWaves>), dim3(count), dim3(64 * kNodeWaves),
                           kNodeWaves * stack * sizeof(int), s, F, ids, first, parity, theta2, sd,
                           kNodeWaves * stack);
}

// Sum over the wave of four values (fixed butterfly).
__device__ __forceinline__ void wave_sum4(long (&s)[kKinds])
{
#pragma unroll
    for (int q = 0; q < kKinds; ++q)
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) s[q] += __shfl_xor(s[q], o);
}

// Scan, first kernel: the four count sums of each block of kScanBlock
// positions of one depth.
__global__ __launch_bounds__(256) void k_fmm_scan_part(FmmDev F, int first, int count)
{
    __shared__ long red[4][kKinds];
    const int tid = threadIdx.x, b = blockIdx.x, nn = F.nn;
    long s[kKinds] = {0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < kScanBlock / 256; ++r) {
        const int pos = b * kScanBlock + r * 256 + tid;
        if (pos < count)
#pragma unroll
            for (int q = 0; q < kKinds; ++q) s[q] += F.lcnt[q * nn + first + pos];
    }
    wave_sum4(s);
    if ((tid & 63) == 0)
#pragma unroll
        for (int q = 0; q < kKinds; ++q) red[tid >> 6][q] = s[q];
    __syncthreads();
    if (tid < kKinds) F.bsum[(long)b * kKinds + tid] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
}

// Scan, second kernel: block b adds the sums of the blocks before it to the
// running totals, scans its positions (4 contiguous per thread) and writes
// every node's offsets; the last block stores the totals for the next depth
// and raises the overflow flag when a list passes its capacity.
__global__ __launch_bounds__(256) void k_fmm_scan_fin(FmmDev F, const int *__restrict__ ids, int first, int count,
                                                      int depth, int nblk)
{
    __shared__ long wsum[4][kKinds];
    __shared__ long bbase[kKinds];
    const int tid = threadIdx.x, b = blockIdx.x, nn = F.nn;
    const int lane = tid & 63, wv = tid >> 6;
    if (wv == 0) {
        long s[kKinds] = {0, 0, 0, 0};
        for (int k = lane; k < b; k += 64)
#pragma unroll
            for (int q = 0; q < kKinds; ++q) s[q] += F.bsum[(long)k * kKinds + q];
        wave_sum4(s);
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < kKinds; ++q) bbase[q] = (q < kPass ? (long)F.tot[tot_at(q, depth)] : 0L) + s[q];
    }
    const int p0 = b * kScanBlock + 4 * tid;
    int v[4][kKinds];
    long s[kKinds] = {0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < kKinds; ++q) {
            v[r][q] = p0 + r < count ? F.lcnt[q * nn + first + p0 + r] : 0;
            s[q] += v[r][q];
        }
    long inc[kKinds];
#pragma unroll
    for (int q = 0; q < kKinds; ++q) inc[q] = s[q];
#pragma unroll
    for (int d = 1; d < 64; d <<= 1)
#pragma unroll
        for (int q = 0; q < kKinds; ++q) {
            const long y = __shfl_up(inc[q], d);
            if (lane >= d) inc[q] += y;
        }
    if (lane == 63)
#pragma unroll
        for (int q = 0; q < kKinds; ++q) wsum[wv][q] = inc[q];
    __syncthreads();
    long o[kKinds];
#pragma unroll
    for (int q = 0; q < kKinds; ++q) {
        long pre = bbase[q];
        for (int w = 0; w < wv; ++w) pre += wsum[w][q];
        o[q] = pre + inc[q] - s[q];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (p0 + r >= count) break;
        const int A = ids[p0 + r];
#pragma unroll
        for (int q = 0; q < kKinds; ++q) {
            F.off[q * nn + A] = (int)min(o[q], (long)INT32_MAX);
            o[q] += v[r][q];
        }
    }
    if (b == nblk - 1 && tid < kKinds) {
        const long run = bbase[tid] + (wsum[0][tid] + wsum[1][tid]) + (wsum[2][tid] + wsum[3][tid]);
        F.tot[tid < kPass ? tot_at(tid, depth + 1) : tot_at(kPass, depth)] = (unsigned long long)run;
        if (run > cap_of(F, tid) || run > (long)INT32_MAX) atomicOr(&F.tot[0], 1ull);
    }
}

// M2L: one wave per node, and a workgroup per wave, since a node's list is what
// it is.  The list is read a step ahead, and the coefficients are summed by
// handing halves on instead of 20 butterflies of 6 shuffles (262144 bodies, 324
// cells per node on average: 236 us with four waves per workgroup and the
// butterflies, 222 us now; the gathers of the cells' records bound it).
__global__ __launch_bounds__(64) void k_fmm_m2l(FmmDev F, float eps2)
{
    const int A = blockIdx.x;
    const int lane = threadIdx.x;
    const unsigned long long over = F.tot[0];
    if (A == 0 && lane == 0) *F.flag = over;
    if (over) return;
    const long o = F.off[kM2L * F.nn + A];
    const int c = (int)min((long)F.cnt[kM2L * F.nn + A], max(0L, F.cap_m2l - o));
    const double4 ca = F.nrec[A].cd;
    const float zx = (float)ca.x, zy = (float)ca.y, zz = (float)ca.z;
    Local L;
#pragma unroll
    for (int k = 0; k < 20; ++k) L.c[k] = 0.0f;
    const int *const list = F.m2l + o;
    int next = lane < c ? list[lane] : -1;  // a step ahead
    for (int k = lane; k < c; k += 64) {
        const int B = next;
        next = k + 64 < c ? list[k + 64] : -1;
        if ((unsigned)B < (unsigned)F.nn) m2l_f32(F.qr + (long)kQuadRec * B, zx, zy, zz, eps2, L);
    }
    const int q = wave_scatter20(L.c, lane);
    if (q >= 0) F.own[20L * A + q] = L.c[0];
}

// Full symmetric K and T of the 20 coefficients (P0, p, K: xx yy zz xy xz yz,
// T: xxx yyy zzz xxy xxz xyy yyz xzz yzz xyz) contracted with d:
// kd = K d, td = T d (3x3), tdd = T(d, d).
__device__ __forceinline__ void fmm_contract(const double *c, const double d[3], double kd[3], double td[3][3],
                                             double tdd[3])
{
    const double K[3][3] = {{c[4], c[7], c[8]}, {c[7], c[5], c[9]}, {c[8], c[9], c[6]}};
    // T[k][l][m] by the stored index of the sorted triple
    auto T = [&](int k, int l, int m) -> double {
        int a = k, b = l, e = m, x;
        if (a > b) { x = a; a = b; b = x; }
        if (b > e) { x = b; b = e; e = x; }
        if (a > b) { x = a; a = b; b = x; }
        if (a == b && b == e) return c[10 + a];                       // xxx yyy zzz
        if (a == 0 && b == 0) return c[e == 1 ? 13 : 14];             // xxy xxz
        if (a == 0 && b == 1 && e == 1) return c[15];                 // xyy
        if (a == 1 && b == 1) return c[16];                           // yyz
        if (a == 0 && b == 2) return c[17];                           // xzz
        if (a == 1 && b == 2) return c[18];                           // yzz
        return c[19];                                                 // xyz
    };
    for (int k = 0; k < 3; ++k) {
        kd[k] = (K[k][0] * d[0] + K[k][1] * d[1]) + K[k][2] * d[2];
        for (int l = 0; l < 3; ++l) td[k][l] = (T(k, l, 0) * d[0] + T(k, l, 1) * d[1]) + T(k, l, 2) * d[2];
        tdd[k] = (td[k][0] * d[0] + td[k][1] * d[1]) + td[k][2] * d[2];
    }
}

// L2L of one node: loc[A] = own[A] + the parent's total re-expanded about
// com_A (the root takes its own sum).
__device__ __forceinline__ void l2l_node(const FmmDev &F, int A)
{
    const int P = F.parent[A];
    double *out = F.loc + 20L * A;
    const float *own = F.own + 20L * A;
    if (P < 0) {
        for (int k = 0; k < 20; ++k) out[k] = (double)own[k];
        return;
    }
    const double *c = F.loc + 20L * P;
    const double4 ca = F.nrec[A].cd, cp = F.nrec[P].cd;
    const double d[3] = {ca.x - cp.x, ca.y - cp.y, ca.z - cp.z};
    double kd[3], td[3][3], tdd[3];
    fmm_contract(c, d, kd, td, tdd);
    const double pd = (c[1] * d[0] + c[2] * d[1]) + c[3] * d[2];
    const double dkd = (d[0] * kd[0] + d[1] * kd[1]) + d[2] * kd[2];
    const double dtdd = (d[0] * tdd[0] + d[1] * tdd[1]) + d[2] * tdd[2];
    out[0] = (c[0] + pd + 0.5 * dkd + dtdd / 6.0) + (double)own[0];
    for (int k = 0; k < 3; ++k) out[1 + k] = (c[1 + k] + kd[k] + 0.5 * tdd[k]) + (double)own[1 + k];
    out[4] = (c[4] + td[0][0]) + (double)own[4];
    out[5] = (c[5] + td[1][1]) + (double)own[5];
    out[6] = (c[6] + td[2][2]) + (double)own[6];
    out[7] = (c[7] + td[0][1]) + (double)own[7];
    out[8] = (c[8] + td[0][2]) + (double)own[8];
    out[9] = (c[9] + td[1][2]) + (double)own[9];
    for (int k = 10; k < 20; ++k) out[k] = c[k] + (double)own[k];
}

// L2L, one thread per node, depth by depth.  Workgroup b takes the subtree of
// the b-th node of its top depth: first[d][b] .. first[d][b + 1] are its
// nodes' positions in the depth order at depth top + d.  One launch for the depths
// of up to kL2lRoots nodes (one workgroup) and one for the depths below (a
// workgroup per node of the last of those): a launch per depth took 103 us at
// 262144 bodies (leaf 8, 16 depths), each a chain of loads and FP64 sums with
// little else in flight; the two take 41 us.
__global__ __launch_bounds__(256) void k_fmm_l2l(FmmDev F, const int *__restrict__ by_depth,
                                                 const int *__restrict__ first, int roots, int depths)
{
    if (F.tot[0]) return;
    for (int d = 0; d < depths; ++d) {
        const int p0 = first[(roots + 1) * d + blockIdx.x], p1 = first[(roots + 1) * d + blockIdx.x + 1];
        for (int p = p0 + threadIdx.x; p < p1; p += blockDim.x) l2l_node(F, by_depth[p]);
        __syncthreads();
    }
}

// P2P of 8 targets in registers against the lane's records of an LDS tile: the
// loop over `cnt` records, `step` bytes apart, of the pair code of pair_f32 (the
// same operations, so the same bits), 4 targets at a time.  By hand for two
// things that the compiler does not do: the reciprocal square roots of
// 4 targets share one raised-priority stretch, and no FMA's accumulator lies in
// the register bank (number mod 4) of one of its multiplicands, where it would
// not issue together with another wave's (a third of the compiler's did).
// Per target t, from v96 + 8 t: dx, dy, dz, r2 then rho, -, m rho, rho^2 then the
// weight (-: free); S + 4 t holds the sums of az, ax, the potential and ay.
#define NB_EACH4(INS) ".irp t,0,1,2,3\n" INS "\n.endr\n"
#define NB_P2P_BATCH(S, X, Y, Z, Q)                                                  \
    NB_EACH4("v_sub_f32 v[96+8*\\t], v[" Q "], v[" X "+\\t]")                        \
    NB_EACH4("v_sub_f32 v[97+8*\\t], v[" Q "+1], v[" Y "+\\t]")                      \
    NB_EACH4("v_sub_f32 v[98+8*\\t], v[" Q "+2], v[" Z "+\\t]")                      \
    NB_EACH4("v_fma_f32 v[99+8*\\t], v[96+8*\\t], v[96+8*\\t], v[103]")              \
    NB_EACH4("v_fmac_f32 v[99+8*\\t], v[97+8*\\t], v[97+8*\\t]")                     \
    NB_EACH4("v_fmac_f32 v[99+8*\\t], v[98+8*\\t], v[98+8*\\t]")                     \
    "s_setprio 1\n"                                                                  \
    NB_EACH4("v_rsq_f32 v[99+8*\\t], v[99+8*\\t]")                                   \
    "s_setprio 0\n"                                                                  \
    NB_EACH4("v_mul_f32 v[102+8*\\t], v[99+8*\\t], v[99+8*\\t]")                     \
    NB_EACH4("v_mul_f32 v[101+8*\\t], v[" Q "+3], v[99+8*\\t]")                      \
    NB_EACH4("v_mul_f32 v[102+8*\\t], v[101+8*\\t], v[102+8*\\t]")                   \
    NB_EACH4("v_fmac_f32 v[" S "+4*\\t+2], v[" Q "+3], v[99+8*\\t]")                 \
    NB_EACH4("v_fmac_f32 v[" S "+4*\\t+1], v[102+8*\\t], v[96+8*\\t]")               \
    NB_EACH4("v_fmac_f32 v[" S "+4*\\t+3], v[102+8*\\t], v[97+8*\\t]")               \
    NB_EACH4("v_fmac_f32 v[" S "+4*\\t], v[102+8*\\t], v[98+8*\\t]")
#define NB_P2P_STEP(Q, P)                                                            \
    "s_waitcnt lgkmcnt(0)\n"                                                         \
    "v_add_u32 %[addr], %[step], %[addr]\n"                                          \
    "ds_read_b128 v[" P ":" P "+3], %[addr]\n"                                       \
    NB_P2P_BATCH("32", "64", "72", "80", Q) NB_P2P_BATCH("48", "68", "76", "84", Q)

constexpr int kTile = 512;  // bodies of a P2P tile
__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

// cnt even; reads one record beyond the last.
__device__ __forceinline__ void p2p_tile8(const float4 *tile, int cnt, int step, Targets<float, 8> &T,
                                          float eps2, Sums<float, 8> &S)
{
    f32x8 x, y, z;
    f32x16 s0, s1;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        x[t] = T.x[t];
        y[t] = T.y[t];
        z[t] = T.z[t];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        s0[4 * t] = S.az[t];
        s0[4 * t + 1] = S.ax[t];
        s0[4 * t + 2] = S.ph[t];
        s0[4 * t + 3] = S.ay[t];
        s1[4 * t] = S.az[t + 4];
        s1[4 * t + 1] = S.ax[t + 4];
        s1[4 * t + 2] = S.ph[t + 4];
        s1[4 * t + 3] = S.ay[t + 4];
    }
    unsigned addr = (unsigned)(size_t)(__attribute__((address_space(3))) const float4 *)tile;
    int turns = cnt / 2;
    asm volatile(
        "ds_read_b128 v[88:91], %[addr]\n"
        ".Lp2p%=:\n"
        NB_P2P_STEP("88", "92") NB_P2P_STEP("92", "88")
        "s_sub_i32 %[turns], %[turns], 1\n"
        "s_cmp_lg_u32 %[turns], 0\n"
        "s_cbranch_scc1 .Lp2p%=\n"
        "s_waitcnt lgkmcnt(0)\n"
        : "+{v[32:47]}"(s0), "+{v[48:63]}"(s1), "+{v[64:71]}"(x), "+{v[72:79]}"(y), "+{v[80:87]}"(z),
          [addr] "+&v"(addr), [turns] "+&s"(turns)  // (the targets pass through, so that one copy of them is live)
        : "{v103}"(eps2), [step] "s"(step)
        : "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95", "v96", "v97", "v98", "v99", "v101", "v102", "v104",
          "v105", "v106", "v107", "v109", "v110", "v112", "v113", "v114", "v115", "v117", "v118", "v120", "v121",
          "v122", "v123", "v125", "v126", "scc", "memory");
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        T.x[t] = x[t];
        T.y[t] = y[t];
        T.z[t] = z[t];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        S.az[t] = s0[4 * t];
        S.ax[t] = s0[4 * t + 1];
        S.ph[t] = s0[4 * t + 2];
        S.ay[t] = s0[4 * t + 3];
        S.az[t + 4] = s1[4 * t];
        S.ax[t + 4] = s1[4 * t + 1];
        S.ph[t + 4] = s1[4 * t + 2];
        S.ay[t + 4] = s1[4 * t + 3];
    }
}

// Leaves: one wave per leaf.  The leaf's P = TPL * NTG target slots (its
// size rounded up to a power of two) form NTG groups of TPL targets; the
// LG = 64 / NTG lanes of a group hold its targets in registers and share its
// sources out, one per lane at a time:
// * P2P, leaves of more than 8 bodies (NTG > 1): through an LDS tile, which each of
//   the NTG groups reads, and the loop of p2p_tile8.  Against the way of the
//   smaller leaves, an FMM force of 300001 bodies (theta 0.5 and 0.6) takes 2119
//   instead of 2268 us with leaves of 16, 2495 instead of 3012 with leaves of
//   32; with leaves of 8, one group, where the tile's LDS traffic is the same per
//   body but serves 8 targets, the two are equal (262144 bodies: 1836 and 1842
//   us), and with leaves of 5 the tile loses 3%.
// * P2P, smaller leaves: up to 64 entries are read at once (a source leaf is stored as its
//   first body; every leaf holds `leaf` bodies except the last, which ends
//   at n); their (entry, body) pairs are numbered e * 2^lb + body and lane v
//   of a group takes v, v + LG, ... (the entry's first body read from the
//   lane that loaded it).  The leaf's own entry is swept apart with the self
//   pair masked.
// * M2P: lane v takes cells v, v + LG, ... as quadrupole cells.
// * Each lane's FP32 partial sums are folded by the precision mode over the
//   group's lanes in lane order (through LDS); each target then adds its
//   leaf's expansion in FP64 and is stored.
template <int MODE, int TPL, int NTG>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(NTG > 1 ? 4 : 1))) void k_fmm_leaf(const float4 *__restrict__ src, FmmDev F,
                                                 const int *__restrict__ leaves, int nleaves, float eps2_in,
                                                 double G, float4 *__restrict__ out, int n, int leaf, int lb)
{
    constexpr int P = TPL * NTG;
    constexpr int LG = 64 / NTG;
    constexpr bool TILE = NTG > 1;  // leaves of more than 8 bodies
    constexpr int UNR = TPL >= 8 ? 2 : (TPL >= 4 ? 4 : 8);  // source loads in flight per lane
    // the P2P tile with the record read beyond it, then the lanes' sums
    __shared__ float4 tile[TILE ? kTile + 64 : 16 * (4 * TPL + 1)];
    float(*const red)[4 * TPL + 1] = (float(*)[4 * TPL + 1]) tile;
    static_assert(sizeof tile >= 64 * sizeof red[0], "the sums of 64 lanes");
    __shared__ double fin[P][4];
    const int w = blockIdx.x;
    if (w >= nleaves || F.tot[0]) return;
    const int lane = threadIdx.x;
    const int g = lane / LG, v = lane % LG;
    const int A = leaves[w];
    const int4 na = F.node[A];
    const int nn = F.nn;
    const float eps2 = lane_copy(eps2_in);
    Targets<float, TPL> T;
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        const int i = na.x + g * TPL + t;
        const float4 p = src[min(i, na.y - 1)];
        T.x[t] = p.x;
        T.y[t] = p.y;
        T.z[t] = p.z;
        T.i[t] = i;
    }
    Sums<float, TPL> S;
    S.zero();
    // P2P
    const int cp = F.cnt[kP2P * nn + A];
    const long op = F.off[kP2P * nn + A];
    const int cpc = (int)min((long)cp, max(0L, F.cap_p2p - op));
    const int bmask = (1 << lb) - 1;
    bool self = false;
    if constexpr (TILE) {
        // Tiles of kTile bodies: the bodies of kTile >> lb entries, gathered 8 per
        // lane.  Where an entry has no body (past the list's or the array's end, the
        // leaf itself) lies a massless record away from every target.
        float most = 0.5f;
#pragma unroll
        for (int t = 0; t < TPL; ++t) most = fmaxf(most, fabsf(T.x[t]));
        most = wave_max(most);
        const float far = most < 1e30f ? 2.0f * most : 1e30f;  // (from where differences would overflow)
        const int per = kTile >> lb;
        auto entries = [&](int base) { return lane < min(per, cpc - base) ? F.p2p[op + base + lane] : -1; };
        int next = entries(0);
        for (int base = 0; base < cpc; base += per) {
            const int k = min(per, cpc - base);
            const int ent = next;
            self = self || __ballot(ent == na.x) != 0ull;
            // (opaque: hoisted out of the loop, the 8 indices would spill)
            int at = lane;
            asm volatile("" : "+v"(at));
            const int sub = at >> lb, body = at & bmask;
            float4 b[kTile / 64];
#pragma unroll
            for (int u = 0; u < kTile / 64; ++u) {
                const int bg = __shfl(ent, u * (64 >> lb) + sub);
                const int len = ((unsigned)bg < (unsigned)n && bg != na.x) ? min(leaf, n - bg) : 0;
                b[u] = src[body < len ? bg + body : 0];
                if (body >= len) b[u] = make_float4(far, 0.0f, 0.0f, 0.0f);
            }
            wave_sync();
#pragma unroll
            for (int u = 0; u < kTile / 64; ++u) tile[u * 64 + lane] = b[u];
            wave_sync();
            next = entries(base + per);
            // records of each lane's: an even number, as many as lie in the tile
            const int cnt = ((k << lb) + 2 * LG - 1) / (2 * LG) * 2;
            p2p_tile8(tile + v, cnt, LG * (int)sizeof(float4), T, eps2, S);
        }
    } else {
        for (int base = 0; base < cpc; base += 64) {
            const int k = min(64, cpc - base);
            const int mybeg = lane < k ? F.p2p[op + base + lane] : -1;
            self = self || __ballot(mybeg == na.x) != 0ull;
            const int npairs = k << lb;
            for (int q0 = 0; q0 < npairs; q0 += LG * UNR) {
                float4 sv[UNR];
                int sj[UNR];
                bool ok[UNR];
#pragma unroll
                for (int r = 0; r < UNR; ++r) {
                    const int q = q0 + r * LG + v;
                    const int bg = __shfl(mybeg, (q >> lb) & 63);
                    const int body = q & bmask;
                    const int len = ((unsigned)bg < (unsigned)n && bg != na.x) ? min(leaf, n - bg) : 0;
                    ok[r] = q < npairs && body < len;
                    sj[r] = bg + body;
                    sv[r] = src[ok[r] ? sj[r] : 0];
                }
#pragma unroll
                for (int r = 0; r < UNR; ++r)
                    if (ok[r]) pair_f32<TPL, false, 1>(sv[r], sj[r], T, eps2, S);
            }
        }
    }
    if (self) {  // the leaf's own bodies, without the self pair
        for (int q = v; q < na.y - na.x; q += LG) pair_f32<TPL, true, 1>(src[na.x + q], na.x + q, T, eps2, S);
    }
    // M2P
    const int cc = F.cnt[kM2P * nn + A];
    const long oc = F.off[kM2P * nn + A];
    const int ccc = (int)min((long)cc, max(0L, F.cap_m2p - oc));
    for (int k = v; k < ccc; k += LG) {
        const int B = F.m2p[oc + k];
        if ((unsigned)B < (unsigned)nn) {
            const float4 *rc = F.qr + (long)kQuadRec * B;
            quad_f32<TPL>(rc[0], rc[1], rc[2], T, eps2, S);
        }
    }
    // fold the group's lanes in lane order
    if constexpr (TILE) __syncthreads();
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
        red[lane][4 * t] = S.ax[t];
        red[lane][4 * t + 1] = S.ay[t];
        red[lane][4 * t + 2] = S.az[t];
        red[lane][4 * t + 3] = S.ph[t];
    }
    __syncthreads();
    for (int s = lane; s < 4 * P; s += 64) {
        const int slot = s >> 2, comp = s & 3;
        const int gg = slot / TPL, t = slot % TPL;
        Run<MODE> R;
        R.zero();
        for (int u = 0; u < LG; ++u) R.fold(red[gg * LG + u][4 * t + comp]);
        fin[slot][comp] = R.get();
    }
    __syncthreads();
    const int i = na.x + lane;
    if (lane >= P || i >= na.y) return;
    double r[4] = {fin[lane][0], fin[lane][1], fin[lane][2], fin[lane][3]};
    // the leaf's expansion at this body, in FP64
    const float4 pt = src[i];
    const double *c = F.loc + 20L * A;
    const double4 ca = F.nrec[A].cd;
    const double y[3] = {(double)pt.x - ca.x, (double)pt.y - ca.y, (double)pt.z - ca.z};
    double ky[3], ty[3][3], tyy[3];
    fmm_contract(c, y, ky, ty, tyy);
    r[0] += c[1] + ky[0] + 0.5 * tyy[0];
    r[1] += c[2] + ky[1] + 0.5 * tyy[1];
    r[2] += c[3] + ky[2] + 0.5 * tyy[2];
    const double py = (c[1] * y[0] + c[2] * y[1]) + c[3] * y[2];
    const double yky = (y[0] * ky[0] + y[1] * ky[1]) + y[2] * ky[2];
    const double ytyy = (y[0] * tyy[0] + y[1] * tyy[1]) + y[2] * tyy[2];
    r[3] += c[0] + py + 0.5 * yky + ytyy / 6.0;
    if constexpr (MODE == M_F32)
        put_f32(out, i, r, (float)G);
    else
        put(out, i, r, G);
}

// Export of one list kind: node a's entries go, in walk order, to
// dst[dst_off[a] ...]; a P2P entry (a leaf's first body) becomes the leaf's
// node id when leaves != nullptr.  One wave per node.
__global__ __launch_bounds__(256) void k_fmm_export(const int *__restrict__ list, const int *__restrict__ cnt,
                                                    const int *__restrict__ off, const long *__restrict__ dst_off,
                                                    int nn, const int *__restrict__ leaves, int leaf,
                                                    int *__restrict__ dst)
{
    const int a = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (a >= nn) return;
    const int c = cnt[a];
    const long o = off[a], t = dst_off[a];
    for (int k = lane; k < c; k += 64) {
        const int v = list[o + k];
        dst[t + k] = leaves ? leaves[v / leaf] : v;
    }
}

__global__ void k_fmm_zero_tot(unsigned long long *tot, int count)
{
    for (int k = threadIdx.x; k < count; k += blockDim.x) tot[k] = 0ull;
}

// ---- host side -----------------------------------------------------------------
struct FmmPlan {
    int n = 0, leaf = 0, dev = -1, nn = 0, depth = 0, max_level = 0;
    int stack = 0;  // LDS stack entries that a walking wave needs at this height
    std::vector<int> parent, by_depth, depth_off;
    int *d_parent = nullptr, *d_by_depth = nullptr, *d_leaves = nullptr;
    // L2L: the depth whose nodes are the second launch's subtrees, and for both
    // launches the subtrees' positions (see k_fmm_l2l; the first launch's first)
    int l2l_depth = 0, l2l_roots = 0;
    int *d_l2l = nullptr;
};

struct FmmBufs {
    int dev = -1, nn = 0, nblk = 0;
    long cap[kKinds] = {0, 0, 0, 0};
    int *cnt = nullptr, *lcnt = nullptr, *off = nullptr, *list[3] = {nullptr, nullptr, nullptr};
    int *pass0 = nullptr, *pass1 = nullptr;
    long *bsum = nullptr;
    unsigned long long *tot = nullptr;
    unsigned long long *flag = nullptr;  // pinned
    hipEvent_t listed = nullptr;         // after the kernel that writes it
    float *own = nullptr;
    double *loc = nullptr;
};

// One-pass slot layout for the current plan: per depth, the room of each
// list per node (grown from the exact counts whenever a walk overflowed).
struct SlotPlan {
    int nn = 0, dev = -1;
    std::vector<SlotDepth> depth;
    long total[kKinds] = {0, 0, 0, 0};  // slots per list kind (pass-down: the larger ping-pong half)
    bool disabled = false;              // the layout outgrew its memory budget: count, scan and fill
    long budget = 0;                    // entries the layout may take: an eighth of the device's memory,
                                        // or NBODY_FMM_SLOT_MB MiB if that is less
};

std::mutex g_fmm_mu;
FmmPlan g_plan;
FmmBufs g_bufs;
SlotPlan g_slots;

void free_plan(FmmPlan &p)
{
    (void)hipFree(p.d_parent);
    (void)hipFree(p.d_by_depth);
    (void)hipFree(p.d_leaves);
    (void)hipFree(p.d_l2l);
    p = FmmPlan();
}

void free_bufs(FmmBufs &b)
{
    (void)hipFree(b.cnt);
    (void)hipFree(b.lcnt);
    (void)hipFree(b.off);
    for (int *l : b.list) (void)hipFree(l);
    (void)hipFree(b.pass0);
    (void)hipFree(b.pass1);
    (void)hipFree(b.bsum);
    (void)hipFree(b.tot);
    (void)hipHostFree(b.flag);
    if (b.listed) (void)hipEventDestroy(b.listed);
    (void)hipFree(b.own);
    (void)hipFree(b.loc);
    b = FmmBufs();
}

int make_plan(const HostTree &h, int n, int leaf, int dev, hipStream_t s)
{
    FmmPlan &p = g_plan;
    if (p.d_parent && p.n == n && p.leaf == leaf && p.dev == dev) return NBODY_OK;
    if (p.d_parent) {
        (void)hipDeviceSynchronize();  // enqueued work may still read the old tables
        free_plan(p);
    }
    const int nn = (int)h.node.size();
    if (64 * (h.height[0] + 2) > kWalkStack || h.height[0] + 2 > kFmmStack) {
        set_error("tree height %d too large for the FMM traversal stack", h.height[0]);
        return NBODY_E_UNSUPPORTED;
    }
    p.stack = 64 * (h.height[0] + 2);
    p.parent.assign(nn, -1);
    std::vector<int> dep(nn, 0);
    for (int a = 0; a < nn; ++a) {  // preorder: parents come first
        const int4 nd = h.node[a];
        if (nd.z >= 0) {
            p.parent[nd.z] = p.parent[nd.w] = a;
            dep[nd.z] = dep[nd.w] = dep[a] + 1;
        }
    }
    p.depth = *std::max_element(dep.begin(), dep.end());
    p.depth_off.assign(p.depth + 2, 0);
    for (int v : dep) ++p.depth_off[v + 1];
    p.max_level = 0;
    for (int k = 0; k <= p.depth; ++k) {
        p.max_level = std::max(p.max_level, p.depth_off[k + 1]);
        p.depth_off[k + 1] += p.depth_off[k];
    }
    p.by_depth.assign(nn, 0);
    std::vector<int> pos(p.depth_off.begin(), p.depth_off.end() - 1);
    for (int a = 0; a < nn; ++a) p.by_depth[pos[dep[a]]++] = a;
    // the L2L launches' tables: one subtree from the root down to the depth of kL2lRoots nodes, then that depth's
    p.l2l_depth = 0;
    while (p.l2l_depth < p.depth && p.depth_off[p.l2l_depth + 1] - p.depth_off[p.l2l_depth] < kL2lRoots) ++p.l2l_depth;
    p.l2l_roots = p.depth_off[p.l2l_depth + 1] - p.depth_off[p.l2l_depth];
    std::vector<int> l2l;
    for (int k = 0; k <= p.l2l_depth; ++k) {
        l2l.push_back(p.depth_off[k]);
        l2l.push_back(p.depth_off[k + 1]);
    }
    for (int k = p.l2l_depth + 1; k <= p.depth; ++k) {
        // the depth order is the preorder within a depth: each root's nodes follow one another
        const auto b = p.by_depth.begin() + p.depth_off[k], e = p.by_depth.begin() + p.depth_off[k + 1];
        for (int r = 0; r < p.l2l_roots; ++r)
            l2l.push_back((int)(std::lower_bound(b, e, p.by_depth[p.depth_off[p.l2l_depth] + r]) - p.by_depth.begin()));
        l2l.push_back(p.depth_off[k + 1]);
    }
    const size_t nl = h.leaves.size();
    if (hipMalloc(&p.d_parent, nn * sizeof(int)) != hipSuccess ||
        hipMalloc(&p.d_by_depth, nn * sizeof(int)) != hipSuccess ||
        hipMalloc(&p.d_leaves, nl * sizeof(int)) != hipSuccess ||
        hipMalloc(&p.d_l2l, l2l.size() * sizeof(int)) != hipSuccess) {
        free_plan(p);
        set_error("cannot allocate the FMM plan");
        return NBODY_E_NOMEM;
    }
    hipError_t e = hipMemcpyAsync(p.d_parent, p.parent.data(), nn * sizeof(int), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(p.d_by_depth, p.by_depth.data(), nn * sizeof(int), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(p.d_leaves, h.leaves.data(), nl * sizeof(int), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(p.d_l2l, l2l.data(), l2l.size() * sizeof(int), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        free_plan(p);
        return hip_fail(e, "FMM plan upload");
    }
    p.n = n;
    p.leaf = leaf;
    p.dev = dev;
    p.nn = nn;
    return NBODY_OK;
}

hipError_t launch_l2l(const FmmDev &F, const FmmPlan &p, hipStream_t s)
{
    hipLaunchKernelGGL(k_fmm_l2l, dim3(1), dim3(256), 0, s, F, p.d_by_depth, p.d_l2l, 1, p.l2l_depth + 1);
    if (p.depth > p.l2l_depth)
        hipLaunchKernelGGL(k_fmm_l2l, dim3(p.l2l_roots), dim3(256), 0, s, F, p.d_by_depth,
                           p.d_l2l + 2 * (p.l2l_depth + 1), p.l2l_roots, p.depth - p.l2l_depth);
    return hipGetLastError();
}

// Buffers for nn nodes (at most max_level on one depth) with at least the
// given list capacities (M2L, P2P, M2P, pass-down).
int make_bufs(int nn, int max_level, int dev, const long (&want)[kKinds])
{
    FmmBufs &b = g_bufs;
    const int nblk = std::max(1, (max_level + kScanBlock - 1) / kScanBlock);
    bool fits = b.cnt && b.dev == dev && b.nn >= nn && b.nblk >= nblk;
    for (int q = 0; q < kKinds; ++q) fits = fits && b.cap[q] >= want[q];
    if (fits) return NBODY_OK;
    long cap[kKinds];
    for (int q = 0; q < kKinds; ++q) cap[q] = std::max(want[q], b.dev == dev ? b.cap[q] : 0L);
    nn = std::max(nn, b.dev == dev ? b.nn : 0);
    const int nb = std::max(nblk, b.dev == dev ? b.nblk : 0);
    if (b.cnt) {
        (void)hipDeviceSynchronize();
        free_bufs(b);
    }
    const size_t per = kKinds * (size_t)nn * sizeof(int);
    bool ok = hipMalloc(&b.cnt, per) == hipSuccess && hipMalloc(&b.lcnt, per) == hipSuccess &&
              hipMalloc(&b.off, per) == hipSuccess;
    for (int q = 0; q < 3 && ok; ++q) ok = hipMalloc(&b.list[q], (size_t)cap[q] * sizeof(int)) == hipSuccess;
    ok = ok && hipMalloc(&b.pass0, (size_t)cap[kPass] * sizeof(int)) == hipSuccess &&
         hipMalloc(&b.pass1, (size_t)cap[kPass] * sizeof(int)) == hipSuccess &&
         hipMalloc(&b.bsum, (size_t)nb * kKinds * sizeof(long)) == hipSuccess &&
         hipMalloc(&b.tot, kTotWords * sizeof(unsigned long long)) == hipSuccess &&
         hipHostMalloc(&b.flag, sizeof(unsigned long long)) == hipSuccess &&
         hipEventCreateWithFlags(&b.listed, hipEventDisableTiming) == hipSuccess &&
         hipMalloc(&b.own, 20 * (size_t)nn * sizeof(float)) == hipSuccess &&
         hipMalloc(&b.loc, 20 * (size_t)nn * sizeof(double)) == hipSuccess;
    if (!ok) {
        free_bufs(b);
        set_error("cannot allocate FMM lists (%ld M2L, %ld P2P, %ld M2P, %ld pass-down entries)", cap[kM2L],
                  cap[kP2P], cap[kM2P], cap[kPass]);
        return NBODY_E_NOMEM;
    }
    b.dev = dev;
    b.nn = nn;
    b.nblk = nb;
    for (int q = 0; q < kKinds; ++q) b.cap[q] = cap[q];
    return NBODY_OK;
}

FmmDev dev_view(const TreeDev &d, const FmmPlan &p, const FmmBufs &b)
{
    FmmDev F;
    F.node = d.node;
    F.nrec = d.nrec;
    F.lo = d.lo;
    F.hi = d.hi;
    F.qr = d.qr;
    F.parent = p.d_parent;
    F.nn = p.nn;
    F.cnt = b.cnt;
    F.lcnt = b.lcnt;
    F.off = b.off;
    F.m2l = b.list[kM2L];
    F.p2p = b.list[kP2P];
    F.m2p = b.list[kM2P];
    F.pass0 = b.pass0;
    F.pass1 = b.pass1;
    F.cap_m2l = b.cap[kM2L];
    F.cap_p2p = b.cap[kP2P];
    F.cap_m2p = b.cap[kM2P];
    F.cap_pass = b.cap[kPass];
    F.bsum = b.bsum;
    F.tot = b.tot;
    F.flag = b.flag;
    F.own = b.own;
    F.loc = b.loc;
    return F;
}

// The traversal: count, scan and fill per depth.
hipError_t launch_traversal(const FmmDev &F, const FmmPlan &p, double theta2, hipStream_t s)
{
    hipLaunchKernelGGL(k_fmm_zero_tot, dim3(1), dim3(256), 0, s, F.tot, kTotWords);
    hipError_t e = hipGetLastError();
    for (int d = 0; d <= p.depth && e == hipSuccess; ++d) {
        const int first = p.depth_off[d], count = p.depth_off[d + 1] - first;
        const int *ids = p.d_by_depth + first;
        const int nblk = (count + kScanBlock - 1) / kScanBlock;
        launch_walk_depth<kWalkCount>(F, ids, first, count, p.stack, d & 1, theta2, SlotDepth{}, s);
        hipLaunchKernelGGL(k_fmm_scan_part, dim3(nblk), dim3(256), 0, s, F, first, count);
        hipLaunchKernelGGL(k_fmm_scan_fin, dim3(nblk), dim3(256), 0, s, F, ids, first, count, d, nblk);
        launch_walk_depth<kWalkFill>(F, ids, first, count, p.stack, d & 1, theta2, SlotDepth{}, s);
        e = hipGetLastError();
    }
    return e;
}

// The one-pass traversal: one walk per depth into the slots of g_slots.
hipError_t launch_traversal_slots(const FmmDev &F, const FmmPlan &p, double theta2, hipStream_t s)
{
    hipLaunchKernelGGL(k_fmm_zero_tot, dim3(1), dim3(256), 0, s, F.tot, kTotWords);
    hipError_t e = hipGetLastError();
    for (int d = 0; d <= p.depth && e == hipSuccess; ++d) {
        const int first = p.depth_off[d], count = p.depth_off[d + 1] - first;
        launch_walk_depth<kWalkSlot>(F, p.d_by_depth + first, first, count, p.stack, d & 1, theta2, g_slots.depth[d],
                                     s);
        e = hipGetLastError();
    }
    return e;
}

// Sets the slot layout from per-depth rooms: cap[d][k] entries per node.
void slots_layout(const FmmPlan &p, const std::vector<std::array<long, kKinds>> &cap)
{
    SlotPlan &S = g_slots;
    S.depth.assign(p.depth + 1, SlotDepth{});
    for (int k = 0; k < kKinds; ++k) S.total[k] = 0;
    for (int d = 0; d <= p.depth; ++d) {
        const long cnt = p.depth_off[d + 1] - p.depth_off[d];
        SlotDepth &sd = S.depth[d];
        for (int k = 0; k < kKinds; ++k) {
            sd.cap[k] = (int)cap[d][k];
            if (k == kPass) {
                sd.base[k] = 0;  // each depth starts its ping-pong half at 0
                S.total[k] = std::max(S.total[k], cnt * cap[d][k]);
            } else {
                sd.base[k] = S.total[k];
                S.total[k] += cnt * cap[d][k];
            }
        }
        sd.prev_pass = d > 0 ? (int)cap[d - 1][kPass] : 0;
    }
}

// Rooms for a first attempt: modest guesses where a depth has the nodes a
// list needs (inner nodes pass down, leaves take M2P and P2P), none elsewhere.
void slots_initial(const FmmPlan &p, const HostTree &h)
{
    std::vector<std::array<long, kKinds>> cap(p.depth + 1);
    for (int d = 0; d <= p.depth; ++d) {
        bool inner = false, leafy = false;
        for (int q = p.depth_off[d]; q < p.depth_off[d + 1]; ++q) (h.node[p.by_depth[q]].z < 0 ? leafy : inner) = true;
        cap[d] = {128, leafy ? 512 : 0, leafy ? 64 : 0, inner ? 512 : 0};
    }
    slots_layout(p, cap);
    g_slots.nn = p.nn;
    g_slots.dev = p.dev;
    g_slots.disabled = false;
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) total_b = 0;
    g_slots.budget = (long)(total_b / 8 / sizeof(int));
    if (const char *mb = std::getenv("NBODY_FMM_SLOT_MB"))  // a smaller budget, in MiB
        g_slots.budget = std::min(g_slots.budget, std::max(0L, std::atol(mb)) * (1L << 20) / (long)sizeof(int));
}

// Entries the current slot layout needs (both pass-down halves).
long slots_need()
{
    long need = 0;
    for (int k = 0; k < kKinds; ++k) need += (k == kPass ? 2 : 1) * g_slots.total[k];
    return need;
}

// After an overflow: every room becomes at least the largest count of its
// depth (exact up to the first depth whose pass-down lists overflowed) plus
// an eighth.  Returns false when the layout would pass its memory budget.
bool slots_regrow(const FmmPlan &p, const std::vector<int> &cnt, long budget_entries)
{
    const int nn = p.nn;
    std::vector<std::array<long, kKinds>> cap(p.depth + 1);
    long need = 0;
    for (int d = 0; d <= p.depth; ++d) {
        for (int k = 0; k < kKinds; ++k) {
            long mx = 0;
            for (int q = p.depth_off[d]; q < p.depth_off[d + 1]; ++q)
                mx = std::max(mx, (long)cnt[(size_t)k * nn + p.by_depth[q]]);
            const long old = g_slots.depth[d].cap[k];
            cap[d][k] = mx > old ? mx + mx / 8 + 8 : old;
        }
    }
    const auto saved = g_slots.depth;
    long saved_total[kKinds];
    std::copy(g_slots.total, g_slots.total + kKinds, saved_total);
    slots_layout(p, cap);
    for (int k = 0; k < kKinds; ++k) need += (k == kPass ? 2 : 1) * g_slots.total[k];
    bool ok = need <= budget_entries;
    for (int k = 0; k < kKinds; ++k) ok = ok && g_slots.total[k] <= (long)INT32_MAX;
    if (!ok) {  // keep the old layout; the caller falls back to count, scan and fill
        g_slots.depth = saved;
        std::copy(saved_total, saved_total + kKinds, g_slots.total);
    }
    return ok;
}

template <int MODE>
hipError_t launch_leaves_mode(const float4 *pm, const FmmDev &F, const FmmPlan &p, int nleaves, int n, int leaf,
                              float eps2, double G, float4 *out, hipStream_t s)
{
    int lb = 0;
    while ((1 << lb) < leaf) ++lb;
    const dim3 grid(nleaves), blk(64);
#define NB_FMM_LEAF(TPL, NTG)                                                                                  \
    hipLaunchKernelGGL((k_fmm_leaf<MODE, TPL, NTG>), grid, blk, 0, s, pm, F, p.d_leaves, nleaves, eps2, G, out, \
                       n, leaf, lb)
    switch (lb) {
    case 0: NB_FMM_LEAF(1, 1); break;
    case 1: NB_FMM_LEAF(2, 1); break;
    case 2: NB_FMM_LEAF(4, 1); break;
    case 3: NB_FMM_LEAF(8, 1); break;
    case 4: NB_FMM_LEAF(8, 2); break;
    case 5: NB_FMM_LEAF(8, 4); break;
    default: NB_FMM_LEAF(8, 8); break;
    }
#undef NB_FMM_LEAF
    return hipGetLastError();
}

// Final list totals (M2L, P2P, M2P) after the deepest depth.
void list_totals(const unsigned long long *tot, int depth, unsigned long long (&out)[3])
{
    for (int q = 0; q < 3; ++q) out[q] = tot[tot_at(q, depth + 1)];
}

// M2L, which tells the host whether the lists fit (g_bufs.listed), L2L and the
// leaves; all of them only if the lists fit.
hipError_t launch_evaluation(const FmmDev &F, const FmmPlan &p, const float4 *pm, int n, int prec, double G, double eps,
                             int leaf, int nleaves, float4 *out, hipStream_t s)
{
    const float eps2 = (float)(eps * eps);
    hipLaunchKernelGGL(k_fmm_m2l, dim3(p.nn), dim3(64), 0, s, F, eps2);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipEventRecord(g_bufs.listed, s);
    if (e == hipSuccess) e = launch_l2l(F, p, s);
    if (e != hipSuccess) return e;
    switch (prec) {
    case NBODY_F32: return launch_leaves_mode<M_F32>(pm, F, p, nleaves, n, leaf, eps2, G, out, s);
    case NBODY_F32_KAHAN: return launch_leaves_mode<M_KAHAN>(pm, F, p, nleaves, n, leaf, eps2, G, out, s);
    default: return launch_leaves_mode<M_F64ACC>(pm, F, p, nleaves, n, leaf, eps2, G, out, s);
    }
}

// Runs the traversal until the lists fit their buffers, with out != nullptr each
// time followed by the evaluation; the host waits until the lists are known to
// fit, not for the evaluation.
// Called with the tree and FMM locks held.
int fmm_run(const void *pm, int n, int prec, double G, double eps, double theta, int leaf, void *out,
            hipStream_t s, TreeDev &d, const HostTree *&h)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        set_error("hipGetDevice failed");
        return NBODY_E_HIP;
    }
    if (leaf > 64) {
        set_error("the FMM takes leaves of at most 64 bodies");
        return NBODY_E_INVAL;
    }
    NB_CHECK_RC(tree_quad_prepare(pm, n, leaf, s, d, h));
    NB_CHECK_RC(make_plan(*h, n, leaf, dev, s));
    const FmmPlan &p = g_plan;
    const int nn = p.nn;
    const int nleaves = (int)h->leaves.size();
    long want[kKinds] = {std::max(1024L, 64L * nn), std::max(1024L, 512L * nleaves), std::max(1024L, 16L * nleaves),
                         std::max(1024L, 16L * nn)};
    if (g_bufs.dev == dev)
        for (int q = 0; q < kKinds; ++q) want[q] = std::max(want[q], g_bufs.cap[q]);
    // One pass into per-node slots while the layout fits its budget;
    // otherwise count, scan and fill into compact lists.
    if (g_slots.nn != nn || g_slots.dev != dev || (int)g_slots.depth.size() != p.depth + 1) slots_initial(p, *h);
    bool slots = !g_slots.disabled && slots_need() <= g_slots.budget;
    // A pass-down list that overflowed truncates what the depths below it see,
    // so each attempt makes at least one more depth exact.
    for (int attempt = 0; attempt < p.depth + 16; ++attempt) {
        if (slots)
            for (int q = 0; q < kKinds; ++q) want[q] = std::max(want[q], std::max(1024L, g_slots.total[q]));
        NB_CHECK_RC(make_bufs(nn, p.max_level, dev, want));
        const FmmDev F = dev_view(d, p, g_bufs);
        hipError_t e = slots ? launch_traversal_slots(F, p, theta * theta, s) : launch_traversal(F, p, theta * theta, s);
        if (e != hipSuccess) return hip_fail(e, "FMM traversal");
        if (out) {
            // The evaluation follows without waiting for the host to see that the
            // lists fit: where they did not, its kernels do nothing and the lists are made again.
            e = launch_evaluation(F, p, (const float4 *)pm, n, prec, G, eps, leaf, nleaves, (float4 *)out, s);
            if (e != hipSuccess) return hip_fail(e, "FMM kernels");
            e = hipEventSynchronize(g_bufs.listed);
            if (e != hipSuccess) return hip_fail(e, "FMM list check");
            if (!*(volatile unsigned long long *)g_bufs.flag) return NBODY_OK;
        }
        unsigned long long tot[kTotWords];
        e = hipMemcpyAsync(tot, g_bufs.tot, sizeof tot, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return hip_fail(e, "FMM list check");
        if (!tot[0]) return NBODY_OK;  // (inspection: the lists fit)
        if (slots) {  // resize the slots from the exact counts and run again
            std::vector<int> cnt(kKinds * (size_t)nn);
            e = hipMemcpyAsync(cnt.data(), g_bufs.cnt, cnt.size() * sizeof(int), hipMemcpyDeviceToHost, s);
            if (e == hipSuccess) e = hipStreamSynchronize(s);
            if (e != hipSuccess) return hip_fail(e, "FMM count download");
            if (!slots_regrow(p, cnt, g_slots.budget)) {
                slots = false;
                g_slots.disabled = true;
            }
            continue;
        }
        // Grow what overflowed and run again.  The totals are exact up to the
        // first depth whose pass-down list overflowed and short beyond it, so
        // every attempt makes at least one more depth exact.
        unsigned long long pass_max = 0, lt[3];
        bool pass_over = false;
        for (int dd = 0; dd <= p.depth; ++dd) {
            pass_max = std::max(pass_max, tot[tot_at(kPass, dd)]);
            pass_over = pass_over || tot[tot_at(kPass, dd)] > (unsigned long long)g_bufs.cap[kPass];
        }
        list_totals(tot, p.depth, lt);
        auto grow = [](long cap, unsigned long long need, bool doubled) {
            long w = std::max(cap, (long)std::min<unsigned long long>(need + need / 4 + 1024, 1ull << 40));
            return doubled ? std::max(w, 2 * cap) : w;
        };
        want[kPass] = grow(g_bufs.cap[kPass], pass_max, pass_over);
        for (int q = 0; q < 3; ++q) want[q] = grow(g_bufs.cap[q], lt[q], false);
        for (int q = 0; q < kKinds; ++q)
            if (want[q] > (long)INT32_MAX) {
                set_error("FMM lists beyond 2^31 entries (M2L %llu, P2P %llu, M2P %llu, pass-down %llu counted so "
                          "far; theta too small for this n and leaf)",
                          lt[0], lt[1], lt[2], pass_max);
                return NBODY_E_UNSUPPORTED;
            }
    }
    set_error("FMM lists did not fit after repeated growth");
    return NBODY_E_NOMEM;
}

}  // namespace

int fmm_accel(const void *pm, int n, int prec, double G, double eps, double theta, int leaf, void *out,
              hipStream_t s)
{
    std::lock_guard<std::mutex> lt(tree_mutex());
    std::lock_guard<std::mutex> lf(g_fmm_mu);
    TreeDev d;
    const HostTree *h = nullptr;
    return fmm_run(pm, n, prec, G, eps, theta, leaf, out, s, d, h);
}

int fmm_lists(const void *pm, int n, int leaf, double theta, int32_t *const cnt_out[3], int32_t *const ids_out[3],
              const int64_t caps[3], hipStream_t s)
{
    std::lock_guard<std::mutex> lt(tree_mutex());
    std::lock_guard<std::mutex> lf(g_fmm_mu);
    TreeDev d;
    const HostTree *h = nullptr;
    NB_CHECK_RC(fmm_run(pm, n, NBODY_F32, 1.0, 0.0, theta, leaf, nullptr, s, d, h));
    const int nn = g_plan.nn;
    std::vector<int> cnt(kKinds * (size_t)nn), off(kKinds * (size_t)nn);
    hipError_t e = hipMemcpyAsync(cnt.data(), g_bufs.cnt, cnt.size() * sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(off.data(), g_bufs.off, off.size() * sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "FMM list download");
    long tl[3] = {0, 0, 0};  // list totals (M2L, P2P, M2P) from the per-node counts
    for (int q = 0; q < 3; ++q)
        for (int a = 0; a < nn; ++a) tl[q] += cnt[(size_t)q * nn + a];
    // the public order is (M2L, M2P, P2P)
    const int kind_of[3] = {kM2L, kM2P, kP2P};
    for (int w = 0; w < 3; ++w) {
        e = hipMemcpyAsync(cnt_out[w], cnt.data() + (size_t)kind_of[w] * nn, nn * sizeof(int), hipMemcpyHostToDevice,
                           s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return hip_fail(e, "FMM count upload");
    }
    for (int w = 0; w < 3; ++w) {
        const int q = kind_of[w];
        int32_t *dst = ids_out[w];
        if (!dst) continue;
        const long total = (long)tl[q];
        if (total > caps[w]) {
            static const char *names[3] = {"M2L", "M2P", "P2P"};
            set_error("%s list of %ld entries exceeds the capacity %lld", names[w], total, (long long)caps[w]);
            return NBODY_E_INVAL;
        }
        std::vector<long> dst_off(nn);
        long o = 0;
        for (int a = 0; a < nn; ++a) {  // node order, each node's entries in walk order
            dst_off[a] = o;
            o += cnt[(size_t)q * nn + a];
        }
        long *d_off = nullptr;
        e = hipMalloc(&d_off, (size_t)nn * sizeof(long));
        if (e == hipSuccess) e = hipMemcpyAsync(d_off, dst_off.data(), (size_t)nn * sizeof(long), hipMemcpyHostToDevice, s);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(k_fmm_export, dim3((nn + 3) / 4), dim3(256), 0, s, g_bufs.list[q],
                               g_bufs.cnt + (size_t)q * nn, g_bufs.off + (size_t)q * nn, (const long *)d_off, nn,
                               q == kP2P ? (const int *)g_plan.d_leaves : nullptr, leaf, dst);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        (void)hipFree(d_off);
        if (e != hipSuccess) return hip_fail(e, "FMM list export");
    }
    return NBODY_OK;
}

void fmm_release()
{
    std::lock_guard<std::mutex> lf(g_fmm_mu);
    free_plan(g_plan);
    free_bufs(g_bufs);
    g_slots = SlotPlan();
}

}  // namespace nbi
