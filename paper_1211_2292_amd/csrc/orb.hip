// Orthogonal Recursive Bisection order on the device (gfx950).
//
// The paper (Section IV.B) divides space into non-overlapping sub-spaces
// holding about equal numbers of bodies by recursive bisection.  Here the
// recursion is carried down to leaves of at most `leaf` bodies and used as a
// body ordering on one device.  The split rule (see nbody.h) depends only on
// the set of bodies in a segment, and the segment sizes depend only on
// (n, leaf), so:
//   * the host computes the whole segment tree (sizes and left counts) once;
//   * the device only decides which bodies go left, by finding the k-th
//     smallest 64-bit key (total-order FP32 coordinate, original index) of
//     each segment exactly, by histograms and rank;
//   * bodies may be partitioned in any order, because every later decision
//     depends on set membership only and every leaf is finally sorted by
//     original index.
// Phase A handles segments larger than kSmall bodies, one level of the tree
// per step, with multi-workgroup kernels over fixed-size chunks.  The three
// axes' keys travel with the index array (two buffers, read and written in
// turn), so every pass reads them coalesced.  A level is: two to four
// histogram passes over the segment's own key range (k_orb_hist; the workgroup
// that finishes a segment picks the bin), one pass that ranks the few keys of
// the last bin (k_orb_pick), and the partition (k_orb_partition), which also
// accumulates each part's key box for the next level.  Phase B (k_orb_block)
// finishes every remaining segment (at most kSmall bodies) inside one
// workgroup: the segment's keys are loaded into LDS once, all nodes of a depth
// are split together, nodes of at most 64 bodies are finished by one wave each,
// and the final order is written.
#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>

#include "internal.h"

namespace nbi {

// Phase A splits segments larger than this: as many as fit phase B's LDS.  A level
// of phase A takes 33 us at 2^20 bodies, one of phase B 10.
constexpr int kSmall = 4096;
constexpr int kMaxBlockSeg = 4096;  // largest leaf
constexpr int kChunk = 4096;        // elements per phase-A workgroup
constexpr int kOrbBlock = 256;
constexpr int kFinBlock = 1024;     // threads of a phase-B workgroup
constexpr int kChunkPer = kChunk / kOrbBlock;  // elements per thread of a phase-A workgroup

namespace {

__device__ __forceinline__ uint32_t tkey(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float untkey(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k);
}

// axis of largest FP32 extent fl32(max - min), ties to the lowest axis
__device__ __forceinline__ int pick_axis(const uint32_t *bb)
{
    float ext[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) ext[a] = untkey(bb[3 + a]) - untkey(bb[a]);
    int axis = 0;
    if (ext[1] > ext[axis]) axis = 1;
    if (ext[2] > ext[axis]) axis = 2;
    return axis;
}

// Total-order keys of the FP32 coordinates in the current order (identity at
// the start).
template <typename V>
__global__ __launch_bounds__(kOrbBlock) void k_orb_coords(const V *__restrict__ pm, int n,
                                                          uint32_t *__restrict__ keys,
                                                          int32_t *__restrict__ cur)
{
    const int i = blockIdx.x * kOrbBlock + threadIdx.x;
    if (i >= n) return;
    const V p = pm[i];
    const float f[3] = {(float)p.x, (float)p.y, (float)p.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) keys[(size_t)a * n + i] = tkey(f[a]);
    cur[i] = i;
}

// Selection of a segment's k-th key (coordinate key in the high half, index in
// the low half): a window of keys [from, from + 2^bits), at first from the
// smallest coordinate to the largest, is divided into kBins bins, the bin that
// holds the k-th key is the next window, and so on; once it holds at most
// kPick keys, or after the last round, one pass gathers and ranks them.  A pass is
// a chain of a few round trips to memory, whatever it counts, so what matters is
// how many there are: four rounds over the coordinate's digits from the top, whose
// first eight bits hardly tell a segment's bodies apart, and a pass for equal
// coordinates took 27 us a level at 2^20 bodies; two rounds over the segment's own
// range, two skipped ones and the pick take 22, without the skipped ones 17.
// (kPick of 32 and 512: 3% and 7% slower.)
constexpr int kDigit = 8;
constexpr int kBins = 1 << kDigit;
constexpr int kRounds = 4;
// The histogram, pick and partition passes run 512 threads per chunk: more
// waves per CU to hide their latency, without more workgroups per segment.
constexpr int kPassBlock = 512;
constexpr int kPassPer = kChunk / kPassBlock;
constexpr int kPick = 128;
constexpr int kPickDigit = 10, kPickBins = 1 << kPickDigit;  // the pick's own rounds
static_assert(kPickBins == 2 * kPassBlock, "two bins per thread");
// Two rounds nearly always leave a few keys.  Where they don't (a dense cluster in
// a wide box, few distinct coordinates), one workgroup takes the rest, which is
// slow for many keys: levels of long segments take up to two rounds more, which
// cost 2.5 us each where every segment is done.  (100000 bodies: 225 us for the
// order with two rounds for short segments, 232 with three.)
constexpr int kShortRounds = 2;
constexpr int kLongSegment = 65536;
static_assert(kBins <= kPassBlock, "one bin per thread");

__device__ __forceinline__ uint64_t body_key(uint32_t key, int32_t id) { return ((uint64_t)key << 32) | (uint32_t)id; }

struct Window {
    uint64_t from;
    int bits;
    __device__ bool holds(uint64_t key) const { return bits == 64 || ((key - from) >> bits) == 0; }
    // the bins of 2^shift keys
    __device__ int shift() const { return max(bits - kDigit, 0); }
    __device__ int bin(uint64_t key) const { return (int)((key - from) >> shift()); }
    __device__ Window of_bin(int b) const { return {from + ((uint64_t)b << shift()), shift()}; }
};

// Per-segment state of one phase-A level.
struct SegState {
    uint32_t bb[6];    // min keys x,y,z then max keys x,y,z
    int krem;          // rank still to find inside the window
    int pick;          // the window's keys are few enough to be ranked
    Window win;        // from the second round on
    uint64_t kth;      // the k-th key
    uint64_t placed;   // partition: bodies placed (high half) and placed left (low half)
    uint32_t arrived;  // workgroups of the current pass done with the segment
    uint32_t picked;   // bodies gathered (k_orb_pick)
};

__device__ __forceinline__ void init_state(SegState *st, int k)
{
    SegState z;
    for (int a = 0; a < 3; ++a) {
        z.bb[a] = 0xFFFFFFFFu;
        z.bb[3 + a] = 0u;
    }
    z.krem = k;
    z.pick = 0;
    z.win = {0, 0};
    z.kth = 0;
    z.placed = 0;
    z.arrived = 0;
    z.picked = 0;
    *st = z;
}

// the segment's split axis, from its key box (complete once the pass that
// accumulated it has ended)
__device__ __forceinline__ int seg_axis(const SegState *st)
{
    uint32_t bb[6];
#pragma unroll
    for (int a = 0; a < 6; ++a) bb[a] = st->bb[a];
    return pick_axis(bb);
}

// Tables: segs (start, size, k) per segment of a level, chunks (segment,
// begin, end), kids (next-level segment of the left and of the right part,
// -1 where that part is finished by phase B).
// First level: its states, and every histogram row cleared (the passes
// leave them cleared after that).  One workgroup per row.
__global__ __launch_bounds__(kOrbBlock) void k_orb_init(const int3 *__restrict__ segs, int nseg,
                                                        SegState *__restrict__ st,
                                                        uint32_t *__restrict__ hist)
{
    const int s = blockIdx.x;
    if (s < nseg && threadIdx.x == 0) init_state(&st[s], segs[s].z);
    for (int j = threadIdx.x; j < kBins; j += kOrbBlock) hist[(size_t)s * kBins + j] = 0u;
}

// Cross-lane moves as operands (DPP): a step of a few clocks, where a shuffle is
// a round trip to the LDS.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);  // (every lane has a source)
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppMirror = 0x140, kDppHalfMirror = 0x141;

// v over the group of W lanes (aligned, a power of two), in every lane of it
template <int W, typename OP>
__device__ __forceinline__ uint32_t group_reduce(uint32_t v, OP op)
{
    if constexpr (W >= 2) v = op(v, dpp<kDppXor1>(v));
    if constexpr (W >= 4) v = op(v, dpp<kDppXor2>(v));
    if constexpr (W >= 8) v = op(v, dpp<kDppHalfMirror>(v));
    if constexpr (W >= 16) v = op(v, dpp<kDppMirror>(v));
    if constexpr (W >= 32) {
        const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = op(p[0], p[1]);
    }
    if constexpr (W >= 64) {
        const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = op(p[0], p[1]);
    }
    return v;
}

__device__ __forceinline__ uint32_t wave_min(uint32_t v)
{
    return group_reduce<64>(v, [](uint32_t x, uint32_t y) { return min(x, y); });
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    return group_reduce<64>(v, [](uint32_t x, uint32_t y) { return max(x, y); });
}

// v plus the v of the lane that CTRL names, in the rows of ROWS (others: v)
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_add(uint32_t v)
{
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
// Inclusive sum over the wave (ROW: over each row of 16 lanes).
template <bool ROW = false>
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v = dpp_add<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    if constexpr (!ROW) {
        v = dpp_add<0x142, 0xa>(v);  // lane 15 to the second row, lane 47 to the fourth
        v = dpp_add<0x143, 0xc>(v);  // lane 31 to the upper two
    }
    return v;
}

// Inclusive sum over the workgroup's threads: within each wave, then the totals
// of the waves before it (scratch: one entry per wave, at most 16).
__device__ __forceinline__ uint32_t block_incl_scan_u32(uint32_t v, uint32_t *scratch)
{
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    v = wave_incl_scan(v);
    __syncthreads();
    if (lane == 63) scratch[w] = v;
    __syncthreads();
    const uint32_t tot = wave_incl_scan<true>(lane < (int)(blockDim.x >> 6) ? scratch[lane & 15] : 0u);
    return v + (w > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)tot, w - 1) : 0u);
}

// Hand-off between the workgroups of one launch, with no cache-wide fence (a
// device-scope fence writes back and invalidates the XCD's whole L2 on this
// GPU, which costs more than the pass it would guard).  Every value that
// another workgroup reads is written by a device-scope atomic whose returned
// value the writing thread waits for (so the update has been performed at the
// device's coherence point before its workgroup arrives), and is read with
// device-scope loads.
template <typename T>
__device__ __forceinline__ T load_dev(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void store_dev(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// waits until v, returned by an atomic, has arrived
template <typename T>
__device__ __forceinline__ void performed(T v)
{
    asm volatile("" ::"v"(v));
}

// Called by every thread of a workgroup after its atomics for segment s: true
// in the workgroup that finishes the segment last.  No workgroup waits for
// another.
__device__ __forceinline__ bool last_of_segment(SegState *__restrict__ st, int s,
                                                const int3 *__restrict__ segs, int *flag)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t nch = (uint32_t)((segs[s].y + kChunk - 1) / kChunk);
        *flag = atomicAdd(&st[s].arrived, 1u) == nch - 1;
    }
    __syncthreads();
    return *flag != 0;
}

__device__ __forceinline__ void box_atomics(uint32_t *bb, const uint32_t *v)
{
    if (threadIdx.x < 3)
        atomicMin(&bb[threadIdx.x], v[threadIdx.x]);
    else if (threadIdx.x < 6)
        atomicMax(&bb[threadIdx.x], v[threadIdx.x]);
}

// Key bounding box of each segment of the first level (the partition
// accumulates it for the later levels).  keys: the three axes' total-order
// keys in the current order (axis a at a * n).
__global__ __launch_bounds__(kOrbBlock) void k_orb_bbox(const int3 *__restrict__ chunks,
                                                        const uint32_t *__restrict__ keys, int n,
                                                        SegState *__restrict__ st)
{
    const int3 c = chunks[blockIdx.x];
    uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
    // a fixed number of elements per thread, so that all their loads are in
    // flight together (positions past the chunk's end read its last element
    // again: no branch around the loads)
#pragma unroll
    for (int u = 0; u < kChunkPer; ++u) {
        const int p = min(c.y + u * kOrbBlock + (int)threadIdx.x, c.z - 1);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const uint32_t k = keys[(size_t)a * n + p];
            lo[a] = min(lo[a], k);
            hi[a] = max(hi[a], k);
        }
    }
    __shared__ uint32_t red[kOrbBlock / 64][6];
    __shared__ uint32_t tot[6];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = wave_min(lo[a]);
        hi[a] = wave_max(hi[a]);
    }
    if (lane == 0)
        for (int a = 0; a < 3; ++a) {
            red[w][a] = lo[a];
            red[w][3 + a] = hi[a];
        }
    __syncthreads();
    if (threadIdx.x < 6) {
        uint32_t v = red[0][threadIdx.x];
        for (int k = 1; k < kOrbBlock / 64; ++k)
            v = threadIdx.x < 3 ? min(v, red[k][threadIdx.x]) : max(v, red[k][threadIdx.x]);
        tot[threadIdx.x] = v;
    }
    __syncthreads();
    box_atomics(st[c.x].bb, tot);
}

// One round of every segment's selection: counts the window's keys by bin; the
// workgroup that finishes the segment finds the bin with rank krem, makes it
// the window and clears the counts.  keys: as for k_orb_bbox; cur: original
// index per position.  The first round also sets up the states of the next
// level (st_next), which the partition fills in.
__global__ __launch_bounds__(kPassBlock) void k_orb_hist(const int3 *__restrict__ chunks,
                                                        const int3 *__restrict__ segs,
                                                        const uint32_t *__restrict__ keys, int n,
                                                        const int32_t *__restrict__ cur,
                                                        SegState *__restrict__ st,
                                                        uint32_t *__restrict__ hist, int round,
                                                        const int3 *__restrict__ segs_next, int nseg_next,
                                                        SegState *__restrict__ st_next)
{
    __shared__ uint32_t h[kBins];
    __shared__ uint32_t red[kPassBlock / 64];
    __shared__ int last;
    if (round == 0 && threadIdx.x == 0)
        for (int s = blockIdx.x; s < nseg_next; s += gridDim.x) init_state(&st_next[s], segs_next[s].z);
    const int3 c = chunks[blockIdx.x];
    // the state was written by earlier launches only
    if (st[c.x].pick) return;  // the whole segment returns: nobody arrives
    const int axis = seg_axis(&st[c.x]);
    const uint32_t *ka = keys + (size_t)axis * n;
    Window win = st[c.x].win;
    if (round == 0) {
        const uint32_t lo = st[c.x].bb[axis], range = st[c.x].bb[3 + axis] - lo;
        win.from = (uint64_t)lo << 32;
        win.bits = 64 - __clz((int)(range | 1u));
    }
    // the index matters once the bins are narrower than a coordinate
    const bool need_idx = win.shift() < 32;
    // positions past the chunk's end read its last element (no branch around
    // the loads, so they are all in flight together) and are masked below
    uint64_t key[kPassPer];
#pragma unroll
    for (int u = 0; u < kPassPer; ++u) {
        const int p = min(c.y + u * kPassBlock + (int)threadIdx.x, c.z - 1);
        key[u] = (uint64_t)ka[p] << 32;
    }
    if (need_idx) {
#pragma unroll
        for (int u = 0; u < kPassPer; ++u)
            key[u] |= (uint32_t)cur[min(c.y + u * kPassBlock + (int)threadIdx.x, c.z - 1)];
    }
    if (threadIdx.x < kBins) h[threadIdx.x] = 0u;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPassPer; ++u) {
        const int p = c.y + u * kPassBlock + threadIdx.x;
        if (p < c.z && win.holds(key[u])) atomicAdd(&h[win.bin(key[u])], 1u);
    }
    __syncthreads();
    uint32_t *hs = hist + (size_t)c.x * kBins;
    if (threadIdx.x < kBins) {
        const uint32_t v = h[threadIdx.x];
        if (v) performed(atomicAdd(&hs[threadIdx.x], v));
    }
    if (!last_of_segment(st, c.x, segs, &last)) return;
    // the last workgroup: thread t < kBins holds bin t
    uint32_t cnt = 0;
    if (threadIdx.x < kBins) {
        cnt = load_dev(&hs[threadIdx.x]);
        store_dev(&hs[threadIdx.x], 0u);
    }
    const uint32_t inc = block_incl_scan_u32(cnt, red);
    const uint32_t krem = (uint32_t)st[c.x].krem;
    __syncthreads();  // (read before the one thread below writes it)
    if (inc >= krem && inc - cnt < krem) {
        st[c.x].win = win.of_bin((int)threadIdx.x);
        st[c.x].krem = (int)(krem - (inc - cnt));
        st[c.x].pick = cnt <= (uint32_t)kPick;
    }
    if (threadIdx.x == 0) store_dev(&st[c.x].arrived, 0u);
}

// After the rounds: the window's bodies (their keys) are gathered into cand, at the segment's own places, and the workgroup that finishes the
// segment finds the k-th key among theirs: by rank, after further rounds of
// its own where they are more than kPick (equal coordinates, mostly).
__global__ __launch_bounds__(kPassBlock) void k_orb_pick(const int3 *__restrict__ chunks,
                                                        const int3 *__restrict__ segs,
                                                        const uint32_t *__restrict__ keys, int n,
                                                        const int32_t *__restrict__ cur,
                                                        SegState *__restrict__ st,
                                                        uint64_t *__restrict__ cand)
{
    __shared__ uint32_t h[kPickBins];
    __shared__ uint32_t red[kPassBlock / 64];
    __shared__ uint64_t few[kPick];
    __shared__ uint32_t nfew, bin_s, krem_s, count_s;
    __shared__ int last;
    const int3 c = chunks[blockIdx.x];
    const int3 sg = segs[c.x];
    const Window win = st[c.x].win;
    const uint32_t *ka = keys + (size_t)seg_axis(&st[c.x]) * n;
    uint32_t kv[kPassPer];
#pragma unroll
    for (int u = 0; u < kPassPer; ++u) kv[u] = ka[min(c.y + u * kPassBlock + (int)threadIdx.x, c.z - 1)];
    // a body whose coordinate the window reaches; its index decides only where
    // the window is narrower than a coordinate
    uint32_t hits = 0;
#pragma unroll
    for (int u = 0; u < kPassPer; ++u) {
        const int p = c.y + u * kPassBlock + threadIdx.x;
        bool hit = p < c.z && kv[u] >= (uint32_t)(win.from >> 32) &&
                   (win.bits >= 32 ? win.holds((uint64_t)kv[u] << 32) : kv[u] == (uint32_t)(win.from >> 32));
        if (hit && win.bits < 32) hit = win.holds(body_key(kv[u], cur[p]));
        hits |= hit ? 1u << u : 0u;
    }
    // one run of slots per workgroup, and one wait for all of a thread's entries
    const uint32_t mine = (uint32_t)__popc(hits), upto = block_incl_scan_u32(mine, red);
    if (threadIdx.x == kPassBlock - 1) bin_s = upto ? atomicAdd(&st[c.x].picked, upto) : 0u;
    __syncthreads();
    if (hits) {
        uint32_t q = bin_s + upto - mine;
        unsigned long long was = 0;
#pragma unroll
        for (int u = 0; u < kPassPer; ++u)
            if (hits >> u & 1u) {
                if (q < (uint32_t)sg.y)
                    was |= __hip_atomic_exchange((unsigned long long *)&cand[sg.x + q],
                                                 body_key(kv[u], cur[c.y + u * kPassBlock + threadIdx.x]),
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ++q;
            }
        performed(was);
    }
    if (!last_of_segment(st, c.x, segs, &last)) return;
    const uint32_t T = min(load_dev(&st[c.x].picked), (uint32_t)sg.y);
    uint64_t from = win.from;
    int bits = win.bits;  // (below 64 after a round)
    // every candidate in the window, several loads in flight
    auto each = [&](auto &&use) {
        constexpr int kAhead = 8;
        for (uint32_t i0 = threadIdx.x; i0 < T; i0 += kAhead * kPassBlock) {
            uint64_t k[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) k[u] = load_dev(&cand[sg.x + min(i0 + u * kPassBlock, T - 1)]);
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (i0 + u * kPassBlock < T && ((k[u] - from) >> bits) == 0) use(k[u]);
        }
    };
    uint32_t krem = (uint32_t)st[c.x].krem, count = T;
    while (count > (uint32_t)kPick && bits > 0) {
        const int sh = max(bits - kPickDigit, 0);
        h[threadIdx.x] = 0u;
        h[threadIdx.x + kPassBlock] = 0u;
        if (threadIdx.x == 0) {
            bin_s = 0u;
            krem_s = krem;
            count_s = 0u;
        }
        __syncthreads();
        each([&](uint64_t k) { atomicAdd(&h[(k - from) >> sh], 1u); });
        __syncthreads();
        const uint32_t c0 = h[2 * threadIdx.x], c1 = h[2 * threadIdx.x + 1];
        const uint32_t to = block_incl_scan_u32(c0 + c1, red), before = to - c0 - c1;
        if (before < krem && to >= krem) {
            const bool second = before + c0 < krem;
            bin_s = 2 * threadIdx.x + second;
            krem_s = krem - before - (second ? c0 : 0u);
            count_s = second ? c1 : c0;
        }
        __syncthreads();
        from += (uint64_t)bin_s << sh;
        bits = sh;
        krem = krem_s;
        count = count_s;
        __syncthreads();
    }
    if (threadIdx.x == 0) nfew = 0u;
    __syncthreads();
    each([&](uint64_t k) {
        const uint32_t q = atomicAdd(&nfew, 1u);
        if (q < (uint32_t)kPick) few[q] = k;
    });
    __syncthreads();
    const uint32_t m = min(nfew, (uint32_t)kPick);
    if (threadIdx.x < m) {
        const uint64_t mine = few[threadIdx.x];
        uint32_t r = 1;
#pragma unroll 8
        for (uint32_t f = 0; f < m; ++f) r += few[f] < mine;
        if (r == krem) st[c.x].kth = mine;
    }
    if (threadIdx.x == 0) store_dev(&st[c.x].arrived, 0u);
}

// Keys <= the k-th key go left.  Each workgroup takes one run of slots per
// side (one 64-bit atomic gives both) and fills it in position order (ballot ranks);
// the order of the runs is irrelevant to the result.  The original indices
// go to cur_out and the three axes' keys to keys_out, both in the new order.
// Each side's key box is accumulated into its next-level state (if it has
// one).
__global__ __launch_bounds__(kPassBlock) void k_orb_partition(const int3 *__restrict__ chunks,
                                                             const int3 *__restrict__ segs,
                                                             const int2 *__restrict__ kids,
                                                             const uint32_t *__restrict__ keys,
                                                             uint32_t *__restrict__ keys_out, int n,
                                                             const int32_t *__restrict__ cur,
                                                             int32_t *__restrict__ cur_out,
                                                             SegState *__restrict__ st,
                                                             SegState *__restrict__ st_next)
{
    constexpr int kW = kPassBlock / 64;
    __shared__ uint32_t cl[kPassPer * kW], cr[kPassPer * kW];
    __shared__ uint32_t bl, br;
    __shared__ uint32_t box[kW][12];
    __shared__ uint32_t tot[12];
    const int3 c = chunks[blockIdx.x];
    const uint64_t kth = st[c.x].kth;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t below = (1ull << lane) - 1ull;
    // all of the thread's loads together, ahead of the split axis
    uint32_t kv[3][kPassPer];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int u = 0; u < kPassPer; ++u)
            kv[a][u] = keys[(size_t)a * n + min(c.y + u * kPassBlock + (int)threadIdx.x, c.z - 1)];
    const int axis = seg_axis(&st[c.x]);
    // this thread's bodies and their sides
    int bod[kPassPer];
    uint32_t rank[kPassPer];
    bool lft[kPassPer];
#pragma unroll
    for (int u = 0; u < kPassPer; ++u) {
        const int p = c.y + u * kPassBlock + threadIdx.x;
        const int q = min(p, c.z - 1);  // loads without a branch, masked below
        const int b = cur[q];
        const uint32_t ka = axis == 0 ? kv[0][u] : (axis == 1 ? kv[1][u] : kv[2][u]);
        lft[u] = (((uint64_t)ka << 32) | (uint32_t)b) <= kth;
        bod[u] = p < c.z ? b : -1;
    }
    // rank inside the (step, wave) group by ballots, group totals in LDS
#pragma unroll
    for (int u = 0; u < kPassPer; ++u) {
        const uint64_t ml = __ballot(bod[u] >= 0 && lft[u]);
        const uint64_t mr = __ballot(bod[u] >= 0 && !lft[u]);
        rank[u] = (uint32_t)__popcll((lft[u] ? ml : mr) & below);
        if (lane == 0) {
            cl[u * kW + w] = (uint32_t)__popcll(ml);
            cr[u * kW + w] = (uint32_t)__popcll(mr);
        }
    }
    __syncthreads();
    // exclusive scans over the kPassPer * kW groups (position order), by wave 0
    static_assert(kPassPer * kW <= 64, "one group per lane of wave 0");
    if (w == 0) {
        const bool g = lane < kPassPer * kW;
        const uint32_t a = g ? cl[lane] : 0u, b = g ? cr[lane] : 0u;
        const uint32_t ia = wave_incl_scan(a), ib = wave_incl_scan(b);
        if (g) {
            cl[lane] = ia - a;
            cr[lane] = ib - b;
        }
        if (lane == 63) {
            // one atomic for both runs: the bodies placed before this
            // workgroup, and how many of them went left
            const unsigned long long was =
                atomicAdd(reinterpret_cast<unsigned long long *>(&st[c.x].placed),
                          ((unsigned long long)(ia + ib) << 32) | ia);
            bl = (uint32_t)was;
            br = (uint32_t)(was >> 32) - (uint32_t)was;
        }
    }
    __syncthreads();
    const int3 sg = segs[c.x];
    // box of each side: min keys x,y,z then max keys x,y,z; left then right
    uint32_t bx[12];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        bx[a] = bx[6 + a] = 0xFFFFFFFFu;
        bx[3 + a] = bx[9 + a] = 0u;
    }
    // destinations; exactly k keys are <= the k-th key, and the guards only
    // keep a violated precondition (non-finite coordinates) inside the segment
    int dst[kPassPer];
#pragma unroll
    for (int u = 0; u < kPassPer; ++u) {
        const uint32_t q = (lft[u] ? bl + cl[u * kW + w] : br + cr[u * kW + w]) + rank[u];
        const bool fits = lft[u] ? q < (uint32_t)sg.z : q < (uint32_t)(sg.y - sg.z);
        dst[u] = bod[u] >= 0 && fits ? sg.x + (lft[u] ? 0 : sg.z) + (int)q : -1;
        if (dst[u] >= 0) cur_out[dst[u]] = bod[u];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        uint32_t *const out = keys_out + (size_t)a * n;
#pragma unroll
        for (int u = 0; u < kPassPer; ++u) {
            const uint32_t v = kv[a][u];
            const bool l = dst[u] >= 0 && lft[u], r = dst[u] >= 0 && !lft[u];
            if (dst[u] >= 0) out[dst[u]] = v;
            bx[a] = min(bx[a], l ? v : 0xFFFFFFFFu);
            bx[3 + a] = max(bx[3 + a], l ? v : 0u);
            bx[6 + a] = min(bx[6 + a], r ? v : 0xFFFFFFFFu);
            bx[9 + a] = max(bx[9 + a], r ? v : 0u);
        }
    }
#pragma unroll
    for (int j = 0; j < 12; ++j) bx[j] = (j % 6) < 3 ? wave_min(bx[j]) : wave_max(bx[j]);
    if (lane == 0)
#pragma unroll
        for (int j = 0; j < 12; ++j) box[w][j] = bx[j];
    __syncthreads();
    if (threadIdx.x < 12) {
        const int j = threadIdx.x;
        uint32_t v = box[0][j];
        for (int k = 1; k < kW; ++k) v = (j % 6) < 3 ? min(v, box[k][j]) : max(v, box[k][j]);
        tot[j] = v;
    }
    __syncthreads();
    const int2 kd = kids[c.x];
    if (kd.x >= 0) box_atomics(st_next[kd.x].bb, tot);
    if (kd.y >= 0) box_atomics(st_next[kd.y].bb, tot + 6);
}

// ---- phase B: one workgroup finishes one segment in LDS --------------------
// The segment's keys are loaded once, coalesced, from the key buffer that
// holds it (phase A leaves them in the segment's order) and stay in their
// slots; the recursion permutes slot numbers only.

// Finishes the recursion of a node of at most 64 bodies (positions
// [lo, lo + m) of pos) with one wave, one position per lane, every node of a
// level split at once.  keys: per-wave LDS of 3 x 64 total-order keys.  The
// k smallest keys of a node are found by ranking (keys and indices are
// distinct), then each leaf is ordered by original index.
constexpr int kWaveSeg = 64;

__device__ void orb_wave(uint16_t *pos, const uint32_t (*skey)[kSmall], const int32_t *gid,
                         uint32_t (*keys)[kWaveSeg], int32_t *wid, int lo, int m, int leaf, int lane)
{
    const int s = lane < m ? pos[lo + lane] : 0;  // this lane's slot
    const uint32_t kx = skey[0][s], ky = skey[1][s], kz = skey[2][s];
    const int b = gid[s];
    int slo = 0, sm = m;  // the node holding this lane's entry (relative to lo)
    int at = lane;        // this lane's entry's current position (relative to lo)
    if (lane < m) {
        keys[0][lane] = kx;
        keys[1][lane] = ky;
        keys[2][lane] = kz;
        wid[lane] = b;
    }
    for (;;) {
        const bool split = lane < m && sm > leaf;
        if (!__any(split)) break;
        wave_sync();
        int to = at;
        int k = sm;
        if (split) {
            uint32_t bb[6] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0u, 0u, 0u};
            // (unrolled so that several LDS reads are in flight per wait)
#pragma unroll 4
            for (int f = slo; f < slo + sm; ++f)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const uint32_t v = keys[a][f];
                    bb[a] = min(bb[a], v);
                    bb[3 + a] = max(bb[3 + a], v);
                }
            const int axis = pick_axis(bb);
            const uint32_t mine = axis == 0 ? kx : (axis == 1 ? ky : kz);
            int r = 0;
#pragma unroll 4
            for (int f = slo; f < slo + sm; ++f) {
                const uint32_t v = keys[axis][f];
                r += (v < mine) || (v == mine && wid[f] < b);
            }
            to = slo + r;
            const int L = (sm + leaf - 1) / leaf;
            k = min(sm, leaf * ((L + 1) / 2));
        }
        wave_sync();
        if (lane < m) {
            keys[0][to] = kx;
            keys[1][to] = ky;
            keys[2][to] = kz;
            wid[to] = b;
            at = to;
            if (split) {
                if (to - slo < k) {
                    sm = k;
                } else {
                    slo += k;
                    sm -= k;
                }
            }
        }
    }
    wave_sync();
    // leaves: ascending original index
    int r = 0;
    if (lane < m)
#pragma unroll 4
        for (int f = slo; f < slo + sm; ++f) r += wid[f] < b;
    if (lane < m) pos[lo + slo + r] = (uint16_t)s;
}


// The same for a leaf size that is a power of two up to 32, in registers.  The
// node's halves then have at most 32 bodies, theirs 16, and so on, so that at
// every level the nodes are groups of W lanes with their bodies first: boxes
// are reductions over the group and ranks counts over it, by cross-lane operands
// instead of an LDS read per pair of lanes (64 nodes of a
// 4096-body segment, four per wave, down to leaves of 4: 75 us by orb_wave, 20 so).
// r += (oh, ol) of another lane < (mh, ml) of this one, one step per cross-lane control:
// the borrow of the difference
#define NB_RANK_STEP(CTRL)                                                                    \
    "v_sub_co_u32_dpp %[t], vcc, %[ol], %[ml] " CTRL " row_mask:0xf bank_mask:0xf\n"          \
    "v_subb_co_u32_dpp %[t], vcc, %[oh], %[mh], vcc " CTRL " row_mask:0xf bank_mask:0xf\n"    \
    "v_addc_co_u32 %[r], vcc, 0, %[r], vcc\n"
#define NB_RANK_OWN                                  \
    "v_sub_co_u32 %[t], vcc, %[ol], %[ml]\n"         \
    "v_subb_co_u32 %[t], vcc, %[oh], %[mh], vcc\n"   \
    "v_addc_co_u32 %[r], vcc, 0, %[r], vcc\n"
#define NB_RANK(STEPS)                                                                                      \
    asm volatile("s_nop 1\n" STEPS                                                                          \
                 : [r] "+&v"(r), [t] "=&v"(t)                                                               \
                 : [oh] "v"(oh), [ol] "v"(ol), [mh] "v"(mh), [ml] "v"(ml)                                   \
                 : "vcc")

__device__ __forceinline__ void rank_row(uint32_t &r, uint32_t oh, uint32_t ol, uint32_t mh, uint32_t ml)
{
    uint32_t t;
    NB_RANK(NB_RANK_OWN ".irp n,1,2,3,4,5,6,7,8,9,10,11,12,13,14,15\n" NB_RANK_STEP("row_ror:\\n") ".endr\n");
}
__device__ __forceinline__ void rank_quad(uint32_t &r, uint32_t oh, uint32_t ol, uint32_t mh, uint32_t ml)
{
    uint32_t t;
    NB_RANK(NB_RANK_OWN NB_RANK_STEP("quad_perm:[1,0,3,2]") NB_RANK_STEP("quad_perm:[2,3,0,1]")
                NB_RANK_STEP("quad_perm:[3,2,1,0]"));
}
__device__ __forceinline__ void rank_pair(uint32_t &r, uint32_t oh, uint32_t ol, uint32_t mh, uint32_t ml)
{
    uint32_t t;
    NB_RANK(NB_RANK_STEP("quad_perm:[1,0,3,2]"));
}

// Rank of (h, l) among the group of W lanes; the pairs of a group are distinct.
template <int W>
__device__ __forceinline__ int group_rank(uint32_t h, uint32_t l)
{
    uint32_t r = 0;
    if constexpr (W == 2) {
        rank_pair(r, h, l, h, l);
    } else if constexpr (W == 4) {
        rank_quad(r, h, l, h, l);
    } else if constexpr (W == 8) {
        rank_quad(r, h, l, h, l);
        rank_quad(r, dpp<kDppHalfMirror>(h), dpp<kDppHalfMirror>(l), h, l);
    } else if constexpr (W == 16) {
        rank_row(r, h, l, h, l);
    } else if constexpr (W == 32) {
        const auto ph = __builtin_amdgcn_permlane16_swap(h, h, false, false);
        const auto pl = __builtin_amdgcn_permlane16_swap(l, l, false, false);
        rank_row(r, ph[0], pl[0], h, l);
        rank_row(r, ph[1], pl[1], h, l);
    } else {
        const auto qh = __builtin_amdgcn_permlane32_swap(h, h, false, false);
        const auto ql = __builtin_amdgcn_permlane32_swap(l, l, false, false);
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const auto ph = __builtin_amdgcn_permlane16_swap(qh[z], qh[z], false, false);
            const auto pl = __builtin_amdgcn_permlane16_swap(ql[z], ql[z], false, false);
            rank_row(r, ph[0], pl[0], h, l);
            rank_row(r, ph[1], pl[1], h, l);
        }
    }
    return (int)r;
}

struct WaveBody {
    uint32_t k[3];  // total-order keys
    uint32_t id;    // original index (an empty lane: above every index, and its own)
    uint32_t slot;
};

// One level: the group's node (its m bodies in the group's first lanes, at slo
// of the whole node's positions) is split in two, whose bodies move to the
// halves' first lanes.
template <int W>
__device__ __forceinline__ void wave_level(WaveBody &b, int &m, int &slo, int leaf_log, int lane)
{
    const int leaf = 1 << leaf_log;
    const int at = lane & (W - 1);
    const bool body = at < m;
    uint32_t bb[6];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        bb[a] = group_reduce<W>(body ? b.k[a] : 0xFFFFFFFFu, [](uint32_t x, uint32_t y) { return min(x, y); });
        bb[3 + a] = group_reduce<W>(body ? b.k[a] : 0u, [](uint32_t x, uint32_t y) { return max(x, y); });
    }
    const int axis = pick_axis(bb);
    const uint32_t key = axis == 0 ? b.k[0] : (axis == 1 ? b.k[1] : b.k[2]);
    const int r = group_rank<W>(body ? key : 0xFFFFFFFFu, b.id);
    const bool split = m > leaf;
    const int L = (m + leaf - 1) >> leaf_log;
    const int k = min(m, ((L + 1) >> 1) << leaf_log);
    // the empty lanes fill up the left half, then the right
    const int q = !split ? at : r < k ? r : r < m ? W / 2 + r - k : r - m < W / 2 - k ? k + r - m : r;
    const int dst = ((lane & ~(W - 1)) + q) * 4;
#pragma unroll
    for (int a = 0; a < 3; ++a) b.k[a] = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)b.k[a]);
    b.id = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)b.id);
    b.slot = (uint32_t)__builtin_amdgcn_ds_permute(dst, (int)b.slot);
    const bool right = (lane & (W / 2)) != 0;
    slo += split && right ? k : 0;
    m = split ? (right ? m - k : k) : (right ? 0 : m);
}

__device__ void orb_wave_pow2(uint16_t *pos, const uint32_t (*skey)[kSmall], const int32_t *gid, int lo, int m0,
                              int leaf_log, int lane)
{
    WaveBody b;
    b.slot = lane < m0 ? pos[lo + lane] : 0u;
#pragma unroll
    for (int a = 0; a < 3; ++a) b.k[a] = skey[a][b.slot];
    b.id = lane < m0 ? (uint32_t)gid[b.slot] : 0xFFFFFF00u | (uint32_t)lane;
    int m = m0, slo = 0;
    wave_level<64>(b, m, slo, leaf_log, lane);
    if (leaf_log <= 4) wave_level<32>(b, m, slo, leaf_log, lane);
    if (leaf_log <= 3) wave_level<16>(b, m, slo, leaf_log, lane);
    if (leaf_log <= 2) wave_level<8>(b, m, slo, leaf_log, lane);
    if (leaf_log <= 1) wave_level<4>(b, m, slo, leaf_log, lane);
    if (leaf_log <= 0) wave_level<2>(b, m, slo, leaf_log, lane);
    // leaves: ascending original index
    int r = 0;
    switch (leaf_log) {
    case 5: r = group_rank<32>(0u, b.id); break;
    case 4: r = group_rank<16>(0u, b.id); break;
    case 3: r = group_rank<8>(0u, b.id); break;
    case 2: r = group_rank<4>(0u, b.id); break;
    case 1: r = group_rank<2>(0u, b.id); break;
    default: break;
    }
    if ((lane & ((1 << leaf_log) - 1)) < m) pos[lo + slo + r] = (uint16_t)b.slot;
}

// Bins of a level's selection, shared by its nodes: node j of depth d has the
// kFinBins >> d from j (kFinBins >> d) on.
constexpr int kFinBins = 4096;
constexpr int kFinDepth = 7;  // a node of depth 7 has at most 64 bodies, whatever the leaf size
constexpr int kFinNodes = 1 << kFinDepth;
constexpr int kFinPer = kSmall / kFinBlock;       // positions per thread
constexpr int kBinPer = kFinBins / kFinBlock;     // bins per thread
constexpr int kCand = 64;                         // keys that one wave ranks
static_assert((kFinBins >> (kFinDepth - 1)) >= kBinPer, "a thread's bins belong to one node");

// A node of the current depth.
struct FinNode {
    int lo, m, k;         // positions [lo, lo + m); the first k keys go left (0: not split)
    uint32_t bb[6];       // key box
    int axis;
    int bits;             // the selection's window: 2^bits keys from `from` on
    int krem;             // rank still to find inside it
    int count;            // keys inside it
    int base;             // keys counted in the bins before the node's
    uint64_t from;
    uint64_t kth;         // the k-th key
    uint32_t cand;        // candidates gathered
    uint32_t put[2];      // partition: entries placed left and right
};

// Bodies of a node of m that go left, 0 if it stays whole.  A leaf of more than
// 64 bodies, which is to be ordered by index, is split along that.
__device__ __forceinline__ int fin_split(int m, int leaf)
{
    if (m <= kWaveSeg) return 0;
    const int unit = m <= leaf ? kWaveSeg : leaf;
    return min(m, unit * (((m + unit - 1) / unit + 1) / 2));
}

// Phase B.  segs: (start, size, which buffer pair holds it).  keys0/1: the
// three axes' keys in the order of cur0/1 (axis a at a * n).
//
// All nodes of a depth are split together: the threads hold kFinPer positions
// each, whatever node they belong to.  Per depth: the nodes' key boxes (LDS
// atomics, one per wave where a wave lies in one node); a histogram of the
// split axis' keys over each node's own range, in kFinBins bins shared out
// among the nodes; the bin that holds the k-th key; the few keys in that bin,
// ranked by one wave (a bin of more than kCand keys is divided again); the
// partition of the slot numbers.  Until every node has at most 64 bodies, which
// one wave per node finishes (orb_wave).  Leaves of more than 64 bodies are
// split on by original index, which is the order their bodies end in.
// A key is the coordinate's total-order key and the index below it, so the
// keys are distinct and every selection ends.
//
// Bound by the latency of its LDS round trips and barriers, some ten per
// depth, and by the VALU work of 16 waves on one CU.  At 2^20 bodies (leaf 4) it
// takes 86 us for 256 segments of 4096; node by node, 1024 segments of 1024
// took 139 us, after two more levels of phase A at 48 us each.
__global__ __launch_bounds__(kFinBlock) void k_orb_block(const int3 *__restrict__ segs,
                                                         const uint32_t *__restrict__ keys0,
                                                         const uint32_t *__restrict__ keys1,
                                                         const int32_t *__restrict__ cur0,
                                                         const int32_t *__restrict__ cur1, int n, int leaf,
                                                         int32_t *__restrict__ perm)
{
    __shared__ uint32_t skey[3][kSmall];   // keys by slot
    __shared__ int32_t gid[kSmall];        // original index by slot
    __shared__ uint16_t posb[2][kSmall];   // slots in the current order, and the partition's target
    __shared__ uint32_t hist[kFinBins];
    __shared__ uint64_t cand[kFinNodes / 2][kCand];
    __shared__ FinNode node[kFinNodes];
    __shared__ uint32_t red[kFinBlock / 64];
    __shared__ int again[2];  // a window is to be divided once more (by the parity of the turn)
    const int3 sg = segs[blockIdx.x];
    const int start = sg.x, size = sg.y;
    const int32_t *cur = sg.z ? cur1 : cur0;
    const uint32_t *keys = sg.z ? keys1 : keys0;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the clamp only keeps a broken invariant (an unfilled slot) from turning
    // into out-of-bounds writes: every slot is filled
    for (int e = tid; e < size; e += kFinBlock) {
        gid[e] = (int32_t)min((uint32_t)cur[start + e], (uint32_t)(n - 1));
        posb[0][e] = (uint16_t)e;
#pragma unroll
        for (int a = 0; a < 3; ++a) skey[a][e] = keys[(size_t)a * n + start + e];
    }
    int lo0 = 0, m0 = size;  // thread j < 2^depth: node j
    const int e0 = tid * kFinPer;  // this thread's positions
    const int ne = max(0, min(kFinPer, size - e0));
    int nid[kFinPer];  // the node of each
#pragma unroll
    for (int u = 0; u < kFinPer; ++u) nid[u] = 0;
    uint16_t *pos = posb[0], *to = posb[1];
    int depth = 0;
    int most = size;  // bodies of the depth's largest node: the leftmost
    for (;; ++depth) {
        const int nn = 1 << depth, bins_log = 12 - depth;
        __syncthreads();
        if (tid == 0) again[0] = again[1] = 0;
        if (tid < nn) {
            FinNode &N = node[tid];
            N.lo = lo0;
            N.m = m0;
            N.k = depth < kFinDepth ? fin_split(m0, leaf) : 0;
            N.cand = 0u;
            N.put[0] = N.put[1] = 0u;
            N.count = kCand + 1;
            N.kth = 0;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                N.bb[a] = 0xFFFFFFFFu;
                N.bb[3 + a] = 0u;
            }
        }
        __syncthreads();
        if (most <= kWaveSeg || depth >= kFinDepth) break;
        most = fin_split(most, leaf);
        // the slots with their keys, and the nodes' boxes.  (A thread's positions lie
        // in one node almost always: what they need of it is read again only
        // where the node changes.)
        int slot[kFinPer];
        int32_t id[kFinPer];
        uint32_t key[kFinPer][3];
        const int first = __shfl(nid[0], 0);
        const bool one = __all((ne == kFinPer) & (nid[0] == first) & (nid[kFinPer - 1] == first)) != 0;
        bool split_u[kFinPer];
        uint32_t bx[6] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0u, 0u, 0u};
        auto box_out = [&](int j, bool split_j) {  // the box so far goes to node j, if that is split
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                if (split_j) {
                    atomicMin(&node[j].bb[a], bx[a]);
                    atomicMax(&node[j].bb[3 + a], bx[3 + a]);
                }
                bx[a] = 0xFFFFFFFFu;
                bx[3 + a] = 0u;
            }
        };
#pragma unroll
        for (int u = 0; u < kFinPer; ++u) {
            if (u == 0 || nid[u] != nid[u - 1])
                split_u[u] = node[nid[u]].k > 0;
            else
                split_u[u] = split_u[u - 1];
            slot[u] = u < ne ? pos[e0 + u] : 0;
            id[u] = gid[slot[u]];
#pragma unroll
            for (int a = 0; a < 3; ++a) key[u][a] = skey[a][slot[u]];
            if (u < ne)
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    bx[a] = min(bx[a], key[u][a]);
                    bx[3 + a] = max(bx[3 + a], key[u][a]);
                }
            if (!one && u < ne && (u + 1 >= ne || nid[u + 1 < kFinPer ? u + 1 : u] != nid[u]))
                box_out(nid[u], split_u[u]);
        }
        if (one && split_u[0]) {
#pragma unroll
            for (int j = 0; j < 6; ++j) bx[j] = j < 3 ? wave_min(bx[j]) : wave_max(bx[j]);
            if (lane == 0) box_out(first, true);
        }
        __syncthreads();
        // the split axes and the first windows: from the smallest key's coordinate
        // to the largest's, all indices
        if (tid < nn && node[tid].k > 0) {
            FinNode &N = node[tid];
            N.krem = N.k;
            if (N.m <= leaf) {  // by index
                N.axis = 3;
                N.from = 0;
                N.bits = 32 - __clz(n);
            } else {
                N.axis = pick_axis(N.bb);
                const uint32_t range = N.bb[3 + N.axis] - N.bb[N.axis];
                N.from = (uint64_t)N.bb[N.axis] << 32;
                N.bits = 64 - __clz((int)(range | 1u));  // (a range of 0 takes the indices' 32 bits and one)
            }
        }
        uint64_t bk[kFinPer];  // the bodies' keys along their nodes' axes
        int axis_u[kFinPer];
        // divide the windows until every node's holds at most kCand keys
        for (int turn = 0;; ++turn) {
            const bool begin = turn == 0;
#pragma unroll
            for (int b = 0; b < kBinPer; ++b) hist[tid * kBinPer + b] = 0u;
            __syncthreads();
            if (tid == 0) again[(turn + 1) & 1] = 0;
            {
                uint64_t from = 0;
                int bits = 0;
                bool open = false;
#pragma unroll
                for (int u = 0; u < kFinPer; ++u) {
                    if (u == 0 || nid[u] != nid[u - 1]) {
                        const FinNode &N = node[nid[u]];
                        open = split_u[u] && N.count > kCand;
                        from = N.from;
                        bits = N.bits;
                        axis_u[u] = N.axis;
                    } else {
                        axis_u[u] = axis_u[u - 1];
                    }
                    if (begin)
                        bk[u] = body_key(axis_u[u] == 0   ? key[u][0]
                                         : axis_u[u] == 1 ? key[u][1]
                                         : axis_u[u] == 2 ? key[u][2]
                                                          : 0u,
                                         id[u]);
                    const uint64_t rel = bk[u] - from;
                    if (open && u < ne && (bits == 64 || (rel >> bits) == 0))
                        atomicAdd(&hist[(nid[u] << bins_log) + (int)(rel >> max(bits - bins_log, 0))], 1u);
                }
            }
            __syncthreads();
            uint32_t c[kBinPer], sum = 0;
#pragma unroll
            for (int b = 0; b < kBinPer; ++b) {
                c[b] = hist[tid * kBinPer + b];
                sum += c[b];
            }
            const uint32_t inc = block_incl_scan_u32(sum, red);
            const int j = (tid * kBinPer) >> bins_log;
            const bool open = node[j].k > 0 && node[j].count > kCand;
            if (open && ((tid * kBinPer) & ((1 << bins_log) - 1)) == 0) node[j].base = (int)(inc - sum);
            const int krem = node[j].krem, bits = node[j].bits;
            const uint64_t from = node[j].from;
            __syncthreads();
            if (open) {
                int before = (int)(inc - sum) - node[j].base;
                if (before < krem && before + (int)sum >= krem) {
#pragma unroll
                    for (int b = 0; b < kBinPer; ++b) {
                        if (before < krem && before + (int)c[b] >= krem) {
                            const int sh = max(bits - bins_log, 0);
                            const int bin = tid * kBinPer + b - (j << bins_log);
                            node[j].from = from + ((uint64_t)bin << sh);
                            node[j].bits = sh;
                            node[j].krem = krem - before;
                            // (a window of one key holds one body)
                            node[j].count = sh > 0 ? (int)c[b] : 1;
                            if (sh > 0 && (int)c[b] > kCand) again[turn & 1] = 1;
                        }
                        before += (int)c[b];
                    }
                }
            }
            __syncthreads();
            if (!again[turn & 1]) break;
        }
        // the keys in the windows, ranked by a wave per node
        {
            uint64_t from = 0;
            int bits = 0;
#pragma unroll
            for (int u = 0; u < kFinPer; ++u) {
                if (u == 0 || nid[u] != nid[u - 1]) {
                    from = node[nid[u]].from;
                    bits = node[nid[u]].bits;
                }
                if (split_u[u] && u < ne && ((bk[u] - from) >> bits) == 0) {
                    const uint32_t q = atomicAdd(&node[nid[u]].cand, 1u);
                    if (q < (uint32_t)kCand) cand[nid[u]][q] = bk[u];
                }
            }
        }
        __syncthreads();
        for (int j = wave; j < nn; j += kFinBlock / 64) {
            FinNode &N = node[j];
            const int cnt = min((int)N.cand, kCand);
            if (N.k == 0 || cnt == 0) continue;
            const uint64_t mine = cand[j][lane < cnt ? lane : 0];
            int r = 1;
#pragma unroll 8
            for (int f = 0; f < cnt; ++f) r += cand[j][f] < mine;
            if (lane < cnt && r == N.krem) N.kth = mine;
        }
        __syncthreads();
        // partition; the order inside a side does not change the result
        bool left[kFinPer];
        int nl = 0, nr = 0;
        int lo_u = 0, k_u = 0, m_u = 0;
        {
            uint64_t kth = 0;
#pragma unroll
            for (int u = 0; u < kFinPer; ++u) {
                if (u == 0 || nid[u] != nid[u - 1]) kth = node[nid[u]].kth;
                left[u] = u < ne && split_u[u] && bk[u] <= kth;
                nl += left[u];
                nr += u < ne && !left[u];
            }
        }
        lo_u = node[nid[0]].lo;
        k_u = node[nid[0]].k;
        m_u = node[nid[0]].m;
        if (one && split_u[0]) {
            // (left and right counts side by side: at most 64 kFinPer each)
            uint32_t v = (uint32_t)nl | ((uint32_t)nr << 16);
            const uint32_t mine = v;
            v = wave_incl_scan(v);
            uint32_t bl = 0, br = 0;
            if (lane == 63) {
                bl = atomicAdd(&node[first].put[0], v & 0xFFFFu);
                br = atomicAdd(&node[first].put[1], v >> 16);
            }
            v -= mine;
            int ql = __builtin_amdgcn_readlane((int)bl, 63) + (int)(v & 0xFFFFu);
            int qr = k_u + __builtin_amdgcn_readlane((int)br, 63) + (int)(v >> 16);
#pragma unroll
            for (int u = 0; u < kFinPer; ++u) {
                const int q = left[u] ? ql++ : qr++;
                if (q < (left[u] ? k_u : m_u)) to[lo_u + q] = (uint16_t)slot[u];
            }
        } else {
            int lo = lo_u, k = k_u, m = m_u;
#pragma unroll
            for (int u = 0; u < kFinPer; ++u) {
                if (u > 0 && nid[u] != nid[u - 1]) {
                    lo = node[nid[u]].lo;
                    k = node[nid[u]].k;
                    m = node[nid[u]].m;
                }
                if (u >= ne) continue;
                if (!split_u[u]) {
                    to[e0 + u] = (uint16_t)slot[u];
                } else {
                    const int q = left[u] ? (int)atomicAdd(&node[nid[u]].put[0], 1u)
                                          : k + (int)atomicAdd(&node[nid[u]].put[1], 1u);
                    if (q < (left[u] ? k : m)) to[lo + q] = (uint16_t)slot[u];
                }
            }
        }
        {
            int lo = lo_u, k = k_u, was = nid[0];
#pragma unroll
            for (int u = 0; u < kFinPer; ++u) {
                if (nid[u] != was) {
                    was = nid[u];
                    lo = node[was].lo;
                    k = node[was].k;
                }
                nid[u] = 2 * nid[u] + (k > 0 && e0 + u >= lo + k);
            }
        }
        // the next depth's nodes: 2 j and 2 j + 1 (an unsplit one stays the left)
        if (tid < 2 * nn) {
            const FinNode &N = node[tid / 2];
            const int k = N.k > 0 ? N.k : N.m;
            lo0 = N.lo + ((tid & 1) ? k : 0);
            m0 = (tid & 1) ? N.m - k : k;
        }
        uint16_t *const t = pos;
        pos = to;
        to = t;
    }
    // (the nodes' table is the last depth's)
    __shared__ uint32_t wkeys[kFinBlock / 64][3][kWaveSeg];
    __shared__ int32_t wgid[kFinBlock / 64][kWaveSeg];
    const int nn = 1 << depth;
    for (int j = wave; j < nn; j += kFinBlock / 64) {
        const int lo = node[j].lo, m = node[j].m;
        if (m == 0) continue;
        if (leaf <= 32 && (leaf & (leaf - 1)) == 0)
            orb_wave_pow2(pos, skey, gid, lo, m, __builtin_ctz(leaf), lane);
        else
            orb_wave(pos, skey, gid, wkeys[wave], wgid[wave], lo, m, leaf, lane);
        wave_sync();
    }
    __syncthreads();
    for (int e = tid; e < size; e += kFinBlock) perm[start + e] = gid[pos[e]];
}

// ---- host side --------------------------------------------------------------
struct Level {
    std::vector<int3> segs;    // (start, size, k)
    std::vector<int3> chunks;  // (segment, begin, end)
    std::vector<int2> kids;    // next-level segment of the left, right part (-1: phase B)
};

// Level l reads the index and key buffers l % 2 and writes (l + 1) % 2, so a
// segment at depth d sits in buffer d % 2: finals are (start, size, d % 2).
void plan_tree(int n, int leaf, std::vector<Level> &levels, std::vector<int3> &finals)
{
    const int cut = std::max(kSmall, leaf);
    std::vector<int2> cur = {make_int2(0, n)};
    for (int depth = 0; !cur.empty(); ++depth) {
        Level lv;
        std::vector<int2> next;
        int nid = 0;  // the next level numbers its segments in the order of `next`
        for (const int2 &s : cur) {
            if (s.y <= cut) {
                finals.push_back(make_int3(s.x, s.y, depth & 1));
                continue;
            }
            const int L = (s.y + leaf - 1) / leaf;
            const int k = std::min(s.y, leaf * ((L + 1) / 2));
            const int id = (int)lv.segs.size();
            lv.segs.push_back(make_int3(s.x, s.y, k));
            for (int b = s.x; b < s.x + s.y; b += kChunk)
                lv.chunks.push_back(make_int3(id, b, std::min(b + kChunk, s.x + s.y)));
            const int kl = k > cut ? nid++ : -1;
            const int kr = s.y - k > cut ? nid++ : -1;
            lv.kids.push_back(make_int2(kl, kr));
            next.push_back(make_int2(s.x, k));
            next.push_back(make_int2(s.x + k, s.y - k));
        }
        if (!lv.segs.empty()) levels.push_back(std::move(lv));
        cur.swap(next);
    }
}

std::mutex g_orb_mu;
void *g_pinned = nullptr;
size_t g_pinned_size = 0;
// An event belongs to one device: one per device, and the one recorded
// after the last upload (on whichever device) guards the shared buffer.
std::map<int, hipEvent_t> g_pinned_evs;
hipEvent_t g_pinned_last = nullptr;

}  // namespace

int orb_order(const void *pm, int prec, int n, int leaf, int32_t *perm, hipStream_t s)
{
    if (leaf > kMaxBlockSeg) {
        set_error("leaf %d larger than the supported %d", leaf, kMaxBlockSeg);
        return NBODY_E_UNSUPPORTED;
    }
    std::vector<Level> levels;
    std::vector<int3> finals;
    plan_tree(n, leaf, levels, finals);
    // one table upload: per level segs, chunks and kids, then the final
    // segments; sections start on 16-byte boundaries (int2 entries need
    // 8-byte alignment)
    std::vector<char> tab;
    auto pad = [&tab]() { tab.resize((tab.size() + 15) & ~size_t(15), 0); };
    auto put = [&tab, &pad](const void *p, size_t bytes) {
        const size_t at = tab.size();
        tab.insert(tab.end(), (const char *)p, (const char *)p + bytes);
        pad();
        return at;
    };
    struct Off {
        size_t segs, chunks, kids;
    };
    std::vector<Off> off;
    size_t maxseg = 1;
    for (const Level &lv : levels) {
        Off o;
        o.segs = put(lv.segs.data(), lv.segs.size() * sizeof(int3));
        o.chunks = put(lv.chunks.data(), lv.chunks.size() * sizeof(int3));
        o.kids = put(lv.kids.data(), lv.kids.size() * sizeof(int2));
        off.push_back(o);
        maxseg = std::max(maxseg, lv.segs.size());
    }
    const size_t foff = put(finals.data(), finals.size() * sizeof(int3));
    const size_t nbytes = (size_t)n * 4;
    // two buffers of the three axes' keys in the current order (each level
    // reads one and writes the other), then the pick pass's candidates
    uint32_t *kmem = (uint32_t *)scratch(kSlotOrb0, 8 * nbytes);
    // original index per position, same two-buffer scheme as the keys
    int32_t *cbuf[2] = {(int32_t *)scratch(kSlotOrb1, nbytes), (int32_t *)scratch(kSlotOrb2, nbytes)};
    char *dtab = (char *)scratch(kSlotOrb3, tab.size() + 16);
    // states of two levels (the partition fills in the next one's), then one
    // histogram row per segment
    const size_t stbytes = (maxseg * sizeof(SegState) + 63) & ~size_t(63);
    char *state = (char *)scratch(kSlotOrb4, 2 * stbytes + maxseg * kBins * 4 + 64);
    if (!kmem || !cbuf[0] || !cbuf[1] || !dtab || !state) {
        set_error("cannot allocate ORB scratch");
        return NBODY_E_NOMEM;
    }
    uint32_t *kbuf[2] = {kmem, kmem + 3 * (size_t)n};
    uint64_t *cand = (uint64_t *)(kmem + 6 * (size_t)n);  // the keys of a window's bodies (k_orb_pick)
    SegState *st[2] = {(SegState *)state, (SegState *)(state + stbytes)};
    uint32_t *hist = (uint32_t *)(state + 2 * stbytes);
    {
        // stage the tables through pinned host memory owned by the library;
        // the previous upload must have completed before the buffer is reused
        std::lock_guard<std::mutex> lk(g_orb_mu);
        if (g_pinned_last) (void)hipEventSynchronize(g_pinned_last);
        if (g_pinned_size < tab.size()) {
            if (g_pinned) (void)hipHostFree(g_pinned);
            g_pinned = nullptr;
            g_pinned_size = 0;
            if (hipHostMalloc(&g_pinned, std::max<size_t>(tab.size(), 4096), hipHostMallocDefault) != hipSuccess) {
                set_error("cannot allocate pinned ORB tables");
                return NBODY_E_NOMEM;
            }
            g_pinned_size = std::max<size_t>(tab.size(), 4096);
        }
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) {
            set_error("hipGetDevice failed");
            return NBODY_E_HIP;
        }
        hipEvent_t &ev = g_pinned_evs[dev];
        if (!ev && hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
            ev = nullptr;
            set_error("cannot create ORB event");
            return NBODY_E_HIP;
        }
        if (!tab.empty()) {
            std::memcpy(g_pinned, tab.data(), tab.size());
            hipError_t e = hipMemcpyAsync(dtab, g_pinned, tab.size(), hipMemcpyHostToDevice, s);
            if (e != hipSuccess) return hip_fail(e, "ORB table upload");
        }
        hipError_t e = hipEventRecord(ev, s);
        if (e != hipSuccess) return hip_fail(e, "ORB event");
        g_pinned_last = ev;
    }
    const int nb = (n + kOrbBlock - 1) / kOrbBlock;
    if (prec == NBODY_F64)
        hipLaunchKernelGGL(k_orb_coords<double4>, dim3(nb), dim3(kOrbBlock), 0, s, (const double4 *)pm, n,
                           kbuf[0], cbuf[0]);
    else
        hipLaunchKernelGGL(k_orb_coords<float4>, dim3(nb), dim3(kOrbBlock), 0, s, (const float4 *)pm, n,
                           kbuf[0], cbuf[0]);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "ORB coordinates");
    for (size_t l = 0; l < levels.size(); ++l) {
        const int nseg = (int)levels[l].segs.size(), nch = (int)levels[l].chunks.size();
        const int3 *segs = (const int3 *)(dtab + off[l].segs);
        const int3 *chunks = (const int3 *)(dtab + off[l].chunks);
        const int2 *kids = (const int2 *)(dtab + off[l].kids);
        const bool more = l + 1 < levels.size();
        const int3 *segs_next = more ? (const int3 *)(dtab + off[l + 1].segs) : nullptr;
        const int nseg_next = more ? (int)levels[l + 1].segs.size() : 0;
        const int i = (int)(l & 1), o = 1 - i;
        if (l == 0) {
            hipLaunchKernelGGL(k_orb_init, dim3((unsigned)maxseg), dim3(kOrbBlock), 0, s, segs, nseg, st[i], hist);
            hipLaunchKernelGGL(k_orb_bbox, dim3(nch), dim3(kOrbBlock), 0, s, chunks, kbuf[i], n, st[i]);
        }
        int longest = 0;
        for (const int3 &sg : levels[l].segs) longest = std::max(longest, sg.y);
        const int rounds = longest > kLongSegment ? kRounds : kShortRounds;
        for (int r = 0; r < rounds; ++r)
            hipLaunchKernelGGL(k_orb_hist, dim3(nch), dim3(kPassBlock), 0, s, chunks, segs, kbuf[i], n, cbuf[i],
                               st[i], hist, r, segs_next, nseg_next, st[o]);
        hipLaunchKernelGGL(k_orb_pick, dim3(nch), dim3(kPassBlock), 0, s, chunks, segs, kbuf[i], n, cbuf[i], st[i],
                           cand);
        hipLaunchKernelGGL(k_orb_partition, dim3(nch), dim3(kPassBlock), 0, s, chunks, segs, kids, kbuf[i], kbuf[o],
                           n, cbuf[i], cbuf[o], st[i], st[o]);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "ORB level");
    }
    hipLaunchKernelGGL(k_orb_block, dim3((unsigned)finals.size()), dim3(kFinBlock), 0, s,
                       (const int3 *)(dtab + foff), kbuf[0], kbuf[1], cbuf[0], cbuf[1], n, leaf, perm);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "ORB leaves");
    return NBODY_OK;
}

void orb_release()
{
    std::lock_guard<std::mutex> lk(g_orb_mu);
    for (auto &kv : g_pinned_evs) {
        (void)hipEventSynchronize(kv.second);
        (void)hipEventDestroy(kv.second);
    }
    g_pinned_evs.clear();
    g_pinned_last = nullptr;
    if (g_pinned) (void)hipHostFree(g_pinned);
    g_pinned = nullptr;
    g_pinned_size = 0;
}

}  // namespace nbi
