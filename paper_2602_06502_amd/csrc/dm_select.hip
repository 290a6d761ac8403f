// SLO-aware candidate selection in request order (Sec. 3.2).
//
// Every request takes its cache-affine candidate unless that candidate's
// TTFT misses the SLO and the other one is less loaded (equal matches: the
// less loaded, first candidate on ties); the chosen instance's load grows by
// the request's uncached tokens before the next request is decided.  The
// batch result is therefore defined by processing the requests one by one.
// The single-criterion rules of the ablation study (Sec. 4.3) run on the same
// machinery: cache affinity is the SLO-aware rule with an unbounded TTFT
// budget, least load is the equal-match rule for every request, and minimum
// TTFT has a bound of its own in the walk's steps (see DM_BOUND_TTFT).
//
// Fast path (uncached counts within 32 bits, live loads within 2^62 of the
// smallest; checked on the device), on 32-bit
// absolute loads when every load stays below 2^31, else on 64-bit loads
// relative to the smallest:
//   sel_prep_kernel   one thread per request packs a 16-byte record: the
//                     affine candidate a and the other o (dense indices),
//                     their uncached tokens, and th such that the rule reads
//                     "take a iff L_a <= max(th, L_o)" (clamped to 32 bits;
//                     the 64-bit walk recomputes it exactly);
//   sel_level_kernel  one wave per block of requests (64 to 2048 by the
//                     batch's size): the dependency
//                     level of every request inside its block (runs of up
//                     to three same-pair requests sharing a level), and the
//                     packing of whole levels into windows of two sets of
//                     64 lanes (one set for the window's even depths, one
//                     for its odd ones);
//   sel_fill_kernel   the windows' places, the walk records of every lane
//                     of both sets of every window and each request's slot;
//   select_walk_kernel one wave picks the path and the load width, then walks
//                     the windows in order and, inside a
//                     window, the levels in order: requests of one level
//                     share no instance, so they run together on loads kept
//                     in LDS, and each sees exactly the loads that the
//                     request-order walk would show it;
//   sel_out_kernel    chosen instance, TTFT and flags of every request from
//                     its recorded pre-update loads, in parallel.
// Slow path: the same rule, one request at a time, on 64-bit loads in LDS.
//
// The windowed path once stopped at 256 live instances (8-bit dense indices);
// a batch on more took the slow path: 65,536 requests on 512 instances
// 14.2 ms, 0.21 us each, against 0.66 ms in windows.
#include <algorithm>
#include <type_traits>

#include "dm_internal.h"

namespace dm {
namespace {

constexpr int kSelSlot = kSlotSelect;  // selection work arrays

// Shared by every selection kernel: the rule given the two candidates'
// pre-update loads.  kind bit0 = compare the loads (equal match, or the
// least-load rule), bit1 = c1 is the cache-affine candidate, bit2 = compare
// the TTFT estimates, bit3 = keep the cache-affine candidate whatever its
// TTFT; th = the affine candidate's load below which its TTFT meets the SLO,
// or for bit2 per * (u2 - u1), so that t1 <= t2 reads
// floor(L1 / 2^q) - floor(L2 / 2^q) <= th.
__device__ __forceinline__ bool pick_first(uint32_t kind, int64_t L1, int64_t L2, int64_t th,
                                           uint32_t qshift)
{
    if (kind & 4)
        return (L1 >> qshift) - (L2 >> qshift) <= th;
    if (kind & 1)
        return L1 <= L2;
    if (kind & 8)
        return (kind & 2) != 0;
    if (kind & 2)
        return L1 < th || !(L2 < L1);
    return !(L2 < th || !(L1 < L2));
}

// One batch and its rule, as the walk and the epilogue read them.
// Requests 0..n-1 here are one part of the batch; the second candidates and
// matches lie `second` entries after the first ones.
struct SelArgs {
    const int64_t* offsets;
    uint64_t n, second;
    uint32_t bshift;
    const uint32_t* cand;
    const uint32_t* match;
    uint8_t* flags;
    uint32_t* chosen;
    int64_t* ttft;
    int64_t* loads;
    const uint32_t* live_ids;
    uint32_t n_live, S;
    int64_t tbase, per;
    uint32_t qshift;
    int64_t slo;
    uint32_t policy;
};

// Per-lane request record for the serial loop and the output epilogue.
struct SelRec {
    uint32_t c1, c2, kind;
    bool eq, aff1;  // equal match; c1 has more cached blocks
    bool a2;        // the fast path's records take c2 as their "a" instance
    int64_t u1, u2, th;
};

__device__ __forceinline__ SelRec load_rec(const SelArgs& g, uint64_t r, bool ok)
{
    SelRec s;
    s.c1 = ok ? g.cand[r] : 0;
    s.c2 = ok ? g.cand[g.second + r] : 0;
    const uint32_t m1 = ok ? g.match[r] : 0, m2 = ok ? g.match[g.second + r] : 0;
    const int64_t len = ok ? g.offsets[r + 1] - g.offsets[r] : 0;
    s.u1 = len - ((int64_t)m1 << g.bshift);
    s.u2 = len - ((int64_t)m2 << g.bshift);
    s.eq = m1 == m2;
    s.aff1 = m1 > m2;
    // T_a <= slo  <=>  floor(L_a / 2^q) <= slo - base - per*u_a  <=>  L_a < th
    s.th = (g.slo - g.tbase - g.per * (s.aff1 ? s.u1 : s.u2) + 1) * ((int64_t)1 << g.qshift);
    s.kind = (s.eq ? 1u : 0u) | (s.aff1 ? 2u : 0u);
    s.a2 = !s.eq && !s.aff1;
    if (g.policy == DM_POLICY_CACHE_AFFINITY) {
        s.kind |= 8u;
    } else if (g.policy == DM_POLICY_LEAST_LOADED) {
        s.kind = 1u;
        s.a2 = false;
    } else if (g.policy == DM_POLICY_MIN_TTFT) {
        s.kind = 4u;
        s.th = g.per * (s.u2 - s.u1);
        s.a2 = false;
    }
    return s;
}

__device__ __forceinline__ void store_out(const SelArgs& g, const SelRec& s, uint64_t r,
                                          int64_t L1, int64_t L2)
{
    const bool pick1 = pick_first(s.kind, L1, L2, s.th, g.qshift);
    const int64_t t1 = g.tbase + g.per * s.u1 + (L1 >> g.qshift);
    const int64_t t2 = g.tbase + g.per * s.u2 + (L2 >> g.qshift);
    uint32_t f = g.flags[r];
    if (t1 > g.slo && t2 > g.slo)
        f |= 2;
    if (s.eq)
        f |= 4;
    else if (pick1 != s.aff1)
        f |= 1;
    g.chosen[r] = pick1 ? s.c1 : s.c2;
    g.ttft[r] = pick1 ? t1 : t2;
    g.flags[r] = (uint8_t)f;
}

// Serial selection by one wave: L holds every slot's load.  All lanes read
// the pair of the request in turn (broadcast) and take its decision; lane 0
// writes the chosen load.  Rules other than minimum TTFT read "take a iff
// L_a <= max(bound, L_o)", a the cache-affine candidate (c1 for equal
// matches and the least-load rule).
template <bool TTFT>
__device__ void select_serial(const SelArgs& g, int64_t* L)
{
    const int lane = lane_id();
    for (uint32_t i = lane; i < g.S; i += kWave)
        L[i] = g.loads[i];
    __syncthreads();
    for (uint64_t r0 = 0; r0 < g.n; r0 += kWave) {
        const uint64_t r = r0 + lane;
        const bool ok = r < g.n;
        const SelRec s = load_rec(g, r, ok);
        const uint32_t pair = s.a2 ? s.c2 | s.c1 << 16 : s.c1 | s.c2 << 16;
        const int64_t ua = s.a2 ? s.u2 : s.u1, uo = s.a2 ? s.u1 : s.u2;
        int64_t bound = s.th;
        if constexpr (!TTFT)
            bound = (s.kind & 1) || s.th == INT64_MIN ? INT64_MIN
                    : (s.kind & 8)                    ? INT64_MAX
                                                      : s.th - 1;
        int64_t myA = 0, myO = 0;
        const int cnt = (int)(g.n - r0 < (uint64_t)kWave ? g.n - r0 : kWave);
        for (int j = 0; j < cnt; j++) {
            const uint32_t P = __builtin_amdgcn_readlane(pair, j), A = P & 0xFFFF, O = P >> 16;
            const int64_t T = (int64_t)readlane_u64((uint64_t)bound, j);
            const int64_t UA = (int64_t)readlane_u64((uint64_t)ua, j);
            const int64_t UO = (int64_t)readlane_u64((uint64_t)uo, j);
            const int64_t La = L[A], Lo = L[O];
            const bool take = TTFT ? (La >> g.qshift) - (Lo >> g.qshift) <= T
                                   : La <= (T > Lo ? T : Lo);
            const int64_t nv = take ? La + UA : Lo + UO;
            __syncthreads();
            if (lane == 0)
                L[take ? A : O] = nv;
            __syncthreads();
            if (lane == j) {
                myA = La;
                myO = Lo;
            }
        }
        if (ok)
            store_out(g, s, r, s.a2 ? myO : myA, s.a2 ? myA : myO);
    }
    __syncthreads();
    for (uint32_t i = lane; i < g.S; i += kWave)
        g.loads[i] = L[i];
}

// ---------------------------------------------------------------------------
// Fast path.
// ---------------------------------------------------------------------------

// A request whose latest earlier request of its block on both of its
// instances is one request with the same pair and cache-affine instance
// joins that request's run while the run holds fewer than kRunMax requests:
// all take the same level, each replays the decisions of the run's earlier
// members (uncached tokens and thresholds copied into its record) before
// its own, and only the run's last member writes the pair's loads.
// Replaying zero increments changes nothing.
constexpr uint32_t kRunMax = 3;

// Per-request record of the packing kernel.
struct SelPack {
    uint32_t w;   // a | o << 16 (dense indices)
    uint32_t ua;  // uncached tokens on a
    uint32_t uo;  // uncached tokens on o
    int32_t th;   // take a iff L_a <= max(th, L_o), relative loads
};

// Per-lane record of one lane set of a window, in the form the window's
// depth steps consume:
// the LDS byte offsets (within the walk's array of 4-byte slots: a spare
// slot per lane, then the loads) of L_a and
// L_o, where the request writes them (its spare slot unless it is the last
// member of its run), rel = its depth in the window (0-based) + the
// window's entry step e, and the window's control word e | (passes - 1) << 4.
// Lanes past a set's requests and the padding windows are inert: every
// offset is the lane's spare slot and rel matches no step.
struct WalkRec {
    uint32_t a4, o4, wa, wo;
    uint32_t rel, ctl;
    uint32_t ua, uo;
    int32_t th;
    uint32_t pua, puo;    // the run's first member: its uncached tokens on a and o
    int32_t pth;          // and its threshold (zeros for a run's first member)
    uint32_t pua2, puo2;  // the run's second member, for its third (else zeros)
    int32_t pth2;
    uint32_t pad;
};
constexpr uint32_t kInertRel = 0xFFFFFFFFu;

// Dense indices fit the level kernel's byte codes up to this many live
// instances; past it, the kernel's wide form (two bytes each).
constexpr uint32_t kByteLive = 256;
constexpr int kPrefetch = 6;  // record windows in flight ahead of the walk
// Lane sets of a window: every lane holds one request for the window's steps
// of even number and one for its steps of odd number.
constexpr uint32_t kSets = 2;

// grow[d] bounds how much live instance d's load can grow in this batch (the
// larger uncached count of every request that has it as a candidate);
// grow[kMaxSlots] is set by a record whose counts do not fit 32 bits.  Both
// start at zero.
__global__ __launch_bounds__(256) void sel_prep_kernel(
    const int64_t* __restrict__ offsets, uint64_t n, uint64_t second, uint32_t bshift,
    const uint32_t* __restrict__ cand, const uint32_t* __restrict__ match,
    const uint32_t* __restrict__ dense, uint32_t n_live, int64_t tbase, int64_t per,
    uint32_t qshift, int64_t slo, uint32_t policy, SelPack* __restrict__ rec,
    unsigned long long* __restrict__ grow)
{
    extern __shared__ unsigned long long sg[];  // [n_live]
    for (uint32_t k = threadIdx.x; k < n_live; k += blockDim.x)
        sg[k] = 0;
    __syncthreads();
    unsigned long long bad = 0;
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n;
         r += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t m1 = match[r], m2 = match[second + r];
        const int64_t len = offsets[r + 1] - offsets[r];
        const int64_t u1 = len - ((int64_t)m1 << bshift), u2 = len - ((int64_t)m2 << bshift);
        // least load: every request as an equal match, c1 as "a"
        const bool eq = m1 == m2 || policy == DM_POLICY_LEAST_LOADED;
        const bool aff2 = m2 > m1 && policy != DM_POLICY_LEAST_LOADED &&
                          policy != DM_POLICY_MIN_TTFT;
        const uint32_t d1 = dense[cand[r]], d2 = dense[cand[second + r]];
        // T_a <= slo  <=>  floor(L_a / 2^q) <= slo - tbase - per*u_a  <=>
        // L_a < (slo - tbase - per*u_a + 1) 2^q, i.e. "take a iff L_a <=
        // max(th, L_o)" with th one less.  The 32-bit walk uses absolute loads
        // in [0, 2^31 - 1), so th is clamped to that range; equal matches:
        // take c1 iff L1 <= L2, th = -2^31; cache affinity: always a,
        // th = 2^31 - 1.
        // Minimum TTFT, a = c1, D = 2^q: floor(L_a / D) - floor(L_o / D) <= d
        // with d = per (u_o - u_a)  <=>  L_a <= (L_o | (D - 1)) + d D; th = d D
        // clamped to 32 bits, which the walk adds saturating (loads are in
        // [0, 2^31), so a saturated sum decides as the exact one).
        int32_t th = INT32_MIN;
        if (policy == DM_POLICY_MIN_TTFT) {
            const int64_t d = per * (u2 - u1), lim = (int64_t)1 << 31;
            const int64_t t = d >= lim ? lim : d <= -lim ? -lim : qshift < 31 ? d * (1ll << qshift)
                              : d > 0  ? lim : d < 0 ? -lim : 0;
            th = (int32_t)(t >= lim ? INT32_MAX : t <= -lim ? INT32_MIN : t);
        } else if (!eq && policy == DM_POLICY_CACHE_AFFINITY) {
            th = INT32_MAX;
        } else if (!eq) {
            const int64_t t = (slo - tbase - per * (aff2 ? u2 : u1) + 1) * ((int64_t)1 << qshift) - 1;
            th = (int32_t)(t < -1 ? -1 : (t > INT32_MAX ? INT32_MAX : t));
        }
        SelPack p;
        p.w = aff2 ? d2 | d1 << 16 : d1 | d2 << 16;
        p.ua = (uint32_t)(aff2 ? u2 : u1);
        p.uo = (uint32_t)(aff2 ? u1 : u2);
        p.th = th;
        rec[r] = p;
        const bool ok = u1 >= 0 && u2 >= 0 && u1 <= INT32_MAX && u2 <= INT32_MAX;
        bad |= ok ? 0ull : 1ull;
        if (ok) {
            const unsigned long long g = (unsigned long long)(u1 > u2 ? u1 : u2);
            atomicAdd(&sg[d1], g);
            if (d2 != d1)
                atomicAdd(&sg[d2], g);
        }
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < n_live; k += blockDim.x)
        if (sg[k])
            atomicAdd(&grow[k], sg[k]);
    if (bad)
        atomicOr(&grow[kMaxSlots], 1ull);
}

// Walk windows from dependency levels.  Requests are grouped in blocks of
// LB requests (request order).  Inside a block, a request's level is 1 + the
// larger level of the latest earlier request of the block on either
// candidate (0 when none), except that a request that joins a run (see
// kRunMax) takes the run's level.
// Along every instance's requests the level strictly grows outside runs, so
// the requests (runs) of one level touch pairwise distinct instances, and
// any order of the levels' requests that keeps levels in order and the
// blocks in order gives every request exactly the loads of the one-by-one
// walk.  A level of more than 64 requests is cut, runs kept whole, into
// parts of at most 64, each part a depth of its own.  Windows take
// consecutive parts, one per depth, and hold two sets of 64 lanes: the
// depths alternate between the sets (steps of even and odd number), so a
// window holds up to 128 requests.  Packing the same parts into windows of
// one set of 64 lanes would close a window only when the next part does not
// fit, so any two consecutive such windows hold more than 64 requests and a
// block needs at most 2 * ceil(LB / 65) + 1 of them; the two-set packing
// needs no more.
//
// Larger blocks give fewer depth steps and windows (on the large batch,
// 78,742 steps in 9,832 windows with blocks of 2048 against 79,786 in
// 10,225 with 1024) but take the level kernel longer per block, in
// proportion.  Batches of at least kLargeFrom requests use blocks of 2048,
// others blocks of 1024, and unpipelined ones of at most kSmallTo requests
// blocks of 256, whose kernel ends in a quarter of the time (124 to 31 us on
// 8 instances) for a walk some 5% longer.  Whole calls, 1024 against 256:
// 1,024 requests 245 and 142 us, 4,096 chat requests 333 and 267, 32,768 on
// 512 instances 417 and 374, 65,536 chat requests 1,804 and 1,780; at 131,072
// the two meet.  Blocks of 64 for at most kTinyTo: 1,024 requests 106 us with
// blocks of 256, 92 with 128, 83 with 64; 4,096 chat requests 236, 223 and 224;
// at 16,384 the three meet, and 65,536 on 512 instances take 561, 595 and 598.
// Just past both lines the smaller blocks would still be ahead, by little: 256
// against 64 on 32 instances, 4,097 chat requests 203 and 194 us, 6,000 231 and
// 225, 8,192 260 and 259, 12,000 315 and 318 (short prompts 206 and 191, 235 and
// 225, 275 and 266, 342 and 334); 1024 against 256 on 128 instances, 65,537
// requests 658 and 629, 80,000 755 and 734, 100,000 892 and 865, 131,072 1,108 and
// 1,089 (short prompts 619 and 591, 712 and 687, 840 and 826, 1,048 and 1,048).
// Pipelined, the kernel runs beside the previous walk, which is what the
// batches wait for.
template <uint32_t LB>
struct LevelShape {
    static constexpr uint32_t block = LB;
    // windows per block
    static constexpr uint32_t wincap = LB == 64 ? 5u : LB == 256 ? 9u : LB == 1024 ? 36u : 66u;
    static_assert(wincap >= 2 * ((LB + 64) / 65) + 1, "room for the windows of a block");
};
constexpr uint64_t kLargeFrom = 1u << 19, kSmallTo = 1u << 16, kTinyTo = 1u << 12;
// The batch limit follows the large layout; the others only serve
// batches whose slots stay far inside 32 bits.
static_assert(LevelShape<2048>::block == kSelBlock &&
                  LevelShape<2048>::wincap == kSelWindowsPerBlock &&
                  kLargeFrom / 1024 * LevelShape<1024>::wincap * kSets * kWave < (1ull << 32),
              "dm_route_batch's batch limit assumes this layout");
// Block size and window capacity of a batch of n requests; hidden: the level
// kernel runs beside an earlier walk.
struct BlockShape {
    uint32_t block, wincap;
};
static BlockShape block_shape(uint64_t n, bool hidden)
{
    if (n >= kLargeFrom)
        return BlockShape{LevelShape<2048>::block, LevelShape<2048>::wincap};
    if (n <= kTinyTo && !hidden)
        return BlockShape{LevelShape<64>::block, LevelShape<64>::wincap};
    if (n <= kSmallTo && !hidden)
        return BlockShape{LevelShape<256>::block, LevelShape<256>::wincap};
    return BlockShape{LevelShape<1024>::block, LevelShape<1024>::wincap};
}

// One wave per block.  Writes, per request, info = depth in its window |
// position in its run << 6 | (not the run's last) << 8 | run's first member
// << 9 | run's second member << 20 (block-local indices); per block, its
// window count, each window's depth and the block-local request index in
// every lane of both sets of every window (0xFFFF for none).  The result is that of taking the
// requests one by one; the wave takes them 64 at a time, in order:
//   - the latest earlier request on each instance: within the chunk from
//     per-instance lane masks, before it from the latest request of the
//     earlier chunks on that instance;
//   - a request whose latest earlier request on both instances is one
//     request of the same pair and orientation is a run candidate; its
//     position in the run is (the predecessor's position + 1) mod kRunMax,
//     0 for any other request (settled along the chunk's candidate chains
//     with wave-wide votes);
//   - levels: the least fixed point of the level rule over the chunk
//     (earlier chunks' levels are final; relaxation from 1, wave-wide votes);
//   - then, with the runs' sizes final, each run reserves its lanes within
//     its level (LDS atomics: any order of a level's runs is valid);
//   - the levels are cut into parts (a lane per level), and the parts placed
//     into windows by one uniform greedy pass over their sizes.
// Every LDS access is by this one wave, so no barrier is needed.
// LIVE: most live instances, kByteLive (pair codes of two bytes) or
// kMaxSlots; the per-instance tables of the larger form take 40 KB more LDS
// (two blocks a compute unit instead of four).
template <uint32_t LB, uint32_t LIVE>
__global__ __launch_bounds__(kWave) void sel_level_kernel(
    const SelPack* __restrict__ prep, uint64_t n, uint32_t* __restrict__ info,
    uint16_t* __restrict__ slotmap, uint8_t* __restrict__ wdepth, uint8_t* __restrict__ wcount,
    uint32_t* __restrict__ status)
{
    constexpr uint32_t kWinCap = LevelShape<LB>::wincap;
    constexpr uint32_t kBits = LIVE <= kByteLive ? 8 : 16, kMask = (1u << kBits) - 1;
    using Code = std::conditional_t<kBits == 8, uint16_t, uint32_t>;
    __shared__ unsigned long long cm[LIVE];  // lanes of the chunk on each instance
    __shared__ uint16_t last[LIVE];          // latest request of earlier chunks, + 1
    __shared__ Code W[LB];                   // a | o << kBits
    __shared__ int16_t P[LB];               // latest earlier request on a
    __shared__ uint8_t psn[LB];             // position in the run
    __shared__ uint16_t hd[LB];             // the run's first member
    __shared__ uint16_t lv[LB];
    __shared__ uint8_t has1[LB], has2[LB];  // a run has a 2nd / 3rd member
    __shared__ __align__(16) uint16_t key[LB];  // a run's first member: level << 2 | size
    __shared__ uint16_t hrank[LB];    // lanes of earlier runs of the same level
    __shared__ uint32_t cnt[LB + 2];  // requests per level (so far), then
                                               // each level's first part
    __shared__ uint16_t lstart[LB + 1];
    __shared__ uint16_t sorted[LB];   // requests by level, runs in order
    __shared__ uint16_t pl_s0[LB];     // part: first index in sorted
    __shared__ uint8_t pl_win[LB], pl_base[LB];  // window, first lane in set
    __shared__ uint16_t wfirst[kWinCap];        // first part of each window
    __shared__ uint16_t smap[kWinCap * kSets * kWave];
    __shared__ uint8_t wdep[kWinCap];
    const uint32_t lane = (uint32_t)lane_id();
    const uint64_t r0 = (uint64_t)blockIdx.x * LB;
    const uint32_t nb = (uint32_t)std::min<uint64_t>(LB, n - r0);
    const unsigned long long below = (1ull << lane) - 1, above = ~below << 1;
    for (uint32_t k = lane; k < LIVE; k += kWave) {
        last[k] = 0;
        cm[k] = 0;
    }
    for (uint32_t k = lane; k < LB + 2; k += kWave)
        cnt[k] = 0;
    for (uint32_t k = lane; k < kWinCap * kSets * kWave; k += kWave)
        smap[k] = 0xFFFF;
    {
        // all pair codes first: 32 loads in flight per lane, one wait
        uint32_t wv[LB / kWave];
#pragma unroll
        for (uint32_t k = 0; k < LB / kWave; k++) {
            const uint32_t t = k * kWave + lane;
            wv[k] = t < nb ? prep[r0 + t].w : 0u;
        }
#pragma unroll
        for (uint32_t k = 0; k < LB / kWave; k++)
            W[k * kWave + lane] = (Code)((wv[k] & kMask) | (wv[k] >> 16) << kBits);
    }
    uint32_t lmax = 0;
    for (uint32_t c0 = 0; c0 < nb; c0 += kWave) {
        const uint32_t t = c0 + lane;
        const bool valid = t < nb;
        const uint32_t w = W[t], a = w & kMask, o = w >> kBits;
        has1[t] = has2[t] = 0;
        if (valid) {
            atomicOr(&cm[a], 1ull << lane);
            if (o != a)
                atomicOr(&cm[o], 1ull << lane);
        }
        const unsigned long long ma = valid ? cm[a] : 0, mo = valid ? cm[o] : 0;
        if (valid)  // read by every lane of the wave above
            cm[a] = cm[o] = 0;
        auto latest = [&](unsigned long long m, uint32_t x) -> int {
            m &= below;
            return m ? (int)(c0 + 63 - __clzll(m)) : (int)last[x] - 1;
        };
        const int pa = valid ? latest(ma, a) : -1, po = valid ? latest(mo, o) : -1;
        P[t] = (int16_t)pa;
        // the last lane of the chunk on an instance records it for later chunks
        if (valid && !(ma & above))
            last[a] = (uint16_t)(t + 1);
        if (valid && o != a && !(mo & above))
            last[o] = (uint16_t)(t + 1);
        const bool cand = valid && pa >= 0 && pa == po && a != o && W[pa] == w;
        // positions: 0 off the candidate chains; a predecessor in an earlier
        // chunk is settled; one in this chunk settles in turn
        const bool inchunk = cand && (uint32_t)pa >= c0;
        uint32_t pos = cand && !inchunk ? (psn[pa] + 1u) % kRunMax : 0u;
        bool done = !inchunk;
        for (;;) {
            const int src = inchunk ? pa - (int)c0 : (int)lane;
            const uint32_t ppos = (uint32_t)__shfl((int)pos, src);
            const bool pdone = __shfl((int)done, src) != 0;
            const bool now = !done && pdone;
            if (now) {
                pos = (ppos + 1u) % kRunMax;
                done = true;
            }
            if (!__any(now))
                break;
        }
        psn[t] = (uint8_t)pos;
        uint32_t h = t;
        for (uint32_t k = 0; k < pos; k++)
            h = (uint32_t)P[h];
        hd[t] = (uint16_t)h;
        if (valid && pos == 1)
            has1[h] = 1;
        if (valid && pos == 2)
            has2[h] = 1;
        // levels of the chunk: the least fixed point, from 1 up; levels of
        // earlier chunks are final (read once), those of this chunk's
        // predecessors come from their lanes
        const bool ina = pa >= (int)c0, ino = po >= (int)c0;
        const uint32_t la0 = !ina && pa >= 0 ? lv[pa] : 0u, lo0 = !ino && po >= 0 ? lv[po] : 0u;
        const int sa = ina ? pa - (int)c0 : (int)lane, so = ino ? po - (int)c0 : (int)lane;
        uint32_t L = valid ? 1u : 0u;
        for (;;) {
            const uint32_t xa = (uint32_t)__shfl((int)L, sa), xo = (uint32_t)__shfl((int)L, so);
            const uint32_t va = ina ? xa : la0, vo = ino ? xo : lo0;
            const uint32_t nl = !valid ? 0u : pos > 0 ? va : 1u + std::max(va, vo);
            const bool ch = nl != L;
            L = nl;
            if (!__any(ch))
                break;
        }
        lv[t] = (uint16_t)L;
        lmax = std::max(lmax, L);
    }
    for (int d = 1; d < kWave; d <<= 1)
        lmax = std::max(lmax, (uint32_t)__shfl_xor((int)lmax, d));
    lmax = (uint32_t)__builtin_amdgcn_readfirstlane((int)lmax);  // uniform from here on
    // inclusive sum over the wave
    auto wave_incl = [&](uint32_t v) -> uint32_t {
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)v, d);
            if ((int)lane >= d)
                v += y;
        }
        return v;
    };
    // the lanes of the runs within their levels, with the runs' sizes final:
    // each run's first member reserves the run's size in its level's count.
    // Requests of one level are independent, so any order of a level's runs
    // is valid; a run's members stay together, in run order.
    for (uint32_t t = lane; t < nb; t += kWave) {
        const bool head = psn[t] == 0;
        const uint32_t L = lv[t], rs = 1u + has1[t] + has2[t];
        key[t] = head ? (uint16_t)(L << 2 | rs) : (uint16_t)0;
        if (head)
            hrank[t] = (uint16_t)atomicAdd(&cnt[L], rs);
    }
    // each level's first index in sorted (a scan of the counts)
    for (uint32_t l0 = 1, start = 0; l0 <= lmax; l0 += kWave) {
        const uint32_t l = l0 + lane, c = l <= lmax ? cnt[l] : 0u, x = wave_incl(c);
        if (l <= lmax)
            lstart[l] = (uint16_t)(start + x - c);
        start += (uint32_t)__builtin_amdgcn_readlane((int)x, kWave - 1);
    }
    for (uint32_t t = lane; t < nb; t += kWave)
        sorted[lstart[lv[t]] + hrank[hd[t]] + psn[t]] = (uint16_t)t;
    // Parts, one lane per level: a level of at most 64 requests is one part;
    // a larger one is cut run by run into parts of at most 64 (its requests
    // are independent, so its parts may take consecutive depths).  The parts
    // cover sorted in order, so part p holds [pl_s0[p], pl_s0[p + 1]); cnt[l]
    // becomes level l's first part (a scan of the part counts).
    auto cut = [&](uint32_t s0, uint32_t c, uint32_t first, bool write) -> uint32_t {
        uint32_t np = 1, part = 0;
        if (write)
            pl_s0[first] = (uint16_t)s0;
        for (uint32_t k = s0; k < s0 + c;) {
            const uint32_t sz = key[sorted[k]] & 3u;  // k is a run's first member
            if (part + sz > kWave) {
                if (write)
                    pl_s0[first + np] = (uint16_t)k;
                np++;
                part = 0;
            }
            part += sz;
            k += sz;
        }
        return np;
    };
    uint32_t npl = 0;
    for (uint32_t l0 = 1; l0 <= lmax; l0 += kWave) {
        const uint32_t l = l0 + lane;
        const bool has = l <= lmax;
        const uint32_t c = has ? cnt[l] : 0u, s0 = has ? lstart[l] : 0u;
        const uint32_t np = !has ? 0u : c <= kWave ? 1u : cut(s0, c, 0, false);
        const uint32_t x = wave_incl(np), first = npl + x - np;
        if (has) {
            cnt[l] = first;
            if (c <= kWave)
                pl_s0[first] = (uint16_t)s0;
            else
                (void)cut(s0, c, first, true);
        }
        npl += (uint32_t)__builtin_amdgcn_readlane((int)x, kWave - 1);
    }
    if (lane == 0)
        cnt[lmax + 1] = npl;
    // Windows of consecutive parts, one depth each: a window of depth D is
    // entered at step e = -D mod 16, so depth t runs on step e + t and takes
    // the lane set of that step's parity, (t + D) & 1.  S0 and S1 sum the
    // parts at an even and an odd distance from the window's last depth;
    // appending a part moves every other part one further, so the window
    // grows while c + S1 <= 64 and the depth stays below 65.  A window that
    // fits holds every window inside it, so closing at the first misfit
    // gives the fewest windows; any window that fits one set of 64 lanes
    // fits the two, so the bound of kWinCap holds.  Parts of one set are
    // those of one depth parity, so a part's first lane is the sum of the
    // earlier parts of its depth parity in the window.  The wave takes the
    // parts 64 at a time, their sizes in lanes; the decisions are uniform.
    uint32_t win = 0, D = 0, S0 = 0, S1 = 0, be = 0, bo = 0;
    for (uint32_t p0 = 0; p0 < npl; p0 += kWave) {
        const uint32_t p = p0 + lane;
        const uint32_t cl = p < npl ? (p + 1 < npl ? (uint32_t)pl_s0[p + 1] : nb) - pl_s0[p] : 0u;
        uint32_t wl = 0, bl = 0;
        const uint32_t m = npl - p0 < (uint32_t)kWave ? npl - p0 : (uint32_t)kWave;
        for (uint32_t i = 0; i < m; i++) {
            const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)cl, (int)i);
            if (D > 0 && (D == kWave || c + S1 > kWave)) {
                if (win < kWinCap) {
                    wdep[win] = (uint8_t)D;
                    wfirst[win] = (uint16_t)(p0 + i - D);
                }
                win++;
                D = S0 = S1 = be = bo = 0;
            }
            const uint32_t base = (D & 1u) ? bo : be;
            if (D & 1u)
                bo += c;
            else
                be += c;
            wl = lane == i ? win : wl;
            bl = lane == i ? base : bl;
            const uint32_t s0n = c + S1;
            S1 = S0;
            S0 = s0n;
            D++;
        }
        if (p < npl) {
            pl_win[p] = (uint8_t)wl;
            pl_base[p] = (uint8_t)bl;
        }
    }
    if (win < kWinCap) {
        wdep[win] = (uint8_t)D;
        wfirst[win] = (uint16_t)(npl - D);
    }
    const uint32_t nwin = win + 1;
    const bool okw = nwin <= kWinCap;
    if (!okw && lane == 0)  // cannot happen (see above); no window of this block is walked
        atomicOr(status, kErrInval);
    if (okw) {
        for (uint32_t t = lane; t < nb; t += kWave) {
            const uint32_t L = lv[t], pos = psn[t], h = hd[t], rs = 1u + has1[h] + has2[h];
            const uint32_t k = lstart[L] + hrank[h] + pos;  // index in sorted
            uint32_t p = cnt[L];
            while (p + 1 < cnt[L + 1] && pl_s0[p + 1] <= k)
                p++;
            const uint32_t w = pl_win[p], d = p - wfirst[w], set = (d + wdep[w]) & 1u;
            const uint32_t ln = pl_base[p] + (k - pl_s0[p]);
            smap[(w * kSets + set) * kWave + ln] = (uint16_t)t;
            const uint32_t m1 = pos == 2 ? (uint32_t)P[t] : 0u;
            info[r0 + t] = d | pos << 6 | (pos + 1 < rs ? 1u << 8 : 0u) | h << 9 | m1 << 20;
        }
    }
    for (uint32_t k = lane; k < kWinCap * kSets * kWave; k += kWave)
        slotmap[(uint64_t)blockIdx.x * kWinCap * kSets * kWave + k] = smap[k];
    if (lane < kWinCap)
        wdepth[(uint64_t)blockIdx.x * kWinCap + lane] = okw && lane < nwin ? wdep[lane] : 0;
    if (lane == 0)
        wcount[blockIdx.x] = (uint8_t)(okw ? nwin : 0);
}

// Exclusive scan of the blocks' window counts (one workgroup); total[0] =
// all windows.  Batches of more than kScanFrom blocks only: below, each wave
// of the fill kernel sums the counts before its block itself (at most 16
// loads a lane), which spares a launch of 4.7 us.
constexpr uint64_t kScanFrom = 1024;
__global__ __launch_bounds__(1024) void sel_scan_kernel(const uint8_t* __restrict__ wcount,
                                                        uint64_t nblk, uint32_t* __restrict__ woff,
                                                        uint32_t* __restrict__ total)
{
    __shared__ uint32_t part[1024 / kWave];
    __shared__ uint32_t carry;
    const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6;
    if (t == 0)
        carry = 0;
    __syncthreads();
    for (uint64_t c0 = 0; c0 < nblk; c0 += 1024) {
        const uint64_t b = c0 + t;
        const uint32_t v = b < nblk ? wcount[b] : 0;
        uint32_t x = v;  // inclusive scan within the wave
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, d);
            if ((int)lane >= d)
                x += y;
        }
        if (lane == 63)
            part[wv] = x;
        __syncthreads();
        uint32_t before = carry;
        for (uint32_t k = 0; k < wv; k++)
            before += part[k];
        if (b < nblk)
            woff[b] = before + x - v;
        __syncthreads();
        if (t == 1023)
            carry = before + x;
        __syncthreads();
    }
    if (t == 0)
        total[0] = carry;
}

// One wave per lane set of every (block, window) of capacity, then of
// 2 * kPrefetch padding windows: the walk records of every lane (inert past
// the set's requests) and each request's slot.  The records of window w's
// set s start at (w * kSets + s) * 64.  woff: the blocks' first windows, or
// null to sum wcount here and write total[0].
__global__ __launch_bounds__(4 * kWave) void sel_fill_kernel(
    const SelPack* __restrict__ prep, uint64_t n, const uint32_t* __restrict__ info,
    const uint16_t* __restrict__ slotmap, const uint8_t* __restrict__ wdepth,
    const uint8_t* __restrict__ wcount, const uint32_t* __restrict__ woff,
    uint32_t* __restrict__ total, uint64_t nblk, BlockShape bs, WalkRec* __restrict__ rec,
    uint32_t* __restrict__ slot_of)
{
    const uint32_t wincap = bs.wincap, bsize = bs.block;
    const int lane = lane_id();
    const uint64_t gw = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint64_t ws = gw / kSets;  // window of capacity
    const uint32_t set = (uint32_t)(gw % kSets);
    const uint32_t sp = 4u * lane;
    auto windows_before = [&](uint64_t b) -> uint32_t {
        if (woff)
            return b < nblk ? woff[b] : total[0];
        uint32_t v = 0;
        for (uint64_t i = lane; i < b; i += kWave)
            v += wcount[i];
        for (int d = 1; d < kWave; d <<= 1)
            v += (uint32_t)__shfl_xor((int)v, d);
        return v;
    };
    uint64_t win;
    uint32_t k = 0xFFFF, depth = 1;
    uint64_t blk = 0;
    if (ws < nblk * wincap) {
        blk = ws / wincap;
        const uint32_t lw = (uint32_t)(ws % wincap);
        if (lw >= wcount[blk])
            return;
        win = (uint64_t)windows_before(blk) + lw;
        k = slotmap[gw * kWave + lane];
        depth = wdepth[ws];
    } else if (ws < nblk * wincap + 2 * kPrefetch) {
        const uint32_t all = windows_before(nblk);
        if (!woff && gw == nblk * wincap * kSets && lane == 0)
            total[0] = all;
        win = (uint64_t)all + (ws - nblk * wincap);
    } else {
        return;
    }
    const uint32_t e = (0u - depth) & 15u, passes = (depth + 15u) >> 4;
    WalkRec q;
    q.ctl = e | (passes - 1) << 4;
    const uint64_t r = blk * bsize + k;
    if (k != 0xFFFF && r < n) {
        const SelPack me = prep[r];
        const uint32_t f = info[r], pos = (f >> 6) & 3;
        const bool not_last = (f >> 8) & 1;
        q.a4 = 4u * (kWave + (me.w & 0xFFFF));
        q.o4 = 4u * (kWave + (me.w >> 16));
        q.wa = not_last ? sp : q.a4;
        q.wo = not_last ? sp : q.o4;
        q.rel = (f & 63) + e;
        q.ua = me.ua;
        q.uo = me.uo;
        q.th = me.th;
        q.pua = q.puo = q.pua2 = q.puo2 = 0;
        q.pth = q.pth2 = 0;
        q.pad = 0;
        if (pos >= 1) {
            const SelPack m0 = prep[blk * bsize + ((f >> 9) & (bsize - 1))];
            q.pua = m0.ua;
            q.puo = m0.uo;
            q.pth = m0.th;
        }
        if (pos >= 2) {
            const SelPack m1 = prep[blk * bsize + ((f >> 20) & (bsize - 1))];
            q.pua2 = m1.ua;
            q.puo2 = m1.uo;
            q.pth2 = m1.th;
        }
        slot_of[r] = (uint32_t)((win * kSets + set) * kWave + lane);
    } else {
        q.a4 = q.o4 = q.wa = q.wo = sp;
        q.rel = kInertRel;
        q.ua = q.uo = q.pua = q.puo = q.pua2 = q.puo2 = q.pad = 0;
        q.th = q.pth = q.pth2 = 0;
    }
    rec[(win * kSets + set) * kWave + lane] = q;
}

// Walks the windows in order; see the file comment.  T is the load type:
// int32_t or int64_t relative loads.  rec holds 2 * kPrefetch inert padding
// windows past the last and lpre kPrefetch, so that the unrolled walk and
// its prefetch stay in bounds; lpre receives the pre-update loads (L_a, L_o)
// of every request relative to the base, as int32 pairs for the 32-bit walk
// and int64 pairs for the 64-bit one, at the request's slot (window w, set
// s, lane l: (w * kSets + s) * 64 + l).
// Byte address of a shared-memory element within the workgroup's LDS.
template <typename T>
__device__ __forceinline__ uint32_t lds_addr(T* p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) T*)p;
}

// One depth step of the 32-bit walk, as asm text for DM_WALK_BLOCK: the
// lanes of set S whose rel equals the inline constant K are on this depth
// (steps of even number take set A, of odd number set B).  The loads of a
// step live in one register pair X = (L_a, L_o): v[240:241] on even steps,
// v[242:243] on odd ones, so that a decision adds both of its increments
// with one 64-bit add.  No carry crosses the halves for a lane on its
// depth: on this path every live load and its growth stay below 2^31.  (A
// lane off its depth may carry; its values only reach its spare slot.)
// Reads X (L_o first), replays the decisions of the run's earlier members
// (no change for zero increments) into X: the loads this request saw;
// captures the previous step's pair XP (lane mask MP) into the other set's
// (La, Lo); M receives this step's lane mask.  Then the lane's own decision
// into v[246:247], and both loads of the pair written back (the second
// instance first, so that a pair of one instance keeps the first's value)
// -- to the lane's write slots (wa, wo) when on the depth, else to its spare
// slot.  The reads of a depth precede its writes in the LDS queue, and the
// writes of one depth precede the reads of the next, so the waits count
// this step's reads only.  Every step has the same instructions with
// fixed-size encodings (operands are registers and inline constants), which
// the computed entry relies on; the assembler checks the sizes.
// BND(T, TH, XO) computes into T the bound that L_a is compared with: the larger
// of the threshold and L_o, or for the minimum-TTFT rule L_o with its low q
// bits set plus the threshold, saturating (one more instruction a decision;
// 16,384 requests on 32 instances route in 0.45 ms against 2.98 ms one at a
// time on the serial path, which this rule took before).
#define DM_BOUND_SLO(T, TH, XO) "v_max_i32_e32 " T ", %[" TH "], " XO "\n\t"
#define DM_BOUND_TTFT(T, TH, XO)                                                               \
    "v_or_b32_e32 " T ", %[low], " XO "\n\t"                                                   \
    "v_add_i32 " T ", " T ", %[" TH "] clamp\n\t"
#define DM_STEP_TEXT(BND, K, XA, XO, X, M, XAP, XOP, MP, S, P)                                      \
    ".Ldmw%=_" #K ":\n\t"                                                                      \
    "ds_read_b32 " XO ", %[o4" S "]\n\t"                                                       \
    "ds_read_b32 " XA ", %[a4" S "]\n\t"                                                       \
    "v_cmp_eq_u32_e64 %[" M "], " #K ", %[rel" S "]\n\t"                                      \
    "v_cndmask_b32_e64 %[La" P "], %[La" P "], " XAP ", %[" MP "]\n\t"                         \
    "v_cndmask_b32_e64 %[Lo" P "], %[Lo" P "], " XOP ", %[" MP "]\n\t"                         \
    "v_cndmask_b32_e64 %[da], %[sp], %[wa" S "], %[" M "]\n\t"                                 \
    "v_cndmask_b32_e64 %[dz], %[sp], %[wo" S "], %[" M "]\n\t"                                 \
    "s_waitcnt lgkmcnt(1)\n\t"                                                                 \
    BND("v244", "pth" S, XO)                                                                   \
    "s_waitcnt lgkmcnt(0)\n\t"                                                                 \
    "v_cmp_le_i32_e32 vcc, " XA ", v244\n\t"                                                   \
    "v_cndmask_b32_e64 v244, 0, %[pua" S "], vcc\n\t"                                          \
    "v_cndmask_b32_e64 v245, %[puo" S "], 0, vcc\n\t"                                          \
    "v_lshl_add_u64 " X ", " X ", 0, v[244:245]\n\t"                                           \
    BND("v244", "pth2" S, XO)                                                                  \
    "v_cmp_le_i32_e32 vcc, " XA ", v244\n\t"                                                   \
    "v_cndmask_b32_e64 v244, 0, %[pua2" S "], vcc\n\t"                                         \
    "v_cndmask_b32_e64 v245, %[puo2" S "], 0, vcc\n\t"                                         \
    "v_lshl_add_u64 " X ", " X ", 0, v[244:245]\n\t"                                           \
    BND("v246", "th" S, XO)                                                                    \
    "v_cmp_le_i32_e32 vcc, " XA ", v246\n\t"                                                   \
    "v_cndmask_b32_e64 v244, 0, %[ua" S "], vcc\n\t"                                           \
    "v_cndmask_b32_e64 v245, %[uo" S "], 0, vcc\n\t"                                           \
    "v_lshl_add_u64 v[246:247], " X ", 0, v[244:245]\n\t"                                      \
    "ds_write_b32 %[dz], v247\n\t"                                                             \
    "ds_write_b32 %[da], v246\n\t"

#define DM_STEP_PAIR(BND, K0, K1)                                                              \
    DM_STEP_TEXT(BND, K0, "v240", "v241", "v[240:241]", "m0", "v242", "v243", "m1", "A", "B")    \
    DM_STEP_TEXT(BND, K1, "v242", "v243", "v[242:243]", "m1", "v240", "v241", "m0", "B", "A")

#define DM_SIZE_CHECK(K0, K1)                                                                  \
    ".if (.Ldmw%=_" #K1 " - .Ldmw%=_" #K0 ") != (.Ldmw%=_1 - .Ldmw%=_0)\n\t"                   \
    ".error \"walk steps differ in size\"\n\t"                                                 \
    ".endif\n\t"

#define DM_SET_OPERANDS(S)                                                                     \
    [a4##S] "v"(a4##S), [o4##S] "v"(o4##S), [wa##S] "v"(wa##S), [wo##S] "v"(wo##S),            \
        [th##S] "v"(c##S.th), [ua##S] "v"(c##S.ua), [uo##S] "v"(c##S.uo),                      \
        [pth##S] "v"(c##S.pth), [pua##S] "v"(c##S.pua), [puo##S] "v"(c##S.puo),                \
        [pth2##S] "v"(c##S.pth2), [pua2##S] "v"(c##S.pua2), [puo2##S] "v"(c##S.puo2)

// All depths of one window of the 32-bit walk in one block of 16 steps
// (K = 0..15), entered at step e by a computed jump (the PC-relative
// sequence of a long branch) and run np1 + 1 times, where the window's
// control word (the same in every lane) is e | np1 << 4; lane l of set A
// (B) is on even (odd) step K of pass j when its rel - 16 j = K.  The
// control word is read inside the block, so that the compiler waits only
// for this window's records.  The first step captures whatever its register
// set held, which is harmless: every lane of the batch is captured again
// after its own depth, and inert lanes' results are never read.  After the
// last pass the last depth's reads (an odd step: set B) are captured into
// (LaB, LoB).  e < 16 and np1 < 4 by the masks, and the assembler checks
// that the 16 steps have one size.
// J0..J3 name the scalar registers of the jump (JP the pair of J0 and J1).
#define DM_WALK_BLOCK(BND, JP, J0, J1, J2, J3)                                                   \
    asm volatile("v_readfirstlane_b32 " J3 ", %[ctl]\n\t"                                       \
                 "s_getpc_b64 " JP "\n"                                                       \
                 ".Ldmw%=_pc:\n\t"                                                             \
                 "s_and_b32 " J2 ", " J3 ", 15\n\t"                                            \
                 "s_mul_i32 " J2 ", " J2 ", (.Ldmw%=_1 - .Ldmw%=_0)\n\t"                       \
                 "s_add_u32 " J2 ", " J2 ", (.Ldmw%=_0 - .Ldmw%=_pc)\n\t"                      \
                 "s_add_u32 " J0 ", " J0 ", " J2 "\n\t"                                        \
                 "s_addc_u32 " J1 ", " J1 ", 0\n\t"                                            \
                 "s_bfe_u32 " J3 ", " J3 ", 0x20004\n\t"                                       \
                 "s_setpc_b64 " JP "\n"                                                       \
                 DM_STEP_PAIR(BND, 0, 1) DM_STEP_PAIR(BND, 2, 3) DM_STEP_PAIR(BND, 4, 5)             \
                 DM_STEP_PAIR(BND, 6, 7) DM_STEP_PAIR(BND, 8, 9) DM_STEP_PAIR(BND, 10, 11)           \
                 DM_STEP_PAIR(BND, 12, 13) DM_STEP_PAIR(BND, 14, 15)                               \
                 ".Ldmw%=_16:\n\t"                                                             \
                 "v_add_u32_e32 %[relA], -16, %[relA]\n\t"                                     \
                 "v_add_u32_e32 %[relB], -16, %[relB]\n\t"                                     \
                 "s_sub_u32 " J3 ", " J3 ", 1\n\t"                                             \
                 "s_cbranch_scc0 .Ldmw%=_0\n\t"                                                \
                 "v_cndmask_b32_e64 %[LaB], %[LaB], v242, %[m1]\n\t"                           \
                 "v_cndmask_b32_e64 %[LoB], %[LoB], v243, %[m1]\n\t"                           \
                 DM_SIZE_CHECK(1, 2) DM_SIZE_CHECK(2, 3) DM_SIZE_CHECK(3, 4)                   \
                 DM_SIZE_CHECK(4, 5) DM_SIZE_CHECK(5, 6) DM_SIZE_CHECK(6, 7)                   \
                 DM_SIZE_CHECK(7, 8) DM_SIZE_CHECK(8, 9) DM_SIZE_CHECK(9, 10)                  \
                 DM_SIZE_CHECK(10, 11) DM_SIZE_CHECK(11, 12) DM_SIZE_CHECK(12, 13)             \
                 DM_SIZE_CHECK(13, 14) DM_SIZE_CHECK(14, 15) DM_SIZE_CHECK(15, 16)             \
                 : [m0] "=&s"(m0), [m1] "=&s"(m1), [LaA] "+v"(LaA), [LoA] "+v"(LoA),          \
                   [LaB] "+v"(LaB), [LoB] "+v"(LoB), [da] "=&v"(da), [dz] "=&v"(dz),          \
                   [relA] "+v"(relA), [relB] "+v"(relB)                                        \
                 : DM_SET_OPERANDS(A), DM_SET_OPERANDS(B), [sp] "v"(sp4), [ctl] "v"(ctl),     \
                   [low] "s"(low)                                                              \
                 : J0, J1, J2, J3, "v240", "v241", "v242", "v243", "v244", "v245", "v246",     \
                   "v247", "vcc", "scc", "memory")

template <typename T, bool TTFT>
__device__ __forceinline__ void walk_windows(const SelArgs& g, const WalkRec* __restrict__ rec,
                                             const uint32_t* __restrict__ nwin, int64_t b0,
                                             longlong2* __restrict__ lpre, T* L)
{
    constexpr bool wide = sizeof(T) == 8;
    const int lane = lane_id();
    // a spare slot per lane, then the loads
    L[lane] = (T)0;
    for (uint32_t d = lane; d < g.n_live; d += kWave)
        L[kWave + d] = (T)(g.loads[g.live_ids[d]] - b0);
    __syncthreads();
    const uint64_t nw = __builtin_amdgcn_readfirstlane(nwin[0]);
    // the records hold offsets within L in 4-byte slots; the LDS address of
    // L itself is a link-time constant (zero when it is the only array)
    const uint32_t lbase = lds_addr(reinterpret_cast<int32_t*>(L));
    const uint32_t sp4 = lbase + 4u * lane;
    // the low q bits (loads of the 32-bit walk are below 2^31)
    const int32_t low = g.qshift < 31 ? (int32_t)((1u << g.qshift) - 1) : INT32_MAX;
    int32_t LaA32 = 0, LoA32 = 0, LaB32 = 0, LoB32 = 0;
    // window w: set A's records cA, set B's cB (same control word)
    auto window = [&](WalkRec& cA, WalkRec& cB, uint64_t w) {
        if constexpr (wide) {
            // the packed bounds are clamped to 32 bits: recompute them
            // exactly, relative to the base (equal matches: -inf; cache
            // affinity: +inf)
            const bool keep_a = g.policy == DM_POLICY_CACHE_AFFINITY;
            auto exact = [&](int32_t packed, uint32_t u) -> T {
                return packed == INT32_MIN ? (T)INT64_MIN
                       : keep_a            ? (T)INT64_MAX
                                           : (T)((g.slo - g.tbase - g.per * (int64_t)u + 1) *
                                                     ((int64_t)1 << g.qshift) -
                                                 1 - b0);
            };
            // take a, on the loads xa and xo relative to b0
            auto takes = [&](T xa, T xo, int32_t packed, uint32_t ua, uint32_t uo) -> bool {
                if constexpr (TTFT)
                    return ((xa + b0) >> g.qshift) - ((xo + b0) >> g.qshift) <=
                           g.per * ((int64_t)uo - (int64_t)ua);
                else
                    return xa <= std::max(exact(packed, ua), xo);
            };
            // Every lane reads and writes at every depth, without branches on
            // lane data; a lane not on the current depth, and a run member
            // other than the last, write their own spare slot.
            const uint32_t ctl = __builtin_amdgcn_readfirstlane(cA.ctl), e = ctl & 15u;
            const uint32_t depth = 16u * (((ctl >> 4) & 3u) + 1u) - e;
            const uint32_t sp = lane;
            T La[kSets] = {0, 0}, Lo[kSets] = {0, 0};
            auto step = [&](const WalkRec& c, uint32_t l, T& la, T& lo) {
                const T ua = (T)c.ua, uo = (T)c.uo, pua = (T)c.pua, puo = (T)c.puo;
                const T pua2 = (T)c.pua2, puo2 = (T)c.puo2;
                const uint32_t a = c.a4 >> 2, o = c.o4 >> 2, wa = c.wa >> 2, wo = c.wo >> 2;
                const bool act = c.rel - e == l;
                const T xa = L[a], xo = L[o];
                const bool p1 = takes(xa, xo, c.pth, c.pua, c.puo);
                const T x0 = xa + (p1 ? pua : (T)0), y0 = xo + (p1 ? (T)0 : puo);
                const bool p2 = takes(x0, y0, c.pth2, c.pua2, c.puo2);
                const T x1 = x0 + (p2 ? pua2 : (T)0), y1 = y0 + (p2 ? (T)0 : puo2);
                const bool take_a = takes(x1, y1, c.th, c.ua, c.uo);
                L[act ? wo : sp] = take_a ? y1 : y1 + uo;
                L[act ? wa : sp] = take_a ? x1 + ua : x1;
                la = act ? x1 : la;
                lo = act ? y1 : lo;
            };
            for (uint32_t l = 0; l < depth; l++) {
                if ((e + l) & 1u)
                    step(cB, l, La[1], Lo[1]);
                else
                    step(cA, l, La[0], Lo[0]);
            }
            lpre[(w * kSets) * kWave + lane] = make_longlong2(La[0], Lo[0]);
            lpre[(w * kSets + 1) * kWave + lane] = make_longlong2(La[1], Lo[1]);
        } else {
            // The same walk in hand-scheduled depth steps (DM_WALK_BLOCK): the
            // ALU work of a step that does not wait for its reads runs in the
            // shadow of the LDS round trip, and the window's depths run as one
            // straight block entered at the step that leaves exactly its
            // depth's steps (a pass of 16 more per further 16 depths).
            const uint32_t a4A = lbase + cA.a4, o4A = lbase + cA.o4;
            const uint32_t waA = lbase + cA.wa, woA = lbase + cA.wo;
            const uint32_t a4B = lbase + cB.a4, o4B = lbase + cB.o4;
            const uint32_t waB = lbase + cB.wa, woB = lbase + cB.wo;
            const uint32_t ctl = cA.ctl;
            uint32_t relA = cA.rel, relB = cB.rel;
            int32_t da, dz;
            uint64_t m0, m1;
            int32_t LaA = LaA32, LoA = LoA32, LaB = LaB32, LoB = LoB32;
            if constexpr (TTFT)
                DM_WALK_BLOCK(DM_BOUND_TTFT, "s[92:93]", "s92", "s93", "s94", "s95");
            else
                DM_WALK_BLOCK(DM_BOUND_SLO, "s[96:97]", "s96", "s97", "s98", "s99");
            (void)m0; (void)m1; (void)da; (void)dz;
            LaA32 = LaA;
            LoA32 = LoA;
            LaB32 = LaB;
            LoB32 = LoB;
            int2* lp = reinterpret_cast<int2*>(lpre);
            lp[(w * kSets) * kWave + lane] = make_int2(LaA, LoA);
            lp[(w * kSets + 1) * kWave + lane] = make_int2(LaB, LoB);
        }
    };
    // Records arrive kPrefetch windows ahead.  The loop is unrolled by
    // kPrefetch so that each slot is used where it was loaded (no register
    // moves, which would wait for every load in flight); windows past the
    // last (inert padded records and outputs) change nothing.  With an odd
    // unroll the compiler's wait at the loop head let only a few loads stay
    // in flight (vmcnt(5)), which cost 12-15% of the walk.
    static_assert(kPrefetch % 2 == 0, "keep the unroll even (see above)");
    auto at = [&](uint64_t w, uint32_t s) { return rec[(w * kSets + s) * kWave + lane]; };
    WalkRec qa[kPrefetch], qb[kPrefetch];
#pragma unroll
    for (int i = 0; i < kPrefetch; i++) {
        qa[i] = at(i, 0);
        qb[i] = at(i, 1);
    }
    // Let the first records land before the loop: the wait the compiler
    // places at the loop head must hold on entry as well as on the
    // back-edge, and with these loads in flight on entry it would wait for
    // every record in flight on each iteration.  (s_waitcnt vmcnt(0),
    // expcnt and lgkmcnt unconstrained, in the gfx9 encoding.)
    __builtin_amdgcn_s_waitcnt(0x0F70);
    for (uint64_t w = 0; w < nw; w += kPrefetch) {
#pragma unroll
        for (int i = 0; i < kPrefetch; i++) {
            window(qa[i], qb[i], w + i);
            qa[i] = at(w + kPrefetch + i, 0);
            qb[i] = at(w + kPrefetch + i, 1);
        }
    }
    __syncthreads();
    for (uint32_t d = lane; d < g.n_live; d += kWave)
        g.loads[g.live_ids[d]] = b0 + (int64_t)L[kWave + d];
}

#undef DM_WALK_BLOCK
#undef DM_SET_OPERANDS
#undef DM_SIZE_CHECK
#undef DM_STEP_PAIR
#undef DM_STEP_TEXT
#undef DM_BOUND_TTFT
#undef DM_BOUND_SLO

// One wave.  First the plan: the windowed path iff every record's uncached
// counts fit 32 bits; its loads are absolute 32-bit values when every live
// load lies in [0, 2^30) and grows by less than 2^30 whatever the decisions,
// else 64-bit values relative to the smallest live load, as long as they stay
// below it + 2^62; otherwise the serial path.  (Three kernels of 4.5 us each
// -- smallest load, plan, an empty serial path -- once ran around the walk.)
// plan[0] = 1 for the windowed path, plan[1] = 1 for its 64-bit loads, and
// base[0] their base, for the epilogue.
template <bool TTFT>
__global__ __launch_bounds__(kWave) void select_walk_kernel(
    SelArgs g, const WalkRec* __restrict__ rec, const uint32_t* __restrict__ nwin,
    const unsigned long long* __restrict__ grow, uint32_t* __restrict__ plan,
    int64_t* __restrict__ base, longlong2* __restrict__ lpre)
{
    // Claim the whole register file of this wave's SIMD (256 + 256
    // registers), so that no wave of another kernel shares its issue slots:
    // this single wave is the serial critical path of a batch, and with
    // pipelining the next batch's kernels run beside it.
    asm volatile("" ::: "v255", "a255");
    __shared__ int64_t L[kWave + kMaxSlots];  // one spare slot per lane, then the loads
    const int lane = lane_id();
    int64_t mn = INT64_MAX, mx = INT64_MIN;
    unsigned long long gmax = 0;
    for (uint32_t d = lane; d < g.n_live; d += kWave) {
        const int64_t v = g.loads[g.live_ids[d]];
        const unsigned long long u = grow[d];
        mn = v < mn ? v : mn;
        mx = v > mx ? v : mx;
        gmax = u > gmax ? u : gmax;
    }
    for (int d = 1; d < kWave; d <<= 1) {
        const int64_t a = (int64_t)shfl_xor_u64((uint64_t)mn, d);
        const int64_t b = (int64_t)shfl_xor_u64((uint64_t)mx, d);
        const unsigned long long u = shfl_xor_u64(gmax, d);
        mn = a < mn ? a : mn;
        mx = b > mx ? b : mx;
        gmax = u > gmax ? u : gmax;
    }
    // mx - mn cannot wrap in unsigned arithmetic
    const bool windowed = __builtin_amdgcn_readfirstlane(
        grow[kMaxSlots] == 0 && (unsigned long long)mx - (unsigned long long)mn < (1ull << 62) &&
        gmax < (1ull << 62));
    const bool narrow =
        __builtin_amdgcn_readfirstlane(mn >= 0 && mx < (1ll << 30) && gmax < (1ull << 30));
    const int64_t b0 = narrow ? 0 : (int64_t)readlane_u64((uint64_t)mn, 0);
    if (lane == 0) {
        plan[0] = windowed ? 1 : 0;
        plan[1] = windowed && !narrow ? 1 : 0;
        base[0] = b0;
    }
    if (!windowed)
        select_serial<TTFT>(g, L);
    else if (!narrow)
        walk_windows<int64_t, TTFT>(g, rec, nwin, b0, lpre, L);
    else
        walk_windows<int32_t, TTFT>(g, rec, nwin, 0, lpre, reinterpret_cast<int32_t*>(L));
}

__global__ void sel_out_kernel(SelArgs g, const longlong2* __restrict__ lpre,
                               const uint32_t* __restrict__ slot_of, uint64_t nslots,
                               const int64_t* __restrict__ base,
                               const uint32_t* __restrict__ plan)
{
    if (!plan[0])
        return;
    const bool wide = plan[1] != 0;
    const int64_t b0 = wide ? base[0] : 0;
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < g.n;
         r += (uint64_t)gridDim.x * blockDim.x) {
        const SelRec s = load_rec(g, r, true);
        const uint32_t q = slot_of[r];
        if (q >= nslots)  // only when the packing failed, which the status reports
            continue;
        int64_t La, Lo;
        if (wide) {
            const longlong2 lp = lpre[q];
            La = lp.x;
            Lo = lp.y;
        } else {
            const int2 lp = reinterpret_cast<const int2*>(lpre)[q];
            La = lp.x;
            Lo = lp.y;
        }
        // the walk records (L_a, L_o); a is c2 when c2 has the longer match
        // (never under the least-load and minimum-TTFT rules)
        store_out(g, s, r, b0 + (s.a2 ? Lo : La), b0 + (s.a2 ? La : Lo));
    }
}

}  // namespace

// Work arrays of one batch in flight: packing records, the level kernel's
// outputs, walk records (room for every block's window capacity, then
// 2 * kPrefetch inert padding windows), pre-update loads (kPrefetch padding
// windows), each request's slot, base/plan words and growth bounds.  Two
// such sets live in the selection slot, one per batch parity.
struct SelBuf {
    SelPack* prep;
    WalkRec* rec;
    longlong2* lpre;
    uint32_t* info;
    uint32_t* slot_of;
    uint16_t* slotmap;
    uint8_t* wdepth;
    uint8_t* wcount;
    uint32_t* woff;
    uint32_t* total;
    int64_t* base;
    uint32_t* plan;
    unsigned long long* grow;
    BlockShape shape;  // requests per block, windows per block
    uint64_t nblk;   // request blocks
    uint64_t nslots; // walk slots that can hold a request
};

static size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

// Sizes of the arrays of m requests in blocks of bs, in layout order.
static void sel_sizes(uint64_t m, BlockShape bs, size_t* sizes)
{
    const uint64_t nblk = (m + bs.block - 1) / bs.block;
    const uint64_t wcap = nblk * bs.wincap;
    const size_t z[] = {
        up256(m * sizeof(SelPack)),                                  // prep
        up256((wcap + 2 * kPrefetch) * kSets * kWave * sizeof(WalkRec)),  // rec
        up256((wcap + kPrefetch) * kSets * kWave * sizeof(longlong2)),    // lpre
        up256(m * sizeof(uint32_t)),                                 // info
        up256(m * sizeof(uint32_t)),                                 // slot_of
        up256(wcap * kSets * kWave * sizeof(uint16_t)),              // slotmap
        up256(wcap),                                                 // wdepth
        up256(nblk),                                                 // wcount
        nblk > kScanFrom ? up256(nblk * sizeof(uint32_t)) : 0,       // woff
        256 + 256 + (kMaxSlots + 1) * sizeof(unsigned long long),   // total, base/plan, grow
    };
    for (int i = 0; i < 10; i++)
        sizes[i] = z[i];
}

// The last array's size is no multiple of 256: sets and parts start aligned.
static uint64_t sel_bytes(uint64_t m, BlockShape bs)
{
    size_t sizes[10], one = 0;
    sel_sizes(m, bs, sizes);
    for (size_t z : sizes)
        one += z;
    return one;
}

uint64_t select_scratch_bytes(uint64_t n) { return sel_bytes(n, block_shape(n, false)); }

// What one set of work arrays is given: the most that any batch of at most n
// requests takes, in one part or in two, pipelined or not.  A form changes with
// the size, the tokens and the streams, and smaller blocks need more room per
// request (4,096 requests take 3.6 MB, 4,097 take 1.9): sized by the form of the
// call, a context warmed by one batch would wait, free and allocate again for a
// smaller one, which a graph under capture cannot do and a captured one does
// not survive.
static uint64_t sel_reserve(uint64_t n)
{
    const BlockShape tiny{LevelShape<64>::block, LevelShape<64>::wincap},
        small{LevelShape<256>::block, LevelShape<256>::wincap},
        mid{LevelShape<1024>::block, LevelShape<1024>::wincap},
        large{LevelShape<2048>::block, LevelShape<2048>::wincap};
    auto early = [&](uint64_t m) -> uint64_t {  // parts whose walk waits for their blocks
        return std::max(sel_bytes(std::min(m, kTinyTo), tiny),
                        sel_bytes(std::min(m, kSmallTo), small));
    };
    const uint64_t below = std::min(n, kLargeFrom - 1);  // the most before the large blocks
    uint64_t one = std::max(early(n), sel_bytes(below, mid));
    if (n >= kLargeFrom)
        one = std::max(one, sel_bytes(n, large));
    if (n < kSplitFrom)
        return up256(one);
    const uint64_t first = n / 4, rest = n - first + kSelBlock;
    uint64_t second = sel_bytes(std::min(rest, below), mid);
    if (n >= kLargeFrom)
        second = std::max(second, sel_bytes(rest, large));
    const uint64_t two = up256(std::max(early(first), sel_bytes(first, mid))) + up256(second);
    return std::max(up256(one), two);
}

// Parts of a batch: the level blocks of a first part of two are those of an
// unpipelined batch (its walk waits for them), but for the shortest; the
// second part's level kernel runs beside the first one's walk.
void select_parts(uint64_t n, bool pipelined, int parts, SelParts* out)
{
    out->count = parts;
    out->bytes = 0;
    out->reserve = sel_reserve(n);
    uint64_t r0 = 0;
    for (int k = 0; k < parts; k++) {
        const uint64_t end = k + 1 == parts ? n : n / 4 & ~(kSelBlock - 1);
        SelPart& q = out->part[k];
        q.r0 = r0;
        q.m = end - r0;
        r0 = end;
        const BlockShape bs = parts == 1 ? block_shape(n, pipelined)
                              : k == 0   ? block_shape(std::min(q.m, kLargeFrom - 1), false)
                                         : block_shape(n, true);
        q.block = bs.block;
        q.wincap = bs.wincap;
        q.at = out->bytes;
        out->bytes += up256(sel_bytes(q.m, bs));
    }
}

static hipError_t sel_buffers(dm_ctx* c, const SelParts& ps, const SelPart& q, int par, SelBuf* b)
{
    hipError_t e = hipSuccess;
    b->shape = BlockShape{q.block, q.wincap};
    b->nblk = (q.m + q.block - 1) / q.block;
    b->nslots = b->nblk * q.wincap * kSets * kWave;
    size_t sizes[10];
    sel_sizes(q.m, b->shape, sizes);
    uint8_t* sw = nullptr;
    if (c->arena.on) {
        // allocation-free call: unpipelined, one set, one part
        sw = static_cast<uint8_t*>(scratch_get(c, kSelSlot, sel_bytes(q.m, b->shape), &e));
    } else {
        // The two sets sit sel_stride apart whatever this batch's size: a
        // smaller batch must not move its set into the other parity's, which
        // the batch before it may still be walking.  A larger batch widens
        // the stride only once every stream is idle.
        if (ps.reserve > c->sel_stride) {
            if ((e = sync_streams(c)) != hipSuccess)
                return e;
            c->sel_stride = ps.reserve;
        }
        sw = static_cast<uint8_t*>(scratch_get(c, kSelSlot, 2 * c->sel_stride, &e));
        if (sw)
            sw += par * c->sel_stride + q.at;
    }
    if (!sw)
        return e;
    uint8_t* at[10];
    for (int i = 0; i < 10; i++) {
        at[i] = sw;
        sw += sizes[i];
    }
    b->prep = reinterpret_cast<SelPack*>(at[0]);
    b->rec = reinterpret_cast<WalkRec*>(at[1]);
    b->lpre = reinterpret_cast<longlong2*>(at[2]);
    b->info = reinterpret_cast<uint32_t*>(at[3]);
    b->slot_of = reinterpret_cast<uint32_t*>(at[4]);
    b->slotmap = reinterpret_cast<uint16_t*>(at[5]);
    b->wdepth = at[6];
    b->wcount = at[7];
    b->woff = reinterpret_cast<uint32_t*>(at[8]);
    uint8_t* tail = at[9];
    b->total = reinterpret_cast<uint32_t*>(tail);
    b->base = reinterpret_cast<int64_t*>(tail + 256);
    b->plan = reinterpret_cast<uint32_t*>(tail + 256 + 128);
    b->grow = reinterpret_cast<unsigned long long*>(tail + 512);
    return hipSuccess;
}

static uint32_t block_shift(const dm_ctx* c)
{
    uint32_t bshift = 0;
    while ((1u << bshift) < c->cfg.block_size)
        bshift++;
    return bshift;
}

hipError_t select_growth(dm_ctx* c, const SelParts& ps, int k, int par, unsigned long long** grow)
{
    SelBuf b;
    const hipError_t e = sel_buffers(c, ps, ps.part[k], par, &b);
    *grow = b.grow;
    return e;
}

// The part's requests as the kernels read them.
static SelArgs part_args(const dm_ctx* c, const int64_t* offsets, uint64_t n, const SelPart& q,
                         const dm_route_out* out, int64_t* loads)
{
    const dm_config& k = c->cfg;
    return SelArgs{offsets + q.r0,     q.m,
                   n,                  block_shift(c),
                   out->cand + q.r0,   out->match + q.r0,
                   out->flags + q.r0,  out->chosen + q.r0,
                   out->ttft_us + q.r0, loads,
                   c->d_live_ids,      c->n_live,
                   k.max_slots,        k.ttft_base_us,
                   k.ttft_per_token_us, c->shift_div,
                   k.slo_us,           c->policy};
}

hipError_t select_prepare(dm_ctx* c, hipStream_t st, const int64_t* offsets, uint64_t n,
                          const dm_route_out* out, const SelParts& ps, int part, int par)
{
    SelBuf b;
    const SelPart& q = ps.part[part];
    hipError_t e = sel_buffers(c, ps, q, par, &b);
    if (e != hipSuccess)
        return e;
    const uint64_t fill_waves = (b.nblk * b.shape.wincap + 2 * kPrefetch) * kSets;
    if (b.nblk > 0x7FFFFFFFull || fill_waves > 0x7FFFFFFFull)
        return hipErrorInvalidValue;
    const uint32_t NL = c->n_live;
    const SelArgs g = part_args(c, offsets, n, q, out, nullptr);
    // few workgroups: each adds its per-instance growth sums to the global
    // ones with one atomic per instance, and those atomics meet on a few lines
    sel_prep_kernel<<<grid_for(q.m, 256, 512), 256, NL * sizeof(unsigned long long), st>>>(
        g.offsets, g.n, g.second, g.bshift, g.cand, g.match, c->d_dense, NL, g.tbase, g.per,
        g.qshift, g.slo, g.policy, b.prep, b.grow);
    if (b.nblk > 0) {
        auto level = [&](auto kernel) {
            kernel<<<(uint32_t)b.nblk, kWave, 0, st>>>(b.prep, q.m, b.info, b.slotmap, b.wdepth,
                                                       b.wcount, c->d_status);
        };
        auto sized = [&](auto live) {
            constexpr uint32_t LIVE = decltype(live)::value;
            if (b.shape.block == LevelShape<2048>::block)
                level(sel_level_kernel<2048, LIVE>);
            else if (b.shape.block == LevelShape<1024>::block)
                level(sel_level_kernel<1024, LIVE>);
            else if (b.shape.block == LevelShape<256>::block)
                level(sel_level_kernel<256, LIVE>);
            else
                level(sel_level_kernel<64, LIVE>);
        };
        if (NL <= kByteLive)
            sized(std::integral_constant<uint32_t, kByteLive>{});
        else
            sized(std::integral_constant<uint32_t, kMaxSlots>{});
    }
    const bool scan = b.nblk > kScanFrom;
    if (scan)
        sel_scan_kernel<<<1, 1024, 0, st>>>(b.wcount, b.nblk, b.woff, b.total);
    sel_fill_kernel<<<(uint32_t)((fill_waves + 3) / 4), 4 * kWave, 0, st>>>(
        b.prep, q.m, b.info, b.slotmap, b.wdepth, b.wcount, scan ? b.woff : nullptr, b.total,
        b.nblk, b.shape, b.rec, b.slot_of);
    return hipGetLastError();
}

hipError_t select_walk(dm_ctx* c, hipStream_t ss, const int64_t* offsets, uint64_t n,
                       const dm_route_out* out, int64_t* loads, const SelParts& ps, int part,
                       int par)
{
    SelBuf b;
    hipError_t e = sel_buffers(c, ps, ps.part[part], par, &b);
    if (e != hipSuccess)
        return e;
    const SelArgs g = part_args(c, offsets, n, ps.part[part], out, loads);
    if (c->policy == DM_POLICY_MIN_TTFT)
        select_walk_kernel<true><<<1, kWave, 0, ss>>>(g, b.rec, b.total, b.grow, b.plan, b.base,
                                                      b.lpre);
    else
        select_walk_kernel<false><<<1, kWave, 0, ss>>>(g, b.rec, b.total, b.grow, b.plan, b.base,
                                                       b.lpre);
    return hipGetLastError();
}

hipError_t select_output(dm_ctx* c, hipStream_t os, const int64_t* offsets, uint64_t n,
                         const dm_route_out* out, const SelParts& ps, int part, int par)
{
    SelBuf b;
    hipError_t e = sel_buffers(c, ps, ps.part[part], par, &b);
    if (e != hipSuccess)
        return e;
    const SelArgs g = part_args(c, offsets, n, ps.part[part], out, nullptr);
    sel_out_kernel<<<grid_for(g.n, 256, 8192), 256, 0, os>>>(g, b.lpre, b.slot_of, b.nslots, b.base,
                                                             b.plan);
    return hipGetLastError();
}

}  // namespace dm
