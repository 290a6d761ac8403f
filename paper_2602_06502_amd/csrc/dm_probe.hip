// Candidates and request groups (Sec. 3.2; Sec. A.1.1).
//
// The owners of a request's two ring keys, with the distinct-candidate
// adjustment, are its candidates (lookup_store also writes the ordering's sort
// input).  Then requests are ordered by the top 16 bits of their first ring key
// (stable radix sort) and grouped: a group is a maximal run of the order
// with equal first ring keys, so its requests have the same first
// candidate and, but for a key collision, the same second one and the same
// first blocks.  Each group's leader is its longest request among its first
// 64; dm_hash.hip probes leaders and resolves every other request against
// its leader's keys.  Grouping is only a matter of speed: any request could
// lead any group and the matches would be the same (a member whose
// candidates differ from its leader's is probed on its own).
#include <algorithm>

#include "dm_internal.h"
#include "dm_sort_tile.h"

namespace dm {
namespace {

static_assert(kOrderBits % 8 == 0, "whole digits");

// Batches on the hotness tree (whose ring keys extend_kernel may rewrite); the
// others are looked up by ring_key_kernel itself.
__global__ void lookup_kernel(uint64_t n, const uint64_t* __restrict__ key, LookupArgs a)
{
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n;
         r += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t x = key[r];
        lookup_store(a, n, r, x, ring_owner(a.r1, x), ring_owner(a.r2, key[n + r]));
    }
}

// Position i starts a group when its first ring key differs from position
// i - 1's; positions past the list act as heads.
__device__ __forceinline__ bool is_head(const uint64_t* skeys, uint64_t m, uint64_t i)
{
    return i >= m || i == 0 || skeys[i] != skeys[i - 1];
}

// Full blocks of request r, capped at 2^32 - 1 (for the leader choice).
__device__ __forceinline__ uint32_t blocks_of(const uint64_t* bstart, bool bad, uint32_t r)
{
    const uint64_t l = bad ? 0 : bstart[(uint64_t)r + 1] - bstart[r];
    return l < 0xFFFFFFFFull ? (uint32_t)l : 0xFFFFFFFFu;
}

// Leader of each group (a head at i leads group gpos[i]): the longest
// request among the group's positions [i, i + 64), ties to the earliest.
// One wave holds positions [64w, 64w + 128), two per lane, as (full blocks <<
// 32 | ~position) so that the larger value is the longer and then earlier
// request.  A segmented suffix maximum by doubling over both halves (each
// lane's span doubles six times, to 64 positions, and stops at the next head)
// gives every head lane of the first half its leader.
__device__ __forceinline__ uint64_t window_leader(int lane, bool h0, bool h1, uint64_t v0,
                                                  uint64_t v1)
{
    const uint64_t H0 = ballot(h0), H1 = ballot(h1);
    // done: this lane's span already ends at a head (or the window end)
    bool done0 = lane < kWave - 1 ? (H0 >> (lane + 1)) & 1 : H1 & 1;
    bool done1 = lane < kWave - 1 ? (H1 >> (lane + 1)) & 1 : true;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int src = (lane + d) & (kWave - 1);
        const bool hi = lane + d >= kWave;  // partner in the second half
        const uint64_t a0 = shfl_u64(v0, src), a1 = shfl_u64(v1, src);
        const uint64_t D0 = ballot(done0), D1 = ballot(done1);
        const uint64_t p0 = hi ? a1 : a0;
        const bool pd0 = hi ? (D1 >> src) & 1 : (D0 >> src) & 1;
        if (!done0) {
            v0 = v0 > p0 ? v0 : p0;
            done0 = pd0;
        }
        if (!done1) {
            if (hi) {
                done1 = true;
            } else {
                v1 = v1 > a1 ? v1 : a1;
                done1 = (D1 >> src) & 1;
            }
        }
    }
    return v0;
}

__device__ __forceinline__ uint64_t lead_value(uint32_t len, uint64_t i)
{
    return ((uint64_t)len << 32) | (uint32_t)~(uint32_t)i;
}

// Groups that start in each tile of kGroupTile positions.
constexpr uint32_t kGroupTile = 1024;
constexpr uint64_t kGroupTiles = 1024;  // as many that a workgroup sums the counts itself

__global__ __launch_bounds__(256) void group_count_kernel(const uint64_t* __restrict__ skeys,
                                                          uint64_t m, uint64_t* __restrict__ cnt)
{
    __shared__ uint32_t part[4];
    uint32_t c = 0;
#pragma unroll
    for (uint32_t q = 0; q < kGroupTile / 256; q++) {
        const uint64_t i = blockIdx.x * (uint64_t)kGroupTile + q * 256 + threadIdx.x;
        c += (uint32_t)__popcll(ballot(i < m && is_head(skeys, m, i)));
    }
    if (lane_id() == 0)
        part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0)
        cnt[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// Leaders and every request's group, a workgroup per tile and a wave per 64
// positions.  The groups before the tile are given (offs) or are the sum of
// the counts before its own.  With the heads found again from the keys
// instead of stored, this and group_count_kernel replace a head kernel, a scan
// over the list and a leader kernel.
__global__ __launch_bounds__(kGroupTile) void group_leader_kernel(
    const uint64_t* __restrict__ skeys, const uint32_t* __restrict__ order, uint64_t m,
    const uint64_t* __restrict__ bstart, const uint32_t* bad_p, const uint64_t* __restrict__ cnt,
    const uint64_t* __restrict__ offs, uint32_t* __restrict__ leader,
    uint32_t* __restrict__ group_of, uint64_t* __restrict__ groups)
{
    constexpr int kWaves = kGroupTile / kWave;
    __shared__ uint32_t here[kWaves];
    __shared__ uint64_t before[kWaves];
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    const bool bad = *bad_p != 0;
    const uint64_t i0 = blockIdx.x * (uint64_t)kGroupTile + threadIdx.x, i1 = i0 + kWave;
    const bool h0 = is_head(skeys, m, i0), h1 = is_head(skeys, m, i1);
    const uint32_t r0 = i0 < m ? order[i0] : 0, r1 = i1 < m ? order[i1] : 0;
    const uint64_t v0 = i0 < m ? lead_value(blocks_of(bstart, bad, r0), i0) : 0;
    const uint64_t v1 = i1 < m ? lead_value(blocks_of(bstart, bad, r1), i1) : 0;
    const uint64_t H = ballot(h0 && i0 < m);
    uint64_t p = !offs && threadIdx.x < blockIdx.x ? cnt[threadIdx.x] : 0;
    for (int d = 1; d < kWave; d <<= 1)
        p += shfl_xor_u64(p, d);
    if (lane == 0) {
        here[wv] = (uint32_t)__popcll(H);
        before[wv] = p;
    }
    __syncthreads();
    uint64_t g0 = offs ? offs[blockIdx.x] : 0;
    uint32_t all = 0;
#pragma unroll
    for (int k = 0; k < kWaves; k++) {
        g0 += before[k] + (k < wv ? here[k] : 0);
        all += here[k];
    }
    if (!offs && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
        *groups = g0 + all;
    const uint64_t v = window_leader(lane, h0, h1, v0, v1);
    if (i0 < m) {
        // the group of position i0, for its request; a head names the
        // group's leader
        const uint64_t g = g0 + __popcll(H & (~0ull >> (63 - lane))) - 1;
        group_of[r0] = (uint32_t)g;
        if (h0)
            leader[g] = order[(uint32_t)~(uint32_t)v];
    }
}

// Batches of at most kOneSort requests, bound by launches: order, groups and
// leaders by one workgroup (requests 0..n-1 with their sort keys), the list in
// LDS throughout: one launch for the sort's, the head kernel's, the scan's and
// the leader kernel's.  With the candidates looked up by the prefix pass and
// the batch's words cleared by the block starts, 1,024 requests on 8 instances
// route in 115 us instead of 123, 4,096 chat requests in 240 instead of 258.
template <int ITEMS>
__global__ __launch_bounds__(kWideThreads) void order_group_kernel(
    const uint64_t* __restrict__ keys, uint32_t n, const uint64_t* __restrict__ bstart,
    const uint32_t* bad_p, uint32_t* __restrict__ leader, uint32_t* __restrict__ group_of,
    uint64_t* __restrict__ groups)
{
    constexpr uint32_t kWindows = kOneSort / kWave;
    static_assert(kWindows == kWave, "one lane per window");
    __shared__ WideTile L;
    __shared__ uint64_t heads[kWindows + 1];
    __shared__ uint32_t gbase[kWindows];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const bool bad = *bad_p != 0;
    uint64_t k[kWideItems];
    uint32_t v[kWideItems];
#pragma unroll
    for (int it = 0; it < ITEMS; it++) {
        v[it] = it * kWideThreads + t;
        k[it] = v[it] < n ? keys[v[it]] : 0;
    }
    for (int shift = 0; shift < kOrderBits; shift += 8) {
        if (shift) {
#pragma unroll
            for (int it = 0; it < ITEMS; it++) {
                const uint32_t i = it * kWideThreads + t;
                if (i < n) {
                    k[it] = L.sk[i];
                    v[it] = L.sv[i];
                }
            }
            __syncthreads();
        }
        order_tile<ITEMS>(L, k, v, n, shift, true);
    }
    // the list is in L.sk / L.sv; the digit counts' room takes the lengths
    uint32_t* len = &L.wcnt[0][0][0];
    static_assert(sizeof(L.wcnt) >= kOneSort * sizeof(uint32_t), "lengths fit");
#pragma unroll
    for (int it = 0; it < ITEMS; it++) {
        const uint32_t i = it * kWideThreads + t;
        if (i < n)
            len[i] = blocks_of(bstart, bad, L.sv[i]);
    }
    for (uint32_t w = wv; w < kWindows; w += kWideWaves) {
        const uint64_t h = ballot(is_head(L.sk, n, w * kWave + lane));
        if (lane == 0)
            heads[w] = h;
    }
    if (t == 0)
        heads[kWindows] = ~0ull;
    __syncthreads();
    if (wv == 0) {
        // heads past the list are not groups
        const uint32_t at = lane * kWave, in = n > at ? n - at : 0;
        const uint32_t c = in == 0 ? 0
                                   : (uint32_t)__popcll(heads[lane] &
                                                        (~0ull >> (in < 64 ? 64 - in : 0)));
        uint32_t x = c;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = __shfl_up(x, d);
            if (lane >= d)
                x += y;
        }
        gbase[lane] = x - c;
        if (lane == kWave - 1)
            *groups = x;
    }
    __syncthreads();
    for (uint32_t w = wv; w * kWave < n; w += kWideWaves) {
        const uint32_t i0 = w * kWave + lane, i1 = i0 + kWave;
        const uint64_t H = heads[w];
        const bool h0 = (H >> lane) & 1, h1 = (heads[w + 1] >> lane) & 1;
        const uint64_t v0 = i0 < n ? lead_value(len[i0], i0) : 0;
        const uint64_t v1 = i1 < n ? lead_value(len[i1], i1) : 0;
        const uint64_t x = window_leader(lane, h0, h1, v0, v1);
        if (i0 < n) {
            const uint32_t g = gbase[w] + (uint32_t)__popcll(H & (~0ull >> (63 - lane))) - 1;
            group_of[L.sv[i0]] = g;
            if (h0)
                leader[g] = L.sv[(uint32_t)~(uint32_t)x];
        }
    }
}

// Work arrays of grouping for m requests, in layout order: sort keys and
// request order (each twice, for the sort's passes), each tile's groups and the
// groups before it, leaders, each request's group, and the group count.
struct GroupWork {
    uint64_t *keys, *ktmp;
    uint32_t *order, *vtmp;
    uint64_t *cnt, *offs;
    uint32_t *leader, *group_of;
    uint64_t* groups;
};

size_t up256z(size_t x) { return (x + 255) & ~size_t(255); }

uint64_t group_tiles(uint64_t m) { return (m + kGroupTile - 1) / kGroupTile; }

size_t group_layout(uint64_t m, uint8_t* w, GroupWork* gw)
{
    const size_t sz[] = {up256z(8 * m), up256z(8 * m), up256z(4 * m), up256z(4 * m),
                         up256z(8 * group_tiles(m)), up256z(8 * group_tiles(m)), up256z(4 * m),
                         up256z(4 * m), 256};
    size_t at[9], off = 0;
    for (int i = 0; i < 9; i++) {
        at[i] = off;
        off += sz[i];
    }
    if (gw) {
        gw->keys = reinterpret_cast<uint64_t*>(w + at[0]);
        gw->ktmp = reinterpret_cast<uint64_t*>(w + at[1]);
        gw->order = reinterpret_cast<uint32_t*>(w + at[2]);
        gw->vtmp = reinterpret_cast<uint32_t*>(w + at[3]);
        gw->cnt = reinterpret_cast<uint64_t*>(w + at[4]);
        gw->offs = reinterpret_cast<uint64_t*>(w + at[5]);
        gw->leader = reinterpret_cast<uint32_t*>(w + at[6]);
        gw->group_of = reinterpret_cast<uint32_t*>(w + at[7]);
        gw->groups = reinterpret_cast<uint64_t*>(w + at[8]);
    }
    return off;
}

}  // namespace

uint64_t probe_scratch_bytes(uint64_t m) { return group_layout(m, nullptr, nullptr); }

hipError_t lookup_args(dm_ctx* c, uint64_t n, uint32_t* cand, uint8_t* flags, LookupArgs* a)
{
    hipError_t e = hipSuccess;
    uint8_t* w = static_cast<uint8_t*>(scratch_get(c, kSlotProbe, probe_scratch_bytes(n), &e));
    if (!w)
        return e;
    GroupWork g;
    group_layout(n, w, &g);
    *a = LookupArgs{view(c->ring[c->cur][0]), view(c->ring[c->cur][1]), c->d_next_live, c->n_live,
                    cand, flags, g.keys, n > kOneSort ? g.order : nullptr};
    return hipSuccess;
}

hipError_t lookup_candidates(dm_ctx* c, uint64_t n, const uint64_t* key, const LookupArgs& a)
{
    lookup_kernel<<<grid_for(n, 256, 8192), 256, 0, c->stream>>>(n, key, a);
    return hipGetLastError();
}

hipError_t group_requests(dm_ctx* c, uint64_t n, const uint64_t* bstart, const uint32_t* bad,
                          GroupView* gv)
{
    hipError_t e = hipSuccess;
    hipStream_t st = c->stream;
    if (n == 0)
        return hipSuccess;
    if (n > 0xFFFFFFFFull)
        return hipErrorInvalidValue;
    uint8_t* w = static_cast<uint8_t*>(scratch_get(c, kSlotProbe, probe_scratch_bytes(n), &e));
    if (!w)
        return e;
    GroupWork g;
    group_layout(n, w, &g);
    *gv = GroupView{g.group_of, g.leader, g.groups};
    if (n <= kOneSort) {
        auto one = n <= kWideThreads       ? order_group_kernel<1>
                   : n <= 2 * kWideThreads ? order_group_kernel<2>
                                           : order_group_kernel<kWideItems>;
        one<<<1, kWideThreads, 0, st>>>(g.keys, (uint32_t)n, bstart, bad, g.leader, g.group_of,
                                        g.groups);
        return hipGetLastError();
    }
    // requests ordered by the top bits of their first ring key (stable radix sort)
    if ((e = radix_sort_kv(c, g.keys, g.order, g.ktmp, g.vtmp, n, kOrderBits)) != hipSuccess)
        return e;
    const uint64_t tiles = group_tiles(n);
    group_count_kernel<<<(uint32_t)tiles, 256, 0, st>>>(g.keys, n, g.cnt);
    const bool many = tiles > kGroupTiles;
    if (many && (e = exclusive_scan_u64(c, g.cnt, tiles, g.offs, g.groups)) != hipSuccess)
        return e;
    group_leader_kernel<<<(uint32_t)tiles, kGroupTile, 0, st>>>(
        g.keys, g.order, n, bstart, bad, g.cnt, many ? g.offs : nullptr, g.leader, g.group_of,
        g.groups);
    return hipGetLastError();
}

}  // namespace dm
