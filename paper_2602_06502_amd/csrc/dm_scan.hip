// Exclusive prefix sums over u64 sequences, used for per-request block
// offsets, stream compaction and the radix sort's digit offsets.
//
// Bound by launches and memory, so the form goes by size:
//   up to kOneScan items     one workgroup;
//   up to kMidTiles tiles    a sum per tile, then each tile's workgroup adds
//                            the sums before its own (8 KB at most) and scans;
//   more                     the tiles' sums are scanned in between, level by
//                            level.
// (One workgroup of 16 items a thread takes longer over 16,384 offsets than the
// two launches: a batch of that size 381 us against 354.)
#include <vector>

#include "dm_internal.h"

namespace dm {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 4;
constexpr uint64_t kTile = kScanThreads * kScanItems;
constexpr uint64_t kOneScan = 4096;    // 4 items a thread of one workgroup
constexpr uint64_t kMidTiles = 1024;   // tile sums a workgroup reads: 4 a thread
constexpr int kScanSlot = kSlotScan;   // tile-sum levels
constexpr uint64_t kBadBit = 1ull << 63;  // of a tile sum: a broken offset in the tile

struct ArrayIn {
    static constexpr bool kChecks = false;
    const uint64_t* p;
    __device__ uint64_t operator()(uint64_t i, uint32_t&) const { return p[i]; }
    __device__ void clear() const {}
    __device__ void result(bool) const {}
};

// Full blocks of request i: floor(len / B), B = 2^shift, for a prompt
// inside [0, n_tokens); a request that breaks 0 <= off[i] <= off[i+1] <=
// n_tokens counts none, and *bad is 1 (else 0) and kErrInval joins the device
// status word.  When every request keeps the rule the offsets never decrease,
// so the prompts are disjoint ranges of the token array and their full blocks
// add up to at most n_tokens / B.
struct FullBlocksIn {
    static constexpr bool kChecks = true;
    const int64_t* off;
    uint32_t shift;
    uint64_t n_tokens;
    uint32_t* bad;
    uint32_t* status;
    BatchClear also;
    __device__ uint64_t operator()(uint64_t i, uint32_t& broken) const
    {
        const int64_t o0 = off[i], o1 = off[i + 1];
        if (o0 < 0 || o1 < o0 || (uint64_t)o1 > n_tokens) {
            broken = 1;
            return 0;
        }
        return (uint64_t)(o1 - o0) >> shift;
    }
    // by one workgroup: the batch's other words, which later kernels add to
    __device__ void clear() const
    {
        for (int p = 0; p < kMaxParts; p++) {
            if (!also.grow[p])
                break;
            for (uint32_t k = threadIdx.x; k < also.n_live; k += blockDim.x)
                also.grow[p][k] = 0;
            if (threadIdx.x == 0)
                also.grow[p][kMaxSlots] = 0;
        }
    }
    // by one thread
    __device__ void result(bool broken) const
    {
        *bad = broken ? 1u : 0u;
        if (broken)
            atomicOr(status, kErrInval);
    }
};

// Block-wide exclusive scan of one u64 per thread; also returns the total.
template <int THREADS>
__device__ uint64_t block_excl_scan(uint64_t v, uint64_t* sh, uint64_t& total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t inc = wave_incl_sum_u64(v, lane);
    if (lane == 63)
        sh[w] = inc;
    __syncthreads();
    uint64_t before = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < THREADS / kWave; k++) {
        if (k < w)
            before += sh[k];
        tot += sh[k];
    }
    __syncthreads();
    total = tot;
    return before + inc - v;
}

// A whole scan of at most THREADS * ITEMS items.
template <typename In, int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void one_scan_kernel(In in, uint64_t n, uint64_t* out,
                                                           uint64_t* total_out)
{
    __shared__ uint64_t sh[THREADS / kWave];
    const uint64_t base = (uint64_t)threadIdx.x * ITEMS;
    uint64_t v[ITEMS], s = 0, total;
    uint32_t broken = 0;
#pragma unroll
    for (int k = 0; k < ITEMS; k++) {
        v[k] = base + k < n ? in(base + k, broken) : 0;
        s += v[k];
    }
    uint64_t run = block_excl_scan<THREADS>(s, sh, total);
#pragma unroll
    for (int k = 0; k < ITEMS; k++) {
        if (base + k < n)
            out[base + k] = run;
        run += v[k];
    }
    if (total_out && threadIdx.x == 0)
        *total_out = total;
    if (In::kChecks) {
        const bool any = __syncthreads_or((int)broken);
        if (threadIdx.x == 0)
            in.result(any);
        in.clear();
    }
}

// sums[tile], for a checked input with kBadBit where the tile is broken.
template <typename In>
__global__ __launch_bounds__(kScanThreads) void tile_sum_kernel(In in, uint64_t n, uint64_t* sums)
{
    __shared__ uint64_t sh[kScanThreads / kWave];
    const uint64_t base = blockIdx.x * kTile + threadIdx.x * kScanItems;
    uint64_t s = 0;
    uint32_t broken = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++)
        if (base + k < n)
            s += in(base + k, broken);
    uint64_t total;
    block_excl_scan<kScanThreads>(s, sh, total);
    const bool any = In::kChecks && __syncthreads_or((int)broken);
    if (threadIdx.x == 0)
        sums[blockIdx.x] = total | (any ? kBadBit : 0);
    if (In::kChecks && blockIdx.x == 0)
        in.clear();
}

// Tile offsets are given scanned (tile_off), or the tiles' sums are (sums),
// at most kMidTiles of them.
template <typename In>
__global__ __launch_bounds__(kScanThreads) void tile_scan_kernel(In in, uint64_t n,
                                                                 const uint64_t* tile_off,
                                                                 const uint64_t* sums,
                                                                 uint64_t* out, uint64_t* total_out)
{
    __shared__ uint64_t sh[kScanThreads / kWave];
    const uint64_t base = blockIdx.x * kTile + threadIdx.x * kScanItems;
    uint64_t v[kScanItems];
    uint64_t s = 0, total, toff = 0;
    uint32_t broken = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        v[k] = base + k < n ? in(base + k, broken) : 0;
        s += v[k];
    }
    if (sums) {
        uint64_t p = 0, bad = broken ? kBadBit : 0;
#pragma unroll
        for (int k = 0; k < (int)(kMidTiles / kScanThreads); k++) {
            const uint32_t t = k * kScanThreads + threadIdx.x;
            const uint64_t x = t < blockIdx.x ? sums[t] : 0;
            p += In::kChecks ? x & ~kBadBit : x;
            bad |= x & kBadBit;
        }
        block_excl_scan<kScanThreads>(p, sh, toff);
        if (In::kChecks && blockIdx.x == gridDim.x - 1) {
            const bool any = __syncthreads_or(bad != 0);
            if (threadIdx.x == 0)
                in.result(any);
        }
    } else if (tile_off) {
        toff = tile_off[blockIdx.x];
    }
    uint64_t run = block_excl_scan<kScanThreads>(s, sh, total) + toff;
#pragma unroll
    for (int k = 0; k < kScanItems; k++) {
        if (base + k < n)
            out[base + k] = run;
        run += v[k];
    }
    if (total_out && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
        *total_out = toff + total;
}

// The broken tiles of a checked scan of many tiles; the sums without the bit.
__global__ __launch_bounds__(1024) void strip_bad_kernel(uint64_t* sums, uint64_t n, FullBlocksIn in)
{
    uint64_t bad = 0;
    for (uint64_t i = threadIdx.x; i < n; i += 1024) {
        const uint64_t x = sums[i];
        bad |= x & kBadBit;
        if (x & kBadBit)
            sums[i] = x & ~kBadBit;
    }
    const bool any = __syncthreads_or(bad != 0);
    if (threadIdx.x == 0)
        in.result(any);
}
inline void strip_bad(dm_ctx*, uint64_t*, uint64_t, const ArrayIn&) {}
inline void strip_bad(dm_ctx* c, uint64_t* sums, uint64_t n, const FullBlocksIn& in)
{
    strip_bad_kernel<<<1, 1024, 0, c->stream>>>(sums, n, in);
}

uint64_t ntiles(uint64_t n) { return (n + kTile - 1) / kTile; }

template <typename In>
hipError_t scan_impl(dm_ctx* c, In in, uint64_t n, uint64_t* out, uint64_t* total_out)
{
    if (n == 0)
        return hipSuccess;
    if (n <= kOneScan) {
        if (n <= kTile)
            one_scan_kernel<In, kScanThreads, kScanItems>
                <<<1, kScanThreads, 0, c->stream>>>(in, n, out, total_out);
        else
            one_scan_kernel<In, 1024, 4><<<1, 1024, 0, c->stream>>>(in, n, out, total_out);
        return hipGetLastError();
    }
    // level d has n_d inputs and tiles_d tiles; n_{d+1} = tiles_d; stop at one tile
    std::vector<uint64_t> nd{n};
    while (ntiles(nd.back()) > 1)
        nd.push_back(ntiles(nd.back()));
    const size_t K = nd.size() - 1;  // levels with more than one tile: 0..K-1
    // scratch: sums_d and scanned_d (tiles_d entries each) for d < K
    std::vector<uint64_t> at(K);
    uint64_t need = 0;
    for (size_t d = 0; d < K; d++) {
        at[d] = need;
        need += 2 * ntiles(nd[d]);
    }
    hipError_t e;
    uint64_t* buf = static_cast<uint64_t*>(scratch_get(c, kScanSlot, scan_scratch_bytes(n), &e));
    if (!buf)
        return e;
    auto sums = [&](size_t d) { return buf + at[d]; };
    auto scanned = [&](size_t d) { return buf + at[d] + ntiles(nd[d]); };
    tile_sum_kernel<In><<<ntiles(nd[0]), kScanThreads, 0, c->stream>>>(in, nd[0], sums(0));
    if (ntiles(n) <= kMidTiles) {
        tile_scan_kernel<In><<<ntiles(n), kScanThreads, 0, c->stream>>>(in, n, nullptr, sums(0), out,
                                                                        total_out);
        return hipGetLastError();
    }
    strip_bad(c, sums(0), ntiles(n), in);
    for (size_t d = 1; d < K; d++)
        tile_sum_kernel<ArrayIn><<<ntiles(nd[d]), kScanThreads, 0, c->stream>>>(
            ArrayIn{sums(d - 1)}, nd[d], sums(d));
    // top level: one tile scans sums_{K-1}
    tile_scan_kernel<ArrayIn><<<1, kScanThreads, 0, c->stream>>>(
        ArrayIn{sums(K - 1)}, nd[K], nullptr, nullptr, scanned(K - 1), nullptr);
    for (size_t d = K - 1; d >= 1; d--)
        tile_scan_kernel<ArrayIn><<<ntiles(nd[d]), kScanThreads, 0, c->stream>>>(
            ArrayIn{sums(d - 1)}, nd[d], scanned(d), nullptr, scanned(d - 1), nullptr);
    tile_scan_kernel<In><<<ntiles(nd[0]), kScanThreads, 0, c->stream>>>(in, nd[0], scanned(0),
                                                                         nullptr, out, total_out);
    return hipGetLastError();
}

}  // namespace

// Words of tile sums a scan of n items keeps: sums and scanned sums of every
// level with more than one tile.
uint64_t scan_scratch_bytes(uint64_t n)
{
    uint64_t need = 0;
    for (uint64_t m = n; ntiles(m) > 1; m = ntiles(m))
        need += 2 * ntiles(m);
    return need * sizeof(uint64_t);
}

hipError_t exclusive_scan_u64(dm_ctx* c, const uint64_t* in, uint64_t n, uint64_t* out,
                              uint64_t* total_out)
{
    return scan_impl(c, ArrayIn{in}, n, out, total_out);
}

// starts[r] = full blocks of requests 0..r-1, for r = 0..n (starts[n] = total).
hipError_t block_starts(dm_ctx* c, const int64_t* offsets, uint64_t n, uint64_t n_tokens,
                        uint64_t* starts, uint32_t* bad, const BatchClear& also)
{
    uint32_t shift = 0;
    while ((1u << shift) < c->cfg.block_size)
        shift++;
    return scan_impl(c, FullBlocksIn{offsets, shift, n_tokens, bad, c->d_status, also}, n,
                     starts, starts + n);
}

}  // namespace dm
