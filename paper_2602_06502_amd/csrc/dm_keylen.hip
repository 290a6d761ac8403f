// Adaptive hash-key length (Sec. 3.2, "How long prefix is appropriate for
// the hash key?"; Sec. A.1.1): the prefix hotness tree's set-up, window
// close and export, and the window's record of each routed batch.  Routing
// reads the tree in ring_key_kernel and extend_kernel (dm_hash.hip).
//
// The tree is the set of its extended prefixes (canonical f1 key of each
// prefix's last block) in an open-addressing table of 8-slot buckets, probed
// like the instance indexes.  The window's record holds every prefix of
// depth >= K of every routed request (its f1 block keys from block K - 1
// on, appended after the batch's members pass).
//
// Closing a window applies the hot and cold rules until nothing changes.
// A prefix's count never exceeds its parent's, so with W routed requests
// and n live instances the result is the set of prefixes with count c
//   extended now:  c * n >= W      (not cold: rho >= 1/n)
//   a leaf now:    c * n >  2 W    (hot: rho > 2/n)
// (extended prefixes the window never saw, c = 0, are dropped).
//
// Counts come from the record's runs (a run is one request's entries, its
// prefixes of growing depth), not from sorting its entries.  A node is a prefix
// with c n >= W, and the runs that carry it:
//   1. the runs meet by their next key (first the depth-K prefix) in a hash
//      table that counts them; the keys with c n >= W are the nodes, at most n,
//      and the other runs are done with;
//   2. one run of each node represents it: every run of the node is compared
//      with it (a wave per run, 64 prefixes a step) and its common length counted;
//   3. suffix sums of the lengths are the counts of every prefix along the
//      representative, which are decided;
//   4. runs that go on past their common length meet again by their next key
//      there, until no node is left (a second node below a first one takes a
//      branch that W / n requests share).
// In the first turns a node's longest run represents it, which settles all runs
// that are cut from one prompt at once (drawn from the second turn on, a window of
// 1,024 chat requests took four turns instead of two).  Past kLongestTurns it is
// drawn: the runs that go on together with a given run are those that share more
// with it than the drawn one does, on average half, so however the branches nest
// the turns are about the logarithm of n.  (Longest every time, a spine whose
// longest runs part first takes a turn a run: 512 requests of 512 to 1,024 blocks
// on 256 instances 22.5 ms instead of 0.6.)
// What bounds it: one read of the hot runs' entries, and launches.  It replaces
// two radix sorts (of the depth-K prefixes and of all entries under hot ones, 64
// bits each): 131,072 requests routed and the window closed, 2.40 to 1.31 ms.
#include <algorithm>

#include "dm_internal.h"

namespace dm {
namespace {

__global__ void kl_fill_kernel(uint64_t* __restrict__ p, uint64_t n, uint64_t v)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Distinct canonical keys into an empty table with room to spare (at most
// half full): the first empty slot along the key's bucket sequence.
__global__ void kl_insert_kernel(uint64_t* __restrict__ tab, uint32_t ls,
                                 const uint64_t* __restrict__ keys, uint64_t n)
{
    const uint32_t nbk = 1u << (ls - 3);
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t k = keys[i];
        uint32_t b = home32(k, ls);
        bool done = false;
        for (uint32_t step = 0; step < nbk && !done; step++, b = (b + 1) & (nbk - 1))
            for (uint32_t s = 0; s < kBucket && !done; s++) {
                const unsigned long long prev =
                    atomicCAS((unsigned long long*)(tab + (uint64_t)b * kBucket + s),
                              (unsigned long long)kEmpty, (unsigned long long)k);
                done = prev == kEmpty || prev == k;
            }
    }
}

// Window record of one batch: request r contributes its block keys from
// block K - 1 on (its prefixes of depth >= K), canonical, at the record's
// current end plus its offset among the batch's entries; *runs += the requests
// that contribute.
__global__ void kl_entries_kernel(const uint64_t* __restrict__ bstart, uint64_t n, uint64_t K,
                                  uint64_t* __restrict__ ent, unsigned long long* __restrict__ runs)
{
    uint32_t mine = 0;
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n;
         r += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t nfull = bstart[r + 1] - bstart[r];
        ent[r] = nfull >= K ? nfull - K + 1 : 0;
        mine += nfull >= K;
    }
    // one add per workgroup, of which there are few: they meet on one word
    __shared__ uint32_t total;
    if (threadIdx.x == 0)
        total = 0;
    __syncthreads();
    for (int d = 1; d < kWave; d <<= 1)
        mine += (uint32_t)__shfl_xor((int)mine, d);
    if (lane_id() == 0)
        atomicAdd(&total, mine);
    __syncthreads();
    if (threadIdx.x == 0 && total)
        atomicAdd(runs, (unsigned long long)total);
}

__global__ void kl_append_kernel(uint64_t n, const uint64_t* __restrict__ bstart,
                                 const uint64_t* __restrict__ epos,
                                 const uint64_t* __restrict__ ent, uint64_t K,
                                 const uint64_t* __restrict__ hkeys, uint64_t* __restrict__ log,
                                 uint32_t* __restrict__ roots, uint64_t cap,
                                 const unsigned long long* __restrict__ log_n)
{
    const uint64_t base = *log_n;
    const uint64_t w = blockIdx.x * (uint64_t)(blockDim.x >> 6) +
                       __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t nw = (uint64_t)gridDim.x * (blockDim.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    for (uint64_t r = w; r < n; r += nw) {
        const uint64_t e = ent[r], at = base + epos[r];
        const uint64_t* src = hkeys + bstart[r] + (K - 1);
        for (uint64_t j = lane; j < e; j += kWave)
            if (at + j < cap)
                log[at + j] = canon_key(src[j]);
        // the request's first entry (its depth-K prefix) starts its run
        if (lane == 0 && e && at < cap)
            atomicOr(&roots[at >> 5], 1u << (at & 31));
    }
}

// Roots of the record: per 32-entry word its root count (for a scan).
__global__ void kl_root_count_kernel(const uint32_t* __restrict__ roots, uint64_t nw,
                                     uint64_t* __restrict__ cnt)
{
    for (uint64_t w = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; w < nw;
         w += (uint64_t)gridDim.x * blockDim.x)
        cnt[w] = __popc(roots[w]);
}

// Start of each run, in record order.
__global__ void kl_runs_kernel(const uint32_t* __restrict__ roots, uint64_t nw,
                               const uint64_t* __restrict__ wpre, uint64_t runs,
                               uint64_t* __restrict__ start)
{
    for (uint64_t w = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; w < nw;
         w += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t at = wpre[w];
        for (uint32_t m = roots[w]; m && at < runs; m &= m - 1)
            start[at++] = w * 32 + (uint32_t)__builtin_ctz(m);
    }
}

// The runs of a window while it is closed, the table that they meet in and
// the nodes found there.
struct KlNode {
    uint64_t rep;    // record position of the node's prefix in its representative
    uint64_t len;    // the representative's entries from there on
    uint64_t base;   // its counts in hist
};
constexpr uint64_t kDone = UINT64_MAX;
constexpr uint32_t kNoNode = UINT32_MAX;  // too few runs share the key
constexpr uint64_t kLongestTurns = 4;
struct KlRuns {
    const uint64_t* log;
    uint64_t m;               // record entries
    const uint64_t* start;    // [runs]
    uint64_t runs;            // how many
    uint32_t* depth;          // [runs] entries of the run that are settled
    uint64_t* slot;           // [runs] where its next key is; kDone
    uint64_t* key;            // [slots] 0: none
    uint64_t* rep;            // [slots] rank among the runs (24 bits, from 1) | ~run (40 bits)
    uint64_t* count;          // [slots]
    uint32_t* node;           // [slots]
    uint64_t mask;            // slots - 1
    KlNode* nodes;            // [n_live]
    uint64_t* hist;           // [m]
    unsigned long long* words;  // nodes, counts used, prefixes kept
    uint64_t W, n_live;
    uint64_t turn;            // from kLongestTurns on a drawn run represents a node
};

__device__ __forceinline__ uint64_t kl_len(const KlRuns& a, uint64_t k)
{
    return (k + 1 < a.runs ? a.start[k + 1] : a.m) - a.start[k];
}

// An empty table and no nodes; FIRST: every run at its first entry.
template <bool FIRST>
__global__ void kl_clear_kernel(KlRuns a)
{
    const uint64_t t0 = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x,
                   nt = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = t0; i <= a.mask; i += nt) {
        a.key[i] = 0;
        a.rep[i] = 0;
        a.count[i] = 0;
    }
    if (FIRST)
        for (uint64_t k = t0; k < a.runs; k += nt) {
            a.depth[k] = 0;
            a.slot[k] = 0;
        }
    if (t0 == 0)
        a.words[0] = a.words[1] = 0;
}

// Slot of a key in the open-addressing table of mask + 1 slots (claimed if
// new); it has at least twice as many slots as there are keys, so this ends.
__device__ __forceinline__ uint64_t kl_claim(uint64_t* tab, uint64_t mask, uint64_t key)
{
    for (uint64_t i = mix64(key) & mask;; i = (i + 1) & mask) {
        uint64_t v = tab[i];
        if (v == 0)
            v = atomicCAS((unsigned long long*)&tab[i], 0ull, (unsigned long long)key);
        if (v == 0 || v == key)
            return i;
    }
}

// Runs meet by their next key, and the run that represents each key is found.  A
// workgroup's runs meet in LDS first: thousands of runs share a popular key, and
// atomics from all over the chip on one address take some 11 ns each
// (131,072 runs: 421 us without this, 18 with it).
constexpr uint32_t kMeet = 1024;

__global__ __launch_bounds__(kMeet) void kl_meet_kernel(KlRuns a)
{
    constexpr uint32_t kSlots = 2 * kMeet;
    __shared__ uint64_t key[kSlots];    // then the key's slot in the table
    __shared__ unsigned long long top[kSlots];
    __shared__ uint32_t count[kSlots];
    for (uint64_t k0 = blockIdx.x * (uint64_t)kMeet; k0 < a.runs; k0 += (uint64_t)gridDim.x * kMeet) {
        const uint64_t k = k0 + threadIdx.x;
        const bool in = k < a.runs && a.slot[k] != kDone;
        if (!__syncthreads_or(in))
            continue;
        for (uint32_t j = threadIdx.x; j < kSlots; j += kMeet) {
            key[j] = 0;
            top[j] = 0;
            count[j] = 0;
        }
        __syncthreads();
        uint32_t j = 0;
        if (in) {
            const uint64_t d = a.depth[k], left = kl_len(a, k) - d;
            j = (uint32_t)kl_claim(key, kSlots - 1, a.log[a.start[k] + d]);
            atomicAdd(&count[j], 1u);
            const uint64_t rank = a.turn >= kLongestTurns ? mix64(k | a.turn << 40) >> 40 | 1
                                  : left < 0xFFFFFFull    ? left
                                                          : 0xFFFFFFull;
            atomicMax(&top[j], (unsigned long long)(rank << 40 | (0xFFFFFFFFFFull - k)));
        }
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < kSlots; q += kMeet)
            if (count[q]) {
                const uint64_t i = kl_claim(a.key, a.mask, key[q]);
                atomicAdd((unsigned long long*)&a.count[i], (unsigned long long)count[q]);
                atomicMax((unsigned long long*)&a.rep[i], top[q]);
                key[q] = i;
            }
        __syncthreads();
        if (in)
            a.slot[k] = key[j];
        __syncthreads();
    }
}

__global__ void kl_node_kernel(KlRuns a)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i <= a.mask;
         i += (uint64_t)gridDim.x * blockDim.x) {
        if (!a.rep[i] || a.count[i] * a.n_live < a.W) {
            a.node[i] = kNoNode;
            continue;
        }
        const uint64_t k = 0xFFFFFFFFFFull - (a.rep[i] & 0xFFFFFFFFFFull);
        const uint64_t d = a.depth[k], len = kl_len(a, k) - d;
        // disjoint sets of at least W / n of at most W runs: at most n nodes,
        // whose representatives are distinct runs: at most m counts
        const uint64_t at = atomicAdd(&a.words[0], 1ull);
        a.nodes[at] = KlNode{a.start[k] + d, len, atomicAdd(&a.words[1], (unsigned long long)len)};
        a.node[i] = (uint32_t)at;
    }
}

__global__ __launch_bounds__(256) void kl_hist_zero_kernel(KlRuns a)
{
    for (uint64_t b = blockIdx.x; b < a.words[0]; b += gridDim.x)
        for (uint64_t j = threadIdx.x; j < a.nodes[b].len; j += blockDim.x)
            a.hist[a.nodes[b].base + j] = 0;
}

// Every run's entries in common with its node's representative: a wave takes
// kAlike runs, whose first 64 entries are loaded together.  The counts meet in
// LDS first, as above (many runs part from their representative where a shared
// prompt ends; 131,072 runs 161 us without this, 36 with it).  A run goes on
// alone, 64 entries a step and after kStep1 of them kAhead steps at once, and few
// runs (kAloneTo) take a wave each, for they may be long: 64 prompts of 7,000
// blocks 195 us with neither, 44 with both.
constexpr uint32_t kCommonWaves = 16, kManyAlike = 8, kAhead = 8;
constexpr uint64_t kAloneTo = 2048, kStep1 = 512;

template <uint32_t kAlike>
__global__ __launch_bounds__(kCommonWaves * kWave) void kl_common_kernel(KlRuns a)
{
    constexpr uint32_t kCommonRuns = kAlike * kCommonWaves;
    constexpr uint32_t kSlots = 2 * kCommonRuns;
    __shared__ uint64_t at[kSlots];  // place in hist + 1
    __shared__ uint32_t count[kSlots];
    if (a.words[0] == 0)
        return;
    const int lane = lane_id();
    const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (uint64_t k0 = blockIdx.x * (uint64_t)kCommonRuns; k0 < a.runs;
         k0 += (uint64_t)gridDim.x * kCommonRuns) {
        for (uint32_t j = threadIdx.x; j < kSlots; j += kCommonWaves * kWave) {
            at[j] = 0;
            count[j] = 0;
        }
        __syncthreads();
        // lane l < kAlike: the wave's l-th run
        const uint64_t k = k0 + wv * kAlike + lane;
        bool in = lane < (int)kAlike && k < a.runs;
        uint64_t mine = 0, rep = 0, lim = 0, left = 0, base = 0, d = 0;
        if (in) {
            const uint64_t i = a.slot[k];
            const uint32_t b = i == kDone ? kNoNode : a.node[i];
            if (i != kDone && b == kNoNode)
                a.slot[k] = kDone;
            in = b != kNoNode;
            if (in) {
                const KlNode nd = a.nodes[b];
                d = a.depth[k];
                left = kl_len(a, k) - d;
                lim = left < nd.len ? left : nd.len;
                mine = a.start[k] + d;
                rep = nd.rep;
                base = nd.base;
            }
        }
        // (lim = 0 for a run that is done with)
        uint64_t x[kAlike], y[kAlike];
#pragma unroll
        for (uint32_t q = 0; q < kAlike; q++) {
            const bool ok = (uint64_t)lane < readlane_u64(lim, q);
            x[q] = ok ? a.log[readlane_u64(mine, q) + lane] : 0;
            y[q] = ok ? a.log[readlane_u64(rep, q) + lane] : 0;
        }
        uint64_t l = lim;
#pragma unroll
        for (uint32_t q = 0; q < kAlike; q++) {
            const uint64_t n = readlane_u64(lim, q);
            uint64_t diff = ballot(x[q] != y[q]), j = 0;
            if (!diff && n > kWave) {
                const uint64_t *m = a.log + readlane_u64(mine, q), *r = a.log + readlane_u64(rep, q);
                for (j = kWave; j < n && j < kStep1; j += kWave) {
                    diff = ballot(j + lane < n && m[j + lane] != r[j + lane]);
                    if (diff)
                        break;
                }
                while (!diff && j < n) {
                    uint64_t u[kAhead], v[kAhead];
#pragma unroll
                    for (uint32_t h = 0; h < kAhead; h++) {
                        const uint64_t p = j + h * kWave + lane;
                        u[h] = p < n ? m[p] : 0;
                        v[h] = p < n ? r[p] : 0;
                    }
#pragma unroll
                    for (uint32_t h = 0; h < kAhead; h++)
                        if (!diff) {
                            diff = ballot(u[h] != v[h]);
                            j += diff ? 0 : kWave;
                        }
                }
            }
            if (diff && lane == (int)q)
                l = j + (uint64_t)__builtin_ctzll(diff);
        }
        if (in) {
            // l > 0: the node's prefix itself is in common
            atomicAdd(&count[kl_claim(at, kSlots - 1, base + l)], 1u);
            a.depth[k] = (uint32_t)(d + l);
            if (l == left)
                a.slot[k] = kDone;
        }
        __syncthreads();
        for (uint32_t j = threadIdx.x; j < kSlots; j += kCommonWaves * kWave)
            if (count[j])
                atomicAdd((unsigned long long*)&a.hist[at[j] - 1], (unsigned long long)count[j]);
        __syncthreads();
    }
}

// A workgroup per node: how many of its runs carry each prefix along its
// representative (suffix sums, from its end up to 2,048 prefixes at a time), and
// the prefixes that the next tree holds: extended now and c n >= W, or a leaf now
// and c n > 2 W.
__global__ __launch_bounds__(256) void kl_decide_kernel(KlRuns a, const uint64_t* __restrict__ tab,
                                                        uint32_t ls, uint64_t* __restrict__ out,
                                                        uint64_t cap)
{
    constexpr uint32_t kMost = 8;  // prefixes of a thread at a time
    __shared__ uint64_t part[256 / kWave];
    const uint32_t wv = threadIdx.x >> 6;
    for (uint64_t b = blockIdx.x; b < a.words[0]; b += gridDim.x) {
        const KlNode nd = a.nodes[b];
        const uint32_t per = nd.len < 256 * kMost ? (uint32_t)((nd.len + 255) / 256) : kMost;
        const uint64_t tile = 256 * per;
        uint64_t after = 0;  // runs that go past the tile
        for (uint64_t t = (nd.len + tile - 1) / tile; t-- > 0;) {
            const uint64_t j0 = t * tile + threadIdx.x * per;
            uint64_t h[kMost], sum = 0;
#pragma unroll
            for (uint32_t q = 0; q < kMost; q++) {
                h[q] = q < per && j0 + q < nd.len ? a.hist[nd.base + j0 + q] : 0;
                sum += h[q];
            }
            const uint64_t upto = wave_incl_sum_u64(sum, lane_id());
            if (lane_id() == kWave - 1)
                part[wv] = upto;
            __syncthreads();
            uint64_t all = 0, before = upto;
#pragma unroll
            for (uint32_t k = 0; k < 256 / kWave; k++) {
                all += part[k];
                before += k < wv ? part[k] : 0;
            }
            __syncthreads();
            uint64_t c = after + all - before;
            after += all;
#pragma unroll
            for (uint32_t q = kMost; q-- > 0;) {
                c += h[q];
                if (q >= per || j0 + q >= nd.len || c * a.n_live < a.W)
                    continue;
                const uint64_t key = a.log[nd.rep + j0 + q];
                if (c * a.n_live > 2 * a.W || table_has(tab, ls, key)) {
                    const uint64_t at = atomicAdd(&a.words[2], 1ull);
                    if (at < cap)
                        out[at] = key;
                }
            }
        }
    }
}

// Nodes and prefixes kept so far, to pinned host memory.
__global__ void kl_post_kernel(const unsigned long long* __restrict__ words,
                               uint64_t* __restrict__ host)
{
    host[0] = words[0];
    host[1] = words[2];
}

__global__ void kl_zero_u32_kernel(uint32_t* __restrict__ p, uint64_t n)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

__global__ void kl_advance_kernel(unsigned long long* __restrict__ log_n,
                                  const uint64_t* __restrict__ total, uint64_t cap,
                                  uint32_t* __restrict__ status)
{
    const unsigned long long v = *log_n + *total;
    *log_n = v;
    if (v > cap)
        atomicOr(status, kErrFull);
}

template <typename T>
T* carve(uint8_t*& p, uint64_t n)
{
    T* r = reinterpret_cast<T*>(p);
    p += ((n * sizeof(T) + 255) / 256) * 256;
    return r;
}

// All work of the context finished (pipelined batches included).
hipError_t quiesce(dm_ctx* c)
{
    hipError_t e = join_selection(c);
    if (e == hipSuccess)
        e = sync_streams(c);
    return e;
}

void reset_window(dm_ctx* c)
{
    KeyLen& k = c->kl;
    k.win = 0;
    kl_fill_kernel<<<1, 64, 0, c->stream>>>(reinterpret_cast<uint64_t*>(k.log_n), 2, 0);
}

size_t up256k(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace

void keylen_free(dm_ctx* c)
{
    KeyLen& k = c->kl;
    for (uint64_t* p : {k.tab[0], k.tab[1], k.list, k.log})
        if (p)
            (void)hipFree(p);
    if (k.roots)
        (void)hipFree(k.roots);
    if (k.log_n)
        (void)hipFree(k.log_n);
    k = KeyLen{};
}

uint64_t keylen_record_bytes(uint64_t n) { return 2 * up256k(8 * n) + 256; }

// (Malformed offsets leave every request with no full block in bstart, so
// such a batch records nothing.)
hipError_t keylen_record(dm_ctx* c, uint64_t n, const uint64_t* bstart, const uint64_t* hkeys,
                         uint64_t* work)
{
    const KeyLen& k = c->kl;
    uint64_t* ent = work;
    uint64_t* epos = work + up256k(8 * n) / 8;
    uint64_t* total = work + 2 * (up256k(8 * n) / 8);
    const uint64_t K = c->cfg.key_blocks;
    kl_entries_kernel<<<grid_for(n, 1024, 128), 1024, 0, c->stream>>>(bstart, n, K, ent,
                                                                      k.log_n + 1);
    hipError_t e = exclusive_scan_u64(c, ent, n, epos, total);
    if (e != hipSuccess)
        return e;
    kl_append_kernel<<<grid_for(n, 4, 16384), 256, 0, c->stream>>>(n, bstart, epos, ent, K, hkeys,
                                                                   k.log, k.roots, k.cap, k.log_n);
    kl_advance_kernel<<<1, 1, 0, c->stream>>>(k.log_n, total, k.cap, c->d_status);
    return hipGetLastError();
}

dm_status keylen_enable(dm_ctx* c, uint64_t max_nodes, uint64_t max_window_blocks)
{
    if (max_nodes > (1ull << 28))
        return fail(c, DM_EINVAL, "dm_keylen_enable: max_nodes must be <= 2^28");
    if (max_nodes && (max_window_blocks == 0 || max_window_blocks >= (1ull << 36)))
        return fail(c, DM_EINVAL, "dm_keylen_enable: max_window_blocks must be in [1, 2^36)");
    hipError_t e = quiesce(c);
    if (e != hipSuccess)
        return hip_fail(c, e, "dm_keylen_enable");
    keylen_free(c);
    if (max_nodes == 0)
        return DM_OK;
    KeyLen k;
    k.max_nodes = max_nodes;
    k.cap = max_window_blocks;
    k.log2 = 6;
    while ((1ull << k.log2) < 2 * max_nodes)
        k.log2++;
    const uint64_t slots = 1ull << k.log2;
    if ((e = hipMalloc(&k.tab[0], slots * 8)) == hipSuccess &&
        (e = hipMalloc(&k.tab[1], slots * 8)) == hipSuccess &&
        (e = hipMalloc(&k.list, max_nodes * 8)) == hipSuccess &&
        (e = hipMalloc(&k.log, k.cap * 8)) == hipSuccess &&
        (e = hipMalloc(&k.roots, (k.cap / 32 + 1) * 4)) == hipSuccess)
        e = hipMalloc(&k.log_n, 16);
    c->kl = k;
    if (e != hipSuccess) {
        keylen_free(c);
        return fail(c, DM_ENOMEM, "dm_keylen_enable: device allocation failed");
    }
    c->kl.on = true;
    kl_fill_kernel<<<grid_for(slots, 256), 256, 0, c->stream>>>(c->kl.tab[0], slots, kEmpty);
    kl_zero_u32_kernel<<<grid_for(k.cap / 32 + 1, 256, 8192), 256, 0, c->stream>>>(
        c->kl.roots, k.cap / 32 + 1);
    reset_window(c);
    if ((e = hipGetLastError()) == hipSuccess)
        e = hipStreamSynchronize(c->stream);
    return e == hipSuccess ? DM_OK : hip_fail(c, e, "dm_keylen_enable");
}

dm_status keylen_window(dm_ctx* c)
{
    KeyLen& k = c->kl;
    if (!k.on)
        return fail(c, DM_ESTATE, "dm_keylen_window: the hotness tree is off");
    if (c->n_live == 0)
        return fail(c, DM_ESTATE, "dm_keylen_window: rings not built");
    hipError_t e = quiesce(c);
    if (e != hipSuccess)
        return hip_fail(c, e, "dm_keylen_window");
    unsigned long long made[2] = {0, 0};
    if ((e = hipMemcpy(made, k.log_n, sizeof(made), hipMemcpyDeviceToHost)) != hipSuccess)
        return hip_fail(c, e, "dm_keylen_window");
    const uint64_t M = made[0], R = made[1], W = k.win;
    hipStream_t st = c->stream;
    if (M > k.cap) {
        reset_window(c);
        kl_zero_u32_kernel<<<grid_for(k.cap / 32 + 1, 256, 8192), 256, 0, st>>>(k.roots,
                                                                              k.cap / 32 + 1);
        if ((e = hipStreamSynchronize(st)) != hipSuccess)
            return hip_fail(c, e, "dm_keylen_window");
        return fail(c, DM_EFULL, "dm_keylen_window: the window held more prefixes than its "
                                 "record (tree unchanged)");
    }
    if (W == 0) {  // no traffic: no change
        reset_window(c);
        e = hipStreamSynchronize(st);
        return e == hipSuccess ? DM_OK : hip_fail(c, e, "dm_keylen_window");
    }
    const uint64_t nw = (M + 31) / 32, outcap = k.max_nodes;
    uint64_t meets = 64;
    while (meets < 2 * R)
        meets *= 2;
    // nodes have disjoint sets of at least W / n runs (more runs than W only
    // where a captured batch was replayed)
    const uint64_t parts = std::min(std::max<uint64_t>(R, 1), std::max(R, W) * c->n_live / W);
    uint8_t* w = static_cast<uint8_t*>(scratch_get(
        c, kSlotMembers,
        2 * up256k(8 * outcap) + 2 * up256k(8 * nw) + 2 * up256k(8 * R) + up256k(4 * R) +
            3 * up256k(8 * meets) + up256k(4 * meets) + up256k(sizeof(KlNode) * parts) +
            up256k(8 * M) + 1024,
        &e));
    if (!w)
        return hip_fail(c, e, "dm_keylen_window");
    uint64_t* out = carve<uint64_t>(w, outcap);
    uint64_t* otmp = carve<uint64_t>(w, outcap);
    uint64_t* wcnt = carve<uint64_t>(w, nw);
    uint64_t* wpre = carve<uint64_t>(w, nw);
    uint64_t* start = carve<uint64_t>(w, R);
    KlRuns a{};
    a.log = k.log;
    a.m = M;
    a.start = start;
    a.slot = carve<uint64_t>(w, R);
    a.depth = carve<uint32_t>(w, R);
    a.key = carve<uint64_t>(w, meets);
    a.rep = carve<uint64_t>(w, meets);
    a.count = carve<uint64_t>(w, meets);
    a.node = carve<uint32_t>(w, meets);
    a.mask = meets - 1;
    a.nodes = carve<KlNode>(w, parts);
    a.hist = carve<uint64_t>(w, M);
    a.words = carve<unsigned long long>(w, 4);
    a.runs = R;
    a.W = W;
    a.n_live = c->n_live;
    kl_fill_kernel<<<1, 64, 0, st>>>(reinterpret_cast<uint64_t*>(a.words), 4, 0);
    uint64_t n_next = 0;
    if (R) {
        kl_root_count_kernel<<<grid_for(nw, 256, 8192), 256, 0, st>>>(k.roots, nw, wcnt);
        if ((e = exclusive_scan_u64(c, wcnt, nw, wpre, nullptr)) != hipSuccess)
            return hip_fail(c, e, "dm_keylen_window");
        kl_runs_kernel<<<grid_for(nw, 256, 8192), 256, 0, st>>>(k.roots, nw, wpre, R, start);
        const uint32_t gs = grid_for(meets, 256, 8192);
        auto meet = [&](bool first) {
            a.turn = first ? 0 : a.turn + 1;
            if (first)
                kl_clear_kernel<true><<<gs, 256, 0, st>>>(a);
            else
                kl_clear_kernel<false><<<gs, 256, 0, st>>>(a);
            kl_meet_kernel<<<grid_for(R, kMeet, 2048), kMeet, 0, st>>>(a);
            kl_node_kernel<<<gs, 256, 0, st>>>(a);
        };
        meet(true);
        // each turn settles the nodes found before it and finds those below; a
        // wait after each of the first, then after every fourth (a turn without
        // nodes does nothing)
        for (uint64_t more = 1; more;) {
            kl_hist_zero_kernel<<<grid_for(parts, 1, 1024), 256, 0, st>>>(a);
            if (R <= kAloneTo)
                kl_common_kernel<1><<<grid_for(R, kCommonWaves, 32768), kCommonWaves * kWave, 0,
                                      st>>>(a);
            else
                kl_common_kernel<kManyAlike><<<grid_for(R, kManyAlike * kCommonWaves, 32768),
                                               kCommonWaves * kWave, 0, st>>>(a);
            kl_decide_kernel<<<grid_for(parts, 1, 1024), 256, 0, st>>>(a, k.tab[k.cur], k.log2, out,
                                                                      outcap);
            meet(false);
            if (a.turn > kLongestTurns && a.turn % 4)
                continue;
            kl_post_kernel<<<1, 1, 0, st>>>(a.words, c->host_words);
            if ((e = hipGetLastError()) != hipSuccess ||
                (e = hipStreamSynchronize(st)) != hipSuccess)
                return hip_fail(c, e, "dm_keylen_window");
            more = c->host_words[0];
            n_next = c->host_words[1];
        }
        kl_zero_u32_kernel<<<grid_for(nw, 256, 8192), 256, 0, st>>>(k.roots, nw);
    }
    reset_window(c);
    if (n_next > k.max_nodes) {
        if ((e = hipStreamSynchronize(st)) != hipSuccess)
            return hip_fail(c, e, "dm_keylen_window");
        return fail(c, DM_EFULL, "dm_keylen_window: the new tree would hold " +
                                     std::to_string(n_next) + " extended prefixes, more than " +
                                     std::to_string(k.max_nodes) + " (tree unchanged)");
    }
    const int nx = 1 - k.cur;
    const uint64_t slots = 1ull << k.log2;
    kl_fill_kernel<<<grid_for(slots, 256), 256, 0, st>>>(k.tab[nx], slots, kEmpty);
    if (n_next) {
        kl_insert_kernel<<<grid_for(n_next, 256, 4096), 256, 0, st>>>(k.tab[nx], k.log2, out, n_next);
        // the list is ascending
        if ((e = radix_sort_kv(c, out, nullptr, otmp, nullptr, n_next, 64)) != hipSuccess ||
            (e = hipMemcpyAsync(k.list, out, n_next * 8, hipMemcpyDeviceToDevice, st)) != hipSuccess)
            return hip_fail(c, e, "dm_keylen_window");
    }
    if ((e = hipGetLastError()) != hipSuccess || (e = hipStreamSynchronize(st)) != hipSuccess)
        return hip_fail(c, e, "dm_keylen_window");
    k.cur = nx;
    k.n_ext = n_next;
    return DM_OK;
}

dm_status keylen_export(dm_ctx* c, uint64_t* keys_host, uint64_t cap, uint64_t* n_host)
{
    const KeyLen& k = c->kl;
    if (!k.on)
        return fail(c, DM_ESTATE, "dm_keylen_export: the hotness tree is off");
    hipError_t e = quiesce(c);
    const uint64_t m = std::min(cap, k.n_ext);
    if (e == hipSuccess && m)
        e = hipMemcpy(keys_host, k.list, m * 8, hipMemcpyDeviceToHost);
    if (e != hipSuccess)
        return hip_fail(c, e, "dm_keylen_export");
    *n_host = k.n_ext;
    return DM_OK;
}

}  // namespace dm
