// KV save with least-recently-used eviction: the serving step after routing
// (the KV query and save of Sec. A.3.2), on the device.  A served request's
// full blocks are touched on its instance, deepest block first; each
// instance's cache is the cap most recently touched distinct keys, and the
// difference is applied to its index (erase, then insert).
//
// The record of saved keys is a flat array of (instance, key, time of the
// latest touch).  One save:
//   1. the record's entries and the batch's touches meet in a hash table with
//      a region per instance (kv_home, kv_record and kv_touch_kernel): a slot
//      holds a key, its latest time and whether the record had it;
//   2. each region's occupied slots are packed to its front
//      (kv_pack_kernel);
//   3. an instance over its cap drops its count - cap least recent keys: the
//      time of the last one dropped is found by a radix select over the
//      times, one histogram and one pick per digit (kv_hist_kernel,
//      kv_pick_kernel; ties, which only a clock that was not advanced can
//      make, go by key: kv_tie_kernel);
//   4. dropped keys that were cached are erased, kept keys that were not are
//      inserted, straight from the regions; the kept keys become the record.
// What bounds it: random accesses to the slots (a touch reads a key word and
// a time word) and the launches.  It replaces sorting record and touches by
// key, instance and time (19 radix passes and 14 scans).  Routing and saving
// 16,384 agent requests, 2.3 M touches on a record of 1 M keys, went from
// 2.39 to 1.27 ms; 4,096 chat requests, 1.1 M touches, from 1.45 to 0.69 ms
// (later steps: 1.19 and 0.55).
#include <algorithm>
#include <vector>

#include "dm_internal.h"

namespace dm {
namespace {

template <typename T>
T* carve(uint8_t*& p, uint64_t n)
{
    T* r = reinterpret_cast<T*>(p);
    p += ((n * sizeof(T) + 255) / 256) * 256;
    return r;
}

size_t up256v(size_t x) { return (x + 255) & ~size_t(255); }

// Regions are whole tiles of kTile slots, so that a workgroup's slots belong
// to one instance.
constexpr uint32_t kTile = 2048, kTileThreads = 256, kPerThread = kTile / kTileThreads;
constexpr uint32_t kDigit0 = 8, kDigit = 12;  // bits of the select's first and later digits

// The hash table.  Instance c's region is slots [first[c] * kTile,
// first[c + 1] * kTile); its last slot is key 0's, the others an
// open-addressing table (key 0 = empty).  word = (latest time + 1) << 1 |
// already in the record; 0 for a slot without a key.  Keys and words are
// separate arrays: side by side, the popular keys' lines are taken by the
// words' atomics while others read the keys (the agent batch's touches 190
// us instead of 153).
struct KvSlots {
    uint64_t* key;
    uint64_t* word;
    const uint32_t* first;  // [S + 1] tiles before each instance's region
};

// The instance whose region holds tile b (every thread of the workgroup).
__device__ __forceinline__ uint32_t tile_instance(const uint32_t* first, uint32_t S, uint32_t b)
{
    __shared__ uint32_t found;
    for (uint32_t c = threadIdx.x; c < S; c += blockDim.x)
        if (first[c] <= b && b < first[c + 1])
            found = c;
    __syncthreads();
    return found;
}

__device__ __forceinline__ uint32_t kv_home(uint32_t size, uint64_t k)
{
    return (uint32_t)(((mix64(k) >> 32) * size) >> 32);
}

// Slot of key k in the region of `size` + 1 slots at base (claimed if new).
__device__ __forceinline__ uint64_t kv_slot(uint64_t* key, uint64_t base, uint32_t size, uint64_t k)
{
    if (k == 0)
        return base + size;
    uint32_t i = kv_home(size, k);
    for (uint32_t step = 0; step < size; step++) {
        uint64_t* p = key + base + i;
        const uint64_t v = *p;
        if (v == k)
            return base + i;
        if (v == 0) {
            // seen empty: the claim finds out whether it still is
            const unsigned long long prev = atomicCAS((unsigned long long*)p, 0ull,
                                                      (unsigned long long)k);
            if (prev == 0 || prev == k)
                return base + i;
        }
        i = i + 1 < size ? i + 1 : 0;
    }
    return base + size;  // not reached: a region has more slots than keys
}

// A wave touches at most kTouchBlocks blocks of a request: each 64 take it some
// 8 us, one after the other.  16 requests of 32,768 blocks, whole save: 6.2 ms by a
// wave each, 0.67 in parts.  (A prompt of the chat and agent workloads is one part.)
constexpr uint32_t kTouchBlocks = 512;

__device__ __forceinline__ uint64_t more_parts(uint64_t nf)
{
    return nf > kTouchBlocks ? (nf - 1) / kTouchBlocks : 0;
}

// What a save's first kernels find: checks, parts of requests past their first
// (counted, then listed).
struct KvFound {
    uint32_t bad, pad;
    unsigned long long parts, listed;
};

// bad |= 2 if a request's instance is out of range; touches[c] = the blocks
// that instance c's requests touch.
__global__ void kv_check_kernel(const uint32_t* __restrict__ inst, uint64_t n, uint32_t S,
                                const uint64_t* __restrict__ bstart, KvFound* __restrict__ found,
                                unsigned long long* __restrict__ touches)
{
    extern __shared__ unsigned long long cnt[];  // [S]
    for (uint32_t c = threadIdx.x; c < S; c += blockDim.x)
        cnt[c] = 0;
    __syncthreads();
    unsigned long long parts = 0;
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n;
         r += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t c = inst[r];
        const uint64_t nf = bstart[r + 1] - bstart[r];
        parts += more_parts(nf);
        if (c >= S)
            atomicOr(&found->bad, 2u);
        else
            atomicAdd(&cnt[c], (unsigned long long)nf);
    }
    for (int d = 1; d < kWave; d <<= 1)
        parts += shfl_xor_u64(parts, d);
    if (lane_id() == 0 && parts)
        atomicAdd(&found->parts, parts);
    __syncthreads();
    for (uint32_t c = threadIdx.x; c < S; c += blockDim.x)
        if (cnt[c])
            atomicAdd(&touches[c], cnt[c]);
}

// Counters that workgroups of many tiles add to lie a line apart: atomics on one
// line take some 11 ns each, wherever they come from (1,237 tiles of 16 instances:
// packing 29 us without this and 18 with it, keeping 36 and 29).
constexpr uint32_t kApart = 128 / sizeof(uint64_t);

// Regions: 1.5 slots per entry that instance c may hold (its record entries
// and its touches), first[c] = tiles before it.  One workgroup; tiles are
// counted in 32 bits, saturating (the host rejects such a save by its entry
// count).
__global__ __launch_bounds__(1024) void kv_region_kernel(const uint32_t* __restrict__ rcount,
                                                         const unsigned long long* __restrict__ touches,
                                                         uint32_t S, uint32_t* __restrict__ first)
{
    __shared__ uint64_t part[1024];
    const uint32_t per = (S + 1023) / 1024, c0 = threadIdx.x * per;
    auto tiles = [&](uint32_t c) -> uint64_t {
        const uint64_t e = rcount[c] + touches[c];
        return e ? (e + e / 2 + 1 + kTile) / kTile : 0;
    };
    uint64_t sum = 0;
    for (uint32_t c = c0; c < c0 + per && c < S; c++)
        sum += tiles(c);
    part[threadIdx.x] = sum;
    __syncthreads();
    for (uint32_t d = 1; d < 1024; d <<= 1) {
        const uint64_t x = threadIdx.x >= d ? part[threadIdx.x - d] : 0;
        __syncthreads();
        part[threadIdx.x] += x;
        __syncthreads();
    }
    uint64_t at = part[threadIdx.x] - sum;
    for (uint32_t c = c0; c < c0 + per && c < S; c++) {
        first[c] = (uint32_t)(at < 0xFFFFFFFFull ? at : 0xFFFFFFFFull);
        at += tiles(c);
    }
    if (threadIdx.x == 1023)
        first[S] = (uint32_t)(part[1023] < 0xFFFFFFFFull ? part[1023] : 0xFFFFFFFFull);
}

// What was found, the table's tiles and the batch's blocks, to pinned host
// memory.
__global__ void kv_post_kernel(const KvFound* __restrict__ found, const uint32_t* __restrict__ tiles,
                               const uint64_t* __restrict__ blocks, uint64_t* __restrict__ host)
{
    host[0] = found->bad;
    host[1] = *tiles;
    host[2] = blocks ? *blocks : 0;
    host[3] = found->parts;
}

// Request (40 bits) and number (24 bits: fewer than 2^32 blocks) of every part
// past a request's first.
__global__ void kv_parts_kernel(uint64_t n, const uint64_t* __restrict__ bstart,
                                KvFound* __restrict__ found, uint64_t* __restrict__ list)
{
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n;
         r += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t more = more_parts(bstart[r + 1] - bstart[r]);
        if (!more)
            continue;
        const uint64_t at = atomicAdd(&found->listed, (unsigned long long)more);
        for (uint64_t p = 1; p <= more; p++)
            list[at + p - 1] = r << 24 | p;
    }
}

__global__ void kv_zero_kernel(unsigned long long* __restrict__ p, uint64_t n)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

__device__ __forceinline__ uint32_t region_size(const KvSlots& h, uint32_t c)
{
    // slots but key 0's; a region never needs 2^32 slots (entries < 2^32)
    const uint64_t slots = (uint64_t)(h.first[c + 1] - h.first[c]) * kTile - 1;
    return (uint32_t)(slots < 0xFFFFFFFFull ? slots : 0xFFFFFFFFull);
}

// The record's keys (distinct) into their home slots, before anything else is in
// the table: where several share one, any of them gets it, and kv_record_kernel
// claims places for the others.  Random claims go at some 3.3 G/s on the whole
// chip, plain stores several times faster: 259,000 entries 80 us by claims
// alone, 14 + 39 us so.
__global__ void kv_home_kernel(const uint64_t* __restrict__ rkey, const uint32_t* __restrict__ rinst,
                               uint64_t nrec, KvSlots h)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < nrec;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t k = rkey[i];
        const uint32_t c = rinst[i];
        if (k)
            __hip_atomic_store(h.key + (uint64_t)h.first[c] * kTile + kv_home(region_size(h, c), k), k,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ void kv_record_kernel(const uint64_t* __restrict__ rkey, const uint64_t* __restrict__ rt,
                                 const uint32_t* __restrict__ rinst, uint64_t nrec, KvSlots h)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < nrec;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t c = rinst[i];
        const uint64_t p = kv_slot(h.key, (uint64_t)h.first[c] * kTile, region_size(h, c), rkey[i]);
        h.word[p] = (rt[i] + 1) << 1 | 1u;  // the record's entries are distinct
    }
}

// One wave per request and part, the last request first: block b of request r
// is touched at time clock + start_r + (nfull_r - 1 - b), so a later request's
// touch of a key makes the earlier ones' atomics unnecessary (popular prefixes
// are touched by thousands of requests).
__global__ void kv_touch_kernel(uint64_t n, const uint64_t* __restrict__ list, uint64_t parts,
                                const uint64_t* __restrict__ bstart,
                                const uint64_t* __restrict__ block_keys,
                                const uint32_t* __restrict__ inst, uint64_t clock, KvSlots h)
{
    const uint64_t w = blockIdx.x * (uint64_t)(blockDim.x >> 6) +
                       __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t nw = (uint64_t)gridDim.x * (blockDim.x >> 6);
    const uint32_t lane = threadIdx.x & 63;
    for (uint64_t i = w; i < parts + n; i += nw) {
        const uint64_t v = i < parts ? list[i] : (n - 1 - (i - parts)) << 24;
        const uint64_t r = v >> 24, b0 = (v & 0xFFFFFF) * kTouchBlocks;
        const uint64_t s = bstart[r], nf = bstart[r + 1] - s;
        const uint32_t c = inst[r];
        const uint64_t base = (uint64_t)h.first[c] * kTile;
        const uint32_t size = nf ? region_size(h, c) : 0;
        const uint64_t end = nf < b0 + kTouchBlocks ? nf : b0 + kTouchBlocks;
        for (uint64_t b = b0 + lane; b < end; b += kWave) {
            const uint64_t p = kv_slot(h.key, base, size, block_keys[s + b]);
            // the record's flag was settled by the kernel before; a time seen
            // late only costs an atomic
            const uint64_t seen = h.word[p];
            const uint64_t mine = (clock + s + (nf - 1 - b) + 1) << 1 | (seen & 1);
            if (seen < mine)
                atomicMax((unsigned long long*)&h.word[p], (unsigned long long)mine);
        }
    }
}

// Sum over the workgroup, in every thread (kTileThreads threads).
__device__ __forceinline__ uint32_t tile_sum(uint32_t v)
{
    __shared__ uint32_t part[kTileThreads / kWave];
    for (int d = 1; d < kWave; d <<= 1)
        v += (uint32_t)__shfl_xor((int)v, d);
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t s = 0;
#pragma unroll
    for (uint32_t k = 0; k < kTileThreads / kWave; k++)
        s += part[k];
    return s;
}

// Exclusive sum over the workgroup's threads; total in every thread.
__device__ __forceinline__ uint32_t tile_excl(uint32_t v, uint32_t& total)
{
    __shared__ uint32_t part[kTileThreads / kWave];
    const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t x = v;
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, d);
        if ((int)lane >= d)
            x += y;
    }
    __syncthreads();
    if (lane == 63)
        part[wv] = x;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (uint32_t k = 0; k < kTileThreads / kWave; k++) {
        before += k < wv ? part[k] : 0;
        total += part[k];
    }
    return before + x - v;
}

// A region's occupied slots to the front of its place in the packed arrays
// (any order); used[c * kApart] = how many.
__global__ __launch_bounds__(kTileThreads) void kv_pack_kernel(KvSlots h, uint32_t S,
                                                               uint64_t* __restrict__ key,
                                                               uint64_t* __restrict__ word,
                                                               unsigned long long* __restrict__ used)
{
    __shared__ uint32_t at0;
    const uint32_t c = tile_instance(h.first, S, blockIdx.x);
    const uint64_t s0 = (uint64_t)blockIdx.x * kTile + threadIdx.x;
    uint64_t w[kPerThread];
    uint32_t mine = 0, total = 0;
#pragma unroll
    for (uint32_t q = 0; q < kPerThread; q++) {
        w[q] = h.word[s0 + q * kTileThreads];
        mine += w[q] != 0;
    }
    uint32_t at = tile_excl(mine, total);
    if (threadIdx.x == 0)
        at0 = total ? (uint32_t)atomicAdd(&used[c * kApart], (unsigned long long)total) : 0;
    __syncthreads();
    uint64_t out = (uint64_t)h.first[c] * kTile + at0 + at;
#pragma unroll
    for (uint32_t q = 0; q < kPerThread; q++)
        if (w[q]) {
            key[out] = h.key[s0 + q * kTileThreads];
            word[out++] = w[q];
        }
}

// State of the select, per instance: keys still to drop among those whose
// leading digits are prefix, and after the last digit how many share that
// time (same) and the largest key dropped among them (last).
struct KvSelect {
    uint32_t* rem;
    uint64_t* prefix;
    uint32_t* same;
    uint64_t* last;
    uint32_t* hist;   // [S << kDigit]: this digit's counts
    uint64_t cap, lo;  // lo: no time is smaller
};

__device__ __forceinline__ uint64_t rel_time(uint64_t word, uint64_t lo) { return (word >> 1) - 1 - lo; }

// Counts of one digit (bits bits above shift) of the times of every instance
// over its cap; of the times that begin with prefix after the first digit.
// A workgroup's counts meet in LDS: times of recent batches next to one old
// entry anywhere share their leading digits, and then every entry counts in a
// few bins (atomics on one line take some 11 ns each: 1 M entries of one
// instance beside an idle one's old entry, whole save 7.9 ms with the later
// digits' counts straight to memory, 0.68 so).  A tile with few times left counts
// straight, which spares clearing and reading the bins.
constexpr uint32_t kFewTimes = 64;

template <bool FIRST>
__global__ __launch_bounds__(kTileThreads) void kv_hist_kernel(const uint32_t* __restrict__ first,
                                                               uint32_t S,
                                                               const unsigned long long* __restrict__ used,
                                                               const uint64_t* __restrict__ word,
                                                               KvSelect s, uint32_t shift,
                                                               uint32_t bits)
{
    constexpr uint32_t kBins = 1u << (FIRST ? kDigit0 : kDigit);
    __shared__ uint32_t cnt[kBins];
    const uint32_t c = tile_instance(first, S, blockIdx.x);
    const uint32_t n = (uint32_t)used[c * kApart];
    const uint64_t i0 = (uint64_t)(blockIdx.x - first[c]) * kTile;
    if (i0 >= n || (FIRST ? n <= s.cap : s.rem[c] == 0))
        return;
    const uint64_t pre = FIRST ? 0 : s.prefix[c];
    uint32_t* const out = s.hist + ((uint64_t)c << kDigit);
    uint32_t d[kPerThread], mine = 0;
    bool in[kPerThread];
#pragma unroll
    for (uint32_t q = 0; q < kPerThread; q++) {
        const uint32_t j = q * kTileThreads + threadIdx.x;
        const bool ok = i0 + j < n;
        const uint64_t v = ok ? rel_time(word[(uint64_t)blockIdx.x * kTile + j], s.lo) : 0;
        in[q] = ok && (FIRST || v >> (shift + bits) == pre);
        d[q] = (uint32_t)(v >> shift) & ((1u << bits) - 1);
        mine += in[q];
    }
    const bool few = !FIRST && tile_sum(mine) <= kFewTimes;
    if (!few) {
        for (uint32_t k = threadIdx.x; k < kBins; k += kTileThreads)
            cnt[k] = 0;
        __syncthreads();
    }
#pragma unroll
    for (uint32_t q = 0; q < kPerThread; q++)
        if (in[q]) {
            if (few)
                atomicAdd(&out[d[q]], 1u);
            else
                atomicAdd(&cnt[d[q]], 1u);
        }
    if (!few) {
        __syncthreads();
        for (uint32_t k = threadIdx.x; k < kBins; k += kTileThreads)
            if (cnt[k])
                atomicAdd(&out[k], cnt[k]);
    }
}

// The digit of the last key dropped, a workgroup per instance; clears the
// counts for the next digit.
template <bool FIRST>
__global__ __launch_bounds__(kTileThreads) void kv_pick_kernel(const unsigned long long* __restrict__ used,
                                                               KvSelect s, uint32_t bits)
{
    const uint32_t c = blockIdx.x;
    const uint64_t held = used[c * kApart];
    const uint32_t rem = FIRST ? (held > s.cap ? (uint32_t)(held - s.cap) : 0) : s.rem[c];
    if (rem == 0) {
        if (FIRST && threadIdx.x == 0)
            s.rem[c] = 0;
        return;
    }
    const uint32_t bins = 1u << bits, per = (bins + kTileThreads - 1) / kTileThreads;
    uint32_t* cnt = s.hist + ((uint64_t)c << kDigit);
    uint32_t mine = 0, total = 0;
    for (uint32_t d = threadIdx.x * per; d < (threadIdx.x + 1) * per && d < bins; d++)
        mine += cnt[d];
    uint32_t before = tile_excl(mine, total);
    for (uint32_t d = threadIdx.x * per; d < (threadIdx.x + 1) * per && d < bins; d++) {
        const uint32_t x = cnt[d];
        cnt[d] = 0;
        if (before < rem && rem <= before + x) {
            s.rem[c] = rem - before;
            s.prefix[c] = (FIRST ? 0 : s.prefix[c] << bits) | d;
            s.same[c] = x;
        }
        before += x;
    }
}

// Of an instance's keys with the time of the last one dropped, the smallest
// go first: the largest of them to drop (all of them: any key).  One workgroup
// per instance lists them (as many as there were saves at that time; few) where
// the instance's hash table was, then picks the key a digit at a time.  Bound by
// the one read of the instance's times: 4 instances of 131,072 entries each at a
// clock that is not advanced, whole save 4.3 ms with a read per bit of the key by
// 256 threads, 0.26 so.
constexpr uint32_t kTieThreads = 1024, kTieAhead = 8, kTieDigit = 8;

__global__ __launch_bounds__(kTieThreads) void kv_tie_kernel(const uint32_t* __restrict__ first,
                                                             const unsigned long long* __restrict__ used,
                                                             const uint64_t* __restrict__ key,
                                                             const uint64_t* __restrict__ word,
                                                             uint64_t* tied, KvSelect s)
{
    constexpr uint32_t kBins = 1u << kTieDigit;
    __shared__ uint32_t cnt[kBins], part[kBins / kWave], len, digit, less;
    const uint32_t c = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    uint32_t rem = s.rem[c];
    if (rem == 0 || rem == s.same[c]) {
        if (t == 0)
            s.last[c] = UINT64_MAX;
        return;
    }
    const uint64_t base = (uint64_t)first[c] * kTile, T = s.prefix[c], n = used[c * kApart];
    if (t == 0)
        len = 0;
    __syncthreads();
    for (uint64_t i0 = t; i0 < n; i0 += kTieThreads * kTieAhead) {
        uint64_t w[kTieAhead];
#pragma unroll
        for (uint32_t q = 0; q < kTieAhead; q++) {
            const uint64_t i = i0 + q * kTieThreads;
            w[q] = i < n ? word[base + i] : 0;
        }
#pragma unroll
        for (uint32_t q = 0; q < kTieAhead; q++) {
            const uint64_t i = i0 + q * kTieThreads;
            if (i < n && rel_time(w[q], s.lo) == T)
                tied[base + atomicAdd(&len, 1u)] = key[base + i];
        }
    }
    __syncthreads();
    const uint32_t m = len;
    uint64_t last = 0;  // the leading digits of the key
    for (int shift = 64 - kTieDigit; shift >= 0; shift -= kTieDigit) {
        if (t < kBins)
            cnt[t] = 0;
        __syncthreads();
        for (uint32_t i = t; i < m; i += kTieThreads) {
            const uint64_t k = tied[base + i] >> shift;
            if (k >> kTieDigit == last)
                atomicAdd(&cnt[k & (kBins - 1)], 1u);
        }
        __syncthreads();
        uint32_t x = t < kBins ? cnt[t] : 0;
        const uint32_t mine = x;
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, d);
            if ((int)lane >= d)
                x += y;
        }
        if (t < kBins && lane == 63)
            part[wv] = x;
        __syncthreads();
        if (t < kBins) {
            for (uint32_t k = 0; k < wv; k++)
                x += part[k];
            if (x - mine < rem && rem <= x) {
                digit = t;
                less = x - mine;
            }
        }
        __syncthreads();
        rem -= less;
        last = last << kTieDigit | digit;
    }
    if (t == 0)
        s.last[c] = last;
}

// Results of a save: per instance the keys to insert and whether its table
// has room for them, its occupied slots afterwards; record entries, erased
// and inserted keys, ~the smallest time kept.  While the tiles are gone through,
// each in a counter of its own per instance (kTallies a line apart).
enum { kPlace, kErased, kInserted, kTime, kTallies };
struct KvOut {
    uint32_t* ins;
    uint32_t* fits;
    uint64_t* occ;
    uint64_t* sum;              // record entries, erased, inserted, ~smallest time
    unsigned long long* tally;  // [S * kTallies * kApart]
};

__device__ __forceinline__ unsigned long long* kv_tally(const KvOut& o, uint32_t c, uint32_t which)
{
    return o.tally + ((uint64_t)c * kTallies + which) * kApart;
}

// Record entries per instance (an instance keeps its cap, or what it has) and
// where they go.
__global__ __launch_bounds__(1024) void kv_place_kernel(const unsigned long long* __restrict__ used,
                                                        uint32_t S, uint64_t cap, KvOut o,
                                                        uint32_t* __restrict__ rcount)
{
    __shared__ uint64_t part[1024];
    const uint32_t per = (S + 1023) / 1024, c0 = threadIdx.x * per;
    uint64_t sum = 0;
    for (uint32_t c = c0; c < c0 + per && c < S; c++) {
        const uint64_t kept = used[c * kApart] < cap ? used[c * kApart] : cap;
        rcount[c] = (uint32_t)kept;
        sum += kept;
    }
    part[threadIdx.x] = sum;
    __syncthreads();
    for (uint32_t d = 1; d < 1024; d <<= 1) {
        const uint64_t x = threadIdx.x >= d ? part[threadIdx.x - d] : 0;
        __syncthreads();
        part[threadIdx.x] += x;
        __syncthreads();
    }
    uint64_t at = part[threadIdx.x] - sum;
    for (uint32_t c = c0; c < c0 + per && c < S; c++) {
        *kv_tally(o, c, kPlace) = at;
        at += rcount[c];
    }
    if (threadIdx.x == 1023)
        o.sum[0] = part[1023];
}

__device__ __forceinline__ bool kv_dropped(const KvSelect& s, uint32_t c, uint32_t rem, uint64_t k,
                                           uint64_t w)
{
    if (rem == 0)
        return false;
    const uint64_t v = rel_time(w, s.lo), T = s.prefix[c];
    return v < T || (v == T && k <= s.last[c]);
}

// The kept keys into the new record, the dropped ones that were cached out
// of their index.
__global__ __launch_bounds__(kTileThreads) void kv_keep_kernel(
    const uint32_t* __restrict__ first, uint32_t S, const unsigned long long* __restrict__ used,
    const uint64_t* __restrict__ key, const uint64_t* __restrict__ word, KvSelect s, KvOut o,
    uint64_t* __restrict__ tables, uint64_t* __restrict__ live, uint32_t log2slots,
    uint64_t* __restrict__ rkey, uint64_t* __restrict__ rt, uint32_t* __restrict__ rinst)
{
    __shared__ unsigned long long at0, tmin;
    const uint32_t c = tile_instance(first, S, blockIdx.x);
    const uint32_t n = (uint32_t)used[c * kApart];
    const uint64_t i0 = (uint64_t)(blockIdx.x - first[c]) * kTile;
    if (i0 >= n)
        return;
    const uint32_t rem = s.rem[c];
    uint64_t k[kPerThread], w[kPerThread];
    uint32_t kept = 0, add = 0, erase = 0, gone = 0, total = 0;
    uint64_t mn = UINT64_MAX;
#pragma unroll
    for (uint32_t q = 0; q < kPerThread; q++) {
        const uint32_t j = q * kTileThreads + threadIdx.x;
        w[q] = 0;
        if (i0 + j >= n)
            continue;
        k[q] = key[(uint64_t)blockIdx.x * kTile + j];
        w[q] = word[(uint64_t)blockIdx.x * kTile + j];
        const bool old = w[q] & 1;
        if (kv_dropped(s, c, rem, k[q], w[q])) {
            if (old) {
                erase++;
                gone += take_key(tables + ((uint64_t)c << log2slots), log2slots, canon_key(k[q]));
            }
            w[q] = 0;
        } else {
            kept++;
            add += !old;
            mn = std::min(mn, (w[q] >> 1) - 1);
        }
    }
    if (threadIdx.x == 0)
        tmin = UINT64_MAX;
    const uint32_t at = tile_excl(kept, total);
    erase = tile_sum(erase);
    add = tile_sum(add);
    gone = tile_sum(gone);
    if (mn != UINT64_MAX)
        atomicMin(&tmin, (unsigned long long)mn);
    __syncthreads();
    if (threadIdx.x == 0) {
        at0 = total ? atomicAdd(kv_tally(o, c, kPlace), (unsigned long long)total) : 0;
        if (erase)
            atomicAdd(kv_tally(o, c, kErased), (unsigned long long)erase);
        if (gone)
            atomicAdd((unsigned long long*)&live[c], 0ull - gone);
        if (add)
            atomicAdd(kv_tally(o, c, kInserted), (unsigned long long)add);
        if (tmin != UINT64_MAX)
            atomicMax(kv_tally(o, c, kTime), ~tmin);
    }
    __syncthreads();
    uint64_t out = at0 + at;
#pragma unroll
    for (uint32_t q = 0; q < kPerThread; q++)
        if (w[q]) {
            rkey[out] = k[q];
            rt[out] = (w[q] >> 1) - 1;
            rinst[out++] = c;
        }
}

// The kept keys that were not cached into the indexes that have room for
// all of theirs (the count words grow once per workgroup).
__global__ __launch_bounds__(kTileThreads) void kv_insert_kernel(
    const uint32_t* __restrict__ first, uint32_t S, const unsigned long long* __restrict__ used,
    const uint64_t* __restrict__ key, const uint64_t* __restrict__ word, KvSelect s, KvOut o,
    uint64_t* __restrict__ tables, uint64_t* __restrict__ counts, uint32_t log2slots,
    uint32_t* __restrict__ status)
{
    const uint32_t c = tile_instance(first, S, blockIdx.x);
    const uint32_t n = (uint32_t)used[c * kApart];
    const uint64_t i0 = (uint64_t)(blockIdx.x - first[c]) * kTile;
    if (i0 >= n || o.ins[c] == 0 || !o.fits[c])
        return;
    const uint32_t rem = s.rem[c];
    uint32_t stored = 0;
    for (uint32_t q = threadIdx.x; q < kTile && i0 + q < n; q += kTileThreads) {
        const uint64_t k = key[(uint64_t)blockIdx.x * kTile + q];
        const uint64_t w = word[(uint64_t)blockIdx.x * kTile + q];
        if ((w & 1) || kv_dropped(s, c, rem, k, w))
            continue;
        const Put p = put_key(tables + ((uint64_t)c << log2slots), log2slots, canon_key(k));
        stored += p == Put::kStored;
        if (p == Put::kNoRoom)
            atomicOr(status, kErrFull);
    }
    stored = tile_sum(stored);
    if (threadIdx.x == 0 && stored) {
        atomicAdd((unsigned long long*)&counts[c], (unsigned long long)stored);
        atomicAdd((unsigned long long*)&counts[S + c], (unsigned long long)stored);
    }
}

// Which tables have room for their keys without a rebuild (the others are
// left to index_insert, with its rebuild and overflow handling), and the
// tallies together.  One workgroup.
__global__ __launch_bounds__(256) void kv_fits_kernel(const uint64_t* __restrict__ counts,
                                                      uint32_t S, uint64_t limit, KvOut o)
{
    __shared__ unsigned long long sum[3];
    if (threadIdx.x < 3)
        sum[threadIdx.x] = 0;
    __syncthreads();
    for (uint32_t c = threadIdx.x; c < S; c += 256) {
        const uint64_t add = *kv_tally(o, c, kInserted);
        o.ins[c] = (uint32_t)add;
        o.fits[c] = counts[S + c] + add <= limit;
        o.occ[c] = counts[S + c] + add;
        atomicAdd(&sum[0], *kv_tally(o, c, kErased));
        atomicAdd(&sum[1], (unsigned long long)add);
        atomicMax(&sum[2], *kv_tally(o, c, kTime));
    }
    __syncthreads();
    if (threadIdx.x < 3)
        o.sum[1 + threadIdx.x] = sum[threadIdx.x];
}

// Instance c's keys to insert, as a list (any order).
__global__ __launch_bounds__(kTileThreads) void kv_list_kernel(
    const uint32_t* __restrict__ first, const unsigned long long* __restrict__ used,
    const uint64_t* __restrict__ key, const uint64_t* __restrict__ word, KvSelect s, uint32_t c,
    uint64_t* __restrict__ list, unsigned long long* __restrict__ len)
{
    const uint32_t rem = s.rem[c];
    const uint64_t base = (uint64_t)first[c] * kTile;
    const uint32_t n = (uint32_t)used[c * kApart];
    for (uint32_t i0 = blockIdx.x * blockDim.x; i0 < n; i0 += gridDim.x * blockDim.x) {
        const uint32_t i = i0 + threadIdx.x;
        const uint64_t k = i < n ? key[base + i] : 0, w = i < n ? word[base + i] : 1;
        const bool add = !(w & 1) && !kv_dropped(s, c, rem, k, w);
        const uint64_t m = ballot(add);
        uint64_t at = 0;
        if (m && lane_id() == 0)
            at = atomicAdd(len, (unsigned long long)__popcll(m));
        at = readlane_u64(at, 0);
        if (add)
            list[at + __popcll(m & ((1ull << lane_id()) - 1))] = k;
    }
}

// Record entries of the given instances dropped (their indexes were emptied):
// the others into the second set of arrays, *n of them.
__global__ __launch_bounds__(kTileThreads) void kv_forget_kernel(
    const uint64_t* __restrict__ k0, const uint64_t* __restrict__ t0,
    const uint32_t* __restrict__ i0, uint64_t n, const uint8_t* __restrict__ gone,
    uint64_t* __restrict__ k1, uint64_t* __restrict__ t1, uint32_t* __restrict__ i1,
    unsigned long long* __restrict__ kept)
{
    __shared__ unsigned long long at0;
    const uint64_t base = (uint64_t)blockIdx.x * kTile;
    uint32_t mine = 0, total = 0;
    bool keep[kPerThread];
#pragma unroll
    for (uint32_t q = 0; q < kPerThread; q++) {
        const uint64_t i = base + q * kTileThreads + threadIdx.x;
        keep[q] = i < n && !gone[i0[i]];
        mine += keep[q];
    }
    const uint32_t at = tile_excl(mine, total);
    if (threadIdx.x == 0)
        at0 = atomicAdd(kept, (unsigned long long)total);
    __syncthreads();
    uint64_t out = at0 + at;
#pragma unroll
    for (uint32_t q = 0; q < kPerThread; q++) {
        const uint64_t i = base + q * kTileThreads + threadIdx.x;
        if (keep[q]) {
            k1[out] = k0[i];
            t1[out] = t0[i];
            i1[out++] = i0[i];
        }
    }
}

__global__ void kv_forget_count_kernel(const uint8_t* __restrict__ gone, uint32_t S,
                                       uint32_t* __restrict__ rcount)
{
    for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c < S; c += gridDim.x * blockDim.x)
        if (gone[c])
            rcount[c] = 0;
}

// The record's arrays not in use hold at least n entries (contents lost).
hipError_t kv_reserve(dm_ctx* c, uint64_t n)
{
    KvRecord& r = c->kv;
    const int o = 1 - r.cur;
    if (n <= r.cap[o])
        return hipSuccess;
    const uint64_t cap = std::max<uint64_t>(n, 2 * r.cap[o]);
    hipError_t e = sync_streams(c);
    if (e != hipSuccess)
        return e;
    (void)hipFree(r.key[o]);
    (void)hipFree(r.t[o]);
    (void)hipFree(r.inst[o]);
    r.key[o] = r.t[o] = nullptr;
    r.inst[o] = nullptr;
    r.cap[o] = 0;
    if ((e = hipMalloc(&r.key[o], cap * 8)) != hipSuccess ||
        (e = hipMalloc(&r.t[o], cap * 8)) != hipSuccess ||
        (e = hipMalloc(&r.inst[o], cap * 4)) != hipSuccess)
        return e;
    r.cap[o] = cap;
    return hipSuccess;
}

}  // namespace

void kv_free(dm_ctx* c)
{
    KvRecord& r = c->kv;
    for (int o = 0; o < 2; o++) {
        (void)hipFree(r.key[o]);
        (void)hipFree(r.t[o]);
        (void)hipFree(r.inst[o]);
    }
    (void)hipFree(r.count);
    r = KvRecord{};
}

hipError_t kv_forget(dm_ctx* c, const uint8_t* d_gone)
{
    KvRecord& r = c->kv;
    if (r.n == 0)
        return hipSuccess;
    const uint64_t n = r.n;
    const uint32_t S = c->cfg.max_slots;
    const int a = r.cur, b = 1 - a;
    hipError_t e = kv_reserve(c, n);
    unsigned long long* kept =
        e == hipSuccess ? static_cast<unsigned long long*>(scratch_get(c, kSlotMembers, 256, &e))
                        : nullptr;
    if (!kept)
        return e;
    kv_zero_kernel<<<1, 64, 0, c->stream>>>(kept, 1);
    kv_forget_kernel<<<(uint32_t)((n + kTile - 1) / kTile), kTileThreads, 0, c->stream>>>(
        r.key[a], r.t[a], r.inst[a], n, d_gone, r.key[b], r.t[b], r.inst[b], kept);
    kv_forget_count_kernel<<<grid_for(S, 256), 256, 0, c->stream>>>(d_gone, S, r.count);
    uint64_t m = 0;
    if ((e = hipGetLastError()) != hipSuccess ||
        (e = hipMemcpyAsync(&m, kept, 8, hipMemcpyDeviceToHost, c->stream)) != hipSuccess ||
        (e = hipStreamSynchronize(c->stream)) != hipSuccess)
        return e;
    r.n = m;
    r.cur = b;
    return hipSuccess;
}

dm_status kv_save(dm_ctx* c, const int64_t* offsets, uint64_t n, const uint64_t* block_keys,
                  const uint32_t* inst, uint64_t clock, uint64_t cap, uint64_t* added,
                  uint64_t* removed)
{
    const uint32_t S = c->cfg.max_slots, log2slots = c->cfg.index_log2_slots;
    auto failed = [&](hipError_t e) { return hip_fail(c, e, "dm_kv_save"); };
    hipError_t e = join_selection(c);
    if (e != hipSuccess)
        return failed(e);
    hipStream_t st = c->stream;
    KvRecord& rec = c->kv;
    if (!rec.count) {
        if ((e = hipMalloc(&rec.count, up256v(4 * (size_t)S))) != hipSuccess) {
            rec.count = nullptr;
            return failed(e);
        }
        if ((e = hipMemsetAsync(rec.count, 0, up256v(4 * (size_t)S), st)) != hipSuccess)
            return failed(e);
    }
    // block starts (offsets checked on the device), each instance's touches
    // and its region of the hash table
    const size_t head = up256v((n + 1) * sizeof(uint64_t));
    uint8_t* w0 = static_cast<uint8_t*>(scratch_get(
        c, kSlotStarts, head + 256 + up256v(8 * (size_t)S) + up256v(4 * ((size_t)S + 1)), &e));
    if (!w0)
        return failed(e);
    uint64_t* bstart = carve<uint64_t>(w0, n + 1);
    unsigned long long* touches = carve<unsigned long long>(w0, S);
    KvFound* found = carve<KvFound>(w0, 1);
    uint32_t* first = carve<uint32_t>(w0, (uint64_t)S + 1);
    kv_zero_kernel<<<grid_for(S + 32, 256), 256, 0, st>>>(
        touches, up256v(8 * (size_t)S) / 8 + sizeof(KvFound) / 8);
    if ((e = block_starts(c, offsets, n, 1ull << 62, bstart, &found->bad)) != hipSuccess)
        return failed(e);
    if (n)
        kv_check_kernel<<<grid_for(n, 256, 256), 256, S * sizeof(unsigned long long), st>>>(
            inst, n, S, bstart, found, touches);
    kv_region_kernel<<<1, 1024, 0, st>>>(rec.count, touches, S, first);
    kv_post_kernel<<<1, 1, 0, st>>>(found, first + S, n ? bstart + n : nullptr, c->host_words);
    if ((e = hipGetLastError()) != hipSuccess || (e = hipStreamSynchronize(st)) != hipSuccess)
        return failed(e);
    const uint32_t badh = (uint32_t)c->host_words[0], tiles = (uint32_t)c->host_words[1];
    const uint64_t E = c->host_words[2], parts = c->host_words[3];
    if (badh & 2)
        return fail(c, DM_EINVAL, "dm_kv_save: an instance id is >= max_slots");
    if (badh)
        return fail(c, DM_EINVAL, "dm_kv_save: offsets must be non-decreasing and non-negative");
    if (E && !block_keys)
        return fail(c, DM_EINVAL, "dm_kv_save: null block keys");
    if (clock + E >= (1ull << 40))
        return fail(c, DM_EINVAL, "dm_kv_save: touch times must stay below 2^40");
    const uint64_t M = rec.n + E;
    if (M >= (1ull << 32))
        return fail(c, DM_EINVAL, "dm_kv_save: more than 2^32 record entries");
    if (M == 0) {
        if (added) *added = 0;
        if (removed) *removed = 0;
        return DM_OK;
    }
    // the hash table and its packed form, the select's state, the results
    const uint64_t slots = (uint64_t)tiles * kTile;
    const size_t apart = 8 * (size_t)kApart * S;  // a counter per instance
    const uint64_t zeroed = 8 * slots * 2 + up256v((4ull * S) << kDigit) + up256v(apart) +
                            up256v(kTallies * apart);
    uint8_t* w = static_cast<uint8_t*>(scratch_get(
        c, kSlotMembers,
        zeroed + 16 * slots + 2 * up256v(8 * (size_t)S) + 4 * up256v(4 * (size_t)S) +
            up256v(8 * (size_t)S) + up256v(8 * parts) + 4096,
        &e));
    if (!w)
        return failed(e);
    uint8_t* const w1 = w;
    KvSlots h{};
    h.key = carve<uint64_t>(w, slots);
    h.word = carve<uint64_t>(w, slots);
    h.first = first;
    KvSelect s{};
    s.hist = carve<uint32_t>(w, (uint64_t)S << kDigit);
    unsigned long long* used = carve<unsigned long long>(w, (uint64_t)S * kApart);
    KvOut o{};
    o.tally = carve<unsigned long long>(w, (uint64_t)S * kApart * kTallies);  // cleared up to here
    o.ins = carve<uint32_t>(w, S);
    o.sum = carve<uint64_t>(w, 8);
    uint64_t* key = carve<uint64_t>(w, slots);
    uint64_t* word = carve<uint64_t>(w, slots);
    s.prefix = carve<uint64_t>(w, S);
    s.last = carve<uint64_t>(w, S);
    s.rem = carve<uint32_t>(w, S);
    s.same = carve<uint32_t>(w, S);
    o.fits = carve<uint32_t>(w, S);
    o.occ = carve<uint64_t>(w, S);
    uint64_t* list = carve<uint64_t>(w, parts);
    uint8_t* const results = reinterpret_cast<uint8_t*>(o.fits);
    const int a = rec.cur, b = 1 - a;
    const uint64_t room = cap && cap < (1ull << 32) ? std::min<uint64_t>(M, cap * S) : M;
    if ((e = kv_reserve(c, room)) != hipSuccess)
        return failed(e);
    s.cap = cap ? cap : UINT64_MAX;
    s.lo = rec.n ? std::min(rec.tmin, clock) : clock;
    const uint64_t tmax = std::max(rec.n ? rec.tmax : 0, clock + (E ? E - 1 : 0));
    kv_zero_kernel<<<grid_for(zeroed / 8, 256, 4096), 256, 0, st>>>(
        reinterpret_cast<unsigned long long*>(w1), zeroed / 8);
    if (rec.n) {
        kv_home_kernel<<<grid_for(rec.n, 256, 8192), 256, 0, st>>>(rec.key[a], rec.inst[a], rec.n, h);
        kv_record_kernel<<<grid_for(rec.n, 256, 8192), 256, 0, st>>>(rec.key[a], rec.t[a],
                                                                     rec.inst[a], rec.n, h);
    }
    if (parts)
        kv_parts_kernel<<<grid_for(n, 256, 256), 256, 0, st>>>(n, bstart, found, list);
    if (E)
        kv_touch_kernel<<<grid_for(parts + n, 4, 8192), 256, 0, st>>>(n, list, parts, bstart,
                                                                      block_keys, inst, clock, h);
    kv_pack_kernel<<<tiles, kTileThreads, 0, st>>>(h, S, key, word, used);
    uint32_t left = 1;
    while (left < 64 && (tmax - s.lo) >> left)
        left++;
    const bool first_all = cap == 0;  // nothing is dropped
    if (first_all) {
        kv_zero_kernel<<<grid_for(S, 256), 256, 0, st>>>(
            reinterpret_cast<unsigned long long*>(s.rem), up256v(4 * (size_t)S) / 8);
    } else {
        uint32_t bits = std::min(left, kDigit0);
        left -= bits;
        kv_hist_kernel<true><<<tiles, kTileThreads, 0, st>>>(first, S, used, word, s, left, bits);
        kv_pick_kernel<true><<<S, kTileThreads, 0, st>>>(used, s, bits);
        while (left) {
            bits = std::min(left, kDigit);
            left -= bits;
            kv_hist_kernel<false><<<tiles, kTileThreads, 0, st>>>(first, S, used, word, s, left,
                                                                  bits);
            kv_pick_kernel<false><<<S, kTileThreads, 0, st>>>(used, s, bits);
        }
        kv_tie_kernel<<<S, kTieThreads, 0, st>>>(first, used, key, word, h.key, s);
    }
    kv_place_kernel<<<1, 1024, 0, st>>>(used, S, s.cap, o, rec.count);
    kv_keep_kernel<<<tiles, kTileThreads, 0, st>>>(first, S, used, key, word, s, o, c->d_tables,
                                                   c->d_counts, log2slots, rec.key[b], rec.t[b],
                                                   rec.inst[b]);
    kv_fits_kernel<<<1, 256, 0, st>>>(c->d_counts, S, 1ull << (log2slots - 1), o);
    kv_insert_kernel<<<tiles, kTileThreads, 0, st>>>(first, S, used, key, word, s, o, c->d_tables,
                                                     c->d_counts, log2slots, c->d_status);
    if ((e = hipGetLastError()) != hipSuccess)
        return failed(e);
    // two copies: keys to insert with the totals, room with occupied slots
    const size_t insb = up256v(4 * (size_t)S), occb = 8 * (size_t)S;
    std::vector<uint64_t> head_h((insb + 64) / 8), tail_h((insb + occb) / 8);
    if ((e = hipMemcpyAsync(head_h.data(), o.ins, insb + 64, hipMemcpyDeviceToHost, st)) !=
            hipSuccess ||
        (e = hipMemcpyAsync(tail_h.data(), results, insb + occb, hipMemcpyDeviceToHost, st)) !=
            hipSuccess ||
        (e = hipStreamSynchronize(st)) != hipSuccess)
        return failed(e);
    const uint32_t* ins = reinterpret_cast<const uint32_t*>(head_h.data());
    const uint64_t* sum = head_h.data() + insb / 8;  // record entries, erased, inserted, ~time
    const uint32_t* fits = reinterpret_cast<const uint32_t*>(tail_h.data());
    const uint64_t* occ = tail_h.data() + insb / 8;
    rec.n = sum[0];
    rec.cur = b;
    rec.tmin = ~sum[3];
    rec.tmax = tmax;
    // tables without room, one at a time: their keys listed where the hash
    // table was
    bool listed = false;
    for (uint32_t i = 0; i < S; i++) {
        if (fits[i]) {
            index_note_occupied(c, i, occ[i]);
            continue;
        }
        listed = true;
        kv_zero_kernel<<<1, 64, 0, st>>>(reinterpret_cast<unsigned long long*>(o.sum), 1);
        kv_list_kernel<<<grid_for(ins[i], 256, 1024), kTileThreads, 0, st>>>(
            first, used, key, word, s, i, h.key, reinterpret_cast<unsigned long long*>(o.sum));
        if ((e = index_insert(c, i, h.key, ins[i])) != hipSuccess)
            return failed(e);
    }
    if (listed && (e = hipStreamSynchronize(st)) != hipSuccess)
        return failed(e);
    if (added) *added = sum[2];
    if (removed) *removed = sum[1];
    return DM_OK;
}

}  // namespace dm
