// One radix pass over a tile of up to 4096 (key, value) pairs by a workgroup of
// 1024 threads, in LDS: the tile sorts of dm_sort.hip and the small batches'
// grouping of dm_probe.hip.
#pragma once
#include "dm_internal.h"

namespace dm {
namespace {

constexpr int kWideThreads = 1024, kWideWaves = kWideThreads / kWave, kWideItems = 4;
constexpr uint64_t kOneSort = (uint64_t)kWideThreads * kWideItems;  // one tile

// LDS of one tile's ordering by one digit.
struct WideTile {
    uint64_t sk[kOneSort];
    uint32_t sv[kOneSort];
    uint32_t wcnt[2][kWideWaves][256];  // as in digit_scatter_kernel
    uint32_t run[256], dbase[256], wsum[4];
};

// Orders the tile's tn items (k, v: item it * 1024 + t) by the digit at shift
// into sk / sv; run[d] = items of digit d, dbase[d] = its first place.
template <int ITEMS>
__device__ __forceinline__ void order_tile(WideTile& L, const uint64_t (&k)[kWideItems],
                                           const uint32_t (&v)[kWideItems], uint32_t tn, int shift,
                                           bool vals)
{
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    uint32_t rk[ITEMS];
    if (t < 256)
        L.run[t] = 0;
    for (int q = t; q < 2 * kWideWaves * 256; q += kWideThreads)
        (&L.wcnt[0][0][0])[q] = 0xFFFFFFFFu;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; it++) {
        const bool ok = (uint32_t)(it * kWideThreads + t) < tn;
        const uint32_t d = (uint32_t)((k[it] >> shift) & 0xFF);
        uint64_t peers = ballot(ok);
#pragma unroll
        for (int b = 0; b < 8; b++) {
            const bool bit = (d >> b) & 1;
            const uint64_t m = ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t pr = __popcll(peers & lt);
        const int buf = it & 1;
        if (ok && pr == 0)
            L.wcnt[buf][w][d] = (uint32_t)__popcll(peers) | ((uint32_t)it << 16);
        __syncthreads();
        if (t < 256) {
            uint32_t r = L.run[t];
#pragma unroll
            for (int ww = 0; ww < kWideWaves; ww++) {
                const uint32_t x = L.wcnt[buf][ww][t];
                const uint32_t c = (x >> 16) == (uint32_t)it ? (x & 0xFFFFu) : 0u;
                L.wcnt[buf][ww][t] = r | ((uint32_t)it << 16);
                r += c;
            }
            L.run[t] = r;
        }
        __syncthreads();
        rk[it] = ok ? (L.wcnt[buf][w][d] & 0xFFFFu) + pr : 0;
    }
    // first place of each digit in the tile (exclusive scan over digits)
    uint32_t x = t < 256 ? L.run[t] : 0;
#pragma unroll
    for (int dlt = 1; dlt < kWave; dlt <<= 1) {
        const uint32_t y = __shfl_up(x, dlt);
        if (lane >= dlt)
            x += y;
    }
    if (t < 256 && lane == kWave - 1)
        L.wsum[w] = x;
    __syncthreads();
    if (t < 256) {
        for (int ww = 0; ww < w; ww++)
            x += L.wsum[ww];
        L.dbase[t] = x - L.run[t];
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; it++)
        if ((uint32_t)(it * kWideThreads + t) < tn) {
            const uint32_t at = L.dbase[(k[it] >> shift) & 0xFF] + rk[it];
            L.sk[at] = k[it];
            if (vals)
                L.sv[at] = v[it];
        }
    __syncthreads();
}

}  // namespace
}  // namespace dm
