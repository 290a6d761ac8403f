// Per-instance cached-block index (the KV metadata of Sec. A.3.2): one
// open-addressing table of 2^k u64 keys per instance slot, probed a bucket
// of 8 slots (one 64-byte line) at a time, buckets in linear order from the
// key's home bucket.  Slot 0 = empty, 1 = erased; stored keys are >= 2.
// An insert takes the first empty slot of the probe sequence, so an empty
// slot seen during a lookup proves the key absent.
//
// Capacity: a table never holds more than 2^(k-1) occupied slots.  A
// workgroup reserves a unit of the occupied count per key that is not there
// before its threads claim empty slots and gives back what they did not use; when that is
// refused at the limit, each of its threads reserves a unit for itself before
// a claim and gives it back if the claim loses (another thread stored the
// same or a different key there).  A single reservation refused is not final,
// since reservations still in flight may be given back: the key goes to an
// overflow list, and once the insert kernel has finished a single wave
// settles the list in order (present already, stored while room is left,
// else dropped with DM_EFULL).  So a batch that fits is stored whole, and a
// batch that does not fills the table to exactly the limit.
#include <algorithm>
#include <vector>

#include "dm_internal.h"

namespace dm {
namespace {

constexpr int kPurgeSlot = kSlotPurge;  // table rebuild work area

struct TableRef {
    uint64_t* slots;
    uint64_t* live;      // live key count
    uint64_t* occupied;  // non-empty slots (live + erased)
    uint32_t log2slots;
    uint64_t limit;      // maximum occupied slots
};

// Overflow list: a count and the keys (room for every key of the batch).
struct Overflow {
    unsigned long long* count;
    uint64_t* keys;
};

// Insert of one canonical key (>= 2); set semantics.  With an overflow list,
// a key whose reservation is refused at the limit is appended to it;
// without one the key is dropped with kErrFull.
__device__ __forceinline__ void insert_one(const TableRef& t, uint64_t k, uint32_t* status,
                                           const Overflow* ovf)
{
    const uint64_t nbk = 1ull << (t.log2slots - 3);
    uint64_t b = home_bucket(k, t.log2slots);
    bool done = false;
    for (uint64_t step = 0; step < nbk && !done; step++, b = (b + 1) & (nbk - 1)) {
        for (uint32_t s = 0; s < kBucket && !done; s++) {
            uint64_t* slot = t.slots + b * kBucket + s;
            uint64_t v = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (v == k) {
                done = true;
            } else if (v == kEmpty) {
                const unsigned long long held =
                    atomicAdd((unsigned long long*)t.occupied, 1ull);
                if (held >= t.limit) {
                    atomicAdd((unsigned long long*)t.occupied, ~0ull);  // give back
                    if (ovf) {
                        const unsigned long long at = atomicAdd(ovf->count, 1ull);
                        ovf->keys[at] = k;
                    } else {
                        atomicOr(status, kErrFull);
                    }
                    return;
                }
                const unsigned long long prev = atomicCAS(
                    (unsigned long long*)slot, (unsigned long long)kEmpty, (unsigned long long)k);
                if (prev == kEmpty) {
                    atomicAdd((unsigned long long*)t.live, 1ull);
                    done = true;
                } else {
                    atomicAdd((unsigned long long*)t.occupied, ~0ull);  // claim lost
                    done = prev == k;  // else another key took the slot: keep walking
                }
            }
        }
    }
    if (!done)
        atomicOr(status, kErrFull);  // every slot scanned: table full
}

// Reserving per workgroup instead of per key took 32,768 keys into an empty
// 2^17-slot table from 54 us to 8.6 us: every key met the others on the two
// count words, where atomics take some 11 ns each.  So a workgroup reserves only
// for its keys that are not there (found before the claims, which go on from
// where the search stopped), and nothing where the host knows that there is room
// for all (ROOM): 1,048,576 keys that are all there, whole call 150 us with a
// reservation for each workgroup and 66 without.
template <bool ROOM>
__global__ __launch_bounds__(256) void insert_kernel(TableRef t, const uint64_t* __restrict__ keys,
                                                     uint64_t n, uint32_t* __restrict__ status,
                                                     Overflow ovf)
{
    __shared__ bool room;
    __shared__ uint32_t absent, stored;
    unsigned long long* const occupied = (unsigned long long*)t.occupied;
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < n;
         base += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = base + threadIdx.x;
        const uint64_t k = i < n ? canon_key(keys[i]) : kEmpty;
        if (threadIdx.x == 0)
            absent = stored = 0;
        __syncthreads();
        PutAt at{home_bucket(k, t.log2slots), 0, 0};
        Put p = i < n ? find_key(t.slots, t.log2slots, k, at) : Put::kThere;
        // a key that many lanes hold is left to one of them (whole wavefronts of one
        // key would meet on its slot: 65,536 copies 782 us instead of 50)
        uint64_t left = ballot(p != Put::kThere);
#pragma unroll
        for (int r = 0; r < 4 && left; r++) {
            const int lead = __builtin_ctzll(left);
            const uint64_t same = ballot(k == readlane_u64(k, lead)) & left;
            if ((same >> lane_id()) & 1 && lane_id() != lead)
                p = Put::kThere;
            left &= ~same;
        }
        const uint64_t m = ballot(p != Put::kThere);
        if (lane_id() == 0 && m)
            atomicAdd(&absent, (uint32_t)__popcll(m));
        __syncthreads();
        const unsigned long long want = absent;
        if (want == 0)
            continue;
        if (!ROOM) {
            if (threadIdx.x == 0) {
                room = atomicAdd(occupied, want) + want <= t.limit;
                if (!room)
                    atomicAdd(occupied, 0ull - want);  // give back
            }
            __syncthreads();
        }
        const bool grouped = ROOM || room;
        if (grouped) {
            if (p == Put::kStored)
                p = claim_key(t.slots, t.log2slots, k, at);
            if (p == Put::kNoRoom)
                atomicOr(status, kErrFull);
            const uint64_t s = ballot(p == Put::kStored);
            if (lane_id() == 0 && s)
                atomicAdd(&stored, (uint32_t)__popcll(s));
        } else if (p != Put::kThere) {
            insert_one(t, k, status, &ovf);
        }
        __syncthreads();
        if (grouped && threadIdx.x == 0) {
            const unsigned long long kept = stored, held = ROOM ? 0 : want;
            if (kept != held)
                atomicAdd(occupied, kept - held);  // give back, or add
            if (kept)
                atomicAdd((unsigned long long*)t.live, kept);
        }
    }
}

// Is canonical key k stored?  Walks k's probe sequence to its first empty slot.
__device__ bool contains(const TableRef& t, uint64_t k)
{
    const uint64_t nbk = 1ull << (t.log2slots - 3);
    uint64_t b = home_bucket(k, t.log2slots);
    for (uint64_t step = 0; step < nbk; step++, b = (b + 1) & (nbk - 1))
        for (uint32_t s = 0; s < kBucket; s++) {
            const uint64_t v = __hip_atomic_load(t.slots + b * kBucket + s, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
            if (v == k)
                return true;
            if (v == kEmpty)
                return false;
        }
    return false;
}

// The overflow list in list order, by one wave after the insert kernel:
// every lane looks up its key, then the absent ones are stored one lane
// at a time while the table has room; the rest are dropped with kErrFull.
// Nothing else writes the table meanwhile, so the counts are exact here.
__global__ void overflow_kernel(TableRef t, Overflow ovf, uint32_t* __restrict__ status)
{
    const int lane = lane_id();
    const uint64_t m = *ovf.count;
    for (uint64_t base = 0; base < m; base += kWave) {
        const uint64_t i = base + lane;
        const uint64_t k = i < m ? ovf.keys[i] : 0;
        bool need = i < m && !contains(t, k);
        if (!__any(need))
            continue;
        for (int j = 0; j < kWave; j++) {
            // lanes in order: an earlier lane may have stored the same key
            if (lane == j && need) {
                if (contains(t, k)) {
                    need = false;
                } else if (__hip_atomic_load(t.occupied, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT) >= t.limit) {
                    atomicOr(status, kErrFull);
                } else {
                    insert_one(t, k, status, nullptr);
                }
            }
            // the next lane sees this lane's store and counts
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "agent");
        }
    }
}

// Erased slots are never reused by inserts (an empty slot must keep proving
// absence), so churn fills a table with them.  Before an insert of n keys
// that could push the occupied count past the limit while erased slots
// exist, the table is rebuilt: live keys gathered, slots cleared, keys
// reinserted.  The decision is taken on the device (plan[0]); every kernel
// of the rebuild returns at once when it is not needed.
__global__ void purge_plan_kernel(TableRef t, uint64_t n, unsigned long long* plan)
{
    const uint64_t occ = *t.occupied, live = *t.live;
    plan[0] = (occ + n > t.limit && occ > live) ? 1ull : 0ull;
    plan[1] = 0;  // live keys gathered
    plan[2] = 0;  // overflow list length
}

__global__ void purge_gather_kernel(TableRef t, const unsigned long long* plan,
                                    unsigned long long* cnt, uint64_t* __restrict__ out)
{
    if (!plan[0])
        return;
    const uint64_t n = 1ull << t.log2slots;
    const uint64_t lt = (1ull << lane_id()) - 1;
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < n;
         base += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = base + threadIdx.x;
        const uint64_t v = i < n ? t.slots[i] : kEmpty;
        const bool keep = v != kEmpty && v != kTomb;
        const uint64_t m = ballot(keep);
        uint64_t first = 0;
        if (m && lane_id() == 0)
            first = atomicAdd(cnt, (unsigned long long)__popcll(m));
        first = readlane_u64(first, 0);
        // live <= occupied <= limit, the buffer's length; bounded all the same
        const uint64_t at = first + __popcll(m & lt);
        if (keep && at < t.limit)
            out[at] = v;
    }
}

__global__ void purge_clear_kernel(TableRef t, const unsigned long long* plan)
{
    if (!plan[0])
        return;
    const uint64_t n = 1ull << t.log2slots;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        t.slots[i] = kEmpty;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *t.live = 0;
        *t.occupied = 0;
    }
}

// The gathered keys into the cleared table (live <= limit: room for all).
__global__ __launch_bounds__(256) void purge_insert_kernel(
    TableRef t, const unsigned long long* plan, const uint64_t* __restrict__ keys,
    uint32_t* __restrict__ status)
{
    if (!plan[0])
        return;
    const uint64_t n = plan[1] < t.limit ? plan[1] : t.limit;
    unsigned long long mine = 0;  // keys stored by this wave
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < n;
         base += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = base + threadIdx.x;
        const Put p = i < n ? put_key(t.slots, t.log2slots, keys[i]) : Put::kThere;
        if (p == Put::kNoRoom)
            atomicOr(status, kErrFull);
        mine += __popcll(ballot(p == Put::kStored));
    }
    if (lane_id() == 0 && mine) {
        atomicAdd((unsigned long long*)t.occupied, mine);
        atomicAdd((unsigned long long*)t.live, mine);
    }
}

__global__ __launch_bounds__(256) void erase_kernel(TableRef t, const uint64_t* __restrict__ keys,
                                                    uint64_t n)
{
    unsigned long long mine = 0;  // keys erased by this wave
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < n;
         base += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = base + threadIdx.x;
        mine += __popcll(ballot(i < n && take_key(t.slots, t.log2slots, canon_key(keys[i]))));
    }
    if (lane_id() == 0 && mine)
        atomicAdd((unsigned long long*)t.live, 0ull - mine);
}

__global__ void clear_kernel(uint64_t* __restrict__ slots, uint64_t n, uint64_t* live,
                             uint64_t* occupied)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        slots[i] = kEmpty;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *live = 0;
        *occupied = 0;
    }
}

// Tables of several instances emptied at once: grid row y clears table
// ids[y] (and its counts).
__global__ void clear_many_kernel(uint64_t* __restrict__ tables, uint32_t log2slots,
                                  const uint32_t* __restrict__ ids, uint64_t* __restrict__ counts,
                                  uint32_t S)
{
    const uint32_t id = ids[blockIdx.y];
    uint64_t* slots = tables + ((uint64_t)id << log2slots);
    const uint64_t n = 1ull << log2slots;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        slots[i] = kEmpty;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        counts[id] = 0;      // live keys
        counts[S + id] = 0;  // occupied slots
    }
}

TableRef table_of(dm_ctx* c, uint32_t id)
{
    const uint32_t k = c->cfg.index_log2_slots;
    return TableRef{c->d_tables + ((uint64_t)id << k), c->d_counts + id,
                    c->d_counts + c->cfg.max_slots + id, k, 1ull << (k - 1)};
}


}  // namespace

// Whether n more keys certainly fit instance id's table, from the host's
// bound on its occupied slots (keys sent to it since it was last empty; the
// bound grows by n).  A captured insert or clear runs whenever its graph is
// replayed, which the host does not see: the bound is then given up for good.
static bool surely_fits(dm_ctx* c, uint32_t id, uint64_t n)
{
    uint64_t& bound = c->occ_bound[id];
    if (stream_capturing(c))
        bound = UINT64_MAX;
    if (bound == UINT64_MAX)
        return false;
    const uint64_t limit = 1ull << (c->cfg.index_log2_slots - 1);
    const bool fits = n <= limit && bound <= limit - n;
    bound = fits ? bound + n : limit;  // a table never holds more
    return fits;
}

static void note_cleared(dm_ctx* c, uint32_t id)
{
    if (stream_capturing(c))
        c->occ_bound[id] = UINT64_MAX;
    if (c->occ_bound[id] != UINT64_MAX)
        c->occ_bound[id] = 0;
}

hipError_t index_insert(dm_ctx* c, uint32_t id, const uint64_t* keys, uint64_t n)
{
    const TableRef t = table_of(c, id);
    // Room for every key whatever they are: one launch (neither a rebuild
    // nor an overflow list can be needed) instead of six.
    if (surely_fits(c, id, n)) {
        if (n)
            insert_kernel<true><<<grid_for(n, 256), 256, 0, c->stream>>>(
                t, keys, n, c->d_status, Overflow{nullptr, nullptr});
        return hipGetLastError();
    }
    hipError_t e = hipSuccess;
    // work area: plan word, gather count, overflow count, then up to `limit`
    // gathered live keys, then up to n overflow keys
    unsigned long long* w = static_cast<unsigned long long*>(
        scratch_get(c, kPurgeSlot, (t.limit + n + 3) * sizeof(uint64_t), &e));
    if (!w)
        return e;
    uint64_t* gathered = reinterpret_cast<uint64_t*>(w + 3);
    const Overflow ovf{w + 2, gathered + t.limit};
    const uint64_t nslots = 1ull << t.log2slots;
    purge_plan_kernel<<<1, 1, 0, c->stream>>>(t, n, w);
    purge_gather_kernel<<<grid_for(nslots, 256, 4096), 256, 0, c->stream>>>(t, w, w + 1, gathered);
    purge_clear_kernel<<<grid_for(nslots, 256, 4096), 256, 0, c->stream>>>(t, w);
    purge_insert_kernel<<<grid_for(t.limit, 256, 4096), 256, 0, c->stream>>>(t, w, gathered,
                                                                            c->d_status);
    insert_kernel<false><<<grid_for(n, 256), 256, 0, c->stream>>>(t, keys, n, c->d_status, ovf);
    overflow_kernel<<<1, kWave, 0, c->stream>>>(t, ovf, c->d_status);
    return hipGetLastError();
}

hipError_t index_erase(dm_ctx* c, uint32_t id, const uint64_t* keys, uint64_t n)
{
    erase_kernel<<<grid_for(n, 256), 256, 0, c->stream>>>(table_of(c, id), keys, n);
    return hipGetLastError();
}

// The host's bound after another kernel's inserts: the table's occupied
// slots as read back (unless the bound was given up).
void index_note_occupied(dm_ctx* c, uint32_t id, uint64_t occupied)
{
    if (c->occ_bound[id] != UINT64_MAX)
        c->occ_bound[id] = occupied;
}

hipError_t index_clear_many(dm_ctx* c, const uint32_t* ids_host, uint32_t n)
{
    if (n == 0)
        return hipSuccess;
    hipError_t e = hipSuccess;
    uint32_t* d = static_cast<uint32_t*>(scratch_get(c, kPurgeSlot, n * sizeof(uint32_t), &e));
    if (!d)
        return e;
    if ((e = hipMemcpyAsync(d, ids_host, n * sizeof(uint32_t), hipMemcpyHostToDevice,
                            c->stream)) != hipSuccess ||
        (e = hipStreamSynchronize(c->stream)) != hipSuccess)
        return e;
    for (uint32_t i = 0; i < n; i++)
        note_cleared(c, ids_host[i]);
    const uint32_t k = c->cfg.index_log2_slots;
    const uint64_t per = std::max<uint64_t>(1, 4096 / n);
    dim3 grid((uint32_t)std::min<uint64_t>(per, ((1ull << k) + 255) / 256), n);
    clear_many_kernel<<<grid, 256, 0, c->stream>>>(c->d_tables, k, d, c->d_counts,
                                                   c->cfg.max_slots);
    return hipGetLastError();
}

hipError_t index_clear(dm_ctx* c, uint32_t id)
{
    const TableRef t = table_of(c, id);
    const uint64_t n = 1ull << t.log2slots;
    note_cleared(c, id);
    clear_kernel<<<grid_for(n, 256, 4096), 256, 0, c->stream>>>(t.slots, n, t.live, t.occupied);
    return hipGetLastError();
}

}  // namespace dm
