// dm_route_batch: batched dual-mapping routing (Sec. 3.2; Sec. A.1.1).
//
//   block_starts   exclusive sum of full blocks per request: where each
//                  request's block keys go; checks the offsets;
//   hash_prefix    both ring keys from the first min(K, full blocks)
//                  blocks, and the candidates on the two rings
//                  (dm_hash.hip);
//   group_requests requests ordered by their first ring key and grouped by
//                  equal ring keys, with a leader per group (dm_probe.hip);
//   hash_leaders   leaders' full chains and longest cached prefixes;
//   hash_members   every other request's full chain and longest cached
//                  prefix, from its leader's keys and its own probes;
//   select_*       SLO-aware choice in request order, loads updated
//                  (dm_select.hip).
// With timing on, events between the stages give the per-stage times that
// dm_route_stage_ms reports.  With pipelining on, the batch's work runs on
// the context's work stream (after the caller's stream and after the batch
// two back), its serial selection on the selection stream (after the
// batch's record packing and the previous selection), and the output
// epilogue on the output stream; the next batch's hashing and probing thus
// overlap this batch's selection.  Unpipelined, a large batch overlaps with
// itself (see kSplitTokens): the selection of its first requests runs beside
// the hashing of the rest.
#include "dm_internal.h"

namespace dm {
namespace {

constexpr int kKeySlot = kSlotKeys;  // block keys when the caller keeps none

// An unpipelined batch of at least kSplitTokens tokens and kSplitFrom requests
// is selected in two parts: the walk of the first, one wave on one
// SIMD, runs on a side stream beside the hashing of the second.  The walk
// claims a whole SIMD's registers, so it starts only on an empty one: its
// records are ready before the second part's member records are written, and
// in the gap between that kernel and the hashing it finds one.  A first part
// of a quarter walks about as long as the rest hashes (a fifth and three
// tenths measured 2 and 1% longer).  The second set of packing kernels and the
// two streams' events cost 40 to 70 us, so both lines are needed: a walk whose
// quarter is worth that, and hashing to run it beside.  In one part and in two
// (us):
//   200 M tokens            128 instances   8              1,000
//   8,192 requests          369    430      586    641     402    471
//   32,768                  512    554      1,332  1,338   533    606
//   65,536                  717    718
//   66,000                  788    730      2,462  2,351   806    742
//   100,000 (305 M)         1,069  982      3,571  3,325   1,073  1,005
//   262,144                 3,495  3,326    7,565  7,381   1,930  1,769
// and with more tokens 262,144 (438 M) 2,030 and 1,800, 1,048,576 (1.75 G) 7,580
// and 6,510, 131,072 with the hotness tree (219 M) 2,550 and 2,490; with fewer,
// 65,536 (109 M) 610 and 670.
}  // namespace

namespace {

uint32_t block_shift_of(const dm_ctx* c)
{
    uint32_t k = 0;
    while ((1u << k) < c->cfg.block_size)
        k++;
    return k;
}

// Block starts [n + 1] and the malformed-offsets word, 256-byte aligned.
uint64_t starts_bytes(uint64_t n) { return ((n + 2) * sizeof(uint64_t) + 255) & ~255ull; }

// The f1 digests the prefix pass keeps for the members pass: K per request,
// when K is small enough that they cost less than a fraction of the tokens
// they replace (always at K <= 16).
uint64_t nh0_bytes(const dm_ctx* c, uint64_t n)
{
    return c->cfg.key_blocks <= 16 ? n * c->cfg.key_blocks * sizeof(uint64_t) : 0;
}

// Routes launches of the helper stages to another stream for one call.
struct StreamSwap {
    dm_ctx* c;
    hipStream_t saved;
    StreamSwap(dm_ctx* ctx, hipStream_t s) : c(ctx), saved(ctx->stream) { c->stream = s; }
    ~StreamSwap() { c->stream = saved; }
};

}  // namespace

void route_scratch_plan(const dm_ctx* c, uint64_t n, uint64_t n_tokens, bool keys_in_scratch,
                        size_t* bytes)
{
    for (int i = 0; i < kScratchSlots; i++)
        bytes[i] = 0;
    // block starts, malformed-offsets word, the first blocks' f1 digests
    bytes[kSlotStarts] = starts_bytes(n) + nh0_bytes(c, n);
    bytes[kSlotProbe] = probe_scratch_bytes(n);       // request order and groups
    bytes[kSlotMembers] = member_scratch_bytes(n);    // members pass records, kept keys
    bytes[kSlotSelect] = select_scratch_bytes(n);     // one set of selection work arrays
    if (keys_in_scratch)                              // block keys
        bytes[kSlotKeys] = ((n_tokens >> block_shift_of(c)) + 1) * sizeof(uint64_t);
    bytes[kSlotSort] = sort_scratch_bytes(n);         // digit counts of the ordering sort
    const uint64_t s1 = scan_scratch_bytes(n), s2 = scan_scratch_bytes(sort_scan_len(n));
    bytes[kSlotScan] = s1 > s2 ? s1 : s2;             // tile sums of both kinds of scan
    if (c->kl.on)  // marks of requests going down the tree; the window record's offsets
        bytes[kSlotRebalance] = ((ext_words(c, n) * sizeof(uint64_t) + 255) & ~255ull) +
                                keylen_record_bytes(n);
}

static hipError_t route_parts(dm_ctx* c, const int32_t* tokens, uint64_t n_tokens,
                              const int64_t* offsets, uint64_t n, int64_t* loads,
                              const dm_route_out* out, bool split)
{
    hipError_t e = hipSuccess;
    const bool pipe = c->pipelined;
    const int par = pipe ? (int)(c->batches & 1) : 0;
    SelParts ps;
    select_parts(n, pipe, split ? 2 : 1, &ps);
    if (pipe) {
        if ((e = hipEventRecord(c->in_ready, c->stream)) != hipSuccess ||
            (e = hipStreamWaitEvent(c->work_stream, c->in_ready, 0)) != hipSuccess)
            return e;
        // outputs and work arrays two batches back may be this batch's
        if (c->batches >= 2 &&
            (e = hipStreamWaitEvent(c->work_stream, c->out_done[par], 0)) != hipSuccess)
            return e;
    }
    StreamSwap swap(c, pipe ? c->work_stream : c->stream);
    hipStream_t st = c->stream;
    hipEvent_t* ev = nullptr;
    if (c->timing) {
        ev = &c->tev[(c->tcount % dm_ctx::kTimingRing) * 5];
        c->tcount++;
    }
    if (ev && (e = hipEventRecord(ev[0], st)) != hipSuccess)
        return e;
    // block starts [n + 1], then the malformed-offsets word, then the f1
    // digests of every request's first min(K, full blocks) blocks
    uint64_t* bstart = static_cast<uint64_t*>(
        scratch_get(c, kSlotStarts, starts_bytes(n) + nh0_bytes(c, n), &e));
    if (!bstart)
        return e;
    uint32_t* bad = reinterpret_cast<uint32_t*>(bstart + n + 1);
    uint64_t* nh0 = nh0_bytes(c, n) ? reinterpret_cast<uint64_t*>(
                                          reinterpret_cast<uint8_t*>(bstart) + starts_bytes(n))
                                    : nullptr;
    // with the hotness tree: marks of the requests going down the tree
    uint64_t* ext = nullptr;
    uint64_t* kl_work = nullptr;
    if (c->kl.on) {
        const uint64_t ext_bytes = (ext_words(c, n) * sizeof(uint64_t) + 255) & ~255ull;
        uint8_t* w = static_cast<uint8_t*>(
            scratch_get(c, kSlotRebalance, ext_bytes + keylen_record_bytes(n), &e));
        if (!w)
            return e;
        ext = reinterpret_cast<uint64_t*>(w);
        kl_work = reinterpret_cast<uint64_t*>(w + ext_bytes);
    }
    BatchClear clear{{}, c->n_live};
    for (int k = 0; k < ps.count; k++)
        if ((e = select_growth(c, ps, k, par, &clear.grow[k])) != hipSuccess)
            return e;
    if ((e = block_starts(c, offsets, n, n_tokens, bstart, bad, clear)) != hipSuccess)
        return e;
    uint64_t* hkeys = out->block_keys;
    // the hotness tree's window records every request's block keys
    const bool write_keys = out->block_keys != nullptr || c->kl.on;
    if (!hkeys) {
        // Requests that pass the offsets check are disjoint ranges of the
        // token array, so they hold at most n_tokens / B full blocks: the
        // scratch is sized without reading the batch's block count back.
        const uint64_t cap = (n_tokens >> block_shift_of(c)) + 1;
        hkeys = static_cast<uint64_t*>(scratch_get(c, kKeySlot, cap * sizeof(uint64_t), &e));
        if (!hkeys)
            return e;
    }
    if (ev && (e = hipEventRecord(ev[1], st)) != hipSuccess)
        return e;
    GroupView gv{};
    LookupArgs look{};
    if ((e = lookup_args(c, n, out->cand, out->flags, &look)) != hipSuccess ||
        (e = hash_prefix(c, tokens, offsets, n, bad, out->key, out->key_len, ext, nh0,
                         c->kl.on ? nullptr : &look)) != hipSuccess)
        return e;
    if (c->kl.on && ((e = hash_extend(c, tokens, offsets, n, bad, out->key, out->key_len,
                                      ext)) != hipSuccess ||
                     (e = lookup_candidates(c, n, out->key, look)) != hipSuccess))
        return e;
    if ((e = group_requests(c, n, bstart, bad, &gv)) != hipSuccess)
        return e;
    if (ev && (e = hipEventRecord(ev[2], st)) != hipSuccess)
        return e;
    if ((e = hash_leaders(c, tokens, offsets, n, bstart, bad, gv, out->cand, hkeys, out->match)) !=
        hipSuccess)
        return e;
    auto order = [&](hipStream_t waits, hipEvent_t event, hipStream_t on) -> hipError_t {
        if (waits == on)
            return hipSuccess;
        const hipError_t r = hipEventRecord(event, on);
        return r != hipSuccess ? r : hipStreamWaitEvent(waits, event, 0);
    };
    for (int k = 0; k < ps.count; k++) {
        const SelPart& q = ps.part[k];
        const bool last = k + 1 == ps.count;
        if ((e = hash_members(c, tokens, offsets, n, q.r0, q.m, k, bstart, bad, gv, out->cand,
                              hkeys, write_keys, out->match, nh0)) != hipSuccess)
            return e;
        if (last && c->kl.on) {
            if ((e = keylen_record(c, n, bstart, hkeys, kl_work)) != hipSuccess)
                return e;
            c->kl.win += n;
        }
        if (last && ev && (e = hipEventRecord(ev[3], st)) != hipSuccess)
            return e;
        if ((e = select_prepare(c, st, offsets, n, out, ps, k, par)) != hipSuccess)
            return e;
        // the walks in order: a first part's on the side stream, the last
        // part's after it (pipelined: all on the selection stream)
        const hipStream_t ss = pipe ? c->sel_stream : last ? st : c->side_stream;
        if ((e = order(ss, c->prep_done, st)) != hipSuccess ||
            (split && last && (e = order(st, c->sel_done, c->side_stream)) != hipSuccess) ||
            (e = select_walk(c, ss, offsets, n, out, loads, ps, k, par)) != hipSuccess)
            return e;
    }
    const hipStream_t os = pipe ? c->out_stream : st;
    if (pipe && (e = order(os, c->sel_done, c->sel_stream)) != hipSuccess)
        return e;
    for (int k = 0; k < ps.count; k++)
        if ((e = select_output(c, os, offsets, n, out, ps, k, par)) != hipSuccess)
            return e;
    if (pipe) {
        if ((e = hipEventRecord(c->out_done[par], os)) != hipSuccess)
            return e;
        c->batches++;
    }
    return ev ? hipEventRecord(ev[4], os) : hipSuccess;
}

hipError_t route(dm_ctx* c, const int32_t* tokens, uint64_t n_tokens, const int64_t* offsets,
                 uint64_t n, int64_t* loads, const dm_route_out* out)
{
    const bool split = !c->pipelined && !c->arena.on && n_tokens >= kSplitTokens &&
                       n >= kSplitFrom && !stream_capturing(c);
    hipError_t e = split ? make_side_stream(c) : hipSuccess;
    if (e == hipSuccess)
        e = route_parts(c, tokens, n_tokens, offsets, n, loads, out, split);
    if (split && e != hipSuccess)
        (void)sync_streams(c);  // nothing stays running behind the caller's stream
    return e;
}

}  // namespace dm
