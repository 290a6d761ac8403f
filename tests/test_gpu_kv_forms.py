"""KV saves against a plain model (a dict of times per instance): touched keys
that repeat within and across requests, key 0, caps above and below, times
over a wide range (several digits of the select), a clock that is not advanced
(equal times: the smaller key goes first), many slots, tables that need their
rebuild, and a cleared instance."""
import numpy as np
import pytest

import workloads
from test_gpu_index_forms import _dev, _held

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _save(model, off, keys, inst, clock, cap, B):
    nf = np.diff(off) // B
    start, added, removed = 0, 0, 0
    before = {c: set(m) for c, m in model.items()}
    for r, f in enumerate(nf):
        m = model.setdefault(int(inst[r]), {})
        for b in range(int(f)):
            k, t = int(keys[start + b]), clock + start + int(f) - 1 - b
            m[k] = max(m.get(k, -1), t)
        start += int(f)
    for c, m in model.items():
        if cap and len(m) > cap:
            for t, k in sorted((t, k) for k, t in m.items())[:len(m) - cap]:
                del m[k]
        old = before.get(c, set())
        added += len(set(m) - old)
        removed += len(old - set(m))
    return added, removed


@pytest.mark.parametrize("slots,log2,steps", [
    (5, 10, [(0, 0), (300, 1), (300, 1), (120, 1), (0, 1)]),          # unbounded, evicting, lower cap
    (5, 10, [(200, 0), (200, 0), (200, 0), (90, 0)]),                 # clock not advanced: ties
    (3, 12, [(700, 1 << 16), (700, 1 << 28), (700, 1 << 39), (5, 1)]),  # times up to 40 bits
    (300, 8, [(40, 1), (40, 1), (3, 1), (40, 1)]),                    # many regions
    (2, 8, [(128, 1), (128, 1), (128, 1), (128, 1), (128, 1)]),       # full tables: rebuilt each time
    (4000, 4, [(8, 1), (2, 1)]),
])
def test_kv_save_matches_lru_dicts(slots, log2, steps):
    import paper_2602_06502_amd as pk
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B = 16
    cfg = dict(workloads.small_random(5, 3, 2, B, 10).route.as_dict(), max_slots=slots, index_log2_slots=log2)
    eng = pk.DualMap(cfg, device="cuda:0")
    eng.build_rings(range(slots))
    rng = np.random.default_rng(slots + len(steps))
    model, clock = {}, 0
    seen = np.zeros(1, np.uint64)
    for i, (cap, ahead) in enumerate(steps):
        n = 60 + 37 * i
        off = np.zeros(n + 1, np.int64)
        off[1:] = np.cumsum(rng.integers(0, 12 * B, size=n))
        nb = int((np.diff(off) // B).sum())
        # popular keys, fresh ones, earlier ones, key 0
        pool = rng.integers(0, 2**64, size=400, dtype=np.uint64)
        keys = np.where(rng.random(nb) < 0.5, pool[rng.integers(0, 40, nb)], pool[rng.integers(0, 400, nb)])
        keys = np.where(rng.random(nb) < 0.2, seen[rng.integers(0, len(seen), nb)], keys).astype(np.uint64)
        inst = rng.integers(0, max(1, slots if i % 2 == 0 else slots // 2), size=n).astype(np.uint32)
        print("[case]", slots, log2, i, "cap", cap, "clock", clock, "blocks", nb, flush=True)
        got = eng.kv_save(_dev(off), _dev(keys), _dev(inst), clock, cap)
        eng.sync()
        assert got == _save(model, off, keys, inst, clock, cap, B), i
        seen = np.unique(np.concatenate([seen, keys]))
        for c in range(0, slots, max(1, slots // 7)):
            assert eng.index_size(c) == len(model.get(c, {})), (i, c)
            held = _held(eng, c, seen)
            assert set(seen[held].tolist()) == set(model.get(c, {})), (i, c)
        clock += nb * min(ahead, 1) + (ahead if ahead > 1 else 0)
        if i == 1:
            eng.index_clear(1)
            model.pop(1, None)


def test_many_equal_times_at_the_cut():
    """More entries of one time than a workgroup has threads: lower caps drop
    the smallest keys first."""
    import paper_2602_06502_amd as pk
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B, saves = 16, 1300
    cfg = dict(workloads.small_random(5, 2, 2, B, 10).route.as_dict(), max_slots=3, index_log2_slots=13)
    eng = pk.DualMap(cfg, device="cuda:0")
    eng.build_rings(range(2))
    rng = np.random.default_rng(3)
    keys = rng.integers(2, 2**63, size=(saves, 2), dtype=np.uint64)
    keys[5, 0], keys[6, 0], keys[7, 1] = 0, 2**64 - 1, 0
    keys[100:160, 0] = keys[100, 0] + np.arange(60, dtype=np.uint64)  # alike but for the last digit
    off, inst = np.array([0, B, 2 * B], np.int64), np.array([0, 1], np.uint32)
    od, idd, kd = _dev(off), _dev(inst), _dev(keys.reshape(-1))
    model = {}
    print("[case] equal times", flush=True)
    for i in range(saves):
        eng.kv_save(od, kd[2 * i:2 * i + 2].contiguous(), idd, 7, 0)
        _save(model, off, keys[i], inst, 7, 0, B)
    seen = np.unique(keys)
    for cap in (1200, 1199, 500, 129, 2, 1):
        print("[case] cap", cap, flush=True)
        got = eng.kv_save(od[:1].contiguous(), kd[:1].contiguous(), idd[:1].contiguous(), 7, cap)
        eng.sync()
        assert got == _save(model, off[:1], keys[0][:0], inst[:0], 7, cap, B), cap
        for c in (0, 1):
            assert set(seen[_held(eng, c, seen)].tolist()) == set(model[c]), (cap, c)


def _median_us(f, reps=7):
    import time
    t = []
    for i in range(reps + 2):
        torch.cuda.synchronize()
        a = time.perf_counter()
        f()
        torch.cuda.synchronize()
        t.append((time.perf_counter() - a) * 1e6)
    return sorted(t[2:])[reps // 2]


def test_equal_times_cost_little():
    """65,536 blocks an instance over a cap of as many and one: the clock not
    advanced (the cut falls between two entries of one time) against advanced.
    One read of the entries more, not one for each bit of a key (8.8 times)."""
    import paper_2602_06502_amd as pk
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S, per, B = 4, 65_536, 16
    cfg = dict(workloads.small_random(5, S, 2, B, 10).route.as_dict(), index_log2_slots=20)
    n = S * 256
    off = torch.arange(n + 1, dtype=torch.int64, device="cuda:0") * (B * (per // 256))
    inst = (torch.arange(n, device="cuda:0") % S).to(torch.int32).view(torch.uint32)
    us = {}
    for ahead in (0, 1):
        eng = pk.DualMap(cfg, device="cuda:0")
        eng.build_rings(range(S))
        g, clock = torch.Generator(device="cuda:0").manual_seed(5), [0]
        batch = [torch.randint(-2**63, 2**63 - 1, (S * per,), dtype=torch.int64, device="cuda:0", generator=g).view(torch.uint64)
                 for _ in range(3)]

        def save():
            batch.insert(0, batch.pop())  # other keys every time
            eng.kv_save(off, batch[0], inst, clock[0], per + 1)
            clock[0] += ahead * S * per
        print("[case] ahead", ahead, flush=True)
        us[ahead] = _median_us(save)
    print(us)
    assert us[0] < 3 * us[1], us


def _saves(S, per, blocks, old, reps=7):
    """Median time of saving `per` fresh blocks on each of S instances over a
    cap of as many, in requests of `blocks`, with or without an old entry on
    one more instance."""
    import paper_2602_06502_amd as pk
    B = 16
    cfg = dict(workloads.small_random(5, S + 1, 2, B, 10).route.as_dict(), index_log2_slots=20)
    eng = pk.DualMap(cfg, device="cuda:0")
    eng.build_rings(range(S + 1))
    n = S * (per // blocks)
    off = torch.arange(n + 1, dtype=torch.int64, device="cuda:0") * (B * blocks)
    inst = (torch.arange(n, device="cuda:0") % S).to(torch.int32).view(torch.uint32)
    g, clock = torch.Generator(device="cuda:0").manual_seed(5), [0]
    batch = [torch.randint(-2**63, 2**63 - 1, (n * blocks,), dtype=torch.int64, device="cuda:0", generator=g)
             .view(torch.uint64) for _ in range(3)]
    if old:
        eng.kv_save(off[:2] // blocks, batch[0][:1].contiguous(), (inst[:1].to(torch.int32) + S).view(torch.uint32), 0, per)
        clock[0] = 1 << 38

    def save():
        batch.insert(0, batch.pop())
        eng.kv_save(off, batch[0], inst, clock[0], per)
        clock[0] += n * blocks
    print("[case] saves", S, per, blocks, old, flush=True)
    us = _median_us(save, reps)
    print(us)
    return us


def test_long_requests_cost_little():
    """As many blocks in 16 requests as in 2,048 (5 times the time with a wave
    for each request)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert _saves(2, 1 << 18, 1 << 15, False) < 2.5 * _saves(2, 1 << 18, 256, False)


@pytest.mark.parametrize("log2", [10, 13])
def test_times_far_apart(log2):
    """Every digit of the select with many entries and with few: an idle
    instance's old entry, then batches long after it, then spread ones."""
    import paper_2602_06502_amd as pk
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S, B = 3, 16
    cfg = dict(workloads.small_random(5, S, 2, B, 10).route.as_dict(), max_slots=S, index_log2_slots=log2)
    eng = pk.DualMap(cfg, device="cuda:0")
    eng.build_rings(range(S))
    rng = np.random.default_rng(log2)
    cap, model, seen = 1 << (log2 - 2), {}, np.zeros(0, np.uint64)
    clock = 0
    for i, (n, ahead) in enumerate([(1, 1 << 38), (700, 0), (700, 1 << 12), (700, 1 << 20), (700, 1 << 24), (3, 1),
                                    (700, 1 << 30), (40, 1 << 33), (700, 1)]):
        f = rng.integers(1, 2 if n == 1 else 12, size=n)
        off = np.zeros(n + 1, np.int64)
        off[1:] = np.cumsum(f) * B
        keys = rng.integers(2, 2**63, size=int(f.sum()), dtype=np.uint64)
        inst = np.full(n, 2, np.uint32) if n == 1 else rng.integers(0, 2, size=n).astype(np.uint32)
        print("[case] far", log2, i, n, clock, flush=True)
        got = eng.kv_save(_dev(off), _dev(keys), _dev(inst), clock, cap)
        eng.sync()
        assert got == _save(model, off, keys, inst, clock, cap, B), i
        seen = np.concatenate([seen, keys])
        for c in range(S):
            assert set(seen[_held(eng, c, seen)].tolist()) == set(model.get(c, {})), (i, c)
        clock += len(keys) + ahead


def test_an_old_entry_costs_little():
    """An idle instance's old entry makes all other times share their leading
    digits (12 times the time with the counts straight to memory)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert _saves(1, 1 << 19, 256, True) < 2.5 * _saves(1, 1 << 19, 256, False)


@pytest.mark.parametrize("cap", [0, 3000])
def test_requests_in_parts(cap):
    """Requests around the number of blocks that one wave touches (512) and its
    multiples, among short ones, with keys that they share."""
    import paper_2602_06502_amd as pk
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S, B = 3, 16
    cfg = dict(workloads.small_random(5, S, 2, B, 10).route.as_dict(), max_slots=S, index_log2_slots=16)
    eng = pk.DualMap(cfg, device="cuda:0")
    eng.build_rings(range(S))
    rng = np.random.default_rng(cap + 1)
    pool = rng.integers(2, 2**63, size=9000, dtype=np.uint64)
    model, clock = {}, 0
    for i in range(3):
        f = np.array([511, 512, 513, 0, 1, 1023, 1024, 1025, 1535, 1536, 1537, 3, 2600], np.int64)[rng.permutation(13)]
        off = np.zeros(14, np.int64)
        off[1:] = np.cumsum(f) * B
        keys = np.concatenate([pool[int(rng.integers(0, 6000)):][:k] for k in f])
        inst = rng.integers(0, S, size=13).astype(np.uint32)
        print("[case] parts", cap, i, f.tolist(), flush=True)
        got = eng.kv_save(_dev(off), _dev(keys), _dev(inst), clock, cap)
        eng.sync()
        assert got == _save(model, off, keys, inst, clock, cap, B), i
        for c in range(S):
            held = _held(eng, c, pool)
            assert set(pool[held].tolist()) == set(model.get(c, {})), (i, c)
        clock += len(keys)
