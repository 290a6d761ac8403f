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
