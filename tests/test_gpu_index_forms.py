"""Index inserts by the form they take: with room whatever the keys are (one
kernel), and without (rebuild, reservations, overflow list), each against a
set model."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _engine(log2):
    import paper_2602_06502_amd as pk
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = workloads.small_random(5, 3, 2, 16, 10)
    cfg = dict(wl.route.as_dict(), index_log2_slots=log2)
    eng = pk.DualMap(cfg, device="cuda:0")
    eng.build_rings(range(3))
    return eng, pk


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _held(eng, inst, keys):
    """Which keys instance inst's index holds, by pricing one queued record per
    key (its chain that key, 16 tokens) on it."""
    n = len(keys)
    S = eng.max_slots
    qoff = np.zeros(S + 1, np.int64)
    qoff[inst + 1:] = n
    z = lambda t: _dev(np.zeros(n, t))
    q = (_dev(qoff), _dev(np.arange(n, dtype=np.uint64)), z(np.uint32), z(np.uint32), z(np.uint32),
         _dev(np.zeros(S, np.int64)))
    out = eng.queue_reprobe(q, _dev(np.arange(n + 1, dtype=np.int64)), _dev(keys),
                            _dev(np.full(n, 16, np.int64)))
    return out[2].cpu().numpy() == 0


@pytest.mark.parametrize("log2,sizes", [(4, (1, 3, 4)), (10, (255, 256, 1)), (10, (257, 200, 400)),
                                        (12, (2048,)), (12, (1500, 500, 400)), (16, (20_000, 12_768))])
def test_inserts_up_to_and_past_the_limit(log2, sizes):
    eng, pk = _engine(log2)
    rng = np.random.default_rng(log2 + len(sizes))
    limit = 1 << (log2 - 1)
    have, sent = set(), []
    for n in sizes:
        keys = rng.integers(0, 2**64, size=n, dtype=np.uint64)
        keys[::7] = keys[0]  # repeated within a batch and across workgroups
        eng.index_insert(1, _dev(keys))
        sent.append(keys)
        want = have | set(keys.tolist())
        if len(want) <= limit:
            eng.sync()
            have = want
            assert eng.index_size(1) == len(have)
        else:
            with pytest.raises(pk.DMError) as ei:
                eng.sync()
            assert ei.value.status == pk.DM_EFULL
            assert eng.index_size(1) == limit
            break
    every = np.unique(np.concatenate(sent))
    held = _held(eng, 1, every)
    assert held.sum() == eng.index_size(1)
    assert set(every[held].tolist()) >= have


def test_rebuild_after_erases_and_clear():
    """Erased slots count against the limit until a rebuild or a clear."""
    eng, _ = _engine(12)
    rng = np.random.default_rng(2)
    keys = rng.integers(2, 2**64, size=6000, dtype=np.uint64)
    live = set()
    for k in range(6):
        part = keys[1000 * k:1000 * (k + 1)]
        eng.index_insert(0, _dev(part))
        live |= set(part.tolist())
        gone = np.array(sorted(live), np.uint64)[::2]
        eng.index_erase(0, _dev(gone))
        live -= set(gone.tolist())
        eng.sync()
        assert eng.index_size(0) == len(live)
        if k == 3:
            eng.index_clear(0)
            live = set()
            eng.sync()
    every = np.unique(keys)
    assert set(every[_held(eng, 0, every)].tolist()) == live


@pytest.mark.parametrize("log2,n", [(4, 3), (10, 200), (12, 1100), (17, 40_000)])
def test_keys_already_there(log2, n):
    """Batches of keys that are there, new ones or both, while the host still
    knows that they fit (first) and once it no longer does, up to the limit."""
    eng, pk = _engine(log2)
    rng = np.random.default_rng(n)
    limit = 1 << (log2 - 1)
    keys = rng.integers(2, 2**63, size=limit + 1, dtype=np.uint64)
    have = 0
    for upto in (n, n, n + 1, n + 1, limit, limit):
        for rep in range(3):
            part = keys[:upto][rng.permutation(upto)]
            eng.index_insert(1, _dev(part))
            have = max(have, upto)
            eng.sync()
            assert eng.index_size(1) == have
    eng.index_insert(1, _dev(keys))
    with pytest.raises(pk.DMError) as ei:
        eng.sync()
    assert ei.value.status == pk.DM_EFULL and eng.index_size(1) == limit
    assert _held(eng, 1, keys)[:limit].all()


def test_keys_already_there_cost_little():
    """4 Mi keys that are all there against 1,024 (16 times the time with a
    reservation on the table's count for every workgroup, 4 for reading their
    buckets)."""
    import time
    eng, _ = _engine(24)
    us = {}
    for n in (1 << 10, 1 << 22):
        k = torch.randint(2, 2**63 - 1, (n,), dtype=torch.int64, device="cuda:0").view(torch.uint64)
        eng.index_insert(2, k)
        t = []
        for _ in range(12):
            eng.sync()
            a = time.perf_counter()
            eng.index_insert(2, k)
            eng.sync()
            t.append((time.perf_counter() - a) * 1e6)
        us[n] = sorted(t[4:])[4]
    print("[case] there", us, flush=True)
    assert us[1 << 22] < 9 * us[1 << 10], us
