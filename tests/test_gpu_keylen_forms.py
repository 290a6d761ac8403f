"""Closing a hotness window over branching prefixes: nodes below nodes, runs
shorter than their representative, few and many workgroups of runs; the tree
against the oracle after every window."""
import dataclasses

import numpy as np
import pytest

import oracle
import oracle.harness as oh
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_06502_amd as pk
    pk.load_library()
    oracle.build(force=False)
    yield


def _branching(rng, B, n, depth):
    """n prompts down a random tree of segments (2 to 4 children a node), cut anywhere."""
    seg = lambda: rng.integers(0, 1000, size=int(rng.integers(1, 40)) * B, dtype=np.int32)
    tree = {(): seg()}

    def walk():
        at, out = (), [tree[()]]
        for _ in range(depth):
            at = at + (int(min(rng.geometric(0.6) - 1, 3)),)
            if at not in tree:
                tree[at] = seg()
            out.append(tree[at])
        p = np.concatenate(out)
        if rng.random() < 0.3:
            p = p[:int(rng.integers(0, len(p) + 1))]
        if rng.random() < 0.5:
            p = np.concatenate([p, rng.integers(0, 1000, size=int(rng.integers(1, 90)), dtype=np.int32)])
        return p
    return [walk() for _ in range(n)]


@pytest.mark.parametrize("n,n_inst,B,K,depth", [(1, 3, 4, 1, 2), (130, 1, 4, 2, 3), (1023, 16, 4, 2, 5), (1025, 5, 8, 3, 4),
                                                (4100, 64, 4, 1, 6), (4096, 200, 16, 4, 3)])
def test_branching_windows(n, n_inst, B, K, depth):
    import paper_2602_06502_amd.harness as gh
    wl = workloads.small_random(91 + n, n_inst, 4, B, 64, slo_us=30_000, key_blocks=K)
    wl = dataclasses.replace(wl, n_prior=0)
    eng, o = gh.engine_for(wl), oh.oracle_for(wl)
    eng.keylen_enable(20_000, 1 << 20)
    assert o.keylen_enable(20_000) == oracle.OK
    rng = np.random.default_rng(n + B)
    L = workloads.initial_loads(wl, wl.route.max_slots)
    Ld = gh.to_dev(L, eng.device)
    most = 0
    for w in range(3):
        print("[case] window", n, n_inst, w, flush=True)
        # the same tree of prompts in every window, then another one
        prompts = _branching(np.random.default_rng(7 if w < 2 else 8), B, n, depth)
        prompts = [prompts[i] for i in rng.permutation(n)]
        off = np.zeros(n + 1, np.int64)
        off[1:] = np.cumsum([len(p) for p in prompts])
        tok = np.concatenate(prompts + [np.zeros(0, np.int32)]).astype(np.int32)
        g = eng.route(gh.to_dev(tok, eng.device), gh.to_dev(off, eng.device), Ld)
        eng.keylen_window()
        r = o.route(tok, off, L)
        L = r["loads"]
        assert o.keylen_window() == oracle.OK
        for k in ("key", "cand", "match", "chosen", "key_len"):
            assert np.array_equal(g[k].cpu().numpy()[:len(r[k])], r[k]), k
        tree = o.keylen_tree()
        assert np.array_equal(eng.keylen_tree(), tree)
        most = max(most, len(tree))
    assert most > 0 or n_inst == 1 or n == 1


def _route(eng, prompts):
    import paper_2602_06502_amd.harness as gh
    off = np.zeros(len(prompts) + 1, np.int64)
    off[1:] = np.cumsum([len(p) for p in prompts])
    tok = np.concatenate(prompts).astype(np.int32)
    return tok, off, gh.to_dev(tok, eng.device), gh.to_dev(off, eng.device)


def _spine(rng, W, B):
    """Run i shares i + 1 blocks with every later one; the longest part first."""
    spine = rng.integers(0, 1000, size=(W + 1) * B, dtype=np.int32)
    return [np.concatenate([spine[:(i + 1) * B], rng.integers(1000, 2000, size=(2 * W - 2 * i) * B, dtype=np.int32)])
            for i in range(W)]


@pytest.mark.parametrize("n,n_inst,K,shuffle", [(300, 200, 1, False), (301, 64, 2, True), (65, 1000, 1, True)])
def test_nested_branches(n, n_inst, K, shuffle):
    """A branch at every block of a spine: a node below a node, hundreds deep."""
    import paper_2602_06502_amd.harness as gh
    B = 4
    wl = dataclasses.replace(workloads.small_random(17 + n, n_inst, 4, B, 64, slo_us=30_000, key_blocks=K), n_prior=0)
    eng, o = gh.engine_for(wl), oh.oracle_for(wl)
    eng.keylen_enable(20_000, 1 << 20)
    assert o.keylen_enable(20_000) == oracle.OK
    L = workloads.initial_loads(wl, wl.route.max_slots)
    Ld = gh.to_dev(L, eng.device)
    rng = np.random.default_rng(n)
    prompts = _spine(rng, n, B)
    if shuffle:
        prompts = [prompts[i] for i in rng.permutation(n)] + prompts[:5]
    tok, off, td, od = _route(eng, prompts)
    for w in range(2):
        print("[case] nested", n, n_inst, w, flush=True)
        g = eng.route(td, od, Ld)
        eng.keylen_window()
        r = o.route(tok, off, L)
        L = r["loads"]
        assert o.keylen_window() == oracle.OK
        assert np.array_equal(g["key_len"].cpu().numpy()[:len(r["key_len"])], r["key_len"])
        tree = o.keylen_tree()
        assert len(tree) > 0 and np.array_equal(eng.keylen_tree(), tree)


def _close_us(prompts, n_inst, B=4, K=1, reps=5):
    """Median time of closing a window of these prompts."""
    import time

    import paper_2602_06502_amd.harness as gh
    wl = dataclasses.replace(workloads.small_random(3, n_inst, 4, B, 64, key_blocks=K), n_prior=0)
    eng = gh.engine_for(wl)
    _, _, td, od = _route(eng, prompts)
    eng.keylen_enable(100_000, int(od[-1]) // B + len(prompts))
    Ld = torch.zeros(wl.route.max_slots, dtype=torch.int64, device=eng.device)
    t = []
    for _ in range(reps + 1):
        eng.route(td, od, Ld)
        eng.sync()
        torch.cuda.synchronize()
        a = time.perf_counter()
        eng.keylen_window()
        t.append((time.perf_counter() - a) * 1e6)
    us = sorted(t[1:])[reps // 2]
    print("[case] close", len(prompts), n_inst, us, flush=True)
    return us


def test_nested_branches_cost_little():
    """A spine of 512 branches against as many prompts that part in one place
    (some 90 times the time with a turn for every branch)."""
    rng = np.random.default_rng(1)
    spine = _spine(rng, 512, 4)
    flat = [np.concatenate([spine[0][:4], p[4:] + 2000]) for p in spine]
    for i, p in enumerate(flat):
        p[4:8] = 5000 + i
    assert _close_us(spine, 256) < 12 * _close_us(flat, 256)


@pytest.mark.parametrize("n,blocks,n_inst", [(3, 2600, 16), (2047, 70, 64), (2049, 70, 64), (40, 1300, 3), (12, 513, 8), (12, 2049, 8)])
def test_long_runs(n, blocks, n_inst):
    """Runs that go on past what a step compares and past what a workgroup sums at
    a time, parting anywhere; few runs (a wave each) and many."""
    import paper_2602_06502_amd.harness as gh
    B = 4
    wl = dataclasses.replace(workloads.small_random(29 + n, n_inst, 4, B, 64, slo_us=30_000, key_blocks=1), n_prior=0)
    eng, o = gh.engine_for(wl), oh.oracle_for(wl)
    eng.keylen_enable(50_000, 1 << 20)
    assert o.keylen_enable(50_000) == oracle.OK
    L = workloads.initial_loads(wl, wl.route.max_slots)
    Ld = gh.to_dev(L, eng.device)
    rng = np.random.default_rng(n + blocks)
    spine = rng.integers(0, 1000, size=blocks * B, dtype=np.int32)
    for w in range(2):
        prompts = []
        for i in range(n):
            k = int(rng.integers(0, blocks + 1)) if i % 3 else blocks
            more = int(rng.integers(0, blocks)) if i % 2 else 0
            prompts.append(np.concatenate([spine[:k * B], rng.integers(1000, 2000, size=more, dtype=np.int32)]))
        tok, off, td, od = _route(eng, prompts)
        print("[case] long", n, blocks, n_inst, w, flush=True)
        g = eng.route(td, od, Ld)
        eng.keylen_window()
        r = o.route(tok, off, L)
        L = r["loads"]
        assert o.keylen_window() == oracle.OK
        assert np.array_equal(g["key_len"].cpu().numpy()[:len(r["key_len"])], r["key_len"])
        tree = o.keylen_tree()
        assert len(tree) > 0 and np.array_equal(eng.keylen_tree(), tree)


def test_long_runs_cost_little():
    """As many blocks in 32 prompts alike but for their ends as in 1,024 (6.7
    times the time with 8 runs a wave and 64 blocks a step; 2.4 now, the deeper
    tree included)."""
    rng = np.random.default_rng(1)
    spine = rng.integers(0, 1000, size=4 * 16_384, dtype=np.int32)
    ends = lambda n, b: [np.concatenate([spine[:4 * (b - 1)], np.full(4, 5000 + i, np.int32)]) for i in range(n)]
    assert _close_us(ends(32, 16_384), 8) < 4 * _close_us(ends(1024, 512), 8)
