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
