"""Forms of a routed batch chosen by its size (block starts, grouping, members
pass), at their edges, each against the oracle element by element."""
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


def _same(g, r, Ld):
    for k in ("key", "cand", "match", "chosen", "ttft", "flags", "key_len", "block_keys"):
        if k in r:
            assert np.array_equal(g[k].cpu().numpy()[:len(r[k])], r[k]), k
    assert np.array_equal(Ld.cpu().numpy(), r["loads"])


@pytest.mark.parametrize("block,key_blocks", [(16, 4), (4, 1), (32, 7)])
@pytest.mark.parametrize("n_req", [1, 63, 64, 65, 1023, 1024, 1025, 2049, 4095, 4096, 4097, 16_383, 16_384, 16_385])
def test_batch_sizes(n_req, block, key_blocks):
    import paper_2602_06502_amd.harness as gh
    wl = dataclasses.replace(workloads.small_random(31 + n_req + block, 5, 3, block, n_req, key_blocks=key_blocks,
                                                    slo_us=20_000), n_prior=min(n_req, 300))
    print("[case] batch", n_req, block, key_blocks, flush=True)
    eng, o = gh.engine_for(wl), oh.oracle_for(wl)
    gh.prefill_from_prior(eng, wl)
    oh.prefill_from_prior(o, wl)
    tok, off = workloads.prompts(wl, n_req, sub=0)
    L0 = workloads.initial_loads(wl, wl.route.max_slots)
    for bk in (False, True):
        Ld = gh.to_dev(L0, eng.device)
        g = eng.route(gh.to_dev(tok, eng.device), gh.to_dev(off, eng.device), Ld, block_keys=bk)
        eng.sync()
        _same(g, o.route(tok, off, L0, block_keys=bk), Ld)


# 1, 2 and 3 launches of the block starts; the broken offset first, inside and last
@pytest.mark.parametrize("n", [1000, 4096, 16_384, 16_385, 1_050_000])
def test_broken_offsets_found_in_every_form(n):
    import paper_2602_06502_amd as pk
    import paper_2602_06502_amd.harness as gh
    wl = workloads.small_random(7, 4, 2, 4, 16)
    eng = gh.engine_for(wl)
    dev = eng.device
    tok = torch.zeros(4 * n, dtype=torch.int32, device=dev)
    good = torch.arange(n + 1, dtype=torch.int64, device=dev) * 4
    for at in (0, n // 2, n):
        print("[case] broken offsets", n, at, flush=True)
        bad = good.clone()
        bad[at] = 4 * n + 1 if at == n else -4 if at == 0 else 4 * n
        L = torch.zeros(wl.route.max_slots, dtype=torch.int64, device=dev)
        out = eng.route(tok, bad, L)
        with pytest.raises(pk.DMError) as ei:
            eng.sync()
        assert ei.value.status == pk.DM_EINVAL
        assert int(out["match"].view(torch.int32).sum()) == 0 and int(out["key"].view(torch.int64).abs().sum()) == 0
    L = torch.zeros(wl.route.max_slots, dtype=torch.int64, device=dev)
    out = eng.route(tok, good, L)
    eng.sync()  # the next batch is whole again
    assert int((out["key"].view(torch.int64) == 0).sum()) == 0


# members within one launch (few requests) and in four (many), every way that a
# member is resolved
@pytest.mark.parametrize("more", [0, 65_536])
def test_member_resolution(more):
    import paper_2602_06502_amd.harness as gh
    B = 16
    cfg = dict(block=B, key_blocks=4, seeds=(3, 9), vnodes=16, max_slots=8, index_log2_slots=14)
    rng = np.random.default_rng(29)
    P = rng.integers(0, 50_000, size=300 * B, dtype=np.int32)
    rnd = lambda nb: rng.integers(0, 50_000, size=nb * B, dtype=np.int32)
    prompts = [np.concatenate([P[:30 * B], rnd(20)]) for _ in range(64)]
    prompts += [P, np.concatenate([P[:33 * B], rnd(5)]), P[:25 * B], np.concatenate([P[:30 * B], rnd(3)]),
                np.concatenate([P[:20 * B], rnd(200)]), prompts[0].copy(), np.concatenate([P, rnd(1)[:7]]),
                np.concatenate([P[:37 * B], rnd(2)]), np.concatenate([P[:38 * B], rnd(2)]),
                np.concatenate([P[:63 * B], rnd(3)]), np.concatenate([P[:64 * B], rnd(3)]),
                np.concatenate([P[:128 * B], rnd(70)]), P[:64 * B], P[:65 * B]]
    at = len(prompts)
    prompts += [rnd(1) for _ in range(more)]
    off = np.zeros(len(prompts) + 1, np.int64)
    off[1:] = np.cumsum([len(p) for p in prompts])
    tok = np.concatenate(prompts).astype(np.int32)
    o, eng = oracle.Oracle(cfg), gh.DualMap(cfg, device="cuda:0")
    o.build_rings(range(8))
    eng.build_rings(list(range(8)))
    keys = o.chain(0, P)
    L0 = np.arange(8, dtype=np.int64) * 1000
    for inst in range(8):
        # every other instance holds a shorter prefix
        have = keys[:len(keys) if inst % 2 else 40]
        o.index_insert(inst, have)
        eng.index_insert(inst, gh.to_dev(have, eng.device))
    for bk in (False, True):
        print("[case] members", more, bk, flush=True)
        Ld = gh.to_dev(L0, eng.device)
        g = eng.route(gh.to_dev(tok, eng.device), gh.to_dev(off, eng.device), Ld, block_keys=bk)
        eng.sync()
        r = o.route(tok, off, L0, block_keys=bk)
        _same(g, r, Ld)
    assert r["match"][:at].max() >= 40
