"""Selection forms chosen by size or rule, each against the oracle, element by
element: dense indices past one byte (more than 256 live instances), the
minimum-TTFT rule's walks, the serial path."""
import dataclasses
import sys

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


def _pair(wl, L0, policy="slo_aware"):
    import paper_2602_06502_amd.harness as gh
    print("[case]", wl.name, wl.route.n_inst, wl.n_req, policy, flush=True)
    sys.stdout.flush()
    eng, o = gh.engine_for(wl), oh.oracle_for(wl)
    gh.prefill_from_prior(eng, wl)
    oh.prefill_from_prior(o, wl)
    eng.set_policy(policy)
    assert o.set_policy(policy) == oracle.OK
    tok, off = workloads.prompts(wl, wl.n_req, sub=0)
    Ld = gh.to_dev(L0, eng.device)
    g = eng.route(gh.to_dev(tok, eng.device), gh.to_dev(off, eng.device), Ld)
    eng.sync()
    r = o.route(tok, off, L0)
    for k in ("key", "cand", "match", "chosen", "ttft", "flags", "key_len"):
        assert np.array_equal(g[k].cpu().numpy()[:len(r[k])], r[k]), k
    assert np.array_equal(Ld.cpu().numpy(), r["loads"])
    return r


@pytest.mark.parametrize("n_inst,n_req,wide", [(256, 1100, False), (257, 1100, False), (257, 1100, True),
                                               (700, 5000, False), (4093, 2100, False), (4093, 2100, True)])
def test_windows_on_many_instances(n_inst, n_req, wide):
    """256 live instances keep the byte codes, more take the wide ones (up to
    every slot of the id space); wide: loads past 2^30 (the 64-bit walk)."""
    wl = workloads.small_random(211 + n_inst, n_inst, 2, 16, n_req, slo_us=6_000_000_000 if wide else 3_000)
    L0 = workloads.initial_loads(wl, wl.route.max_slots)
    if wide:
        L0[::3] += 1 << 40
    _pair(wl, L0)


@pytest.mark.parametrize("n_inst,div,wide", [(1, 4, 0), (3, 4, 0), (8, 1, 0), (8, 1 << 14, 0), (8, 1 << 31, 0),
                                             (200, 4, 0), (300, 4, 0), (8, 4, 1), (8, 1 << 33, 1), (300, 4, 1),
                                             (8, 4, 2)])
def test_min_ttft_windows(n_inst, div, wide):
    """The minimum-TTFT rule: 32-bit walk (its bound in the steps), 64-bit walk
    (wide=1) and serial path (wide=2: loads spread past 2^62), under queue
    divisors from none to past every load."""
    wl = workloads.small_random(91 + n_inst, n_inst, 3, 16, 2600)
    wl = dataclasses.replace(wl, n_prior=300, route=dataclasses.replace(wl.route, queue_div=div))
    L0 = workloads.initial_loads(wl, wl.route.max_slots)
    if wide:
        L0[::3] += 1 << 40
        L0[1] = (1 << 62) + ((1 << 50) if wide == 2 else -(1 << 50))
    _pair(wl, L0, "min_ttft")


@pytest.mark.parametrize("policy", ["slo_aware", "cache_affinity", "least_loaded", "min_ttft"])
@pytest.mark.parametrize("n_inst", [2, 64, 260])
def test_serial_path(n_inst, policy):
    """Loads spread past 2^62: one request at a time, whatever the rule."""
    wl = workloads.small_random(17 + n_inst, n_inst, 3, 16, 200, slo_us=3_000)
    L0 = workloads.initial_loads(wl, wl.route.max_slots)
    L0[1] = (1 << 62) + (1 << 50)
    _pair(wl, L0, policy)


@pytest.mark.parametrize("n_inst,n_req", [(1, 255), (2, 256), (3, 257), (8, 511), (64, 513), (200, 1024),
                                          (300, 700), (40, 65_536), (40, 65_537)])
def test_small_level_blocks(n_inst, n_req):
    """Blocks of 256 requests at their edges (one to three instances: every
    level one pair, 64-depth windows), and both sides of the line to blocks
    of 1024."""
    wl = workloads.small_random(131 + n_inst, n_inst, 4, 16, n_req, slo_us=3_000)
    wl = dataclasses.replace(wl, n_prior=300)
    _pair(wl, workloads.initial_loads(wl, wl.route.max_slots))


@pytest.mark.parametrize("policy", ["slo_aware", "min_ttft"])
@pytest.mark.parametrize("n_inst,n_req", [(1, 63), (2, 64), (3, 65), (8, 127), (64, 1025), (200, 4095), (300, 4096),
                                          (1, 4097), (2, 4351), (3, 4352), (8, 4353), (64, 4609), (300, 4700)])
def test_tiny_level_blocks(n_inst, n_req, policy):
    """Blocks of 64 requests at their edges, and both sides of the line to blocks of 256."""
    wl = workloads.small_random(171 + n_inst, n_inst, 4, 16, n_req, slo_us=3_000)
    wl = dataclasses.replace(wl, n_prior=300)
    _pair(wl, workloads.initial_loads(wl, wl.route.max_slots), policy)


@pytest.mark.parametrize("n_inst,n_req,policy", [(300, 65_537, "slo_aware"), (4093, 66_000, "min_ttft"),
                                                 (300, 524_287, "slo_aware"), (300, 524_288, "slo_aware"),
                                                 (1000, 526_500, "min_ttft")])
def test_large_level_blocks_on_many_instances(n_inst, n_req, policy):
    """Blocks of 1024 and of 2048 requests with two bytes an instance."""
    wl = workloads.small_random(311 + n_inst, n_inst, 2, 16, n_req, slo_us=3_000)
    wl = dataclasses.replace(wl, n_prior=3000)
    _pair(wl, workloads.initial_loads(wl, wl.route.max_slots), policy)


@pytest.mark.parametrize("n_inst,n_req,policy", [(257, 63, "slo_aware"), (300, 5000, "min_ttft"), (4093, 4097, "slo_aware"),
                                                 (300, 70_000, "slo_aware"), (700, 525_000, "slo_aware")])
def test_pipelined_on_many_instances(n_inst, n_req, policy):
    """Consecutive pipelined batches (blocks of 1024 at every size below the
    largest) on more than 256 instances, the loads carried on."""
    import paper_2602_06502_amd.harness as gh
    wl = workloads.small_random(331 + n_inst, n_inst, 2, 16, n_req, slo_us=3_000)
    wl = dataclasses.replace(wl, n_prior=3000)
    eng, o = gh.engine_for(wl), oh.oracle_for(wl)
    gh.prefill_from_prior(eng, wl)
    oh.prefill_from_prior(o, wl)
    eng.set_policy(policy)
    assert o.set_policy(policy) == oracle.OK
    L = workloads.initial_loads(wl, wl.route.max_slots)
    Ld = gh.to_dev(L, eng.device)
    data = [workloads.prompts(wl, n_req, sub=k) for k in (0, 2, 3)]
    dev = [(gh.to_dev(tok, eng.device), gh.to_dev(off, eng.device)) for tok, off in data]
    outs = [eng.alloc_route_out(n_req) for _ in data]
    print("[case] pipelined", n_inst, n_req, policy, flush=True)
    eng.set_pipelining(True)
    for (tok, off), out in zip(dev, outs):
        eng.route_into(tok, off, Ld, out)
    eng.sync()
    eng.set_pipelining(False)
    for (tok, off), out in zip(data, outs):
        r = o.route(tok, off, L)
        L = r["loads"]
        for k in ("key", "cand", "match", "chosen", "ttft", "flags"):
            assert np.array_equal(out[k].cpu().numpy()[:len(r[k])], r[k]), k
    assert np.array_equal(Ld.cpu().numpy(), L)


@pytest.mark.parametrize("n_req,mean,kl,n_inst,policy", [
    (8192, 24_500, False, 40, "slo_aware"), (20_000, 10_100, True, 40, "slo_aware"), (33_333, 6100, False, 40, "slo_aware"),
    (65_537, 3100, False, 40, "slo_aware"), (70_001, 2900, True, 300, "slo_aware"), (90_000, 2250, False, 40, "min_ttft"),
    (131_072, 1550, False, 1000, "cache_affinity")])
def test_batch_overlapping_itself(n_req, mean, kl, n_inst, policy):
    """Unpipelined batches of at least 200 M tokens, those of more than 65,536
    requests selected in two parts beside the hashing: outputs, loads, block keys
    and the hotness tree's windows against the oracle, twice in a row on the same
    buffers, then pipelined."""
    import paper_2602_06502_amd.harness as gh
    B = 16
    wl = workloads.small_random(7, n_inst, 8, B, 64, slo_us=30_000)
    eng, o = gh.engine_for(wl), oh.oracle_for(wl)
    eng.set_policy(policy)
    assert o.set_policy(policy) == oracle.OK
    rng = np.random.default_rng(n_req)
    tpl = [rng.integers(0, 1 << 20, size=B * 90, dtype=np.int32) for _ in range(12)]
    lens = rng.integers(mean // 2, mean * 3 // 2 + 200, size=n_req)
    off = np.zeros(n_req + 1, np.int64)
    off[1:] = np.cumsum(lens)
    tok = rng.integers(0, 1 << 20, size=int(off[-1]), dtype=np.int32)
    for r in range(n_req):
        t = tpl[int(rng.integers(0, 12))]
        k = min(len(t), int(lens[r]))
        tok[off[r]:off[r] + k] = t[:k]
    assert len(tok) >= 200_000_000
    if kl:
        eng.keylen_enable(4096, int((lens // B).sum()) + n_req)
        assert o.keylen_enable(4096) == oracle.OK
    L = workloads.initial_loads(wl, wl.route.max_slots)
    Ld = gh.to_dev(L, eng.device)
    td, od = gh.to_dev(tok, eng.device), gh.to_dev(off, eng.device)
    for step in range(3):
        print("[case] overlap", n_req, len(tok), n_inst, policy, step, flush=True)
        eng.set_pipelining(step == 2)
        g = eng.route(td, od, Ld, block_keys=True)
        if step == 2:
            eng.sync()
        g2 = {k: v.clone() for k, v in g.items()}  # unpipelined: on the caller's stream, no wait
        r = o.route(tok, off, L, block_keys=True)
        for k in ("key", "cand", "match", "chosen", "ttft", "flags", "key_len", "block_keys"):
            assert np.array_equal(g2[k].cpu().numpy()[:len(r[k])], r[k]), k
        assert np.array_equal(Ld.cpu().numpy(), r["loads"])
        L = r["loads"]
        if kl:
            eng.keylen_window()
            assert o.keylen_window() == oracle.OK
            assert np.array_equal(eng.keylen_tree(), o.keylen_tree())
    eng.sync()
