"""The radix sort's forms by size (one workgroup, tiles of 4096, tiles of 1024),
through the queue append that orders a batch by its chosen instances: the
records against numpy's stable order."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 2, 63, 1023, 1024, 1025, 2047, 2049, 4095, 4096, 4097, 8191, 70_001, 262_143,
                               262_144, 262_145])
@pytest.mark.parametrize("slots", [3, 700])
def test_append_orders_by_instance(n, slots):
    import paper_2602_06502_amd as pk
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B = 16
    cfg = dict(workloads.small_random(5, 2, 2, B, 10).route.as_dict(), max_slots=slots, index_log2_slots=4)
    eng = pk.DualMap(cfg, device="cuda:0")
    eng.build_rings(range(slots))
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    rng = np.random.default_rng(n + slots)
    chosen = np.minimum(rng.geometric(0.02, size=n) - 1, slots - 1).astype(np.uint32)  # a few hot ones
    other = ((chosen + 1 + rng.integers(0, slots - 1, size=n)) % slots).astype(np.uint32)
    first = rng.random(n) < 0.5
    cand = np.concatenate([np.where(first, chosen, other), np.where(first, other, chosen)])
    match = rng.integers(0, 3, size=2 * n).astype(np.uint32)
    lens = rng.integers(2 * B, 9 * B, size=n)
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(lens)
    z = lambda k, t: d(np.zeros(k, t))
    routed = dict(key=z(2 * n, np.uint64), cand=d(cand), match=d(match), chosen=d(chosen), ttft=z(n, np.int64),
                  flags=z(n, np.uint8))
    base = rng.integers(0, 99, size=slots)
    empty = (z(slots + 1, np.int64), z(0, np.uint64), z(0, np.uint32), z(0, np.uint32), z(0, np.uint32), d(base))
    print("[case] append", n, slots, flush=True)
    q = [x.cpu().numpy() for x in eng.queue_append(empty, d(off), routed, 5)]
    order = np.argsort(chosen, kind="stable")
    u = [lens - B * match[:n].astype(np.int64), lens - B * match[n:].astype(np.int64)]
    here, there = np.where(first, u[0], u[1]), np.where(first, u[1], u[0])
    assert np.array_equal(q[0], np.searchsorted(chosen[order], np.arange(slots + 1)))
    assert np.array_equal(q[1], order.astype(np.uint64) + 5)
    assert np.array_equal(q[2], here[order]) and np.array_equal(q[3], other[order])
    assert np.array_equal(q[4], there[order]) and np.array_equal(q[5], base)
