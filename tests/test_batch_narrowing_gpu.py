"""GPU parity of the narrowed sorts of batch selection and eviction at the
sizes where their form changes (512 and 1024 kept entries), with ties that
one narrowing round cannot split, and with keys too wide to pack. Exact."""

import numpy as np
import pytest

from oracle import evict, select_batch
from tests._lib import ensure_built, gpu_available
from tests.test_batch_gpu import dev, instance, run_select

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


def run_evict(p, l, cached, kv, usage, capacity, demands):
    import paper_2506_12204_amd as ss
    v, u = ss.evict(dev(p, np.uint8), dev(l, np.int32), dev(cached, np.int32), dev(kv, np.int64),
                    usage, capacity, dev(demands, np.int64))
    return v.cpu().numpy().tolist(), u.cpu().numpy().tolist()


# one distinct key (only ids differ), a few, many
@pytest.mark.parametrize("classes,max_len", [(1, 1), (2, 3), (5, 4000)])
@pytest.mark.parametrize("b,buffer,ongoing", [
    (0, 600, 5), (1, 512, 0), (64, 513, 64), (512, 512, 512), (512, 4096, 513), (513, 1024, 512),
    (1000, 1049, 1024), (1024, 1025, 1025), (1024, 4096, 1), (1025, 4096, 600)])
def test_select(b, buffer, ongoing, classes, max_len):
    print(f"[gpu] select b={b} buffer={buffer} ongoing={ongoing} {classes}x{max_len}", flush=True)
    p, l, stage, heap, buf, ong = instance(b + buffer, 30000, 3000, buffer, ongoing, classes,
                                           max_len)
    want = select_batch(p.tolist(), l.tolist(), stage.tolist(), heap.tolist(), buf.tolist(),
                        ong.tolist(), b)
    assert run_select(p, l, stage, heap, buf, ong, b) == want


@pytest.mark.parametrize("classes,max_len", [(1, 1), (2, 3), (5, 4000)])
@pytest.mark.parametrize("cached,share", [
    (1, 1.0), (64, 0.5), (512, 0.9), (513, 0.1), (1024, 1.0), (1025, 0.4), (1025, 0.6),
    (8192, 0.0), (8192, 0.01), (8192, 0.07), (8192, 0.13), (8192, 0.9), (8192, 1.0), (8192, 2.0)])
def test_evict(cached, share, classes, max_len):
    # the demands take about `share` of the cached KV; some requests hold none
    rng = np.random.default_rng(cached)
    n = 30000
    print(f"[gpu] evict cached={cached} share={share} {classes}x{max_len}", flush=True)
    p = rng.integers(0, classes, n).astype(np.uint8)
    l = rng.integers(0, max_len, n).astype(np.int32)
    ids = rng.permutation(n)[:cached]
    kv = rng.integers(0, 5000, cached)
    kv[rng.random(cached) < 0.1] = 0
    nd = 37
    demands = rng.multinomial(int(share * kv.sum()), np.full(nd, 1 / nd))
    usage = int(kv.sum())
    want = evict(p.tolist(), l.tolist(), ids.tolist(), kv.tolist(), usage, usage,
                 demands.tolist())
    assert run_evict(p, l, ids, kv, usage, usage, demands) == (want[0], want[1])


def test_keys_beyond_63_bits():
    # 2^25 ids, ranks to 255, lengths to 2^31 - 1: 64 bits, so the lists are
    # sorted whole
    n = 1 << 25
    rng = np.random.default_rng(1)
    p = np.zeros(n, np.uint8)
    l = np.zeros(n, np.int32)
    stage = np.ones(n, np.uint8)
    ids = np.unique(rng.integers(0, n, 9000))
    rng.shuffle(ids)
    p[ids] = rng.integers(0, 256, ids.size)
    l[ids] = rng.integers(0, 2**31 - 1, ids.size)
    p[ids[0]], l[ids[0]] = 255, 2**31 - 1
    p[ids[3000]], l[ids[3000]] = 255, 2**31 - 1
    buf, ong, cached = ids[:2000], ids[2000:2300], ids[2300:8000]
    heap = np.zeros(0, np.int32)
    pk, lk = dict(zip(ids, p[ids])), dict(zip(ids, l[ids]))
    small = {i: k for k, i in enumerate(sorted(ids.tolist()))}  # same order, fewer ids
    back = {k: i for i, k in small.items()}
    ps = [int(pk[back[k]]) for k in range(len(back))]
    ls = [int(lk[back[k]]) for k in range(len(back))]
    want = select_batch(ps, ls, [1] * len(ps), [], [small[i] for i in buf.tolist()],
                        [small[i] for i in ong.tolist()], 100)
    got = run_select(p, l, stage, heap, buf, ong, 100)
    assert got == ([back[k] for k in want[0]], [back[k] for k in want[1]])
    kv = rng.integers(1, 5000, cached.size)
    usage = int(kv.sum())
    demands = [usage // 50] * 3
    want = evict(ps, ls, [small[i] for i in cached.tolist()], kv.tolist(), usage, usage, demands)
    got = run_evict(p, l, cached, kv, usage, usage, demands)
    assert got == ([back[k] for k in want[0]], want[1])


# Sizes that are narrowed, and sizes whose lists are known to be sorted whole: a
# bad id (and a negative KV size) is found in either form, and a good call after
# it is right
@pytest.mark.parametrize("b,buffer,ongoing", [(64, 600, 64), (800, 3000, 300), (800, 700, 300),
                                              (1500, 700, 300), (64, 600, 1500)])
@pytest.mark.parametrize("where", ["buffer", "ongoing"])
def test_select_bad_id(b, buffer, ongoing, where):
    import paper_2506_12204_amd as ss
    n = 30000
    p, l, stage, heap, buf, ong = instance(b, n, 3000, buffer, ongoing, 5, 4000)
    bad = {"buffer": buf, "ongoing": ong}[where].copy()
    for value in (n, -1):
        bad[-1] = value
        print(f"[gpu] select b={b} buffer={buffer} ongoing={ongoing}: {where} {value}", flush=True)
        with pytest.raises(ss.SemschedError):
            run_select(p, l, stage, heap, bad if where == "buffer" else buf,
                       bad if where == "ongoing" else ong, b)
    want = select_batch(p.tolist(), l.tolist(), stage.tolist(), heap.tolist(), buf.tolist(),
                        ong.tolist(), b)
    assert run_select(p, l, stage, heap, buf, ong, b) == want


@pytest.mark.parametrize("cached,nd", [(300, 5), (700, 5), (700, 600), (1024, 1024), (3000, 5)])
@pytest.mark.parametrize("share", [0.0, 0.3, 0.95])
def test_evict_forms(cached, nd, share):
    import paper_2506_12204_amd as ss
    rng = np.random.default_rng(cached + nd)
    n = 30000
    p = rng.integers(0, 5, n).astype(np.uint8)
    l = rng.integers(0, 4000, n).astype(np.int32)
    ids = rng.permutation(n)[:cached]
    kv = rng.integers(1, 5000, cached)
    demands = rng.multinomial(int(share * kv.sum()), np.full(nd, 1 / nd))
    usage = int(kv.sum())
    print(f"[gpu] evict cached={cached} demands={nd} share={share}", flush=True)
    for change, error in ((lambda i, k: i.__setitem__(-1, n), ss.SemschedError),
                          (lambda i, k: k.__setitem__(-1, -1), ss.SemschedRangeError)):
        bad_ids, bad_kv = ids.copy(), kv.copy()
        change(bad_ids, bad_kv)
        with pytest.raises(error):
            run_evict(p, l, bad_ids, bad_kv, usage, usage, demands)
    want = evict(p.tolist(), l.tolist(), ids.tolist(), kv.tolist(), usage, usage,
                 demands.tolist())
    assert run_evict(p, l, ids, kv, usage, usage, demands) == (want[0], want[1])
