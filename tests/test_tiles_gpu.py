"""GPU parity of the two paths a queue above the LDS size can take: one tile
per workgroup (up to 2^21 requests) and big tiles (SEMSCHED_NO_TILES=1 sends
the same queues there). Integers throughout, so every comparison is exact."""

import numpy as np
import pytest

from oracle import c_oracle_policy, c_oracle_queue
from tests._lib import assert_same, ensure_built, gpu_available, gpu_queue, to_gpu
from workloads import fuzz_queue

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

# one past the LDS size; around the limits of the tile sizes (64 tiles of 1024
# and 2048, 128 of 4096, 256 of 8192); a last tile of one request; the last
# size of the path and the first beyond it
SIZES = [16385, 65536, 65537, 131073, 262145, 524288, 524289, (1 << 20) - 1, 1 << 20,
         (1 << 20) + 1, (1 << 21) - 1, 1 << 21, (1 << 21) + 1]


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


def check(p, l, label, monkeypatch, paths=("0", "1")):
    want = c_oracle_queue(p, l)
    for no_tiles in paths:
        monkeypatch.setenv("SEMSCHED_NO_TILES", no_tiles)
        print(f"[gpu] {label} n={len(p)} no_tiles={no_tiles}", flush=True)
        assert_same(gpu_queue(p, l), want, f"{label} no_tiles={no_tiles}")


@pytest.mark.parametrize("n", SIZES)
def test_sizes(n, monkeypatch):
    p, l = fuzz_queue(n, seed=n, classes=5, max_len=4096, tie_frac=0.3)
    check(p, l, "sizes", monkeypatch)


# final digits: 1, up to 64, up to 256, 1024; then one and two middle passes;
# with 256 ranks and 31-bit lengths the key is 39 bits (above 32: the id below
# it takes its own width)
@pytest.mark.parametrize("classes,max_len", [(1, 1000), (9, 4096), (5, 32768), (256, 4095),
                                             (9, 2_000_000), (5, 2**31 - 1), (256, 2**31 - 1)])
@pytest.mark.parametrize("n", [20001, 150000, 1_200_000])
def test_key_widths(n, classes, max_len, monkeypatch):
    p, l = fuzz_queue(n, seed=classes, classes=classes, max_len=max_len, tie_frac=0.1, min_len=0)
    check(p, l, f"widths {classes}x{max_len}", monkeypatch)
    monkeypatch.setenv("SEMSCHED_SPLIT_MID", "1")
    check(p, l, f"widths {classes}x{max_len} split", monkeypatch)


def test_largest_sums(monkeypatch):
    # 2^21 lengths of 2^31 - 1: wave sums near 2^61, totals above 2^64
    n = 1 << 21
    check(np.zeros(n, np.uint8), np.full(n, 2**31 - 1, np.int32), "largest sums", monkeypatch)


@pytest.mark.parametrize("n", [30000, 1 << 19])
def test_sjf(n, monkeypatch):
    import paper_2506_12204_amd as ss
    p, l = fuzz_queue(n, seed=3, classes=7, max_len=9000, tie_frac=0.2)
    want = c_oracle_policy(p, l, ss.POLICY_SJF)
    for no_tiles in ("0", "1"):
        monkeypatch.setenv("SEMSCHED_NO_TILES", no_tiles)
        o, w, t = ss.schedule_policy(*to_gpu(p, l), ss.POLICY_SJF)
        assert_same((o.cpu().numpy(), w.cpu().numpy(), t), want, f"sjf no_tiles={no_tiles}")


@pytest.mark.parametrize("no_tiles", ["0", "1"])
def test_range_error_and_next_call(no_tiles, monkeypatch):
    import paper_2506_12204_amd as ss
    monkeypatch.setenv("SEMSCHED_NO_TILES", no_tiles)
    p, l = fuzz_queue(70000, seed=2)
    bad = l.copy()
    bad[69999] = -1
    s = ss.Scheduler(70000)
    s.run(*to_gpu(p, bad))
    with pytest.raises(ss.SemschedRangeError):
        s.check()
    s.run(*to_gpu(p, l))  # the same workspace
    s.check()
    assert_same((s.order.cpu().numpy(), s.wait.cpu().numpy(), ss.totals_to_ints(s.totals)),
                c_oracle_queue(p, l), "after an error")


@pytest.mark.parametrize("no_tiles", ["0", "1"])
def test_barrier_give_up_then_separate_launches(no_tiles, monkeypatch):
    # no polls: the barrier of the middle passes gives up at once, and the
    # blocking call runs them again as separate launches
    import ctypes
    import torch
    import paper_2506_12204_amd as ss
    monkeypatch.setenv("SEMSCHED_NO_TILES", no_tiles)
    monkeypatch.setenv("SEMSCHED_MID_SPIN", "0")
    n = 100_000
    p, l = fuzz_queue(n, seed=8, classes=200, max_len=2**31 - 1)
    tp, tl = to_gpu(p, l)
    order = torch.empty(n, dtype=torch.int32, device="cuda")
    wait = torch.empty(n, dtype=torch.int64, device="cuda")
    totals = torch.empty((257, 2), dtype=torch.int64, device="cuda")
    ss.lib.sem_set_stream(ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    rc = ss.lib.sem_schedule(*(ctypes.c_void_p(t.data_ptr())
                               for t in (tp, tl)), n,
                             *(ctypes.c_void_p(t.data_ptr()) for t in (order, wait, totals)))
    assert rc == ss.SEM_OK
    assert_same((order.cpu().numpy(), wait.cpu().numpy(), ss.totals_to_ints(totals)),
                c_oracle_queue(p, l), "give up")


def test_replayed_graph_equals_eager():
    import torch
    import paper_2506_12204_amd as ss
    n = 300_001
    s = ss.Scheduler(n)
    tp = torch.empty(n, dtype=torch.uint8, device="cuda")
    tl = torch.empty(n, dtype=torch.int32, device="cuda")
    p, l = fuzz_queue(n, seed=0, classes=6, max_len=20000)
    tp.copy_(torch.from_numpy(p))
    tl.copy_(torch.from_numpy(l))
    s.run(tp, tl)  # before the capture: sizes and occupancy are looked up once
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.run(tp, tl)
    for seed in range(4):
        p, l = fuzz_queue(n, seed=seed, classes=6, max_len=20000 if seed % 2 else 2**31 - 1)
        tp.copy_(torch.from_numpy(p))
        tl.copy_(torch.from_numpy(l))
        g.replay()
        torch.cuda.synchronize()
        got = (s.order.cpu().numpy(), s.wait.cpu().numpy(), ss.totals_to_ints(s.totals))
        assert_same(got, c_oracle_queue(p, l), f"replay {seed}")


# The tiles' rows lie in parts of the workspace that this path leaves unused: the
# most rows of every tile size, and nothing written past the workspace's end
@pytest.mark.parametrize("n", [16385, 65535, 65537, 1 << 17, (1 << 17) + 1, 1 << 19,
                               (1 << 19) + 1, 1 << 21])
@pytest.mark.parametrize("classes,max_len", [(5, 4096), (256, 2**31 - 1)])
def test_rows_inside_the_workspace(n, classes, max_len):
    import torch
    import paper_2506_12204_amd as ss
    p, l = fuzz_queue(n, seed=n, classes=classes, max_len=max_len)
    tp, tl = to_gpu(p, l)
    size = ss.workspace_bytes(n, 1)
    ws = torch.full((size + 65536,), 0xA5, dtype=torch.uint8, device="cuda")
    order = torch.empty(n, dtype=torch.int32, device="cuda")
    wait = torch.empty(n, dtype=torch.int64, device="cuda")
    totals = torch.empty((257, 2), dtype=torch.int64, device="cuda")
    stream = ss._stream_handle(ws.device)
    print(f"[gpu] rows n={n} {classes}x{max_len}", flush=True)
    rc = ss.lib.sem_schedule_async(ss._ptr(tp), ss._ptr(tl), n, ss._ptr(order), ss._ptr(wait),
                                   ss._ptr(totals), ss._ptr(ws), size, stream)
    assert rc == ss.SEM_OK and ss.lib.sem_check(ss._ptr(ws), stream) == ss.SEM_OK
    assert bool((ws[size:] == 0xA5).all())
    assert_same((order.cpu().numpy(), wait.cpu().numpy(), ss.totals_to_ints(totals)),
                c_oracle_queue(p, l), "rows")
