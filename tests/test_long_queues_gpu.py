"""GPU parity of the batched call's long queues (more than 16,384 requests) at
the edges of their tiles and scans. Integers throughout: exact."""

import numpy as np
import pytest

from oracle import c_oracle_batched
from tests._lib import assert_same, ensure_built, gpu_available, gpu_batched
from workloads import fuzz_segments

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

TILE = 8192


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


def check(sizes, label, classes=5, max_len=32768, seed=1):
    p, l, off = fuzz_segments(sizes, seed=seed, classes=classes, max_len=max_len)
    want = c_oracle_batched(p, l, off, classes)
    room = sum(s for s in sizes if s > 16384)
    for blocking, long_requests in ((False, room), (True, None)):
        print(f"[gpu] {label} sizes={list(sizes)[:6]} blocking={blocking}", flush=True)
        got = gpu_batched(p, l, off, classes, blocking=blocking, long_requests=long_requests)
        assert_same(got, want, label)


# one request past the LDS size; whole tiles and one request either side; the
# last queue scanned as one item (32 tiles), the first scanned in parts; runs
# of more than one batch of rows per lane (1100 tiles)
@pytest.mark.parametrize("m", [16385, 3 * TILE, 3 * TILE + 1, 32 * TILE, 32 * TILE + 1,
                               100 * TILE - 1, 1100 * TILE + 5])
def test_one_queue(m):
    check([m], "one")


def test_mixed_with_short_queues():
    check([0, 16385, 1, 5000, 40 * TILE + 3, 256, 16384, 20000, 0, 300], "mixed")


# digits of one value, up to 64, 256 and 1024; one and two middle passes; keys
# above 32 bits
@pytest.mark.parametrize("classes,max_len", [(1, 1000), (3, 9000), (256, 4095), (9, 2_000_000),
                                             (5, 2**31 - 1), (256, 2**31 - 1)])
def test_key_widths(classes, max_len):
    check([50001, 17000, 35 * TILE], f"widths {classes}x{max_len}", classes, max_len)


# Elements without the first digit, whose lengths are read through the id (keys and
# ids beyond 64 bits together, here forced): several queues, tiles of two queues
# in one workgroup's run, tile edges
@pytest.mark.parametrize("sizes", [[16385], [50001, 17000, 35 * TILE], [3 * TILE + 1, 40 * TILE - 1],
                                   [16385 + 13 * i for i in range(300)]])
@pytest.mark.parametrize("classes,max_len", [(1, 1000), (5, 32768), (9, 2_000_000),
                                             (256, 2**31 - 1)])
def test_lengths_read_through_the_id(sizes, classes, max_len, monkeypatch):
    monkeypatch.setenv("SEMSCHED_FORCE_WIDE", "1")
    check(sizes, f"gather {classes}x{max_len}", classes, max_len)


def test_workgroups_that_span_queues():
    # more tiles than workgroups, so that one takes tiles of several queues
    check([16385 + 13 * i for i in range(400)], "span")


def test_largest_sums():
    # waits whose sums over a wave reach 2^64, and class totals above it
    sizes = np.array([1 << 21])
    off = np.array([0, 1 << 21], np.int64)
    p = np.repeat(np.array([0, 3], np.uint8), 1 << 20)
    l = np.full(1 << 21, 2**31 - 1, np.int32)
    got = gpu_batched(p, l, off, 4, long_requests=int(sizes.sum()))
    assert_same(got, c_oracle_batched(p, l, off, 4), "largest sums")


def folds(room, queues):
    """Whether the passes sum the count rows themselves: the library's tiles for
    that room (a partial one per queue, and one) against its limits."""
    tiles = -(-room // TILE) + min(queues, room // 16385) + 1
    return tiles <= min(256, 96 * queues)


# The same queues with their exact room (the passes sum the count rows
# themselves, up to the last size that does) and with room for 300 tiles more
# (the rows' prefixes are launched)
@pytest.mark.parametrize("sizes,exact_folds", [
    ([16385], True), ([94 * TILE - 1], True), ([94 * TILE], True), ([94 * TILE + 1], False),
    ([96 * TILE - 1], False), ([30 * TILE, 17000, 65 * TILE + 1], True),
    ([84 * TILE] * 2 + [84 * TILE], True), ([84 * TILE] * 2 + [84 * TILE + 1], False),
    ([3 * TILE] * 60 + [4 * TILE] * 3, True), ([3 * TILE] * 60 + [4 * TILE] * 2 + [4 * TILE + 1], False)])
@pytest.mark.parametrize("classes,max_len", [(5, 32768), (9, 2_000_000), (256, 2**31 - 1)])
def test_both_sides_of_the_fold_rule(sizes, exact_folds, classes, max_len):
    assert folds(sum(sizes), len(sizes)) == exact_folds
    assert not folds(sum(sizes) + 300 * TILE, len(sizes))
    p, l, off = fuzz_segments(sizes, seed=len(sizes), classes=classes, max_len=max_len)
    want = c_oracle_batched(p, l, off, classes)
    for more in (0, 300 * TILE):
        print(f"[gpu] fold sizes={sizes} {classes}x{max_len} more={more}", flush=True)
        got = gpu_batched(p, l, off, classes, long_requests=sum(sizes) + more)
        assert_same(got, want, f"fold more={more}")


# A range error in one long queue: found in the first or the last tile, by the
# lengths or by the ranks, with the scans of many workgroups running beside the
# one that raises it; then the next call on the same workspace
@pytest.mark.parametrize("sizes", [[16385], [17000] * 60, [40 * TILE, 16385, 100, 33 * TILE + 1]])
@pytest.mark.parametrize("where", ["first", "last"])
@pytest.mark.parametrize("what", ["length", "rank"])
def test_range_error_and_next_call(sizes, where, what):
    import torch
    import paper_2506_12204_amd as ss
    from tests._lib import to_gpu
    classes = 5
    p, l, off = fuzz_segments(sizes, seed=7, classes=classes, max_len=32768)
    n, s = len(p), len(sizes)
    ws = torch.empty(ss.workspace_bytes(n, s), dtype=torch.uint8, device="cuda")
    order = torch.empty(n, dtype=torch.int32, device="cuda")
    wait = torch.empty(n, dtype=torch.int64, device="cuda")
    totals = torch.empty((s, 1 + classes, 2), dtype=torch.int64, device="cuda")
    stream = ss._stream_handle(ws.device)

    def call(pri, length):
        tp, tl, to = to_gpu(pri, length, off.astype(np.int64))
        rc = ss.lib.sem_schedule_batched_async(
            ss._ptr(tp), ss._ptr(tl), ss._ptr(to), s, classes, ss._ptr(order), ss._ptr(wait),
            ss._ptr(totals), ss._ptr(ws), ws.numel(), stream)
        assert rc == ss.SEM_OK
        return ss.lib.sem_check(ss._ptr(ws), stream)

    print(f"[gpu] range error sizes={sizes[:4]} {where} {what}", flush=True)
    bp, bl = p.copy(), l.copy()
    at = 0 if where == "first" else n - 1
    if what == "length":
        bl[at] = -1
    else:
        bp[at] = classes
    assert call(bp, bl) == ss.SEM_ERANGE
    assert call(p, l) == ss.SEM_OK
    got = (order.cpu().numpy(), wait.cpu().numpy(), ss.totals_to_ints(totals))
    assert_same(got, c_oracle_batched(p, l, off, classes), "after an error")


# A kernel of several phases hands its shares out as workgroups start: with one
# poll a workgroup that is done early takes the shares of those that have not
# started, and has several in all phases
@pytest.mark.parametrize("sizes", [[16385], [95 * TILE + 7], [20000] * 70, [17000 + i for i in range(400)]])
@pytest.mark.parametrize("classes,max_len", [(5, 32768), (9, 2_000_000), (256, 2**31 - 1)])
def test_shares_taken_over(sizes, classes, max_len, monkeypatch):
    monkeypatch.setenv("SEMSCHED_CLAIM_POLLS", "1")
    check(sizes, f"claims {classes}x{max_len}", classes, max_len, seed=classes)


# Launches of a batch in a workspace with room for long queues, whether it has
# any or not: every one costs a caller 3 to 4 us on the host
@pytest.mark.parametrize("n,segments,most", [(131072, 512, 9), (1 << 22, 4096, 13)])
def test_launches_with_room_for_long_queues(n, segments, most):
    import ctypes
    import torch
    import paper_2506_12204_amd as ss
    p, l, off = fuzz_segments([n // segments] * segments, seed=1, classes=4)
    from tests._lib import to_gpu
    tp, tl, to = to_gpu(p, l, off.astype(np.int64))
    ws = torch.empty(ss.workspace_bytes(n, segments), dtype=torch.uint8, device="cuda")
    order = torch.empty(n, dtype=torch.int32, device="cuda")
    wait = torch.empty(n, dtype=torch.int64, device="cuda")
    totals = torch.empty((segments, 5, 2), dtype=torch.int64, device="cuda")

    def call():
        rc = ss.lib.sem_schedule_batched_async(
            ss._ptr(tp), ss._ptr(tl), ss._ptr(to), segments, 4, ss._ptr(order), ss._ptr(wait),
            ss._ptr(totals), ss._ptr(ws), ws.numel(), ss._stream_handle(ws.device))
        assert rc == ss.SEM_OK
    call()  # before the capture: occupancies are looked up once
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    nodes = ctypes.c_size_t(0)
    rc = ctypes.CDLL("libamdhip64.so").hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None,
                                                        ctypes.byref(nodes))
    assert rc == 0
    print(f"[gpu] {segments} queues: {nodes.value} launches", flush=True)
    assert nodes.value <= most
