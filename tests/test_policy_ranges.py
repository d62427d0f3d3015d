"""The ranges of the comparison policies: 512 to 4096 positions per wave, by
the queue's size. Schedules on both sides of every edge against the C oracle
(whole numbers, so bit-exact), and the workspace never shrinks with the size."""

import numpy as np
import pytest

import paper_2506_12204_amd as ss
from oracle import POLICY_FCFS, POLICY_HPJF, POLICY_SJF, c_oracle_policy
from tests._lib import assert_same, ensure_built, gpu_available
from workloads import fuzz_queue

POLICIES = [POLICY_FCFS, POLICY_SJF, POLICY_HPJF]
EDGES = [1 << 19, 1 << 21, 1 << 23]  # twice the range from here on


@pytest.mark.parametrize("policy", POLICIES)
def test_workspace_never_shrinks(policy):
    ensure_built()
    sizes = sorted(n for e in EDGES for n in (e // 2, e - 1, e, e + 1, e + 5000, e + e // 2))
    need = [int(ss._load().sem_policy_workspace_bytes(policy, n)) for n in sizes]
    assert need == sorted(need)


# Sizes that a caller may have kept from when all ranges were 4096 positions
KEPT = {(POLICY_FCFS, 1000): 5120, (POLICY_FCFS, 50003): 17408, (POLICY_FCFS, 524288): 132864,
        (POLICY_FCFS, 3000000): 760320, (POLICY_SJF, 1000): 5888, (POLICY_SJF, 16384): 21248,
        (POLICY_SJF, 16385): 2607616, (POLICY_SJF, 524288): 16940032,
        (POLICY_SJF, 3000000): 86899456, (POLICY_HPJF, 1000): 11008, (POLICY_HPJF, 50003): 60160,
        (POLICY_HPJF, 524288): 528128, (POLICY_HPJF, 3000000): 3009280}


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("policy,n", sorted(KEPT))
def test_kept_workspace_size(policy, n):
    import torch
    ensure_built()
    p, l = fuzz_queue(n, seed=n % 1009 + policy, classes=70, max_len=5000, tie_frac=0.2)
    dev = torch.device("cuda")
    tp = torch.from_numpy(np.ascontiguousarray(p, dtype=np.uint8)).to(dev)
    tl = torch.from_numpy(np.ascontiguousarray(l, dtype=np.int32)).to(dev)
    size = KEPT[policy, n]
    print(f"[gpu] policy {policy} n={n} in {size} bytes", flush=True)
    ws = torch.full((size + 65536,), 0xA5, dtype=torch.uint8, device=dev)
    order = torch.empty(n, dtype=torch.int32, device=dev)
    wait = torch.empty(n, dtype=torch.int64, device=dev)
    totals = torch.empty((257, 2), dtype=torch.int64, device=dev)
    stream = ss._stream_handle(dev)
    rc = ss.lib.sem_schedule_policy_async(policy, ss._ptr(tp), ss._ptr(tl), n, ss._ptr(order),
                                          ss._ptr(wait), ss._ptr(totals), ss._ptr(ws), size,
                                          stream)
    assert rc == ss.SEM_OK and ss.lib.sem_check(ss._ptr(ws), stream) == ss.SEM_OK
    assert bool((ws[size:] == 0xA5).all())
    assert_same((order.cpu().numpy(), wait.cpu().numpy(), ss.totals_to_ints(totals)),
                c_oracle_policy(p, l, policy), f"policy {policy} n={n} kept size")


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("policy", [POLICY_FCFS, POLICY_HPJF])
@pytest.mark.parametrize("n,classes", [
    (511, 6), (512, 6), (513, 6), (2047, 40), (2049, 6),
    (EDGES[0] - 1, 6), (EDGES[0], 40), (EDGES[0] + 1, 6),
    (EDGES[1] - 1, 6), (EDGES[1], 6), (EDGES[1] + 1023, 9),
    (EDGES[2] - 1, 6), (EDGES[2], 6), (EDGES[2] + 2047, 9)])
def test_range_edges(policy, n, classes):
    import torch
    ensure_built()
    p, l = fuzz_queue(n, seed=n % 1009 + policy, classes=classes, max_len=5000, tie_frac=0.2)
    print(f"[gpu] policy {policy} n={n} classes={classes}", flush=True)
    dev = torch.device("cuda")
    order, wait, totals = ss.schedule_policy(
        torch.from_numpy(np.ascontiguousarray(p, dtype=np.uint8)).to(dev),
        torch.from_numpy(np.ascontiguousarray(l, dtype=np.int32)).to(dev), policy)
    assert_same((order.cpu().numpy(), wait.cpu().numpy(), totals),
                c_oracle_policy(p, l, policy), f"policy {policy} n={n}")
