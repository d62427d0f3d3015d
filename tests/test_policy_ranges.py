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
