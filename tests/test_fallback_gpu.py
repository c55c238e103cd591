"""Orders against the sampling where each path meets them: batches and replayed
batch graphs whose levels are chased (the bounded fallback with a batch's outputs
and with sizes from the device), and independent walks with more than one level,
alone and above a chased level: rulers after or before all other elements, of the
first level or of the second. Rulers first leave the last of them before a long
stretch without any, which the doubling of the rulers gives up on and the
downward passes finish."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_09318_amd as lr
import workloads
from adversarial import level_seed, sampled
from gpu_util import dev, host_u32

pytestmark = pytest.mark.gpu


def spacings(n, w=lr.LR_W_NONE, opts=None):
    p = lr.lr_plan_query(n, w, opts)
    return [int(p.spacing[i]) for i in range(p.levels)]


def rulers_and_others(n, k, seed_l, first):
    r = sampled(n, k, seed_l)
    is_r = np.zeros(n, bool)
    is_r[r] = True
    others = np.nonzero(~is_r)[0].astype(np.uint32)
    parts = [others[workloads.perm(others.size, 5, 1)], r[workloads.perm(r.size, 5, 2)]]
    return np.concatenate(parts[::-1] if first else parts).astype(np.uint32)


def level0_order(n, ks, first):
    return rulers_and_others(n, ks[0], level_seed(0, 0), first)


def level1_order(n, ks, first):
    """Rulers evenly among the other elements, but the second level's rulers
    before or after all others of theirs."""
    r0 = sampled(n, ks[0], level_seed(0, 0))
    rseq = r0[rulers_and_others(r0.size, ks[1], level_seed(0, 1), first)]
    is_r = np.zeros(n, bool)
    is_r[r0] = True
    others = np.nonzero(~is_r)[0].astype(np.uint32)
    others = others[workloads.perm(others.size, 6, 1)]
    cuts = (np.arange(1, r0.size + 1, dtype=np.int64) * others.size) // r0.size
    return np.insert(others, cuts, rseq)


# independent walks of one level | of two | above a chased level | of two above it
@pytest.mark.parametrize("n", [300_007, (1 << 20) + 3, 3_000_001, 12_000_007])
@pytest.mark.parametrize("make", [level0_order, level1_order])
@pytest.mark.parametrize("first", [False, True])
def test_rank(n, make, first):
    print(f"case: against the sampling, {make.__name__} first={first} n={n}", flush=True)
    succ = workloads.link_order(make(n, spacings(n), first))
    r, t = lr.rank(dev(succ), opts=lr.make_opts(flags=lr.LR_PROFILE))
    fell_back = lr.lr_profile_last()[7]
    torch.cuda.synchronize()
    _, er, et, _ = oracle.rank(succ)
    assert np.array_equal(host_u32(r), er) and np.array_equal(host_u32(t), et)
    assert make is not level0_order or fell_back == 1.0


@pytest.mark.parametrize("n", [100_003, (1 << 19) - 1, (1 << 19) + 3, 3_000_001])
@pytest.mark.parametrize("make", [level0_order, level1_order])
@pytest.mark.parametrize("first", [False, True])
def test_prefix_sums(n, make, first):
    print(f"case: against the sampling, sums, {make.__name__} first={first} n={n}", flush=True)
    succ = workloads.link_order(make(n, spacings(n, lr.LR_W_I64), first))
    w = workloads.weights(n, seed=5, stream=1, lo=-(1 << 40), hi=1 << 40)
    s, r, t = lr.prefix_sum(dev(succ), dev(w))
    torch.cuda.synchronize()
    _, er, et, es = oracle.rank(succ, w)
    assert np.array_equal(s.cpu().numpy(), es)
    assert np.array_equal(host_u32(r), er) and np.array_equal(host_u32(t), et)


def batch_inputs(sizes, N, k0, at):
    """Random requests, that number `at` with the rulers of its ids in the
    concatenation after its other elements."""
    inputs = [workloads.random_list(n, seed=70 + i).succ for i, n in enumerate(sizes)]
    lo, n = sum(sizes[:at]), sizes[at]
    r = sampled(N, k0, level_seed(0, 0))
    r = r[(r >= lo) & (r < lo + n)] - lo
    is_r = np.zeros(n, bool)
    is_r[r] = True
    others = np.nonzero(~is_r)[0].astype(np.uint32)
    order = np.concatenate([others[workloads.perm(others.size, 7, 1)], r[workloads.perm(r.size, 7, 2)]])
    inputs[at] = workloads.link_order(order.astype(np.uint32))
    return inputs


def run_batch(inputs, launch):
    items = [(dev(a), torch.full((a.size,), -1, dtype=torch.int32, device="cuda"),
              torch.full((a.size,), -1, dtype=torch.int32, device="cuda")) for a in inputs]
    reqs = lr.requests(items)
    torch.cuda.synchronize()
    assert launch(reqs, len(items)) == lr.LR_OK
    torch.cuda.synchronize()
    for a, (_, r, t) in zip(inputs, items):
        _, er, et, _ = oracle.rank(a)
        assert np.array_equal(host_u32(r), er) and np.array_equal(host_u32(t), et)


@pytest.mark.parametrize("sizes", [[5000, 1 << 18, 70_001, 3, 1_900_000], [2_300_000], [1, 1_500_000, 1_500_000]])
def test_chased_batch(sizes):
    N = sum(sizes)
    at = int(np.argmax([0 if n == 1_900_000 else n for n in sizes]))
    print(f"case: chased batch {sizes}, request {at} against the sampling", flush=True)
    assert N >= 1 << 21
    o = lr.make_opts(flags=lr.LR_PROFILE)
    run_batch(batch_inputs(sizes, N, spacings(N)[0], at),
              lambda reqs, k: lr.lr_rank_batch(reqs, k, lr.workspace(lr.lr_batch_workspace_bytes(reqs, k, o)), o))
    assert lr.lr_profile_last()[7] == 1.0


def test_chased_batch_graph_with_sizes_from_the_device():
    cap = (1 << 21) + 5
    print(f"case: chased batch graph, capacity {cap}, against the sampling", flush=True)
    cfg = lr.batch_graph_config(cap, 4, True)
    g = lr.BatchGraph(cfg, lr.workspace(lr.lr_batch_graph_workspace_bytes(cfg)))
    k0 = spacings(cap, opts=lr.make_opts(flags=lr.LR_NO_LOCAL))[0]
    for sizes, at in (([5000, 1 << 18, 3], 1), ([cap], 0), ([70_001, 12], 0)):
        run_batch(batch_inputs(sizes, sum(sizes), k0, at), g.launch)
        run_batch([workloads.random_list(n, seed=n % 9).succ for n in sizes], g.launch)  # and an ordinary replay after it
    g.close()
