"""Independent walks (lists below about 2^20 elements and the levels above a
chased one): the sizes where their levels, tiles and dispatch change, orders
against the sampling, cycles, and the same inputs through the chased levels
(a plan named by its spacings is followed down to the base case)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2606_09318_amd as lr
import workloads
from adversarial import rulers_last
from gpu_util import dev, host_u32

pytestmark = pytest.mark.gpu


def make(kind, n, seed):
    if kind == "forest":
        return workloads.forest(n, mean=5, n_long=1, long_len=n // 3, seed=seed).succ
    if kind == "identity":
        return workloads.identity_list(n).succ
    if kind == "reversed":
        return np.maximum(np.arange(n, dtype=np.int64) - 1, 0).astype(np.uint32)
    if kind == "singletons":
        return np.arange(n, dtype=np.uint32)
    return workloads.random_list(n, seed=seed).succ


def check(succ_np, weight_np=None, opts=None):
    n = succ_np.size
    _, er, et, es = oracle.rank(succ_np, weight_np)
    succ = dev(succ_np)
    if weight_np is None:
        r, t = lr.rank(succ, opts=opts)
    else:
        s, r, t = lr.prefix_sum(succ, dev(weight_np), opts=opts)
    torch.cuda.synchronize()
    if weight_np is not None:
        assert np.array_equal(s.cpu().numpy(), es), n
    assert np.array_equal(host_u32(r), er) and np.array_equal(host_u32(t), et), n


# base case (its columns) | doubling alone | one level of walks | two levels | chased above
SIZES = [1, 1024, 1025, 2049, 4096, 4097, 8192, 8193, 65535, 65536, 65537, 131072 + 5, (1 << 18) - 1, (1 << 19) + 255, (1 << 19) + 257, (1 << 20) + 1,
         (1 << 21) - 1, 1 << 21, (1 << 21) + 1, (1 << 23) - 1, 1 << 23]


@pytest.mark.parametrize("kind", ["random", "forest", "identity", "reversed", "singletons"])
@pytest.mark.parametrize("n", SIZES)
def test_rank_at_the_edges(kind, n):
    print(f"case: independent walks {kind} n={n}", flush=True)
    succ = make(kind, n, n % 97)
    check(succ)
    if 1 < n < (1 << 20):
        check(succ, opts=lr.make_opts(spacing=(4, 2), base_max=8192))


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("kind", ["random", "forest", "identity"])
@pytest.mark.parametrize("n", [1, 1025, 2049, 4097, 8192, 8193, 16384, 16385, 32768, 131072 + 7, (1 << 18) + 1, (1 << 19) - 1, 1 << 19,
                               (1 << 22) + 3])
def test_prefix_sums_at_the_edges(n, kind, dtype):
    print(f"case: independent walks sums {kind} {dtype.__name__} n={n}", flush=True)
    lo, hi = (-(1 << 31), (1 << 31) - 1) if dtype == np.int32 else (-(1 << 40), 1 << 40)  # both halves of a sum
    w = workloads.weights(n, seed=n % 89, stream=3, lo=lo, hi=hi, dtype=dtype)
    check(make(kind, n, n % 97), w)


@pytest.mark.parametrize("n", [100_003, (1 << 19) + 3, (1 << 20) + 7])
@pytest.mark.parametrize("weighted", [False, True])
def test_order_against_the_sampling(n, weighted):
    """Every sampled ruler after all other elements: the downward pass finds a
    stretch of almost the whole list without a ruler."""
    print(f"case: independent walks, rulers last, n={n} weighted={weighted}", flush=True)
    k0 = int(lr.lr_plan_query(n, lr.LR_W_I64 if weighted else lr.LR_W_NONE).spacing[0])
    L = rulers_last(n, k0)
    w = workloads.weights(n, seed=5, stream=1, lo=-(1 << 33), hi=1 << 33) if weighted else None
    check(L.succ, w)


@pytest.mark.parametrize("n", [5000, 70_001, 300_007, (1 << 20) + 3])
@pytest.mark.parametrize("weighted", [False, True])
def test_cycles_end_and_are_reported(n, weighted):
    """One list and one cycle over the other half of the elements, and a
    cycle over all of them: the call ends, and LR_VALIDATE reports it."""
    print(f"case: independent walks, cycles, n={n} weighted={weighted}", flush=True)
    L = workloads.random_list(n, seed=11)
    for start in (0, n // 2):
        a = L.succ.copy()
        a[L.order[-1]] = L.order[start]
        if start:
            a[L.order[start - 1]] = L.order[start - 1]
        succ = dev(a)
        w = torch.ones(n, dtype=torch.int64, device="cuda") if weighted else None
        for flags in (0, lr.LR_VALIDATE):
            o = lr.make_opts(flags=flags)
            ws = lr.workspace(lr.lr_workspace_bytes(n, lr.LR_W_I64 if weighted else lr.LR_W_NONE, o))
            r = torch.empty(n, dtype=torch.int32, device="cuda")
            if weighted:
                s = torch.empty(n, dtype=torch.int64, device="cuda")
                st = lr.lr_prefix_sum(succ, w, s, r, None, ws, o)
            else:
                st = lr.lr_rank(succ, r, None, ws, o)
            torch.cuda.synchronize()
            assert st == (lr.LR_ERR_BAD_LIST if flags else lr.LR_OK)


def test_plans_named_by_their_own_spacings_take_the_same_route():
    """Options that spell out the planner's plan are ranked like the defaults."""
    n = 300_001
    p = lr.lr_plan_query(n)
    o = lr.make_opts(spacing=[p.spacing[i] for i in range(p.levels)], base_max=p.base_max)
    print("case: named plan", flush=True)
    check(make("random", n, 3), opts=o)
    q = lr.lr_plan(); assert lr.load().lr_plan_query(n, 0, ctypes.byref(o), ctypes.byref(q)) == 0
    assert [q.spacing[i] for i in range(q.levels)] == [p.spacing[i] for i in range(p.levels)]


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


@pytest.mark.parametrize("count,n", [(1, 1), (1, 8192), (2, 4097), (96, 80), (97, 90), (200, 41), (96, 700), (97, 10_007)])
def test_batches_read_in_place(count, n):
    """Batches that are ranked from their requests' arrays, around the table
    sizes of one launch (96 requests), with an empty request among them."""
    print(f"case: independent walks, batch of {count} x {n}", flush=True)
    inputs = [make("forest" if i % 3 == 2 and n > 100 else "random", n + i % 5, i) for i in range(count)]
    if count > 2:
        inputs[1] = np.zeros(0, np.uint32)
    run_batch(inputs, lambda reqs, k: lr.lr_rank_batch(reqs, k, lr.workspace(lr.lr_batch_workspace_bytes(reqs, k))))


@pytest.mark.parametrize("cap", [3000, 20_000, 120_000, 900_000])
def test_batch_graph_sizes_from_the_device(cap):
    """A graph planned for `cap` elements replayed with fewer."""
    print(f"case: independent walks, graph capacity {cap}", flush=True)
    cfg = lr.batch_graph_config(cap, 8, True)
    g = lr.BatchGraph(cfg, lr.workspace(lr.lr_batch_graph_workspace_bytes(cfg)))
    for k, sizes in enumerate([[cap], [1, cap // 3, cap // 2], [2], [cap // 5, 7, cap // 4 + 1]]):
        inputs = [make("forest" if (i + k) % 3 == 2 and n > 100 else "random", n, 31 * k + i) for i, n in enumerate(sizes)]
        run_batch(inputs, g.launch)
    g.close()


def local_forest(n, seed, gamma):
    """Lists stored mostly in id order: the identity order with a share gamma
    of its positions permuted, cut into lists at random."""
    order = workloads.gamma_order(n, gamma, seed)
    rng = np.random.default_rng(seed)
    ends = rng.random(n) < 1e-4
    ends[-1] = True
    succ = np.empty(n, np.uint32)
    succ[order] = np.where(ends, order, np.roll(order, -1))
    return succ


# contracted lists that are not chased (short), that are, and one handed back
# to the plain path; around the sizes where the contracted plan gains a level
@pytest.mark.parametrize("n,gamma", [((1 << 21) + 9, 0.01), (6_710_000, 0.1), (6_720_000, 0.1), (7_000_001, 0.001),
                                     (1 << 24, 0.05), ((1 << 24) + 3, 0.1), (30_000_001, 0.002), (30_000_001, 0.1)])
@pytest.mark.parametrize("weighted", [False, True])
def test_contracted_lists(n, gamma, weighted):
    if weighted and n > (1 << 24):
        n = (1 << 24) + 3
    print(f"case: contracted lists n={n} gamma={gamma} weighted={weighted}", flush=True)
    succ = local_forest(n, n % 83, gamma)
    w = workloads.weights(n, seed=4, stream=2, lo=-(1 << 30), hi=1 << 30) if weighted else None
    check(succ, w)
    check(succ, w, opts=lr.make_opts(flags=lr.LR_LOCAL))


def test_contracted_path_on_a_list_that_is_too_long():
    """Forced contraction of a random list: nothing contracts, the list has as
    many elements as the input and its levels are chased."""
    n = (1 << 22) + 1
    print("case: contracted random list", flush=True)
    check(make("random", n, 5), opts=lr.make_opts(flags=lr.LR_LOCAL))
