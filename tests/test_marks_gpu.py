"""Grouped predecessor marks: forests ranked through the visit log, whose
initial elements come from one grouping pass and LDS bitmaps. Whole numbers,
compared for equality with the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_09318_amd as lr
import workloads

pytestmark = pytest.mark.gpu


def check(succ, weight=None):
    o = lr.make_opts(flags=lr.LR_VISIT_LOG | lr.LR_NO_LOCAL)
    d = torch.from_numpy(succ.view(np.int32)).to("cuda:0")
    if weight is None:
        r, t = lr.rank(d, want_root=True, opts=o)
        st, er, et, _ = oracle.rank(succ)
    else:
        s, r, t = lr.prefix_sum(d, torch.from_numpy(weight).to("cuda:0"), opts=o)
        st, er, et, es = oracle.rank(succ, weight)
    torch.cuda.synchronize()
    assert st == 0
    assert np.array_equal(r.cpu().numpy().view(np.uint32), er)
    assert np.array_equal(t.cpu().numpy().view(np.uint32), et)
    if weight is not None:
        assert np.array_equal(s.cpu().numpy(), es)


# groups of 8192 ids up to 2^22 elements, of 16384 above; a grouping tile holds 16384 targets
@pytest.mark.parametrize("n", [65536, 65537, 73727, 73728, 8192 * 9 + 15, 8192 * 9 + 33, 1 << 20, (1 << 22) - 1,
                               (1 << 22) + 1, 16384 * 300 + 31])
def test_forests(n):
    print(f"case: grouped marks n={n}", flush=True)
    F = workloads.forest(n, mean=64, n_long=1, long_len=1024, seed=n)
    check(F.succ)
    check(F.succ, F.weight)


@pytest.mark.parametrize("n", [65536, 100_003])
@pytest.mark.parametrize("shape", ["all terminals", "two lists", "pairs", "one full group"])
def test_few_and_many_targets(n, shape):
    """No target at all; every id but two a target; every other id; the
    targets all in one group."""
    print(f"case: grouped marks {shape} n={n}", flush=True)
    i = np.arange(n, dtype=np.uint32)
    succ = i.copy()
    if shape == "two lists":
        succ = np.minimum(i + 1, n - 1).astype(np.uint32)
        succ[n // 2] = n // 2
    elif shape == "pairs":
        succ = (i | 1).astype(np.uint32)
        succ[succ >= n] = n - 1
    elif shape == "one full group":
        succ[8192:16384] = i[:8192]
    check(succ)


@pytest.mark.parametrize("n", [(1 << 20) - 1, 1 << 20, (1 << 20) + 33, (5 << 19) - 1, 5 << 19, (5 << 19) + 33])
def test_slot_array_forests(n):
    """Without the visit log: byte stores below, groups in the slot array from
    2^20 elements on."""
    print(f"case: grouped marks without the log n={n}", flush=True)
    F = workloads.forest(n, mean=64, n_long=1, long_len=4096, seed=n)
    d = torch.from_numpy(F.succ.view(np.int32)).to("cuda:0")
    s, r, t = lr.prefix_sum(d, torch.from_numpy(F.weight).to("cuda:0"))
    r2, t2 = lr.rank(d, want_root=True)
    torch.cuda.synchronize()
    st, er, et, es = oracle.rank(F.succ, F.weight)
    assert st == 0
    assert np.array_equal(s.cpu().numpy(), es)
    for got, ex in ((r, er), (t, et), (r2, er), (t2, et)):
        assert np.array_equal(got.cpu().numpy().view(np.uint32), ex)
