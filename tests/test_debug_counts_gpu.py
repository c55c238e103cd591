"""What the write-counting debug build counts under default options: inputs that
the release build ranks by independent walks, and forests whose predecessor
marks are grouped, are still refused when an element has two predecessors."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2606_09318_amd as lr
import workloads
from paper_2606_09318_amd import build as lr_build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dbg():
    lr.load()  # torch's HIP runtime first, as the binding does
    L = ctypes.CDLL(lr_build.DEBUG_LIB)
    L.lr_workspace_bytes.restype = ctypes.c_size_t
    vp, u64, sz = ctypes.c_void_p, ctypes.c_uint64, ctypes.c_size_t
    L.lr_workspace_bytes.argtypes = [u64, ctypes.c_int, vp]
    L.lr_rank.argtypes = [vp, vp, vp, u64, vp, sz, vp, vp]
    L.lr_prefix_sum.argtypes = [vp, vp, ctypes.c_int, vp, vp, vp, u64, vp, sz, vp, vp]
    return L


def run(L, succ_np, weight_np, flags):
    n = succ_np.size
    succ = torch.from_numpy(succ_np.view(np.int32)).cuda()
    r, t = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    o = ctypes.byref(lr.make_opts(flags=flags)) if flags else None
    w = lr.LR_W_NONE if weight_np is None else lr.LR_W_I64
    ws = torch.empty(L.lr_workspace_bytes(n, w, o), dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    if weight_np is None:
        rc = L.lr_rank(succ.data_ptr(), r.data_ptr(), t.data_ptr(), n, ws.data_ptr(), ws.numel(), o, st)
        s = None
    else:
        wt = torch.from_numpy(weight_np).cuda()
        s = torch.empty(n, dtype=torch.int64, device="cuda")
        rc = L.lr_prefix_sum(succ.data_ptr(), wt.data_ptr(), w, s.data_ptr(), r.data_ptr(), t.data_ptr(), n,
                             ws.data_ptr(), ws.numel(), o, st)
    torch.cuda.synchronize()
    return rc, r.cpu().numpy().view(np.uint32), t.cpu().numpy().view(np.uint32), None if s is None else s.cpu().numpy()


@pytest.mark.parametrize("kind,n,flags", [("random", 20_001, 0), ("random", 300_007, 0), ("random", (1 << 20) + 3, 0),
                                          ("forest", 20_001, 0), ("forest", (1 << 20) - 1, 0),
                                          ("forest", (1 << 20) + 3, 0), ("forest", 1 << 18, lr.LR_VISIT_LOG)])
@pytest.mark.parametrize("weighted", [False, True])
def test_two_predecessors_are_refused_and_forests_are_not(dbg, kind, n, flags, weighted):
    print(f"case: debug counts {kind} n={n} flags={flags} weighted={weighted}", flush=True)
    if kind == "forest":
        a = workloads.forest(n, mean=16, n_long=1, long_len=n // 8, seed=n % 97).succ
    else:
        a = workloads.random_list(n, seed=n % 97).succ
    w = workloads.weights(n, seed=2, stream=0, lo=-9, hi=9) if weighted else None
    rc, r, t, s = run(dbg, a, w, flags)
    assert rc == lr.LR_OK
    _, er, et, es = oracle.rank(a, w)
    assert np.array_equal(r, er) and np.array_equal(t, et) and (s is None or np.array_equal(s, es))
    b = a.copy()
    links = np.nonzero(a != np.arange(n, dtype=np.uint32))[0]
    x, y = int(links[n // 50]), int(links[n // 3])
    b[y] = b[x]
    assert run(dbg, b, w, flags)[0] == lr.LR_ERR_BAD_LIST
