"""lr_autotune where the planner's own plan does not fit the trial workspace: it
returns the fastest of the others but stores nothing, so default calls keep the
planner's plan; with room for it the winner is stored."""
import pytest
import torch

import paper_2606_09318_amd as lr
import workloads
from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def empty_cache():
    lr.autotune_cache_clear()
    yield
    lr.autotune_cache_clear()


@pytest.mark.parametrize("n", [20_000, 1 << 20])
@pytest.mark.parametrize("weighted", [False, True])
def test_winner_is_stored_only_if_it_beat_the_planners_plan(n, weighted):
    print(f"case: autotune without room for the planner's plan, n={n} weighted={weighted}", flush=True)
    succ = dev(workloads.random_list(n, seed=3).succ)
    w = torch.ones(n, dtype=torch.int64, device="cuda") if weighted else None
    wt = lr.LR_W_I64 if weighted else lr.LR_W_NONE
    out = n * (8 if weighted else 4) + 4096
    own, named = lr.lr_workspace_bytes(n, wt), lr.lr_workspace_bytes(n, wt, lr.make_opts(spacing=(16, 8)))
    assert own > named + 4096
    before = lr.lr_plan_query(n, wt)
    st, best, ms = lr.lr_autotune(succ, w, lr.workspace(named + out))
    assert st == lr.LR_OK and len(ms) >= 4 and best.spacing[0] >= 2
    assert lr.autotune_cache_entries() == 0
    after = lr.lr_plan_query(n, wt)
    assert [after.spacing[i] for i in range(after.levels)] == [before.spacing[i] for i in range(before.levels)]
    assert after.base_max == before.base_max
    st, _, _ = lr.lr_autotune(succ, w, lr.workspace(own + out))
    assert st == lr.LR_OK and lr.autotune_cache_entries() == 1
