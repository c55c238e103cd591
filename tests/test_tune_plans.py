"""The autotune cache and the planner's own plan (host-only): an entry that keeps
the planner's spacings (k0 = k1 = 0, as a winning plan without a ruling-set level
has) is loaded and saved like any other."""
import pytest

import paper_2606_09318_amd as lr


@pytest.fixture(autouse=True)
def empty_cache():
    lr.autotune_cache_clear()
    yield
    lr.autotune_cache_clear()


def levels(n, w=lr.LR_W_NONE):
    p = lr.lr_plan_query(n, w)
    return [int(p.spacing[i]) for i in range(p.levels)], int(p.base_max)


def write(path, rows):
    with open(path, "w") as fh:
        for r in rows:
            fh.write(" ".join(str(x) for x in r) + "\n")


@pytest.mark.parametrize("base_max", [0, 16384])
def test_entry_with_the_planners_spacings_round_trips(tmp_path, base_max):
    arch = lr.autotune_arch()
    f, g = str(tmp_path / "a.txt"), str(tmp_path / "b.txt")
    default = levels(12_000)
    write(f, [(arch, 13, 0, 0, 0, base_max, 1, 1, 0.5), (arch, 20, 0, 32, 8, 4096, 1, 1, 0.5)])
    assert lr.autotune_cache_load(f) == lr.LR_OK and lr.autotune_cache_entries() == 2
    assert levels(12_000) == default
    assert levels(1 << 20)[0][:2] == [32, 8]
    assert lr.autotune_cache_save(g) == lr.LR_OK
    lr.autotune_cache_clear()
    assert lr.autotune_cache_load(g) == lr.LR_OK and lr.autotune_cache_entries() == 2
    assert levels(12_000) == default


def test_second_spacing_needs_a_first(tmp_path):
    f = str(tmp_path / "a.txt")
    write(f, [(lr.autotune_arch(), 20, 0, 0, 8, 4096, 1, 1, 0.5)])
    assert lr.autotune_cache_load(f) == lr.LR_ERR_INVALID_ARG and lr.autotune_cache_entries() == 0
