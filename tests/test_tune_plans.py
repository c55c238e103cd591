"""The autotune cache and the planner's own plan (host-only): an entry that keeps
the planner's spacings (k0 = k1 = 0, as a winning plan without a ruling-set level
has) is loaded and saved like any other, and an entry whose levels are the planner's
leaves every call of its size bucket the planner's own route. The route (which
levels are chased, which are ranked by independent walks) is read from the
library's plans by tests/plan_probe.cpp."""
import os
import subprocess

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


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    pkg, exe = os.path.join(root, "paper_2606_09318_amd"), str(tmp_path_factory.mktemp("probe") / "plan_probe")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(root, "include"),
                    "-I", os.path.join(pkg, "csrc"), os.path.join(root, "tests", "plan_probe.cpp"), "-o", exe,
                    lr.LIB_PATH, "-L/opt/rocm/lib", "-lamdhip64",
                    f"-Wl,-rpath,{os.path.dirname(lr.LIB_PATH)}:/opt/rocm/lib"], check=True)

    def run(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, (args, r.returncode, r.stderr)
        return r.stdout

    return run


# sizes at both ends of a bucket in which the planner changes its spacings or its base size
@pytest.mark.parametrize("n0,n", [(1 << 22, 1 << 22), (1 << 22, (1 << 23) - 1), ((1 << 23) - 1, 1 << 22),
                                  (1 << 27, (1 << 28) - 1), ((1 << 28) - 1, 1 << 27), (12_000, 8193), (12_000, 16_383),
                                  (1 << 17, (1 << 18) - 1), (1 << 20, (1 << 21) - 1)])
@pytest.mark.parametrize("weighted", [0, 1])
def test_planners_own_entry_leaves_the_planners_route(probe, n0, n, weighted):
    assert probe("store", n0, n, weighted, 0, 0, 0) == probe("opts", n, weighted, 0, 0)


@pytest.mark.parametrize("weighted", [0, 1])
def test_a_tuned_base_size_stays_with_the_plain_levels(probe, weighted):
    n = 1 << 24
    default, tuned = (probe(*a).splitlines() for a in (("opts", n, weighted, 0, 0),
                                                       ("store", n, n, weighted, 64, 16, 2048)))
    assert tuned[0].startswith("plain") and " iw=0 " in tuned[0] and "base=2048 k=64,16" in tuned[0]
    assert tuned[1:] == default[1:] and " iw=1 " in tuned[1]


def test_options_that_spell_out_the_planners_levels_take_its_route(probe):
    n = 1 << 22
    p = lr.lr_plan_query(n)
    assert probe("opts", n, 0, 0, p.base_max, *[p.spacing[i] for i in range(p.levels)]) == probe("opts", n, 0, 0, 0)
    # a base size that changes the levels is followed by both paths
    other = probe("opts", n, 0, 0, 2048).splitlines()
    assert len(other) >= 2 and all(" iw=0 " in ln and "base=2048" in ln for ln in other)


@pytest.mark.parametrize("weighted", [0, 1])
def test_every_path_samples_with_the_seed_of_the_call(probe, weighted):
    """Another seed samples other rulers: the way out of an order against the
    sampling, on short contracted lists too."""
    seeds = [[ln.split("seed=")[1] for ln in probe("seed", 1 << 24, weighted, s).splitlines()] for s in (0, 12345)]
    assert len(seeds[0]) == 3 and all(len(set(x)) == 1 for x in seeds) and seeds[0] != seeds[1]
