// Prints the plans of one call (host code of liblr.so): levels, how many of them
// are chased, whether the rest is ranked by independent walks, spacings, base,
// the first level's sampling seed.
//   plan_probe load FILE n weighted          after loading a cache file
//   plan_probe store n0 n weighted k0 k1 bm  after storing that plan, tuned at n0
//   plan_probe opts n weighted flags bm k... with explicit options
//   plan_probe seed n weighted seed          with another sampling seed
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "plan.hpp"

using namespace lr;

static void show(const char* name, const Plan& p) {
    printf("%s levels=%u run=%u iw=%d top=%u base=%u k=", name, p.levels, p.run, p.iw, p.iw ? p.top : 0, p.base_max);
    for (uint32_t l = 0; l < p.levels; ++l) printf("%s%u", l ? "," : "", 1u << p.log2k[l]);
    printf(" lw=%u refill=%u seed=%08x\n", p.lane_walks, p.refill, p.levels ? p.lseed[0] : 0u);
}

int main(int argc, char** argv) {
    auto num = [&](int i) { return i < argc ? strtoull(argv[i], nullptr, 10) : 0ull; };
    uint64_t n;
    bool weighted;
    lr_opts o{};
    bool named = false;
    if (argc > 4 && !strcmp(argv[1], "load")) {
        if (lr_autotune_cache_load(argv[2]) != LR_OK) return 2;
        n = num(3), weighted = num(4) != 0;
    } else if (argc > 7 && !strcmp(argv[1], "store")) {
        n = num(3), weighted = num(4) != 0;
        lr_opts best{};
        best.spacing[0] = (uint32_t)num(5), best.spacing[1] = (uint32_t)num(6), best.base_max = (uint32_t)num(7);
        best.lane_walks = best.refill = 1;
        if (!best.base_max) {  // the planner's own, spelt out as lr_autotune returns it
            PlanSet ps;
            if (make_plans(num(2), weighted, nullptr, 0, &ps) != LR_OK) return 2;
            for (uint32_t l = 0; l < ps.p.levels; ++l) best.spacing[l] = 1u << ps.p.log2k[l];
            best.base_max = ps.p.base_max;
        }
        tune_store(num(2), weighted, best, 1.0);
    } else if (argc > 5 && !strcmp(argv[1], "opts")) {
        n = num(2), weighted = num(3) != 0, o.flags = (uint32_t)num(4), o.base_max = (uint32_t)num(5);
        for (int i = 6; i < argc && i - 6 < LR_MAX_LEVELS; ++i) o.spacing[i - 6] = (uint32_t)num(i);
        named = true;
    } else if (argc > 4 && !strcmp(argv[1], "seed")) {
        n = num(2), weighted = num(3) != 0, o.seed = num(4);
        named = true;
    } else {
        return 3;
    }
    PlanSet ps;
    if (make_plans(n, weighted, named ? &o : nullptr, 0, &ps) != LR_OK) return 4;
    show("plain", ps.p);
    if (ps.autol) show("contracted", ps.lp);
    if (ps.small) show("short", ps.sp);
    return 0;
}
