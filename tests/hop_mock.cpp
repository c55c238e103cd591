// The stopping rule of the pointer-doubling loops (csrc/hop.hpp) on the CPU:
// lanes compose records in place in a random order, as the kernels do, over
// lists, over cycles and over arbitrary memory (records that input which is not
// a forest leaves unwritten). Every lane must end within as many hops as the
// input has elements, and on lists with the right rank.
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "hop.hpp"

static const uint32_t TERM = 0x80000000u;
struct Rec { uint32_t nxt, c; };

// Runs all lanes; false: some lane took more than `climit` hops.
template <class Stuck>
static bool run(std::vector<Rec> nodes, uint32_t climit, std::mt19937& rng, Stuck stuck, std::vector<Rec>* out = nullptr) {
    const uint32_t m = (uint32_t)nodes.size();
    std::vector<uint32_t> hops(m, 0), open;
    for (uint32_t i = 0; i < m; ++i)
        if (!(nodes[i].nxt & TERM)) open.push_back(i);
    while (!open.empty()) {
        const uint32_t k = rng() % open.size(), i = open[k];
        Rec r = nodes[i];
        bool bad = r.nxt >= m;
        if (!bad) {
            const uint32_t before = r.c;
            const Rec q = nodes[r.nxt];
            r.c += q.c;
            r.nxt = q.nxt;
            bad = stuck(before, r.c, (r.nxt & TERM) != 0, climit);
        }
        if (bad) r = {TERM | 0x7fffffffu, 0xffffffffu};
        nodes[i] = r;
        if (++hops[i] > climit + 1) return false;
        if (r.nxt & TERM) {
            open[k] = open.back();
            open.pop_back();
        }
    }
    if (out) *out = nodes;
    return true;
}

int main() {
    std::mt19937 rng(7);
    auto rule = [](uint32_t b, uint32_t a, bool e, uint32_t l) { return lr::hop_stuck(b, a, e, l); };
    auto counts_only = [](uint32_t, uint32_t a, bool, uint32_t l) { return a >= l; };
    int fails = 0;
    // lists: the rule never stops a valid one
    for (uint32_t n : {1u, 2u, 3u, 100u, 1000u}) {
        std::vector<uint32_t> order(n);
        for (uint32_t i = 0; i < n; ++i) order[i] = i;
        for (uint32_t i = n; i > 1; --i) std::swap(order[i - 1], order[rng() % i]);
        std::vector<Rec> a(n), o;
        for (uint32_t i = 0; i + 1 < n; ++i) a[order[i]] = {order[i + 1], 1};
        a[order[n - 1]] = {TERM | order[n - 1], 0};
        bool ok = run(a, n, rng, rule, &o);
        for (uint32_t i = 0; ok && i < n; ++i) ok = o[order[i]].c == n - 1 - i && o[order[i]].nxt == (TERM | order[n - 1]);
        if (!ok) ++fails, std::printf("list %u\n", n);
    }
    // a record that leads to itself and counts nothing: the count alone never ends it
    const std::vector<Rec> self = {{0, 0}, {0, 0}, {0, 3}};
    if (!run(self, 4096, rng, rule)) ++fails, std::printf("zero counts\n");
    if (run(self, 4096, rng, counts_only)) ++fails, std::printf("the count alone ended zero counts\n");
    // two records whose counts sum to 2^32
    const std::vector<Rec> wrap = {{1, 1}, {0, 0xffffffffu}, {0, 1}};
    if (!run(wrap, 4096, rng, rule)) ++fails, std::printf("wrapping counts\n");
    // arbitrary memory
    for (int t = 0; t < 4000; ++t) {
        const uint32_t m = 1 + rng() % 60, climit = m + rng() % 200;
        std::vector<Rec> a(m);
        for (auto& r : a) {
            const uint32_t kind = rng() % 8;
            r.nxt = kind == 0 ? TERM | (rng() % m) : kind == 1 ? rng() : rng() % m;
            r.c = (rng() % 3 == 0) ? 0u : (rng() % 3 == 0) ? 0u - rng() % 5 : (rng() % 5 == 0) ? rng() : rng() % 4;
        }
        if (!run(a, climit, rng, rule)) { ++fails; std::printf("random records %d\n", t); break; }
    }
    if (!fails) std::printf("ok\n");
    return fails != 0;
}
