// HIP kernels for gfx950 (wave64) and the launch sequences that chain them.
//
// Sparse ruling set (Section 2.1, Fig. 1), per level l of the recursion:
//   detect   (level 0 only) mark every element that has a predecessor;
//            unmarked elements are the initial elements (findInit). One list:
//            its head from a streaming sum (headsum). Forests from 2^20
//            elements on: link targets grouped by range (mark1), marks and
//            initial elements from LDS bitmaps (mark_bits), no heads pass.
//   heads    compact the initial elements that are not sampled rulers into a
//            walk list (tile count -> one-workgroup scan -> tile write).
//   chase    one lane per walk: from its start, follow succ and record in
//            slot[x] the walk id and the weight from the start to x, until the
//            next sampled ruler or a terminal (the ruler chasing loop). The
//            walk's end and total weight form the next level's element (for a
//            sampled ruler) or a parked record (for an initial element).
//   iw       the first level of at most about 2^21 elements and those above it
//            are ranked by independent walks: every element to the next ruler
//            (iw_first, iw_walk), asynchronous doubling on the last level
//            (iw_double), downward passes (iw_down). Inputs of that size take
//            the same kernels alone.
//   base     inputs of at most 8192 elements, and the last level of plans that
//            name their own levels, are ranked by pointer doubling in LDS by
//            one workgroup (the base case).
//   resolve  walks of initial elements take the result of the ruler (or
//            terminal) they ended on.
//   expand   every element takes rank = rank(walk) - offset and the walk's
//            root (ruler propagation).
// Walks run forward along succ, so ranks toward the terminal come out
// directly and no list reversal is needed.
//
// Level 0 of large inputs (n >= 2^25) logs the chase's visits and places the
// results by element range (place1/2/3) instead of storing at random
// addresses, and weighted inputs are interleaved into one record per element
// first (pair).
//
// Tile-local contraction (Section 2.3): chains of links inside 4096-id tiles
// are contracted first (lc_chain, lc_scan, lc_compact), the levels above rank
// the contracted list with sizes read from the device, and lc_expand restores
// every element. By default a sample of the tiles chooses on the device
// between this path and the plain one (lsample, ldecide; the exact count in
// lc_scan can still hand over to the plain path); both are enqueued and the
// kernels of the path not taken return at once (Gate).
//
// Ruler spawning (Section 2.2, LR_SPAWN): the input level is chased in two
// rounds (sp_chase1 capped at 2k steps; sp_count/scan/write spawn rulers at
// the cap targets and among the unreached elements; sp_chase2 walks from
// them), and all walks form the list the levels above rank (run_clevels, as
// for the contracted list); sp_expand restores every element.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device.hpp"
#include "hop.hpp"
#include "runner.hpp"

namespace lr {

constexpr int TPB = 256;
#ifndef LR_CHASE_TPB
#define LR_CHASE_TPB 256
#endif
constexpr int CHASE_TPB = LR_CHASE_TPB;
constexpr int BASE_TPB = 1024;
constexpr int BASE_PER = BASE_MAX_LIMIT / BASE_TPB;  // 16 elements per lane
constexpr int EXPAND_CH = 8;                         // elements per lane per wave tile
#ifndef LR_CHASE_POOL
#define LR_CHASE_POOL 2   // sixteenths of a level's walks handed out from a shared pool at the end
#endif
constexpr uint32_t CHASE_GRAB = 64;  // walks a wavefront takes from the pool at a time
#ifndef LR_XCD_GROUPS
#define LR_XCD_GROUPS 1   // second grouping pass: the tiles of one coarse range on one XCD
#endif
static_assert(LR_XCD_GROUPS == 0 || LR_XCD_GROUPS == 1, "XCD grouping is on (1) or off (0)");
static_assert(CHASE_TPB % 64 == 0 && CHASE_TPB >= 64 && CHASE_TPB <= 1024, "chase workgroup width");
static_assert(LR_CHASE_POOL >= 0 && LR_CHASE_POOL < 16, "pool share of the walks, in sixteenths");

// ----------------------------------------------------------- debug writes --
// Debug builds (LR_DEBUG_WRITES): the stores that rely on having one writer
// per address (a slot per visited element, a predecessor mark per element)
// also count themselves, per level, into counters the call sets up; a check
// after the call wants every slot of a chased level written exactly once and
// every mark at most once. Null pointers (release builds, and calls outside
// the plain path) count nothing.
struct DbgWrites {
    uint32_t* slot[MAXL];
    uint32_t* mark[MAXL];
};
struct DbgSizes {
    uint32_t m[MAXL];
};
#if LR_DEBUG_WRITES
__device__ DbgWrites g_dbg;
#define LR_DBG_COUNT(kind, lvl, i)                  \
    do {                                            \
        uint32_t* c_ = g_dbg.kind[(lvl)];           \
        if (c_) atomicAdd(&c_[(i)], 1u);            \
    } while (0)
#else
#define LR_DBG_COUNT(kind, lvl, i) \
    do {                           \
    } while (0)
#endif

// ------------------------------------------------------------------ fill --
__global__ __launch_bounds__(TPB) void k_fill(uint32_t* __restrict__ p, uint64_t words, uint32_t val,
                                              const Ctrl* skip_if_single, Gate gate) {
    if (gate.off()) return;
    if (skip_if_single && skip_if_single->single) return;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t n4 = words / 4;
    uint4 v = make_uint4(val, val, val, val);
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride)
        reinterpret_cast<uint4*>(p)[i] = v;
    for (uint64_t i = n4 * 4 + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride) p[i] = val;
}

// ---------------------------------------------------------------- detect --
// hp[succ[i]] = 1 for every non-terminal i. In a forest each element has at
// most one predecessor, so every byte has at most one writer and plain byte
// stores suffice (no atomics, no cross-XCD coherence traffic).
template <bool VEC>
__global__ __launch_bounds__(TPB) void k_detect(const uint32_t* __restrict__ succ, uint32_t m,
                                                uint8_t* __restrict__ hp, const Ctrl* ctrl, const uint32_t* dm,
                                                Gate gate) {
    if (gate.off()) return;
    if (ctrl->single) return;
    if (dm) m = dm[0];
    const uint32_t stride = gridDim.x * blockDim.x;
    const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t done = 0;
    if constexpr (VEC) {
        const uint32_t m4 = m / 4;
        for (uint32_t i = g; i < m4; i += stride) {
            const uint4 s = reinterpret_cast<const uint4*>(succ)[i];
            const uint32_t x = 4 * i;
            if (s.x != x && s.x < m) { hp[s.x] = 1; LR_DBG_COUNT(mark, 0, s.x); }
            if (s.y != x + 1 && s.y < m) { hp[s.y] = 1; LR_DBG_COUNT(mark, 0, s.y); }
            if (s.z != x + 2 && s.z < m) { hp[s.z] = 1; LR_DBG_COUNT(mark, 0, s.z); }
            if (s.w != x + 3 && s.w < m) { hp[s.w] = 1; LR_DBG_COUNT(mark, 0, s.w); }
        }
        done = m4 * 4;
    }
    for (uint32_t i = done + g; i < m; i += stride) {
        const uint32_t s = succ[i];
        if (s != i && s < m) {
            hp[s] = 1;
            LR_DBG_COUNT(mark, 0, s);
        }
    }
}

// One list shortcut for finding the initial elements. Every non-head element
// has exactly one predecessor, so over a forest
//   sum(all ids) - sum(succ[x] over non-terminals x) = sum of the heads,
// and the number of terminals is the number of lists. With one list this
// sum IS the head, found by one streaming reduction instead of a random
// store per element; the marking passes then do nothing.
template <bool VEC>
__global__ __launch_bounds__(TPB) void k_headsum(const uint32_t* __restrict__ succ, uint32_t m,
                                                 uint32_t* __restrict__ partial, Gate gate) {
    if (gate.off()) return;
    const uint32_t stride = gridDim.x * blockDim.x;
    const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t hs = 0;
    uint32_t nt = 0;
    auto one = [&](uint32_t x, uint32_t s) {
        if (s == x || s >= m) { ++nt; hs += x; }
        else hs += (uint64_t)x - s;
    };
    uint32_t done = 0;
    if constexpr (VEC) {
        const uint32_t m4 = m / 4;
        for (uint32_t i = g; i < m4; i += stride) {
            const uint4 s = reinterpret_cast<const uint4*>(succ)[i];
            one(4 * i, s.x);
            one(4 * i + 1, s.y);
            one(4 * i + 2, s.z);
            one(4 * i + 3, s.w);
        }
        done = m4 * 4;
    }
    for (uint32_t i = done + g; i < m; i += stride) one(i, succ[i]);
    __shared__ uint64_t shs[TPB / 64];
    __shared__ uint32_t snt[TPB / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        hs += __shfl_xor(hs, o);
        nt += __shfl_xor(nt, o);
    }
    if ((threadIdx.x & 63) == 0) { shs[threadIdx.x >> 6] = hs; snt[threadIdx.x >> 6] = nt; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < TPB / 64; ++i) { hs += shs[i]; nt += snt[i]; }
        partial[4 * blockIdx.x] = nt;
        partial[4 * blockIdx.x + 1] = 0;
        reinterpret_cast<uint64_t*>(partial)[2 * blockIdx.x + 1] = hs;
    }
}

// Automatic contraction, the guess: local links counted on every
// LOCAL_SAMPLE_STRIDE-th tile (one workgroup per sampled tile at a time);
// partial[4b] = local links, partial[4b + 1] = elements looked at.
template <bool VEC>
__global__ __launch_bounds__(TPB) void k_lsample(const uint32_t* __restrict__ succ, uint32_t m,
                                                 uint32_t* __restrict__ partial) {
    const uint32_t ntiles = (m + LOCAL_TILE - 1) / LOCAL_TILE;
    const uint32_t nsamp = (ntiles + LOCAL_SAMPLE_STRIDE - 1) / LOCAL_SAMPLE_STRIDE;
    uint32_t loc = 0, seen = 0;
    for (uint32_t q = blockIdx.x; q < nsamp; q += gridDim.x) {
        const uint32_t b = q * LOCAL_SAMPLE_STRIDE * LOCAL_TILE;
        const uint32_t len = min(LOCAL_TILE, m - b);
        for (uint32_t i = threadIdx.x; i < len; i += TPB) {
            const uint32_t s = succ[b + i];
            loc += s != b + i && s < m && (s >> LOCAL_SHIFT) == (b >> LOCAL_SHIFT);
        }
        seen += len;
    }
    __shared__ uint32_t sl[TPB / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) loc += __shfl_xor(loc, o);
    if ((threadIdx.x & 63) == 0) sl[threadIdx.x >> 6] = loc;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < TPB / 64; ++i) loc += sl[i];
        partial[4 * blockIdx.x] = loc;
        partial[4 * blockIdx.x + 1] = seen;
    }
}

// The guess: contract when the sampled tiles extrapolate to a contracted
// list of at most thr elements. The contracted path's scan checks the exact
// size against its capacity and falls back to the plain path if it is larger.
__global__ __launch_bounds__(TPB) void k_ldecide(const uint32_t* __restrict__ partial, uint32_t nparts, uint32_t m,
                                                 uint32_t thr, Ctrl* ctrl) {
    uint64_t loc = 0, seen = 0;
    for (uint32_t i = threadIdx.x; i < nparts; i += TPB) {
        loc += partial[4 * i];
        seen += partial[4 * i + 1];
    }
    __shared__ uint64_t sl[TPB / 64], ss[TPB / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        loc += __shfl_xor(loc, o);
        seen += __shfl_xor(seen, o);
    }
    if ((threadIdx.x & 63) == 0) { sl[threadIdx.x >> 6] = loc; ss[threadIdx.x >> 6] = seen; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < TPB / 64; ++i) { loc += sl[i]; seen += ss[i]; }
        const uint64_t est_local = seen ? loc * (uint64_t)m / seen : 0;
        ctrl->mode = (seen && (uint64_t)m - est_local <= thr) ? 1u : 0u;
        ctrl->single = 0;  // set by the plain path's head sum if that path runs
        ctrl->multi = 0;
    }
}

// Sums the partials (plain path). With exactly one terminal (and a head
// inside the range) it publishes the head as the level's only
// initial-element walk; multi says whether predecessor marks are needed.
__global__ __launch_bounds__(TPB) void k_headsum_final(const uint32_t* __restrict__ partial, uint32_t nparts,
                                                       Ctrl* ctrl, Sampler smp, char* __restrict__ eb, uint32_t S,
                                                       uint32_t rec_bytes, int lvl, uint32_t mode, Gate gate) {
    if (gate.off()) return;
    uint64_t hs = 0;
    uint32_t nt = 0;
    for (uint32_t i = threadIdx.x; i < nparts; i += TPB) {
        nt += partial[4 * i];
        hs += reinterpret_cast<const uint64_t*>(partial)[2 * i + 1];
    }
    __shared__ uint64_t shs[TPB / 64];
    __shared__ uint32_t snt[TPB / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        hs += __shfl_xor(hs, o);
        nt += __shfl_xor(nt, o);
    }
    if ((threadIdx.x & 63) == 0) { shs[threadIdx.x >> 6] = hs; snt[threadIdx.x >> 6] = nt; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < TPB / 64; ++i) { hs += shs[i]; nt += snt[i]; }
        ctrl->nterm = nt;
        ctrl->hsum = hs;
        ctrl->hc_done = 0;  // the head-count kernels' workgroup counter starts the call at zero
        if (mode != NONE) ctrl->mode = mode;
        const bool single = nt == 1 && hs < smp.m;
        ctrl->single = single ? 1u : 0u;
        ctrl->multi = single ? 0u : 1u;
        uint32_t H = 0;  // more than one list: the marks' pass adds its heads
        if (single && !smp.sampled((uint32_t)hs)) {
            *reinterpret_cast<uint32_t*>(eb + (size_t)S * rec_bytes) = (uint32_t)hs;
            H = 1;
        }
        ctrl->lv[lvl].H = H;
        ctrl->lv[lvl].q = 0;
        ctrl->chunks = 0;
        ctrl->conts = 0;
    }
}

// Validation: counts[s]++ per link (counts zeroed before); any element with
// two predecessors or an out-of-range successor sets an error bit.
__global__ __launch_bounds__(TPB) void k_validate_in(const uint32_t* __restrict__ succ, uint32_t m,
                                                     uint32_t* __restrict__ counts, uint32_t* err) {
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const uint32_t s = succ[i];
        if (s >= m) { atomicOr(err, 1u); continue; }
        if (s != i && atomicAdd(&counts[s], 1u) != 0) atomicOr(err, 2u);
    }
}

// Result check (lr_verify): the local equations of the ranking, each
// element against its successor (one gather per output). err |= 1 for a
// successor out of range, 2 for a terminal whose values are not (0, itself,
// 0), 4 for an element whose values do not follow from its successor's.
template <int WT>
__global__ __launch_bounds__(TPB) void k_verify(const uint32_t* __restrict__ succ, const void* __restrict__ weight,
                                                const uint32_t* __restrict__ rank, const uint32_t* __restrict__ root,
                                                const int64_t* __restrict__ sum, uint32_t m, uint32_t* err) {
    const uint32_t stride = gridDim.x * blockDim.x;
    uint32_t bad = 0;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const uint32_t s = succ[i];
        if (s >= m) { bad |= 1u; continue; }
        if (s == i) {
            if ((rank && rank[i] != 0) || (root && root[i] != i) || (sum && sum[i] != 0)) bad |= 2u;
            continue;
        }
        if (rank && rank[i] != rank[s] + 1u) bad |= 4u;
        if (root && root[i] != root[s]) bad |= 4u;
        if (sum) {
            int64_t w = 1;
            if constexpr (WT == 1) w = static_cast<const int32_t*>(weight)[i];
            if constexpr (WT == 2) w = static_cast<const int64_t*>(weight)[i];
            // two's complement wrap, as the prefix sums themselves
            if ((uint64_t)sum[i] != (uint64_t)sum[s] + (uint64_t)w) bad |= 4u;
        }
    }
    if (bad) atomicOr(err, bad);
}


// ----------------------------------------------------------------- heads --
// A tile of TILE elements per block: each lane owns 16 consecutive bytes of
// the hp bytemap. An element starts a walk of its own when it has no
// predecessor and is not the sampled ruler of its block.
__device__ __forceinline__ uint32_t tile_heads(const uint8_t* __restrict__ hp, const Sampler& smp, uint32_t x0,
                                               uint32_t& bits) {
    bits = 0;
    const uint32_t m = smp.m;
    if (x0 >= m) return 0;
    uint8_t b[16];
    if (x0 + 16 <= m) {
        const uint4 v = *reinterpret_cast<const uint4*>(hp + x0);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 16; ++j) b[j] = (uint8_t)(w[j >> 2] >> (8 * (j & 3)));
    } else {
#pragma unroll
        for (int j = 0; j < 16; ++j) b[j] = (x0 + j < m) ? hp[x0 + j] : 1;
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const uint32_t x = x0 + j;
        if (b[j] == 0 && x < m && !smp.sampled(x)) bits |= 1u << j;
    }
    return __popc(bits);
}

__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t* sh) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    const uint32_t wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sh[wv] = v;
    __syncthreads();
    uint32_t t = 0;
    for (uint32_t i = 0; i < blockDim.x / 64; ++i) t += sh[i];
    return t;
}

constexpr int SPL = MAXL - 1;  // Ctrl level entry of the spawning path's input level

// Counts, per tile of TILE elements, the initial elements that are not
// sampled rulers. With scan_last (levels of at most HEADS_SCAN_LAST_TILES
// tiles) the last workgroup to finish then scans the counts in place
// (exclusive) and publishes the walk count of the level, which saves a launch;
// larger levels leave that to k_heads_scan's wider workgroup. Ctrl.hc_done
// counts finished workgroups: each writes its tiles' counts, fences, and
// takes a ticket; the one with the last ticket fences again, sees every
// count, and resets the counter for the next level. The first kernels of
// every path (head sum, batch heads, contraction scan) clear it at the start
// of a call.
constexpr uint32_t HEADS_SCAN_LAST_TILES = 1024;
__global__ __launch_bounds__(TPB) void k_heads_count(const uint8_t* __restrict__ hp, Sampler smp,
                                                     uint32_t* __restrict__ tilecnt, uint32_t ntiles, uint32_t* zero_p,
                                                     uint32_t zero_words, uint32_t skip_single, uint32_t scan_last,
                                                     Ctrl* ctrl, int lvl, const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    __shared__ uint32_t sh[TPB / 64];
    __shared__ uint32_t last;
    if (dm) smp.m = dm[0];
    // clear the next level's predecessor marks (free memory at this point)
    if (zero_p) {
        const uint32_t stride = gridDim.x * blockDim.x;
        for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < zero_words; i += stride) zero_p[i] = 0;
    }
    // one list: its head is known (head sum) and no workgroup counts or scans
    if (skip_single && ctrl->single) return;
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        uint32_t bits;
        const uint32_t c = tile_heads(hp, smp, tile * TILE + threadIdx.x * 16, bits);
        const uint32_t t = block_sum(c, sh);
        if (threadIdx.x == 0) tilecnt[tile] = t;
        __syncthreads();  // sh is reused by the next tile
    }
    if (!scan_last) return;
    if (threadIdx.x == 0) {
        __threadfence();  // this workgroup's counts before its ticket
        last = atomicAdd(&ctrl->hc_done, 1u) == gridDim.x - 1u;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();  // every other workgroup's counts after the last ticket
    const uint32_t total = wg_exscan_inplace(tilecnt, ntiles, sh);
    if (threadIdx.x == 0) {
        ctrl->hc_done = 0;
        ctrl->lv[lvl].H = total;
        ctrl->lv[lvl].q = 0;
        if (lvl == 0) {
            ctrl->chunks = 0;
            ctrl->conts = 0;
        }
    }
}

// One workgroup: exclusive scan of the tile counts in place (levels of more
// than HEADS_SCAN_LAST_TILES tiles); publishes the walk count and resets the
// chase queue of this level.
__global__ __launch_bounds__(1024) void k_heads_scan(uint32_t* __restrict__ tilecnt, uint32_t ntiles,
                                                     Ctrl* ctrl, int lvl, uint32_t skip_single, Gate gate) {
    if (gate.off()) return;
    __shared__ uint32_t sh[1024 / 64];
    if (skip_single && ctrl->single) return;
    const uint32_t total = wg_exscan_inplace(tilecnt, ntiles, sh);
    if (threadIdx.x == 0) {
        ctrl->lv[lvl].H = total;
        ctrl->lv[lvl].q = 0;
        if (lvl == 0) {
            ctrl->chunks = 0;
            ctrl->conts = 0;
        }
    }
}

// Writes walk start j into the first word of walk record S + j.
__global__ __launch_bounds__(TPB) void k_heads_write(const uint8_t* __restrict__ hp, Sampler smp,
                                                     const uint32_t* __restrict__ tileoff, uint32_t ntiles,
                                                     char* __restrict__ eb, uint32_t S, uint32_t rec_bytes,
                                                     const Ctrl* skip_if_single, const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    __shared__ uint32_t sh[TPB / 64];
    if (skip_if_single && skip_if_single->single) return;
    if (dm) { smp.m = dm[0]; S = dm[1]; }
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const uint32_t x0 = tile * TILE + threadIdx.x * 16;
        uint32_t bits;
        const uint32_t c = tile_heads(hp, smp, x0, bits);
        uint32_t total;
        uint32_t pos = tileoff[tile] + block_exscan(c, sh, &total);
        while (bits) {
            const int j = __ffs(bits) - 1;
            bits &= bits - 1;
            *reinterpret_cast<uint32_t*>(eb + (size_t)(S + pos) * rec_bytes) = x0 + j;
            ++pos;
        }
        __syncthreads();  // sh is reused by the next tile
    }
}

// ----------------------------------------------------------------- chase --
// Pads the rest of a wavefront's visit-log chunk with records that name no
// element (x = NONE wide, all ones packed).
template <int LOG, bool W>
__device__ __forceinline__ void pad_chunk(const LogArrays<W>& lg, uint32_t cbase, uint32_t cfill, uint32_t lane) {
    for (uint32_t q = cfill + lane; q < LOG_CHUNK; q += 64) {
        if constexpr (LOG == 2) lg.r[cbase + q] = ~0ull;
        else lg.x[cbase + q] = NONE;
    }
}

// The record of x is fetched as soon as x is known, at the end of the step
// before, and decoded only after the step's bookkeeping (refill, log position,
// stores), so that work runs while the read is in flight; the last walks, with
// few reads in flight, are bound by that chain (2^28 elements 10.49 -> 10.33 ms a
// call, 2^24 862 -> 820 us, 3 M 245 -> 235, weighted 600,003 137 -> 127).
// Fetching before the ruler test as well gains nothing from 2^24 on and loses
// 3 % at 5 M (one read in k is wasted).
//
// Persistent kernel: each lane holds one walk; a wavefront refills its idle
// lanes from its own range of walk ids (ballot + mbcnt hand out consecutive
// ids) once `refill` lanes are idle. Each step is
// one dependent gather (the record of x), one store (slot[x]) and a few ALU
// operations for the ruler test, so the loop is bound by memory latency and
// the lanes resident on the chip keep that many gathers in flight.
//
// LOG mode (level 0 of large inputs): instead of storing slot[x] at a random
// address, the active lanes of a wavefront append their (x, walk, offset)
// records to a chunk of the visit log that the wavefront owns, at consecutive
// positions (mbcnt over the active lanes), so every step writes whole lines.
// A chunk that cannot take another step's records is padded and a new one is
// taken with one atomic. LOG = 1 writes wide records, LOG = 2 packed ones.
//
// NW walks per lane: the lane issues the loads of all its walks before it
// uses any of them, so NW independent gathers are in flight per lane.
// At most 80 scalar registers: the persistent grid is 8 waves per SIMD, and
// waves allocated 96 scalar registers (the next granule) measured 1.5-2 %
// slower at 2^28 elements, although the compiler's occupancy estimate is 8
// either way.
template <bool W, class Src, int LOG, int NW>
__global__ __launch_bounds__(CHASE_TPB) __attribute__((amdgpu_num_sgpr(80))) void k_chase(Src src, Sampler smp, uint32_t S, Ctrl* ctrl, int lvl,
                                                     typename Lay<W>::Slot* __restrict__ slot,
                                                     typename Lay<W>::Rec* __restrict__ eb,
                                                     uint8_t* __restrict__ hp_next, uint32_t refill,
                                                     LogArrays<W> lg, uint32_t max_chunks, const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    using L = Lay<W>;
    using Val = typename L::Val;
    if (dm) { smp.m = src.m = dm[0]; S = dm[1]; }
    const uint32_t lane = lane_id();
    const uint32_t total = S + ctrl->lv[lvl].H;
    const uint32_t m = smp.m;
    const uint32_t cap = walk_cap(m, smp.log2k);
    uint32_t w[NW], x[NW], steps[NW];
    Val off[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        w[k] = NONE;
        x[k] = 0;
        steps[k] = 0;
        off[k] = L::zero();
    }
    // Each wavefront owns a contiguous range of walk ids and refills its lanes
    // from it, so no queue is contended while the chip is busy. In LOG mode
    // with at least 64 walks per wavefront (level 0 of large inputs) the last
    // LR_CHASE_POOL sixteenths of the walk ids form a pool instead: a
    // wavefront done with its own range takes CHASE_GRAB of them at a time
    // with one atomic, so the wavefronts finish closer together. With few walks
    // per wavefront (upper levels, short contracted lists) every wavefront
    // would reach the pool at once, and the contended counter costs more than
    // the balance gains.
    const uint32_t gwave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint32_t nwave = (gridDim.x * blockDim.x) >> 6;
    const uint32_t pool16 = (LOG != 0 && total >= 64u * nwave) ? LR_CHASE_POOL : 0u;  // many walks per wavefront
    const uint32_t own = (uint32_t)((uint64_t)total * (16u - pool16) / 16u);
    const uint32_t per = own / nwave + 1;
    uint32_t whi = (uint32_t)min<uint64_t>((uint64_t)(gwave + 1) * per, own);
    uint32_t cursor = (uint32_t)min<uint64_t>((uint64_t)gwave * per, own);
    bool exhausted = false;
    uint32_t cbase = 0, cfill = LOG_CHUNK;  // visit-log chunk held by this wavefront (LOG mode)
    bool have = false, dead = false;
    // packed records (LOG == 2): field widths, and per walk slot the id its
    // records carry (the walk, or its current continuation) and the offset
    // that id's records count from; continuation ids come from a block of
    // CONT_GRAB held by the wavefront
    const LogFmt fmt(m, total, lg.ccap, lg.bocap);
    uint32_t rw[NW], rb[NW];
    uint32_t kbase = 0, kfill = CONT_GRAB;
    typename Src::Raw raw[NW];  // the record of x, in flight while the step's bookkeeping runs
    for (;;) {
        uint64_t idle[NW];
        uint32_t nidle = 0;
        bool all_idle = true;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            idle[k] = __ballot(w[k] == NONE);
            nidle += __popcll(idle[k]);
            all_idle &= idle[k] == ~0ull;
        }
        const bool want = nidle >= refill || all_idle;
        if (!exhausted && want && cursor >= whi && own >= total) exhausted = true;  // no pool
        if (!exhausted && want && cursor >= whi) {  // own range (or last grab) used up: the pool
            uint32_t g = 0;
            if (lane == 0) g = atomicAdd(&ctrl->lv[lvl].q, CHASE_GRAB);
            g = __shfl(g, 0);
            if ((uint64_t)own + g < total) {
                cursor = own + g;
                whi = (uint32_t)min<uint64_t>((uint64_t)cursor + CHASE_GRAB, total);
            } else {
                exhausted = true;
            }
        }
        if (all_idle && exhausted) break;
        if (!exhausted && want) {
            const uint32_t base = cursor;
            cursor = min(cursor + nidle, whi);
            uint32_t acc = base;
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                if (w[k] == NONE) {
                    const uint32_t my = acc + mbcnt(idle[k]);
                    if (my < whi) {
                        w[k] = my;
                        off[k] = L::zero();
                        steps[k] = 0;
                        rw[k] = my;
                        rb[k] = 0;
                        x[k] = (my < S) ? smp.start(my) : reinterpret_cast<const uint32_t*>(eb + my)[0];
                        if (x[k] >= m) {  // corrupt start (cannot happen for valid input)
                            eb[w[k]] = L::rec(TERM | IDX, L::zero());
                            atomicOr(&ctrl->err, 8u);
                            w[k] = NONE;
                        } else {
                            raw[k] = src.fetch(x[k]);
                        }
                    }
                }
                acc += __popcll(idle[k]);
            }
        }
        uint32_t pos[NW];
        if constexpr (LOG != 0) {
            uint64_t act[NW];
            uint32_t na = 0;
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                act[k] = __ballot(w[k] != NONE);
                na += __popcll(act[k]);
            }
            if (na && !dead) {
                if (cfill + na > LOG_CHUNK) {
                    if (have) pad_chunk<LOG>(lg, cbase, cfill, lane);
                    uint32_t c = 0;
                    if (lane == 0) c = atomicAdd(&ctrl->chunks, 1u);
                    c = __shfl(c, 0);
                    if (c >= max_chunks) {  // more visits than elements: the input is not a forest
                        dead = true;
                        have = false;
                        if (lane == 0) atomicOr(&ctrl->err, 32u);
                    } else {
                        cbase = c * LOG_CHUNK;
                        cfill = 0;
                        have = true;
                    }
                }
                uint32_t acc = cbase + cfill;
#pragma unroll
                for (int k = 0; k < NW; ++k) {
                    pos[k] = acc + mbcnt(act[k]);
                    acc += __popcll(act[k]);
                }
                cfill += na;
            }
            if constexpr (LOG == 2) {
                // walks whose offset no longer fits the field take a continuation id
                uint64_t nc[NW];
                uint32_t ncs = 0;
#pragma unroll
                for (int k = 0; k < NW; ++k) {
                    nc[k] = __ballot(!dead && w[k] != NONE && off[k].c - rb[k] >= (1u << fmt.bo));
                    ncs += __popcll(nc[k]);
                }
                if (ncs) {
                    if (kfill + ncs > CONT_GRAB) {
                        uint32_t b = 0;
                        if (lane == 0) b = atomicAdd(&ctrl->conts, CONT_GRAB);
                        kbase = __shfl(b, 0);
                        kfill = 0;
                    }
                    if ((uint64_t)kbase + kfill + ncs > lg.ccap) {
                        // cannot happen: the table holds every continuation a full log can need
                        if (lane == 0) atomicOr(&ctrl->err, 32u);
                        dead = true;
                    } else {
                        uint32_t acc = kbase + kfill;
#pragma unroll
                        for (int k = 0; k < NW; ++k) {
                            if ((nc[k] >> lane) & 1ull) {
                                const uint32_t j = acc + mbcnt(nc[k]);
                                lg.cont[j] = make_uint2(w[k], off[k].c);
                                rw[k] = total + j;
                                rb[k] = off[k].c;
                            }
                            acc += __popcll(nc[k]);
                        }
                        kfill += ncs;
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            if (w[k] == NONE) continue;
            if constexpr (LOG == 1) {
                if (!dead) {
                    lg.x[pos[k]] = x[k];
                    lg.w[pos[k]] = w[k];
                    lg.c[pos[k]] = off[k].c;
                    if constexpr (W) lg.s[pos[k]] = off[k].s;
                }
            } else if constexpr (LOG == 2) {
                if (!dead) {
                    lg.r[pos[k]] = fmt.pack(x[k], rw[k], off[k].c - rb[k]);
                    if constexpr (W) lg.s[pos[k]] = off[k].s;
                }
            } else {
                slot[x[k]] = L::slot(w[k], off[k]);
                LR_DBG_COUNT(slot, lvl, x[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            if (w[k] == NONE) continue;
            uint32_t nxt;
            Val v;
            src.decode(x[k], raw[k], nxt, v);
            if (nxt & TERM) {                       // x is a terminal: the walk ends on it
                eb[w[k]] = L::rec(nxt, L::add(off[k], v));
                w[k] = NONE;
            } else {
                off[k] = L::add(off[k], v);
                // steps so far: on the input level every record is one link,
                // so the walk's count is its step count and no counter is kept
                uint32_t walked;
                if constexpr (Src::kLinks) walked = off[k].c;
                else walked = ++steps[k];
                if (walked >= cap) {                // too long (or a cycle): the bounded fallback takes over
                    eb[w[k]] = L::rec(TERM | IDX, off[k]);
                    ctrl->mode = MODE_FALLBACK;
                    w[k] = NONE;
                } else if (smp.sampled(nxt)) {      // reached the next ruler
                    const uint32_t c = nxt >> smp.log2k;
                    eb[w[k]] = L::rec(c, off[k]);
                    if (hp_next && w[k] < S) {
                        hp_next[c] = 1;
                        LR_DBG_COUNT(mark, lvl + 1, c);  // hp_next exists below the last level only
                    }
                    w[k] = NONE;
                } else {
                    x[k] = nxt;
                    raw[k] = src.fetch(nxt);
                }
            }
        }
    }
    if constexpr (LOG != 0) {
        if (have) pad_chunk<LOG>(lg, cbase, cfill, lane);
    }
}

// A record (nxt, count) as one word.
__device__ __forceinline__ uint64_t iw_word(uint32_t f, uint32_t v) { return ((uint64_t)v << 32) | f; }

// ------------------------------------------------------------------ base --
// Pointer doubling (Wyllie) on <= 16384 elements in LDS by one workgroup.
//
// Unweighted levels: a record (nxt, count) per element, 8 B in LDS, as in the
// independent walks: nxt = TERM | t once the list's end is reached, its count
// then including the terminal's own value. Lane t holds the records of slots
// t + j * BASE_TPB for j < COLS (1, 2, 4, 8 or 16 columns, the fewest that
// cover the planned size) in registers and composes them, in place and without
// barriers, until all have ended: a record stays true whatever the others do, so
// a neighbour's older record only jumps less far, and no wavefront waits for
// another. On a cycle the count reaches climit. Slots past m hold ended records
// and ended slots read themselves, so a round has no per-lane branch and the
// lane's COLS gathers are in flight together.
// Bound by the launch, a global read and the LDS rounds. A call against
// synchronised rounds (two barriers each): 1000 elements 11.2 -> 8.7 us, which is
// the rate the host enqueues at, 4096 13.7 -> 8.5; 8192 take 12.5 (independent
// walks 16.6), 16384 24.7 (18), which is why the planner's line lies between.
template <int COLS, class Src, class Out>
__global__ __launch_bounds__(BASE_TPB) void k_base_unweighted(Src src, Out out, uint32_t m, uint32_t climit, Ctrl* ctrl,
                                                              const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    using Val = typename Lay<false>::Val;
    extern __shared__ __align__(16) unsigned char lds[];
    if (dm) m = src.m = min(dm[0], m);  // a device-side size is at most the planned one
    uint64_t* fd = reinterpret_cast<uint64_t*>(lds);
    const uint32_t t = threadIdx.x;
    auto get = [&](uint32_t i) { return __hip_atomic_load(fd + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
    auto put = [&](uint32_t i, uint64_t v) {
        __hip_atomic_store(fd + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    uint64_t e[COLS];
#pragma unroll
    for (int j = 0; j < COLS; ++j) {
        const uint32_t i = t + j * BASE_TPB;
        e[j] = TERM | IDX;
        if (i < m) {
            uint32_t nxt;
            Val v;
            src.bind(i).load(i, nxt, v);
            e[j] = iw_word(nxt, v.c);
        }
    }
#pragma unroll
    for (int j = 0; j < COLS; ++j) put(t + j * BASE_TPB, e[j]);
    __syncthreads();
    for (;;) {
        uint32_t open = 0;
#pragma unroll
        for (int j = 0; j < COLS; ++j) open |= ~(uint32_t)e[j] & TERM;
        if (!open) break;
        uint64_t w[COLS];
#pragma unroll
        for (int j = 0; j < COLS; ++j) w[j] = get(((uint32_t)e[j] & TERM) ? t + j * BASE_TPB : (uint32_t)e[j]);
#pragma unroll
        for (int j = 0; j < COLS; ++j) {
            const uint32_t b = (uint32_t)(e[j] >> 32), c = b + (uint32_t)(w[j] >> 32);
            // more links than the input has: a cycle
            const uint64_t n = hop_stuck(b, c, (uint32_t)w[j] & TERM, climit) ? ~0ull : iw_word((uint32_t)w[j], c);
            e[j] = ((uint32_t)e[j] & TERM) ? e[j] : n;
            put(t + j * BASE_TPB, e[j]);
        }
    }
#pragma unroll
    for (int j = 0; j < COLS; ++j) {
        const uint32_t i = t + j * BASE_TPB;
        if (i < m) {
            if (e[j] == ~0ull) atomicOr(&ctrl->err, 16u);
            auto cur = out.begin(i);
            out.store(cur, i, Val{(uint32_t)(e[j] >> 32)}, (uint32_t)e[j] & IDX);
        }
    }
}

// Weighted levels of at most 8192 elements, the same way with two words per
// element (16 B): the count, the 64-bit sum and, in both words, the slot they
// lead to. A record is taken only if both words name the same slot (which
// determines the values), so halves of two records are never combined.
//   word 0: slot and ended bit (14 bits) | count (31) | sum bits 0-18
//   word 1: slot and ended bit (14 bits) | sum bits 19-63
// An ended record names its terminal's slot, whose own value and id are read
// from the source again at the end.
// Bound as above (against synchronised rounds: 600 elements 14.5 -> 8.9 us a
// call, 3000 20.5 -> 12.2, 8192 33.8 -> 28.2).
constexpr uint32_t BW_END = 1u << 13;
template <int COLS, class Src, class Out>
__global__ __launch_bounds__(BASE_TPB) void k_base_weighted(Src src, Out out, uint32_t m, uint32_t climit, Ctrl* ctrl,
                                                            const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    using L = Lay<true>;
    using Val = typename L::Val;
    static_assert(COLS * BASE_TPB <= BW_END, "13-bit slots");
    extern __shared__ __align__(16) unsigned char lds[];
    if (dm) m = src.m = min(dm[0], m);  // a device-side size is at most the planned one
    uint64_t* w0 = reinterpret_cast<uint64_t*>(lds);
    uint64_t* w1 = w0 + COLS * BASE_TPB;
    const uint32_t t = threadIdx.x;
    auto get = [&](const uint64_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
    auto put = [&](uint32_t i, uint32_t f, uint32_t c, uint64_t s) {
        __hip_atomic_store(w0 + i, (uint64_t)f | ((uint64_t)c << 14) | (s << 45), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(w1 + i, (uint64_t)f | ((s >> 19) << 14), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    uint32_t f[COLS], c[COLS];
    uint64_t s[COLS];
    uint32_t cyc = 0;  // columns that never reached a terminal
#pragma unroll
    for (int j = 0; j < COLS; ++j) {
        const uint32_t i = t + j * BASE_TPB;
        f[j] = BW_END | i;
        c[j] = 0;
        s[j] = 0;
        if (i < m) {
            uint32_t nxt;
            Val v;
            src.load(i, nxt, v);
            if (!(nxt & TERM) && nxt < m) {
                f[j] = nxt;
                c[j] = v.c;
                s[j] = (uint64_t)v.s;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < COLS; ++j) put(t + j * BASE_TPB, f[j], c[j], s[j]);
    __syncthreads();
    for (;;) {
        uint32_t open = 0;
#pragma unroll
        for (int j = 0; j < COLS; ++j) open |= ~f[j] & BW_END;
        if (!open) break;
        uint64_t a[COLS], b[COLS];
#pragma unroll
        for (int j = 0; j < COLS; ++j) {
            const uint32_t q = f[j] & (BW_END - 1);
            a[j] = get(w0 + q);
            b[j] = get(w1 + q);
        }
#pragma unroll
        for (int j = 0; j < COLS; ++j) {
            const uint32_t i = t + j * BASE_TPB;
            const uint32_t fa = (uint32_t)a[j] & (2 * BW_END - 1);
            if ((f[j] & BW_END) || fa != ((uint32_t)b[j] & (2 * BW_END - 1))) continue;  // ended, or caught half stored
            const uint32_t before = c[j];
            c[j] += (uint32_t)(a[j] >> 14) & IDX;
            s[j] += (a[j] >> 45) | ((b[j] >> 14) << 19);
            f[j] = fa;
            if (hop_stuck(before, c[j], fa & BW_END, climit)) {  // more links than the input has: a cycle
                cyc |= 1u << j;
                f[j] = BW_END | i;
                c[j] = 0;
            }
            put(i, f[j], c[j], s[j]);
        }
    }
    Val rv[COLS];
    uint32_t rr[COLS];
#pragma unroll
    for (int j = 0; j < COLS; ++j) {
        if (t + j * BASE_TPB >= m) continue;
        uint32_t nxt;
        Val v;
        src.load(f[j] & (BW_END - 1), nxt, v);
        rv[j] = L::add(Val{c[j], (int64_t)s[j]}, v);
        rr[j] = nxt & IDX;
        if (!(nxt & TERM) || ((cyc >> j) & 1u)) {
            rv[j] = L::junk();
            rr[j] = NONE;
            atomicOr(&ctrl->err, 16u);
        }
    }
    __syncthreads();  // every read of the level's records happens before any in-place write
#pragma unroll
    for (int j = 0; j < COLS; ++j) {
        const uint32_t i = t + j * BASE_TPB;
        if (i < m) {
            auto cur = out.begin(i);
            out.store(cur, i, rv[j], rr[j]);
        }
    }
}

// Larger weighted levels (a user base size above 8192), in rounds: d[i] is the
// weight from i up to (not including) f[i]; terminals point to themselves with
// d = 0, so a round d[i] += d[f[i]], f[i] = f[f[i]] leaves them fixed, and after
// ceil(log2 len) rounds f[i] is i's terminal. 8 B sum, 4 B count and 2 B
// successor arrays.
template <class Src, class Out>
__global__ __launch_bounds__(BASE_TPB) void k_base_weighted_large(Src src, Out out, uint32_t m, Ctrl* ctrl,
                                                                  const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    using L = Lay<true>;
    using Val = typename L::Val;
    extern __shared__ __align__(16) unsigned char lds[];
    if (dm) m = src.m = min(dm[0], m);  // a device-side size is at most the planned one
    const uint32_t t = threadIdx.x;
    uint32_t f_[BASE_PER], dc_[BASE_PER];
    int64_t ds_[BASE_PER];
    {
        int64_t* ds = reinterpret_cast<int64_t*>(lds);
        uint32_t* dc = reinterpret_cast<uint32_t*>(lds + 8 * (size_t)m);
        uint16_t* f = reinterpret_cast<uint16_t*>(lds + 12 * (size_t)m);
        for (uint32_t i = t; i < m; i += BASE_TPB) {
            uint32_t nxt;
            Val v;
            src.load(i, nxt, v);
            const bool term = (nxt & TERM) || nxt >= m;
            f[i] = (uint16_t)(term ? i : nxt);
            dc[i] = term ? 0u : v.c;
            ds[i] = term ? 0 : v.s;
        }
        __syncthreads();
        for (int round = 0; round < 40; ++round) {
            uint16_t ff[BASE_PER];
            uint32_t fc[BASE_PER];
            int64_t fs[BASE_PER];
            int changed = 0;
#pragma unroll
            for (int j = 0; j < BASE_PER; ++j) {
                const uint32_t i = t + j * BASE_TPB;
                if (i < m) {
                    const uint32_t fi = f[i];
                    ff[j] = f[fi];
                    fc[j] = dc[fi];
                    fs[j] = ds[fi];
                    changed |= (ff[j] != fi);
                }
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < BASE_PER; ++j) {
                const uint32_t i = t + j * BASE_TPB;
                if (i < m) {
                    f[i] = ff[j];
                    dc[i] += fc[j];
                    ds[i] += fs[j];
                }
            }
            if (!__syncthreads_or(changed)) break;
        }
#pragma unroll
        for (int j = 0; j < BASE_PER; ++j) {
            const uint32_t i = t + j * BASE_TPB;
            if (i < m) {
                f_[j] = f[i];
                dc_[j] = dc[i];
                ds_[j] = ds[i];
            }
        }
    }
    Val rv[BASE_PER];
    uint32_t rr[BASE_PER];
#pragma unroll
    for (int j = 0; j < BASE_PER; ++j) {
        const uint32_t i = t + j * BASE_TPB;
        if (i < m) {
            const uint32_t ti = f_[j];
            uint32_t nxt;
            Val v;
            src.load(ti, nxt, v);
            Val d;
            d.c = dc_[j];
            d.s = ds_[j];
            if (nxt & TERM) {
                rv[j] = L::add(d, v);
                rr[j] = nxt & IDX;
            } else {  // never reached a terminal: the input has a cycle
                rv[j] = L::junk();
                rr[j] = NONE;
                atomicOr(&ctrl->err, 16u);
            }
        }
    }
    __syncthreads();  // every read of the level's records happens before any in-place write
#pragma unroll
    for (int j = 0; j < BASE_PER; ++j) {
        const uint32_t i = t + j * BASE_TPB;
        if (i < m) {
            auto cur = out.begin(i);
            out.store(cur, i, rv[j], rr[j]);
        }
    }
}

// ----------------------------------------------------- independent walks --
// Lists of up to about a million elements (the input itself, or a level of a
// larger one) without heads, marks, slots or a one-workgroup base case:
//   k_iw_first  every element walks the list by itself, up to `cap` steps, to
//               the next ruler (the level's stratified sample) or to its end.
//               That is about k steps per element where the ruling-set chase
//               takes one, but the reads hit the caches, nothing is scattered,
//               and no walk is longer than the cap.
//   k_iw_walk   the same on the rulers, to the rulers of the next level.
//   k_iw_double on the last level: asynchronous pointer doubling, every
//               element's record composed with the record it points to until
//               it has reached a terminal.
//   k_iw_down   then, level by level downward, every element composes its
//               record with its ruler's (solved) one.
// Nodes: one record (nxt, value) per element of every level, in one array;
// level j's nodes start at base_j. A record says that following the list from
// its element for `value` leads to node nxt or, with nxt = TERM | t, to the
// terminal t. That stays true whatever the others do, so records are updated
// in place without any barrier: a reader that finds an older record only jumps
// less far. A walk that stopped at its cap points to an element that is no
// ruler, whose own record leads on; a reader just takes one more hop.
//   - In the doubling the records are read and written with device-scope
//     accesses, which pass the (per-XCD, not coherent) L2s, so the lanes see
//     each other's progress; an element's record has one writer per kernel.
//   - No lane waits for another: a lane alone still moves at least one link a
//     hop, so the kernels end however their workgroups are scheduled.
//   - On a cycle (input that is not a forest) the count reaches climit, more
//     links than a list can have, and the lane stops; so it does where a hop
//     counts no link (hop_stuck), as unwritten records of such input may.
//   - An order built against the sampling leaves long stretches without a
//     ruler. The downward pass over the input then turns into doubling itself:
//     after IW_PATIENCE hops (a random order needs 1.5 on average and stays
//     below 16) a lane stores its progress after every further hop and reads
//     device-scope, and its stretch's lanes halve the rest with every hop: all
//     of them are resident, but for weighted contracted lists above 3 * 2^19
//     elements (see IW_PER), of which the rest is followed at about 12 links a
//     hop. The last level's doubling stops after IW_TOP_CAP hops for the same
//     reason and leaves the rest to that pass.
// Bound by latency: cap cached reads, about log2(m) device-scope reads (0.7 us
// each up to 2^15 lanes, then 50 G/s), a few cached reads, and a launch (4.5
// us) for each kernel. A cap of 12 steps (random lists of 1.5 * 2^18 elements:
// 8 steps 73 us, 12 60, 16 59; weighted 1.4 * 2^19: 181, 168, 172).
constexpr uint32_t IW_PATIENCE = 32;
constexpr uint32_t IW_TOP_CAP = 128;
#ifndef LR_IW_CAP
#define LR_IW_CAP 12
#endif
constexpr uint32_t IW_CAP_ALONE = 8;  // steps of a list that the doubling takes alone

template <bool DEV>
__device__ __forceinline__ uint64_t iw_get(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, DEV ? __HIP_MEMORY_SCOPE_AGENT : __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void iw_put(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A node's record. Unweighted: one word (nxt, count), the layout of a level's
// records. Weighted: three words (nxt, count), (nxt, low half of the sum),
// (nxt, high half), stored one by one; a record is taken only if all three
// name the same nxt (which determines the values), so halves of two records
// are never combined.
template <bool W> struct IwRec;
template <> struct IwRec<false> {
    using Val = Lay<false>::Val;
    static constexpr uint32_t WORDS = 1;
    template <bool DEV>
    static __device__ __forceinline__ bool load(const uint64_t* p, uint32_t i, uint32_t& nxt, Val& v) {
        const uint64_t e = iw_get<DEV>(p + i);
        nxt = (uint32_t)e;
        v.c = (uint32_t)(e >> 32);
        return true;
    }
    static __device__ __forceinline__ void store(uint64_t* p, uint32_t i, uint32_t nxt, Val v) {
        iw_put(p + i, iw_word(nxt, v.c));
    }
};
template <> struct IwRec<true> {
    using Val = Lay<true>::Val;
    static constexpr uint32_t WORDS = 3;
    template <bool DEV>
    static __device__ __forceinline__ bool load(const uint64_t* p, uint32_t i, uint32_t& nxt, Val& v) {
        const uint64_t* q = p + 3 * (size_t)i;
        const uint64_t a = iw_get<DEV>(q), b = iw_get<DEV>(q + 1), c = iw_get<DEV>(q + 2);
        nxt = (uint32_t)a;
        v.c = (uint32_t)(a >> 32);
        v.s = (int64_t)((b >> 32) | (c & 0xffffffff00000000ull));
        return (uint32_t)b == nxt && (uint32_t)c == nxt;
    }
    static __device__ __forceinline__ void store(uint64_t* p, uint32_t i, uint32_t nxt, Val v) {
        uint64_t* q = p + 3 * (size_t)i;
        iw_put(q, iw_word(nxt, v.c));
        iw_put(q + 1, iw_word(nxt, (uint32_t)v.s));
        iw_put(q + 2, iw_word(nxt, (uint32_t)((uint64_t)v.s >> 32)));
    }
};

// Level 0 of the nodes from the source's records. SAMPLE = false: no rulers,
// every element walks `cap` steps (the list is small enough for the doubling
// alone).
template <bool W, bool SAMPLE, class Src>
__device__ __forceinline__ void iw_first(const Src& src, const Sampler& smp, uint64_t* __restrict__ nodes,
                                         uint32_t base1, uint32_t i, uint32_t cap) {
    using L = Lay<W>;
    const auto sr = src.bind(i);
    uint32_t nxt;
    typename L::Val acc;
    sr.load(i, nxt, acc);
    bool ruler = false;
    for (uint32_t t = 1; !(nxt & TERM); ++t) {
        if constexpr (SAMPLE) ruler = smp.sampled(nxt);
        if (ruler || t >= cap) break;
        typename L::Val v;
        uint32_t nn;
        sr.load(nxt, nn, v);
        acc = L::add(acc, v);
        nxt = nn;
    }
    uint32_t at = i;
    if constexpr (SAMPLE) {
        if (ruler) nxt = base1 + (nxt >> smp.log2k);
        if (smp.sampled(i)) at = base1 + (i >> smp.log2k);
    }
    IwRec<W>::store(nodes, at, nxt, acc);
}

// The input itself: its first kernel sets the path word.
template <bool W, bool SAMPLE, class Src>
__global__ __launch_bounds__(TPB) void k_iw_first(Src src, Sampler smp, uint64_t* __restrict__ nodes, uint32_t base1,
                                                  uint32_t m, uint32_t cap, Ctrl* ctrl, const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    if (dm) m = min(dm[0], m);
    smp.m = src.m = m;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) ctrl->mode = MODE_PLAIN;
    if (i < m) iw_first<W, SAMPLE>(src, smp, nodes, base1, i, cap);
}

// Composes (nxt, acc) with the record of node nxt; false: caught between two
// of its stores (nothing changed), look again device-scope.
template <bool W, bool DEV>
__device__ __forceinline__ bool iw_hop(const uint64_t* nodes, uint32_t& nxt, typename Lay<W>::Val& acc) {
    uint32_t nn;
    typename Lay<W>::Val v;
    if (!IwRec<W>::template load<DEV>(nodes, nxt, nn, v)) return false;
    acc = Lay<W>::add(acc, v);
    nxt = nn;
    return true;
}

// Level j >= 1: every node's record hops on to the next of level j's rulers,
// which are the nodes of level j + 1. total: nodes in all.
template <bool W>
__device__ __forceinline__ void iw_walk(uint64_t* __restrict__ nodes, const Sampler& smp, uint32_t base, uint32_t basen,
                                        uint32_t total, uint32_t c, uint32_t cap) {
    using L = Lay<W>;
    uint32_t nxt;
    typename L::Val acc;
    while (!IwRec<W>::template load<true>(nodes, base + c, nxt, acc)) {}  // own record: written by the last kernel
    for (uint32_t t = 1; nxt < total; ++t) {
        if (nxt >= base && nxt < basen && smp.sampled(nxt - base)) {
            nxt = basen + ((nxt - base) >> smp.log2k);
            break;
        }
        // another lane may have stored its node's new record already: then nxt
        // is a ruler's node
        if (nxt >= basen || t >= cap) break;
        if (!iw_hop<W, false>(nodes, nxt, acc)) while (!iw_hop<W, true>(nodes, nxt, acc)) {}
    }
    IwRec<W>::store(nodes, smp.sampled(c) ? basen + (c >> smp.log2k) : base + c, nxt, acc);
}

template <bool W>
__global__ __launch_bounds__(TPB) void k_iw_walk(uint64_t* __restrict__ nodes, Sampler smp, uint32_t base,
                                                 uint32_t basen, uint32_t total, uint32_t m, uint32_t cap,
                                                 const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    if (dm) m = min(dm[0], m);
    smp.m = m;
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < m) iw_walk<W>(nodes, smp, base, basen, total, c, cap);
}

// The doubling of the last level, nodes [base, base + m). OUTS: the results go
// to `out`, else they stay in the nodes. cap: hops after which an element is
// left to the downward pass. A hop's stores are awaited before the next hop's
// load: a load that runs ahead of the others' stores finds the records of the
// round before, and its element needs a hop more (2^16 elements 28 us, 31
// without the wait; weighted 100,003 43 against 49). Single-wave workgroups
// spread a few hundred waves over all CUs (weighted 100,003 elements 43 us, 51
// with 256 lanes; unweighted 1 us).
constexpr uint32_t IW_DBL_TPB = 64;
template <bool W>
__device__ __forceinline__ void iw_double(uint64_t* __restrict__ nodes, uint32_t base, uint32_t total, uint32_t c,
                                          uint32_t climit, uint32_t cap, Ctrl* ctrl, uint32_t& nxt,
                                          typename Lay<W>::Val& acc) {
    using L = Lay<W>;
    while (!IwRec<W>::template load<true>(nodes, base + c, nxt, acc)) {}
    for (uint32_t hop = 0; !(nxt & TERM) && hop < cap; ++hop) {
        bool bad = nxt >= total;
        if (!bad) {
            const uint32_t before = acc.c;
            if (!iw_hop<W, true>(nodes, nxt, acc)) continue;
            bad = hop_stuck(before, acc.c, nxt & TERM, climit);
        }
        if (bad) {  // more links than the input has: a cycle (or no forest at all)
            nxt = TERM | IDX;
            acc = L::junk();
            atomicOr(&ctrl->err, 16u);
        }
        IwRec<W>::store(nodes, base + c, nxt, acc);
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    }
}

template <bool W, bool OUTS, class Out>
__global__ __launch_bounds__(IW_DBL_TPB) void k_iw_double(uint64_t* __restrict__ nodes, uint32_t base, uint32_t total,
                                                          uint32_t m, uint32_t climit, uint32_t cap, Ctrl* ctrl,
                                                          Out out, const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    if (dm) m = min(dm[0], m);
    const uint32_t c = blockIdx.x * IW_DBL_TPB + threadIdx.x;
    if (c >= m) return;
    uint32_t nxt;
    typename Lay<W>::Val acc;
    iw_double<W>(nodes, base, total, c, climit, cap, ctrl, nxt, acc);
    if constexpr (OUTS) {
        auto cur = out.begin(c);
        out.store(cur, c, acc, nxt & IDX);
    }
}

// The downward pass of a level: every element composes its record with its
// ruler's solved one; an element that is a ruler takes the record of its node
// one level up. OUTS: the results go to `out`, else to the nodes. last: the
// pass over the whole list, which must solve every element (any other may
// leave some of them to it). PER elements a lane, the loads of all issued
// before any is used.
template <bool W, int PER>
__device__ __forceinline__ void iw_down(uint64_t* __restrict__ nodes, const Sampler& smp, uint32_t base, uint32_t basen,
                                        uint32_t total, uint32_t m, uint32_t c0, uint32_t climit, uint32_t last,
                                        uint32_t set_mode, Ctrl* ctrl, uint32_t (&nxt)[PER],
                                        typename Lay<W>::Val (&acc)[PER]) {
    using L = Lay<W>;
    uint32_t at[PER], nn[PER];
    typename L::Val v[PER];
    bool ok[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const uint32_t c = c0 + r * TPB;
        nxt[r] = TERM | IDX;
        at[r] = base + c;
        ok[r] = true;
        if (c < m) {
            if (smp.sampled(c)) at[r] = basen + (c >> smp.log2k);
            ok[r] = IwRec<W>::template load<false>(nodes, at[r], nxt[r], acc[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < PER; ++r)
        while (!ok[r]) ok[r] = IwRec<W>::template load<true>(nodes, at[r], nxt[r], acc[r]);
    // the record each element looks at next
    auto look = [&](int r, bool dbl) {
        ok[r] = false;
        if (nxt[r] < total) ok[r] = dbl ? IwRec<W>::template load<true>(nodes, nxt[r], nn[r], v[r])
                                        : IwRec<W>::template load<false>(nodes, nxt[r], nn[r], v[r]);
    };
    const uint32_t cap = last ? NONE : IW_TOP_CAP;
#pragma unroll
    for (int r = 0; r < PER; ++r) look(r, false);
    for (uint32_t hop = 0; hop < cap; ++hop) {
        bool any = false;
#pragma unroll
        for (int r = 0; r < PER; ++r) any |= !(nxt[r] & TERM);
        if (!any) break;
        const bool dbl = hop >= IW_PATIENCE;
        if (hop == IW_PATIENCE && set_mode) ctrl->mode = MODE_FALLBACK;
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            if (nxt[r] & TERM) continue;
            bool bad = nxt[r] >= total;
            // caught between two of its stores (weighted): look again
            if (!bad && !ok[r] && !IwRec<W>::template load<true>(nodes, nxt[r], nn[r], v[r])) continue;
            if (!bad) {
                const uint32_t before = acc[r].c;
                acc[r] = L::add(acc[r], v[r]);
                nxt[r] = nn[r];
                bad = hop_stuck(before, acc[r].c, nxt[r] & TERM, climit);
            }
            if (bad) {
                nxt[r] = TERM | IDX;
                acc[r] = L::junk();
                atomicOr(&ctrl->err, 16u);
            }
            if (dbl) IwRec<W>::store(nodes, at[r], nxt[r], acc[r]);
        }
#pragma unroll
        for (int r = 0; r < PER; ++r) look(r, dbl);
    }
}

template <bool W, bool OUTS, int PER, class Out>
__global__ __launch_bounds__(TPB) void k_iw_down(uint64_t* __restrict__ nodes, Sampler smp, uint32_t base,
                                                 uint32_t basen, uint32_t total, uint32_t m, uint32_t climit,
                                                 uint32_t last, uint32_t set_mode, Ctrl* ctrl, Out out,
                                                 const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    if (dm) m = min(dm[0], m);
    smp.m = m;
    const uint32_t c0 = blockIdx.x * (TPB * PER) + threadIdx.x;
    if (c0 >= m) return;
    uint32_t nxt[PER];
    typename Lay<W>::Val acc[PER];
    iw_down<W, PER>(nodes, smp, base, basen, total, m, c0, climit, last, set_mode, ctrl, nxt, acc);
    [[maybe_unused]] typename Out::Cur cur{};
    if constexpr (OUTS) cur = out.begin(c0);
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const uint32_t c = c0 + r * TPB;
        if (c >= m) continue;
        if constexpr (OUTS) out.store(cur, c, acc[r], nxt[r] & IDX);
        else IwRec<W>::store(nodes, base + c, nxt[r], acc[r]);
    }
}

// The same on a level's records, whose results replace them. A call that
// enqueues more than one path passes the list of each, and the path word
// selects: the launches are shared by the plain path's list (0), the
// contracted one's level above its chases (1), and the contracted list itself
// where it is short (2).
template <bool W>
struct IwArg {
    typename Lay<W>::Rec* rec;  // the records, where this launch reads or replaces them
    uint64_t* nodes;
    const uint32_t* dm;         // the level's size, if only the device knows it (m is then a capacity)
    uint32_t m;                 // 0: nothing to do in this launch
    uint32_t base, basen, total, log2k, seed, climit;
};
template <bool W>
struct IwArgs {
    IwArg<W> a[3];
    const uint32_t* mode;  // null: a[0]
};
// f on the list that the path word selects, if it has something to do here.
// (One copy of f per list: a list picked into a variable would be copied
// through scratch memory, which cost every launch 20 us.)
template <bool W, class F>
__device__ __forceinline__ void iw_pick(const IwArgs<W>& s, F f) {
    auto on = [&](const IwArg<W>& a) {
        uint32_t m = a.m;
        if (m && a.dm) m = min(*a.dm, m);
        if (m) f(a, m);
    };
    const uint32_t md = s.mode ? *s.mode : (uint32_t)MODE_PLAIN;
    if (md == MODE_PLAIN) on(s.a[0]);
    else if (md == MODE_LOCAL) on(s.a[1]);
    else if (md == MODE_LOCAL_SMALL) on(s.a[2]);
}

template <bool W>
__global__ __launch_bounds__(TPB) void k_iwl_first(IwArgs<W> s) {
    iw_pick(s, [](const IwArg<W>& a, uint32_t m) {
        const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
        if (i >= m) return;
        const SrcLvl<W> src{a.rec, m};
        const Sampler smp{m, a.log2k, a.seed};
        if (a.log2k) iw_first<W, true>(src, smp, a.nodes, a.basen, i, LR_IW_CAP);
        else iw_first<W, false>(src, smp, a.nodes, a.basen, i, IW_CAP_ALONE);
    });
}

template <bool W>
__global__ __launch_bounds__(TPB) void k_iwl_walk(IwArgs<W> s) {
    iw_pick(s, [](const IwArg<W>& a, uint32_t m) {
        const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
        if (c < m) iw_walk<W>(a.nodes, Sampler{m, a.log2k, a.seed}, a.base, a.basen, a.total, c, LR_IW_CAP);
    });
}

// rec: the doubling alone, whose results are final (unweighted ones are in
// place already).
template <bool W>
__global__ __launch_bounds__(IW_DBL_TPB) void k_iwl_double(IwArgs<W> s, Ctrl* ctrl) {
    iw_pick(s, [ctrl](const IwArg<W>& a, uint32_t m) {
        const uint32_t c = blockIdx.x * IW_DBL_TPB + threadIdx.x;
        if (c >= m) return;
        uint32_t nxt;
        typename Lay<W>::Val acc;
        iw_double<W>(a.nodes, a.base, a.total, c, a.climit, a.base ? IW_TOP_CAP : NONE, ctrl, nxt, acc);
        if constexpr (W) {
            if (a.rec) a.rec[c] = Lay<W>::res(acc, nxt & IDX);
        }
    });
}

template <bool W, int PER>
__global__ __launch_bounds__(TPB) void k_iwl_down(IwArgs<W> s, Ctrl* ctrl) {
    iw_pick(s, [ctrl](const IwArg<W>& a, uint32_t m) {
        const uint32_t c0 = blockIdx.x * (TPB * PER) + threadIdx.x;
        if (c0 >= m) return;
        uint32_t nxt[PER];
        typename Lay<W>::Val acc[PER];
        iw_down<W, PER>(a.nodes, Sampler{m, a.log2k, a.seed}, a.base, a.basen, a.total, m, c0, a.climit,
                        a.base ? 0u : 1u, 0u, ctrl, nxt, acc);
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            const uint32_t c = c0 + r * TPB;
            if (c >= m) continue;
            if (a.base) IwRec<W>::store(a.nodes, a.base + c, nxt[r], acc[r]);
            else a.rec[c] = Lay<W>::res(acc[r], nxt[r] & IDX);
        }
    });
}

// --------------------------------------------------------------- resolve --
// Walk S + j of an initial element: its result is its own weight plus the
// result of the ruler it ended on, or plus nothing when it ended on a
// terminal (whose weight the chase already added).
template <bool W>
__global__ __launch_bounds__(TPB) void k_resolve(char* __restrict__ eb_raw, uint32_t S, const Ctrl* ctrl, int lvl,
                                                 const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    using L = Lay<W>;
    if (dm) S = dm[1];
    auto* rec = reinterpret_cast<typename L::Rec*>(eb_raw);
    auto* res = reinterpret_cast<typename L::Res*>(eb_raw);
    const uint32_t H = ctrl->lv[lvl].H;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < H; j += stride) {
        const typename L::Rec r = rec[S + j];
        typename L::Res o;
        if (r.nxt & TERM) {
            o = L::res(L::val(r), r.nxt & IDX);
        } else if (r.nxt < S) {
            const typename L::Res b = res[r.nxt];
            o = L::res(L::add(L::val(r), L::val(b)), L::root(b));
        } else {
            o = L::res(L::junk(), NONE);
        }
        res[S + j] = o;
    }
}

// ---------------------------------------------------------------- expand --
// rank(x) = result(walk(x)) - offset(x); root(x) = root(walk(x)).
// Wave tiles of 64 * EXPAND_CH elements, lane-strided (coalesced slot reads
// and output writes); the result gather hits the small per-walk table.
template <bool W, class Out>
__global__ __launch_bounds__(TPB) void k_expand(const typename Lay<W>::Slot* __restrict__ slot, uint32_t m,
                                                const typename Lay<W>::Res* __restrict__ res, uint32_t S,
                                                Ctrl* ctrl, int lvl, Out out, const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    using L = Lay<W>;
    if (dm) { m = dm[0]; S = dm[1]; }
    const uint32_t nw = S + ctrl->lv[lvl].H;
    const uint32_t lane = lane_id();
    const uint32_t wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint32_t nwaves = (gridDim.x * blockDim.x) >> 6;
    const uint32_t ntile = (m + 64 * EXPAND_CH - 1) / (64 * EXPAND_CH);
    bool bad = false;
    for (uint32_t tile = wave; tile < ntile; tile += nwaves) {
        const uint32_t base = tile * 64 * EXPAND_CH;
        if (base + lane >= m) continue;
        auto cur = out.begin(base + lane);
        typename L::Slot sv[EXPAND_CH];
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const uint32_t i = base + j * 64 + lane;
            if (i < m) sv[j] = slot[i];
        }
        // all gathers before any store: the outputs may alias nothing here,
        // but the compiler cannot know that and would order each gather
        // after the previous element's store
        typename L::Res rv[EXPAND_CH];
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const uint32_t i = base + j * 64 + lane;
            if (i < m && sv[j].w < nw) rv[j] = res[sv[j].w];
        }
        // all values first, then the stores (see k_lc_expand)
        typename L::Val ov[EXPAND_CH];
        uint32_t orr[EXPAND_CH];
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const typename L::Slot s = sv[j];
            const bool ok = s.w < nw;
            bad |= !ok && (base + j * 64 + lane < m);
            ov[j] = ok ? L::sub(L::val(rv[j]), L::val(s)) : L::junk();
            orr[j] = ok ? L::root(rv[j]) : NONE;
        }
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const uint32_t i = base + j * 64 + lane;
            if (i < m) out.store(cur, i, ov[j], orr[j]);
        }
    }
    if (__ballot(bad) && lane == 0) atomicOr(&ctrl->err, 4u);
}

// ---------------------------------------------------------- placement ----
// Log mode, after the recursion: every visit-log record (x, walk, offset)
// becomes (x, rank[, root][, sum]) and must land at x. Records are grouped by
// element range in two passes and a third pass writes each range of 2^s2
// elements from LDS, so every output line is written whole:
//   place1  resolve each record against its walk's result (records of one
//           walk sit close together in the log, so these gathers mostly hit
//           the caches) and group by x >> s1 (coarse ranges);
//   place2  within each coarse range, group by x >> s2 (fine ranges);
//   place3  one workgroup per fine range: scatter into LDS by x, then write
//           the outputs in order.
// Every element is visited exactly once, so range r receives exactly as many
// records as it has ids; its group starts at r << shift and a fill counter per
// range hands out positions inside it. All tiles append at the same few
// frontiers, so the partially written lines there complete quickly.
// Element and rank of a record are one 8 B word, in memory and in LDS: every run
// is written in half as many pieces and every record takes half the accesses of
// two arrays (2^28 elements: place1 1.35 -> 1.15 ms, place2 1.15 -> 0.99, a call 10.31 ->
// 9.95 ms; weighted records of 2^27: 1.20 -> 1.17 and 1.28 -> 1.20).
template <bool W>
struct PlaceArrays {
    uint32_t* x;   // grouping element ids only
    uint2* xr;     // (element, rank), over the same memory
    uint32_t* t;   // root
    int64_t* s;    // weighted rank (weighted levels only)
};

template <bool W, bool ROOT>
constexpr int place_per() { return (int)place_tile_records(W, ROOT) / place_tpb(W, ROOT); }

// LDS bytes of one grouping tile over nb ranges (device and host agree).
__host__ __device__ constexpr size_t place_lds_bytes(bool weighted, bool root, uint32_t nb) {
    const size_t T = place_tile_records(weighted, root);
    size_t o = 8 * (size_t)nb + (root ? 12 : 8) * T;
    if (weighted) o = ((o + 7) & ~(size_t)7) + 8 * T;
    return o;
}

// LDS counting sort of one tile by range, then coalesced writes of each
// range's run at [group(lo_bucket + b) + reserved, ...), space reserved with
// one atomic per range and tile. TWO: the ranges' two-sided counters (front
// and back, one line each), the tile taking the given side. Bound by
// instructions and LDS accesses next to the bytes, so the write loop adds one
// word per range to the record's place in the tile and nothing else; a range
// that overflows (some element was visited twice) keeps the whole tile back.
template <bool W, bool ROOT, int PER, bool VALS = true, bool TWO = false>
__device__ void place_tile(const uint32_t (&xs)[PER], const uint32_t (&rs)[PER], const uint32_t (&ts)[PER],
                           const int64_t (&ss)[PER], const uint32_t (&bs)[PER], uint32_t nb, uint32_t shift,
                           uint32_t lo_bucket, uint32_t n, uint32_t* __restrict__ fill, PlaceArrays<W> out,
                           Ctrl* ctrl, unsigned char* lds, uint32_t side = 0) {
    constexpr int TPB_ = place_tpb(W, ROOT);
    constexpr uint32_t T = (uint32_t)PER * TPB_;
    size_t o = 0;
    uint32_t* hist = reinterpret_cast<uint32_t*>(lds + o);  // counts, then the range's first record in the tile
    o += 4 * (size_t)nb;
    uint32_t* gdst = reinterpret_cast<uint32_t*>(lds + o);  // record i of the tile goes to gdst + i
    o += 4 * (size_t)nb;
    uint32_t* sx = reinterpret_cast<uint32_t*>(lds + o);
    uint2* sxr = reinterpret_cast<uint2*>(lds + o);
    o += (VALS ? 8 : 4) * (size_t)T;
    uint32_t* st = nullptr;
    if constexpr (ROOT) {
        st = reinterpret_cast<uint32_t*>(lds + o);
        o += 4 * (size_t)T;
    }
    int64_t* sw = nullptr;
    if constexpr (W) {
        o = (o + 7) & ~(size_t)7;
        sw = reinterpret_cast<int64_t*>(lds + o);
        o += 8 * (size_t)T;
    }
    __shared__ uint32_t scan_sh[TPB_ / 64];
    __shared__ uint32_t tile_total, over;
    const uint32_t t = threadIdx.x;
    uint32_t lr[PER];
    for (uint32_t b = t; b < nb; b += TPB_) hist[b] = 0;
    if (t == 0) over = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (xs[j] < n) lr[j] = atomicAdd(&hist[bs[j]], 1u);
    __syncthreads();
    // exclusive scan of hist (each lane owns a run of consecutive ranges) and reservations
    const uint32_t chunk = (nb + TPB_ - 1) / TPB_;
    const uint32_t a = min(t * chunk, nb), e = min(a + chunk, nb);
    uint32_t sum = 0;
    for (uint32_t b = a; b < e; ++b) sum += hist[b];
    uint32_t total;
    uint32_t run = block_exscan(sum, scan_sh, &total);
    for (uint32_t b = a; b < e; ++b) {
        const uint32_t h = hist[b];
        uint32_t g = 0;
        if (h) {
            const uint32_t r = lo_bucket + b;
            const uint32_t lo = r << shift;
            const uint32_t len = min(1u << shift, n - lo);
            const uint32_t old = atomicAdd(&fill[TWO ? (2 * r + side) * FILL_LINE : r], h);
            // the back side's run ends where the previous back run began
            g = lo + ((TWO && side) ? len - old - h : old);
            if (old > len || h > len - old) over = 1;
        }
        gdst[b] = g - run;
        hist[b] = run;
        run += h;
    }
    if (t == 0) tile_total = total;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (xs[j] < n) {
            const uint32_t p = hist[bs[j]] + lr[j];
            if constexpr (VALS) sxr[p] = make_uint2(xs[j], rs[j]);
            else sx[p] = xs[j];
            if constexpr (ROOT) st[p] = ts[j];
            if constexpr (W) sw[p] = ss[j];
        }
    }
    __syncthreads();
    const uint32_t cnt = over ? 0u : tile_total;
    if (over && t == 0) atomicOr(&ctrl->err, 64u);
    for (uint32_t i = t; i < cnt; i += TPB_) {
        uint2 v;
        if constexpr (VALS) v = sxr[i];
        else v.x = sx[i];
        const uint32_t p = gdst[(v.x >> shift) - lo_bucket] + i;
        if constexpr (VALS) out.xr[p] = v;
        else out.x[p] = v.x;
        if constexpr (ROOT) out.t[p] = st[i];
        if constexpr (W) out.s[p] = sw[i];
    }
    __syncthreads();
}

template <bool W, bool ROOT, bool PACK>
__global__ __launch_bounds__(place_tpb(W, ROOT)) void k_place1(LogArrays<W> lg, uint32_t max_chunks,
                                                const typename Lay<W>::Res* __restrict__ res, uint32_t S,
                                                Ctrl* ctrl, uint32_t n, uint32_t s1, uint32_t nb1,
                                                uint32_t* __restrict__ fill1, PlaceArrays<W> out, const uint32_t* dm,
                                                Gate gate) {
    if (gate.off()) return;
    if (dm) { n = dm[0]; S = dm[1]; }
    using L = Lay<W>;
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int PER = place_per<W, ROOT>();
    constexpr int TPB_ = place_tpb(W, ROOT);
    constexpr uint32_t T = PER * TPB_;
    const uint32_t used = min(ctrl->chunks, max_chunks) * LOG_CHUNK;
    const uint32_t nw = S + ctrl->lv[0].H;
    const uint32_t tiles = (used + T - 1) / T;
    // The fields of every record of a tile in one round of loads (a padding
    // record names no element and is read like the others: it shares their
    // lines). The next tile's round is issued before this tile is grouped:
    // the grouping's barriers wait for LDS only, so those loads stay in
    // flight meanwhile. Packed records are decoded when they are used.
    const LogFmt fmt(n, nw, lg.ccap, lg.bocap);
    uint32_t nx[PER], nwl[PER];
    uint64_t nr[PER];
    typename L::Val noff[PER];
    auto load_tile = [&](uint32_t tile) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint32_t i = tile * T + j * TPB_ + threadIdx.x;
            if constexpr (PACK) {
                nr[j] = ~0ull;
                if (i < used) {
                    nr[j] = lg.r[i];
                    if constexpr (W) noff[j].s = lg.s[i];
                }
            } else {
                nx[j] = NONE;
                nwl[j] = NONE;
                if (i < used) {
                    nx[j] = lg.x[i];
                    nwl[j] = lg.w[i];
                    noff[j].c = lg.c[i];
                    if constexpr (W) noff[j].s = lg.s[i];
                }
            }
        }
    };
    if (blockIdx.x < tiles) load_tile(blockIdx.x);
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        uint32_t xs[PER], rs[PER], ts[PER], bs[PER], wl[PER];
        int64_t ss[PER];
        typename L::Val offs[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if constexpr (PACK) {
                xs[j] = fmt.x(nr[j]);
                wl[j] = fmt.w(nr[j]);
                offs[j].c = fmt.o(nr[j]);
                if constexpr (W) offs[j].s = noff[j].s;
            } else {
                xs[j] = nx[j];
                wl[j] = nwl[j];
                offs[j] = noff[j];
            }
        }
        if constexpr (PACK) {
            // a continuation id stands for (walk, offset its records count from)
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                if (xs[j] < n && wl[j] >= nw) {
                    const uint32_t cid = wl[j] - nw;
                    if (cid < lg.ccap) {
                        const uint2 e = lg.cont[cid];
                        wl[j] = e.x;
                        offs[j].c += e.y;
                    } else {
                        wl[j] = NONE;
                    }
                }
            }
        }
        // every walk result (the records of a walk sit together, so these
        // mostly hit the caches), all issued before any is used
        typename L::Res bres[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (xs[j] < n && wl[j] < nw) bres[j] = res[wl[j]];
        if (tile + gridDim.x < tiles) load_tile(tile + gridDim.x);
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (xs[j] < n) {
                const uint32_t w = wl[j];
                const typename L::Val off = offs[j];
                if (w < nw) {
                    const typename L::Res b = bres[j];
                    const typename L::Val v = L::sub(L::val(b), off);
                    rs[j] = v.c;
                    ts[j] = L::root(b);
                    if constexpr (W) ss[j] = v.s;
                } else {
                    rs[j] = NONE;
                    ts[j] = NONE;
                    if constexpr (W) ss[j] = INT64_MIN;
                    atomicOr(&ctrl->err, 4u);
                }
                bs[j] = xs[j] >> s1;
            }
        }
        place_tile<W, ROOT, PER, true, true>(xs, rs, ts, ss, bs, nb1, s1, 0, n, fill1, out, ctrl, lds, tile & 1u);
    }
}

// fill1: the coarse ranges' two-sided counters. Every coarse range is full: its
// front and back counts must add up to its length.
template <bool W, bool ROOT>
__global__ __launch_bounds__(place_tpb(W, ROOT)) void k_place2(PlaceArrays<W> in, Ctrl* ctrl, uint32_t n, uint32_t s1, uint32_t s2,
                                                uint32_t* __restrict__ fill2, PlaceArrays<W> out, const uint32_t* dm,
                                                const uint32_t* __restrict__ fill1, Gate gate) {
    if (gate.off()) return;
    if (dm) n = dm[0];
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int PER = place_per<W, ROOT>();
    constexpr int TPB_ = place_tpb(W, ROOT);
    constexpr uint32_t T = PER * TPB_;
    const uint32_t tiles = (n + T - 1) / T;
    const uint32_t fan = 1u << (s1 - s2);
    // All tiles of one coarse range append to the same fan frontiers. Workgroup
    // i runs on XCD i mod 8, so the tiles of coarse range c go to workgroups
    // on XCD c mod 8: the partial lines at a frontier then meet in one L2.
    const uint32_t tpc = (1u << s1) / T;                        // tiles per coarse range
    const bool xcd = LR_XCD_GROUPS && (gridDim.x % 8) == 0;
    const uint32_t lane8 = blockIdx.x % 8, step = xcd ? gridDim.x / 8 : gridDim.x;
    // the workgroup's tiles in order: q advances by step; NONE when done
    uint32_t q = xcd ? blockIdx.x / 8 : blockIdx.x;
    auto next_tile = [&]() -> uint32_t {
        for (;; q += step) {
            if (!xcd) return q < tiles ? q : NONE;
            const uint32_t c = lane8 + 8 * (q / tpc);
            if (c * tpc >= tiles) return NONE;
            const uint32_t tile = c * tpc + q % tpc;
            if (tile < tiles) return tile;
        }
    };
    // every field of a tile's records in one round of loads (the value loads
    // do not wait for the element id); the next tile's round is issued while
    // this tile is grouped (the grouping's barriers wait for LDS only)
    uint32_t nx[PER], nr[PER], nt[PER];
    int64_t ns[PER];
    auto load_tile = [&](uint32_t tile) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint32_t i = tile * T + j * TPB_ + threadIdx.x;
            nx[j] = NONE;
            if (i < n) {
                const uint2 e = in.xr[i];
                nx[j] = e.x;
                nr[j] = e.y;
                if constexpr (ROOT) nt[j] = in.t[i];
                if constexpr (W) ns[j] = in.s[i];
            }
        }
    };
    uint32_t tile = next_tile();
    if (tile != NONE) load_tile(tile);
    while (tile != NONE) {
        const uint32_t c = (tile * T) >> s1;  // coarse range of this tile (T divides 2^s1)
        if (threadIdx.x == 0 && tile % tpc == 0) {
            // the range's two sides met exactly (otherwise some element was
            // visited twice or not at all)
            const uint32_t len = min(1u << s1, n - (c << s1));
            const uint64_t got = (uint64_t)fill1[2 * c * FILL_LINE] + fill1[(2 * c + 1) * FILL_LINE];
            if (got != len) atomicOr(&ctrl->err, 64u);
        }
        uint32_t xs[PER], rs[PER], ts[PER], bs[PER];
        int64_t ss[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            xs[j] = nx[j];
            rs[j] = nr[j];
            if constexpr (ROOT) ts[j] = nt[j];
            if constexpr (W) ss[j] = ns[j];
        }
        q += step;
        const uint32_t nxt_tile = next_tile();
        if (nxt_tile != NONE) load_tile(nxt_tile);
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (xs[j] < n && (xs[j] >> s1) != c) {  // stale record: the input is not a forest
                atomicOr(&ctrl->err, 64u);
                xs[j] = NONE;
            }
            if (xs[j] < n) bs[j] = (xs[j] >> s2) - c * fan;
        }
        place_tile<W, ROOT, PER>(xs, rs, ts, ss, bs, fan, s2, c * fan, n, fill2, out, ctrl, lds);
        tile = nxt_tile;
    }
}

// One workgroup per fine range of 2^s2 elements: place the records by x in
// LDS, then write the outputs in element order.
template <bool W, bool ROOT, class Out>
__global__ __launch_bounds__(place_tpb(W, ROOT)) void k_place3(PlaceArrays<W> in, Ctrl* ctrl, uint32_t n, uint32_t s2, uint32_t nb2,
                                                const uint32_t* __restrict__ fill2, int check, Out out,
                                                const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    if (dm) {  // a device-side size: only the ranges it covers
        n = dm[0];
        nb2 = (n + (1u << s2) - 1) >> s2;
    }
    using L = Lay<W>;
    extern __shared__ __align__(16) unsigned char lds[];
    const uint32_t R = 1u << s2;
    int64_t* ls = reinterpret_cast<int64_t*>(lds);
    uint32_t* lr = reinterpret_cast<uint32_t*>(lds + (W ? 8 * (size_t)R : 0));
    uint32_t* lt = lr + R;
    const uint32_t t = threadIdx.x;
    for (uint32_t f = blockIdx.x; f < nb2; f += gridDim.x) {
        const uint32_t base = f << s2;
        const uint32_t len = min(R, n - base);
        for (uint32_t i = t; i < len; i += place_tpb(W, ROOT)) {
            lr[i] = NONE;
            if constexpr (ROOT) lt[i] = NONE;
            if constexpr (W) ls[i] = INT64_MIN;
        }
        if (check && t == 0 && fill2[f] != len) atomicOr(&ctrl->err, 128u);
        __syncthreads();
        // four records per lane per round, every field loaded before any LDS
        // store (the value loads do not wait for the element id)
        constexpr int U = 4;
        for (uint32_t i0 = t; i0 < len; i0 += U * place_tpb(W, ROOT)) {
            uint32_t kk[U], rv[U], tv[U];
            int64_t sv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = i0 + u * place_tpb(W, ROOT);
                kk[u] = NONE;
                if (i < len) {
                    const uint2 e = in.xr[base + i];
                    kk[u] = e.x - base;
                    rv[u] = e.y;
                    if constexpr (ROOT) tv[u] = in.t[base + i];
                    if constexpr (W) sv[u] = in.s[base + i];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (kk[u] < len) {
                    lr[kk[u]] = rv[u];
                    if constexpr (ROOT) lt[kk[u]] = tv[u];
                    if constexpr (W) ls[kk[u]] = sv[u];
                }
            }
        }
        __syncthreads();
        if (t < len) {
            auto cur = out.begin(base + t);
            for (uint32_t i = t; i < len; i += place_tpb(W, ROOT)) {
                typename L::Val v;
                v.c = lr[i];
                if constexpr (W) v.s = ls[i];
                out.store(cur, base + i, v, ROOT ? lt[i] : NONE);
            }
        }
        __syncthreads();
    }
}

// Interleave successor and weight (weighted level 0 in log mode).
template <int WT>
__global__ __launch_bounds__(TPB) void k_pair(const uint32_t* __restrict__ succ, const void* __restrict__ weight,
                                              uint32_t n, PairRec<WT>* __restrict__ out, Gate gate) {
    if (gate.off()) return;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        PairRec<WT> r{};
        r.s = succ[i];
        if constexpr (WT == 1) r.w = static_cast<const int32_t*>(weight)[i];
        if constexpr (WT == 3) r.w = static_cast<const int8_t*>(weight)[i];
        if constexpr (WT == 2) r.w = static_cast<const int64_t*>(weight)[i];
        out[i] = r;
    }
}

// ------------------------------------------------- predecessor marks ----
// Level 0 in log mode with more than one list: instead of one random byte
// store per link, the link targets are grouped by element range with the first
// placement pass (ids only) and written range by range from LDS. Every id is the
// target of at most one link, so no range receives more targets than it has ids.
// The grouping counts a link's target in debug builds.
constexpr int MARK_TPB = 1024;
// ids a lane holds in the grouping: a tile's run in a group is 32 ids on average
// at 512 groups (2^27 ids: 16 a lane 522 us, 32 360)
constexpr int MARK_PER = 32;
constexpr uint32_t MARK_TILE = MARK_PER * place_tpb(false, false);
static_assert(8 * PLACE_MAX_RANGES + 4 * MARK_TILE <= LDS_MAX, "a tile of targets fits one workgroup's LDS");
// TGT: the input is a plain list of nin target ids (those not below n are
// skipped) instead of a successor array of n entries.
template <bool TGT>
__global__ __launch_bounds__(place_tpb(false, false)) void k_mark1(const uint32_t* __restrict__ succ, uint32_t n, uint32_t s1,
                                                            uint32_t nb1, uint32_t* __restrict__ fill1,
                                                            PlaceArrays<false> out, Ctrl* ctrl, Gate gate,
                                                            const uint32_t* dm, uint32_t nin = 0) {
    if (gate.off()) return;
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int PER = MARK_PER;
    constexpr int TPB_ = place_tpb(false, false);
    constexpr uint32_t T = PER * TPB_;
    if (dm) n = dm[0];
    if constexpr (!TGT) nin = n;
    const uint32_t tiles = (nin + T - 1) / T;
    // the next tile's successors are loaded while this tile is grouped (the
    // grouping's barriers wait for LDS only)
    uint32_t ns[PER];
    auto load_tile = [&](uint32_t tile) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint32_t i = tile * T + j * TPB_ + threadIdx.x;
            ns[j] = (i < nin) ? succ[i] : NONE;
        }
    };
    if (blockIdx.x < tiles) load_tile(blockIdx.x);
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        uint32_t xs[PER], rs[PER], ts[PER], bs[PER];
        int64_t ss[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint32_t i = tile * T + j * TPB_ + threadIdx.x;
            const uint32_t s = ns[j];
            if constexpr (TGT) xs[j] = s < n ? s : NONE;  // a target id
            else xs[j] = (s != i && s < n) ? s : NONE;    // the target of a link
            bs[j] = xs[j] >> s1;
            if constexpr (!TGT) if (xs[j] != NONE) LR_DBG_COUNT(mark, 0, xs[j]);
        }
        if (tile + gridDim.x < tiles) load_tile(tile + gridDim.x);
        place_tile<false, false, PER, false, true>(xs, rs, ts, ss, bs, nb1, s1, 0, n, fill1, out, ctrl, lds, tile & 1u);
    }
}

// One workgroup per group of 2^s1 ids: its targets (fill1 holds how many lie at
// the group's two ends) set bits in LDS. The ids left without one that are no
// rulers are the level's initial elements: they start walks S + j, j counted up
// in Ctrl.lv[0].H with one atomic a group. With DIR the bits become a bitmap with
// running counts instead: word w of `dir` holds the bits of ids [32 w, 32 w + 32)
// and the marked ids before them in their range of 2^PLACE_FINE_SHIFT ids; cnt[f]
// is that range's count. With a bit per id a group is 2^18 ids in 32 KB, so one
// grouping pass is enough. Bound by the LDS atomics: two workgroups a CU take 192
// us for 2^27 ids, one (groups of 2^19) 301; loading ahead gains nothing.
// Against a second grouping pass (375 us) and byte marks of 8192 ids a workgroup
// (155): a 2^27 forest 6.28 -> 6.11 ms, int64 sums over it 9.51 -> 9.33, a forest of
// 9 * 10^7 4.37 -> 4.27, a 2^26-vertex tree 8.91 -> 8.76. Against marks written as
// bytes, with the heads counted, scanned and written by three more kernels: a 5 M
// forest 335 -> 324 us, 33 M 1856 -> 1807, 2^27 int64 9.33 -> 9.17 ms.
template <bool DIR>
__global__ __launch_bounds__(MARK_TPB) void k_mark_bits(const uint32_t* __restrict__ tx, uint32_t n, uint32_t s1,
                                                        uint32_t nb1, const uint32_t* __restrict__ fill1,
                                                        Sampler smp, char* __restrict__ eb, uint32_t S,
                                                        uint32_t rec_bytes, uint2* __restrict__ dir,
                                                        uint32_t* __restrict__ cnt, Ctrl* ctrl, Gate gate,
                                                        const uint32_t* dm) {
    if (gate.off()) return;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ uint32_t sh[MARK_TPB / 64];
    __shared__ uint32_t first;
    uint32_t* bits = reinterpret_cast<uint32_t*>(lds);
    if (dm) { n = smp.m = dm[0]; S = dm[1]; }
    const uint32_t t = threadIdx.x;
    for (uint32_t g = blockIdx.x; g < nb1; g += gridDim.x) {
        const uint32_t lo = g << s1;
        if (lo >= n) break;  // device-side size: the groups past it hold no ids
        const uint32_t len = min(1u << s1, n - lo);
        const uint32_t words = (len + 31) / 32;
        for (uint32_t i = t; i < words; i += MARK_TPB) bits[i] = 0;
        const uint32_t f0 = fill1[2 * g * FILL_LINE], f1 = fill1[(2 * g + 1) * FILL_LINE];
        if (t == 0 && (uint64_t)f0 + f1 > len) atomicOr(&ctrl->err, 64u);  // a target has two links
        const uint32_t front = min(f0, len), c = front + min(f1, len - front);
        const uint32_t gap = len - c;  // between the two ends
        __syncthreads();
        constexpr int U = 8;  // loads in flight per lane
        for (uint32_t i0 = t; i0 < c; i0 += U * MARK_TPB) {
            uint32_t u[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const uint32_t i = i0 + j * MARK_TPB;
                u[j] = (i < c) ? tx[lo + i + (i < front ? 0u : gap)] - lo : NONE;
            }
#pragma unroll
            for (int j = 0; j < U; ++j)
                if (u[j] < len) atomicOr(&bits[u[j] >> 5], 1u << (u[j] & 31));
        }
        __syncthreads();
        if constexpr (DIR) {
            constexpr uint32_t RW = (1u << PLACE_FINE_SHIFT) / 32;  // words of a counted range
            static_assert(MARK_TPB % RW == 0 && RW % 64 == 0, "whole ranges a round, whole wavefronts a range");
            for (uint32_t w0 = 0; w0 < words; w0 += MARK_TPB) {
                const uint32_t w = w0 + t;
                const uint32_t v = w < words ? bits[w] : 0u;
                uint32_t in = __popc(v);
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const uint32_t y = __shfl_up(in, o);
                    if ((t & 63) >= o) in += y;
                }
                if ((t & 63) == 63) sh[t >> 6] = in;
                __syncthreads();
                uint32_t pre = in - __popc(v);
                for (uint32_t q = t / RW * (RW / 64); q < (t >> 6); ++q) pre += sh[q];
                if (w < words) {
                    dir[(lo >> 5) + w] = make_uint2(v, pre);
                    if (w % RW == RW - 1 || w == words - 1) cnt[(lo >> PLACE_FINE_SHIFT) + w / RW] = pre + __popc(v);
                }
                __syncthreads();  // sh is reused by the next round
            }
        } else {
            uint32_t mine = 0;
            for (uint32_t w = t; w < words; w += MARK_TPB) {
                const uint32_t x0 = lo + 32 * w, left = n - x0;
                uint32_t no = bits[w];  // marked ids and rulers
                const uint32_t blk = x0 >> smp.log2k;
                const uint32_t blks = smp.log2k < 5 ? 32u >> smp.log2k : 1u;
                for (uint32_t j = 0; j < blks && ((blk + j) << smp.log2k) < n; ++j) {
                    const uint32_t d = smp.start(blk + j) - x0;
                    if (d < 32) no |= 1u << d;
                }
                const uint32_t h = ~no & (left < 32 ? (1u << left) - 1u : ~0u);
                bits[w] = h;
                mine += __popc(h);
            }
            uint32_t total;
            block_exscan(mine, sh, &total);
            if (t == 0) first = total ? atomicAdd(&ctrl->lv[0].H, total) : 0u;
            __syncthreads();
            uint32_t run = S + first;
            for (uint32_t w0 = 0; total && w0 < words; w0 += MARK_TPB) {
                const uint32_t w = w0 + t;
                uint32_t h = w < words ? bits[w] : 0u, tot;
                uint32_t pos = run + block_exscan(__popc(h), sh, &tot);
                for (; h; h &= h - 1)
                    *reinterpret_cast<uint32_t*>(eb + (size_t)pos++ * rec_bytes) = lo + 32 * w + __ffs(h) - 1;
                run += tot;
                __syncthreads();  // sh is reused by the next round
            }
            __syncthreads();  // LDS is reused by the next ids
        }
    }
}

// ---------------------------------------------------------------- Wyllie --
template <bool W, class Src>
__global__ __launch_bounds__(TPB) void k_wy_init(Src src, typename Lay<W>::Rec* __restrict__ a, uint32_t m) {
    using L = Lay<W>;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        uint32_t nxt;
        typename L::Val v;
        src.load(i, nxt, v);
        a[i] = (nxt & TERM) ? L::rec(i, L::zero()) : L::rec(nxt, v);
    }
}

// One doubling round: d[i] += d[f[i]]; f[i] = f[f[i]] (ping-pong buffers).
// The last round writes the outputs instead (terminal weight is 0 here).
template <bool W, bool LAST>
__global__ __launch_bounds__(TPB) void k_wy_round(const typename Lay<W>::Rec* __restrict__ a,
                                                  typename Lay<W>::Rec* __restrict__ b, uint32_t m,
                                                  OutUser<W, true, true, true> out) {
    using L = Lay<W>;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const typename L::Rec r = a[i];
        const typename L::Rec q = a[r.nxt];
        const typename L::Val d = L::add(L::val(r), L::val(q));
        if constexpr (LAST) {
            typename OutUser<W, true, true, true>::Cur c;
            out.store(c, i, d, q.nxt);
        } else {
            b[i] = L::rec(q.nxt, d);
        }
    }
}

template <bool W>
__global__ __launch_bounds__(TPB) void k_wy_copy(const typename Lay<W>::Rec* __restrict__ a, uint32_t m,
                                                 OutUser<W, true, true, true> out) {
    using L = Lay<W>;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const typename L::Rec r = a[i];
        typename OutUser<W, true, true, true>::Cur c;
        out.store(c, i, L::val(r), r.nxt);
    }
}

// ------------------------------------------------------------- fallback --
// The bounded fallback, run only when a walk of the ruling-set path reached
// its step cap (an order built against the sampling): pointer doubling over
// the whole input, whatever the order. Its kernels are enqueued with every call
// and return at once unless the cap was hit (about 2 us each), so there are two:
// first records of up to FB_HOPS links, then the asynchronous doubling of the
// independent walks (see there) by as many lanes as the chip holds, each going
// round its share of the elements, one hop each, until all have reached a
// terminal. All elements move together, so a pass about doubles what is
// left: 28 passes at the most, of one random read per element. On orders with
// every ruler last (the other side: rounds of pointer doubling with 16- or
// 128-fold jumps, three to eight launches): 2^18 elements 0.65 -> 0.18 ms, 2^20
// 2.33 -> 0.51, 2^22 5.0 -> 1.7, 2^24 25.5 -> 7.9, int64 sums over 2^23 14.5 -> 9.0.
constexpr uint32_t FB_HOPS = 16;

template <bool W, class Src>
__global__ __launch_bounds__(TPB) void k_fb_first(Src src, uint64_t* __restrict__ nodes, uint32_t m,
                                                  const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    if (dm) m = src.m = dm[0];
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride)
        iw_first<W, false>(src, Sampler{}, nodes, 0u, i, FB_HOPS);
}

// err: where to report a path that never reaches a terminal (more links than
// elements: a cycle), or null. An element that catches another's record between
// two of its stores (weighted) takes one link from the input instead, so every
// element moves in every pass and the end waits for no other lane's stores.
template <bool W, class Src, class Out>
__global__ __launch_bounds__(TPB) void k_fb_double(Src src, uint64_t* __restrict__ nodes, uint32_t m, Out out,
                                                   uint32_t* err, const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    if (dm) m = src.m = dm[0];
    using L = Lay<W>;
    const uint32_t stride = gridDim.x * blockDim.x;
    const uint32_t i0 = blockIdx.x * blockDim.x + threadIdx.x;
    if (i0 >= m) return;
    for (bool open = true; open;) {
        open = false;
        for (uint32_t i = i0; i < m; i += stride) {
            uint32_t nxt;
            typename L::Val acc;
            IwRec<W>::template load<true>(nodes, i, nxt, acc);  // its own stores, in order
            if (nxt & TERM) continue;
            bool bad = nxt >= m;
            const uint32_t before = acc.c;
            if (!bad && !iw_hop<W, true>(nodes, nxt, acc)) {
                typename L::Val v;
                uint32_t nn;
                src.load(nxt, nn, v);
                acc = L::add(acc, v);
                nxt = nn;
            }
            bad |= hop_stuck(before, acc.c, nxt & TERM, m);
            if (bad) {
                nxt = TERM | IDX;
                acc = L::junk();
                if (err) atomicOr(err, ERR_FALLBACK_CYCLE);
            }
            IwRec<W>::store(nodes, i, nxt, acc);
            open |= !(nxt & TERM);
        }
    }
    auto cur = out.begin(i0);
    for (uint32_t i = i0; i < m; i += stride) {
        uint32_t nxt;
        typename L::Val acc;
        IwRec<W>::template load<true>(nodes, i, nxt, acc);
        out.store(cur, i, acc, nxt & IDX);
    }
}

// Per level, log2 of the ruler spacing (device-side level sizes follow from them).
struct LevelShifts { uint8_t lg[MAXL]; };

// ----------------------------------------------------------------- batch --
// The request table is built on the device: k_batch_desc copies descriptors
// passed by value (up to BATCH_ARG_DESC per launch) into the workspace, and
// k_batch_index scans their sizes into the request bases and first chunks and
// fills the header. With device-side sizes (a batch planned for a capacity,
// as a replayed graph is) it also publishes the level sizes.
struct BatchDescArg {
    BatchDesc d[BATCH_ARG_DESC];
    uint32_t first;  // table index of d[0]
    uint32_t cnt;    // descriptors in this launch
    uint32_t count;  // requests of the whole batch (written to the header)
};
static_assert(sizeof(BatchDescArg) <= 4096, "kernel arguments");

__global__ __launch_bounds__(64) void k_batch_desc(BatchDescArg a, BatchDesc* __restrict__ dst,
                                                   BatchHdr* __restrict__ hdr) {
    for (uint32_t i = threadIdx.x; i < a.cnt; i += 64) dst[a.first + i] = a.d[i];
    if (a.first == 0 && threadIdx.x == 0) hdr->count = a.count;
}

// One workgroup: bases[q] = elements before request q, boff[q] = chunks
// before it (count + 1 entries each); the header's chunk and element totals;
// dm[0] = total; with levels > 0 (device-side sizes) also dm[l + 1] =
// ceil(dm[l] / k_l).
__device__ __forceinline__ void batch_index(const BatchDesc* d, uint32_t count, uint32_t* __restrict__ bases,
                                            uint32_t* __restrict__ boff, BatchHdr* __restrict__ hdr,
                                            Ctrl* ctrl, uint32_t levels, const LevelShifts& ks) {
    __shared__ uint32_t sh[2 * (1024 / 64)];
    const uint32_t per = (count + 1023u) >> 10;
    const uint32_t lo = min(threadIdx.x * per, count), hi = min(lo + per, count);
    uint32_t sn = 0, sc = 0;
    for (uint32_t q = lo; q < hi; ++q) {
        const uint32_t n = (uint32_t)d[q].n;
        sn += n;
        sc += (n + BATCH_CHUNK - 1) / BATCH_CHUNK;
    }
    uint32_t tn, tc;
    uint32_t an = block_exscan(sn, sh, &tn);
    uint32_t ac = block_exscan(sc, sh + 1024 / 64, &tc);
    for (uint32_t q = lo; q < hi; ++q) {
        const uint32_t n = (uint32_t)d[q].n;
        bases[q] = an;
        boff[q] = ac;
        an += n;
        ac += (n + BATCH_CHUNK - 1) / BATCH_CHUNK;
    }
    if (threadIdx.x == 0) {
        bases[count] = tn;
        boff[count] = tc;
        hdr->nchunks = tc;
        hdr->total = tn;
        uint32_t m = tn;
        ctrl->dm[0] = m;
        if (levels) {
            for (uint32_t l = 0; l < levels; ++l) {
                m = (m + (1u << ks.lg[l]) - 1u) >> ks.lg[l];
                ctrl->dm[l + 1] = m;
            }
        }
    }
}

__global__ __launch_bounds__(1024) void k_batch_index(const BatchDesc* __restrict__ d, uint32_t* __restrict__ bases,
                                                      uint32_t* __restrict__ boff, BatchHdr* __restrict__ hdr,
                                                      Ctrl* ctrl, uint32_t levels, LevelShifts ks) {
    batch_index(d, hdr->count, bases, boff, hdr, ctrl, levels, ks);
}

// k_batch_desc and k_batch_index in one launch, for a table of at most
// BATCH_ARG_DESC requests.
__global__ __launch_bounds__(1024) void k_batch_table(BatchDescArg a, BatchDesc* __restrict__ dst,
                                                      uint32_t* __restrict__ bases, uint32_t* __restrict__ boff,
                                                      BatchHdr* __restrict__ hdr, Ctrl* ctrl, uint32_t levels,
                                                      LevelShifts ks) {
    if (threadIdx.x < a.cnt) dst[threadIdx.x] = a.d[threadIdx.x];
    if (threadIdx.x == 0) hdr->count = a.count;
    __syncthreads();
    batch_index(dst, a.count, bases, boff, hdr, ctrl, levels, ks);
}

// One workgroup per chunk of BATCH_CHUNK ids of one request:
// concat[g] = base(q) + succ_q[g - base(q)]; out-of-range successors become
// terminals (no list leaves its request). The chunk also sums, for the one-list
// head test, ids minus successors of non-terminals and counts terminals.
__global__ __launch_bounds__(TPB) void k_batch_gather(const BatchDesc* __restrict__ d,
                                                      const uint32_t* __restrict__ bases,
                                                      const uint32_t* __restrict__ boff, const BatchHdr* hdr,
                                                      uint32_t* __restrict__ concat, uint2* __restrict__ part) {
    __shared__ uint64_t shs[TPB / 64];
    __shared__ uint32_t snt[TPB / 64];
    const uint32_t count = hdr->count, nchunks = hdr->nchunks;
    for (uint32_t b = blockIdx.x; b < nchunks; b += gridDim.x) {
        const uint32_t q = batch_find(boff, count, b);  // the request whose chunks hold b
        const uint32_t lo = bases[q], nq = bases[q + 1] - lo;
        const uint32_t start = (b - boff[q]) * BATCH_CHUNK;
        const uint32_t end = min(start + BATCH_CHUNK, nq);
        const uint32_t* sq = d[q].succ;
        uint64_t hs = 0;
        uint32_t nt = 0;
        for (uint32_t i = start + threadIdx.x; i < end; i += TPB) {
            const uint32_t s = sq[i];
            const uint32_t g = lo + i;
            const uint32_t c = (s < nq) ? lo + s : g;
            concat[g] = c;
            if (c == g) { ++nt; hs += g; }
            else hs += (uint64_t)g - c;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            hs += __shfl_xor(hs, o);
            nt += __shfl_xor(nt, o);
        }
        if ((threadIdx.x & 63) == 0) { shs[threadIdx.x >> 6] = hs; snt[threadIdx.x >> 6] = nt; }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int i = 1; i < TPB / 64; ++i) { hs += shs[i]; nt += snt[i]; }
            part[2 * b] = make_uint2((uint32_t)hs, (uint32_t)(hs >> 32));
            part[2 * b + 1] = make_uint2(nt, 0u);
        }
        __syncthreads();  // shs, snt are reused by the next chunk
    }
}

// One workgroup per request: its chunks' partial sums -> (head sum, terminals).
__global__ __launch_bounds__(TPB) void k_batch_reduce(const uint2* __restrict__ part,
                                                      const uint32_t* __restrict__ boff, const BatchHdr* hdr,
                                                      uint2* __restrict__ sums, Gate gate) {
    if (gate.off()) return;
    __shared__ uint64_t shs[TPB / 64];
    __shared__ uint32_t snt[TPB / 64];
    const uint32_t count = hdr->count;
    for (uint32_t q = blockIdx.x; q < count; q += gridDim.x) {
        uint64_t hs = 0;
        uint32_t nt = 0;
        for (uint32_t b = boff[q] + threadIdx.x; b < boff[q + 1]; b += TPB) {
            const uint2 h = part[2 * b];
            hs += (uint64_t)h.x | ((uint64_t)h.y << 32);
            nt += part[2 * b + 1].x;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            hs += __shfl_xor(hs, o);
            nt += __shfl_xor(nt, o);
        }
        if ((threadIdx.x & 63) == 0) { shs[threadIdx.x >> 6] = hs; snt[threadIdx.x >> 6] = nt; }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int i = 1; i < TPB / 64; ++i) { hs += shs[i]; nt += snt[i]; }
            sums[2 * q] = make_uint2((uint32_t)hs, (uint32_t)(hs >> 32));
            sums[2 * q + 1] = make_uint2(nt, 0u);
        }
        __syncthreads();
    }
}

// One workgroup, in place of the head-sum pass for a batch: if every
// non-empty request holds exactly one terminal, each is one list whose head is
// its head sum (the one-list shortcut per request). Then the heads that are
// not sampled rulers become the level-0 walk list in request order, and the
// level-0 marking and compaction are skipped as for a single list; otherwise
// the forest path runs. dm (device-side sizes) gives the level-0 size and
// walk count.
__global__ __launch_bounds__(1024) void k_batch_heads(const uint2* __restrict__ sums,
                                                      const uint32_t* __restrict__ bases, const BatchHdr* hdr,
                                                      Ctrl* ctrl, Sampler smp, char* __restrict__ eb, uint32_t S,
                                                      uint32_t rec_bytes, const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    __shared__ uint32_t sh[1024 / 64];
    if (threadIdx.x == 0) ctrl->hc_done = 0;  // the head-count kernels' workgroup counter
    if (dm) { smp.m = dm[0]; S = dm[1]; }
    const uint32_t count = hdr->count;
    int ok = 1;
    for (uint32_t q = threadIdx.x; q < count; q += 1024) {
        const uint32_t lo = bases[q], hi = bases[q + 1];
        if (lo == hi) continue;
        const uint64_t hs = (uint64_t)sums[2 * q].x | ((uint64_t)sums[2 * q].y << 32);
        if (sums[2 * q + 1].x != 1 || hs < lo || hs >= hi) ok = 0;
    }
    if (!__syncthreads_and(ok)) {
        if (threadIdx.x == 0) {
            ctrl->single = 0;
            ctrl->multi = 1;
            ctrl->mode = MODE_PLAIN;
            ctrl->lv[0].H = 0;  // the marks' pass adds the heads
            ctrl->lv[0].q = 0;
            ctrl->chunks = 0;
            ctrl->conts = 0;
        }
        return;
    }
    uint32_t run = 0;  // heads written so far
    for (uint32_t q0 = 0; q0 < count; q0 += 1024) {
        const uint32_t q = q0 + threadIdx.x;
        uint32_t h = NONE;
        if (q < count && bases[q] != bases[q + 1]) {
            h = sums[2 * q].x;  // < 2^31: the check above
            if (smp.sampled(h)) h = NONE;
        }
        uint32_t tot;
        const uint32_t pos = run + block_exscan(h != NONE ? 1u : 0u, sh, &tot);
        if (h != NONE) *reinterpret_cast<uint32_t*>(eb + (size_t)(S + pos) * rec_bytes) = h;
        run += tot;
        __syncthreads();  // sh is reused by the next round
    }
    if (threadIdx.x == 0) {
        ctrl->single = 1;
        ctrl->multi = 0;
        ctrl->mode = MODE_PLAIN;
        ctrl->lv[0].H = run;
        ctrl->lv[0].q = 0;
        ctrl->chunks = 0;
        ctrl->conts = 0;
    }
}

// ------------------------------------------------ tile-local contraction --
// Section 2.3: sublists whose links stay inside one tile of LOCAL_TILE
// consecutive ids are contracted before the ruling-set levels run. A local
// chain starts at an element that no element of its tile links to and ends at
// the first element whose successor lies outside the tile (or that is a
// terminal). The contracted list has one element per chain start, linked to
// the start that the chain's exit leads to, with the chain's link count (and
// weight) as its value; after it is ranked, every element takes the rank of
// its chain start minus its distance from that start.
//   chain    one workgroup per tile: chains by pointer jumping in LDS; per
//            element its chain start and distance; per 32 ids the start
//            bits; per chain its record, staged at the tile's own offset
//   scan     start counts -> compact ids of the first start of every tile
//   compact  staged records -> compact positions, exit successors -> compact
//            ids, predecessor marks for the first ruling-set level
//   expand   every element from its chain start's result
// Elements are owned lane-strided (element j * LC_TPB + lane), so every
// global access of the tile kernels is coalesced.
constexpr int LC_TPB = 512;  // 2^26 ids 589 us a call; 256 lanes 624, 1024 the same (weighted 25 % slower)
#ifndef LR_LC_GRID_PER_CU
#define LR_LC_GRID_PER_CU 64  // chain kernel workgroups per CU, each looping over tiles; 0 = one per tile
#endif
static_assert(LR_LC_GRID_PER_CU >= 0 && LR_LC_GRID_PER_CU <= 1024, "chain kernel workgroups per CU");
constexpr uint32_t LC_T = LOCAL_TILE;
constexpr int LC_PER = LC_T / LC_TPB;   // elements per lane
constexpr int LC_ROUNDS = 14;           // > log2(LC_T): chains of a tile converge within this many rounds
constexpr int LC_CHUNKS = LC_T / 64;    // 64-id chunks of a tile (one wave ballot each)
constexpr uint32_t LC_TGT = 0xffffu;    // jump entry: target (tile-relative id); link count in bits 16-31

static_assert(LC_T == (1u << LOCAL_SHIFT) && LC_T <= LC_TGT + 1 && LC_CHUNKS <= 64, "local tile");

// start ids are compact: tile base (scanned start counts) + starts before the
// element in its tile (word prefix + bits below it in its 32-id word)
__device__ __forceinline__ uint32_t lc_below(uint2 d, uint32_t y) {
    return d.y + __popc(d.x & ((1u << (y & 31)) - 1u));
}

// Chains by pointer jumping toward their starts. PD packs the current jump
// target (low 16 bits, tile-relative) and the link count to it (high 16
// bits); starts point to themselves. Writes pos (start's tile-relative
// compact index << 16 | distance, NONE on a cycle inside the tile), wd (weight
// from the start, weighted only), the tile's start bits and word prefixes
// (dir), its start count (cnt), and per chain its record at stage[tile *
// LC_T + index] with the exit's successor still a global id.
template <bool W, int WT>
__global__ __launch_bounds__(LC_TPB) void k_lc_chain(const uint32_t* __restrict__ succ, const void* __restrict__ weight,
                                                     uint32_t n, uint32_t ntiles, uint32_t* __restrict__ cnt,
                                                     uint2* __restrict__ dir,
                                                     typename Lay<W>::Rec* __restrict__ stage,
                                                     uint32_t* __restrict__ pos, int64_t* __restrict__ wd,
                                                     Ctrl* ctrl, Gate gate) {
    if (gate.off()) return;
    using L = Lay<W>;
    using Val = typename L::Val;
    __shared__ uint32_t PD[LC_T];
    __shared__ int64_t WS[W ? LC_T : 1];
    __shared__ uint2 DIR[LC_T / 32];
    __shared__ uint32_t CH[LC_CHUNKS];
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const uint32_t b = tile * LC_T;
        const uint32_t len = min(LC_T, n - b);
        const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        uint32_t sv[LC_PER];
        int64_t wv[LC_PER];
#pragma unroll
        for (int j = 0; j < LC_PER; ++j) {
            const uint32_t i = j * LC_TPB + threadIdx.x;
            sv[j] = NONE;
            wv[j] = 1;
            if (i < len) {
                sv[j] = succ[b + i];
                if constexpr (WT == 1) wv[j] = static_cast<const int32_t*>(weight)[b + i];
                if constexpr (WT == 3) wv[j] = static_cast<const int8_t*>(weight)[b + i];
                if constexpr (WT == 2) wv[j] = static_cast<const int64_t*>(weight)[b + i];
                if constexpr (W) WS[i] = 0;
            }
            PD[i] = i;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < LC_PER; ++j) {
            const uint32_t i = j * LC_TPB + threadIdx.x;
            const uint32_t d = sv[j] - b;
            if (i < len && d < len && d != i) {
                PD[d] = i | (1u << 16);
                if constexpr (W) WS[d] = wv[j];
            }
        }
        __syncthreads();
        uint32_t v[LC_PER];
        int64_t ws[LC_PER];
#pragma unroll
        for (int j = 0; j < LC_PER; ++j) {
            const uint32_t i = j * LC_TPB + threadIdx.x;
            v[j] = (i < len) ? PD[i] : i;
            ws[j] = 0;
            if constexpr (W) if (i < len) ws[j] = WS[i];
            // chunk j * 8 + wave covers ids [64 (j * 8 + wave), +64), lane = id offset
            const uint64_t starts = __ballot(i < len && (v[j] >> 16) == 0);
            if (lane == 0) CH[j * (LC_TPB / 64) + wave] = __popcll(starts);
            if (lane < 2) DIR[2 * (j * (LC_TPB / 64) + wave) + lane] = make_uint2((uint32_t)(starts >> (32 * lane)), 0u);
        }
        __syncthreads();
        if (wave == 0) {  // exclusive scan of the 64 chunk counts, then the word prefixes
            const uint32_t c = (lane < (uint32_t)LC_CHUNKS) ? CH[lane] : 0u;
            uint32_t inc = c;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(inc, o);
                if (lane >= (uint32_t)o) inc += y;
            }
            if (lane < (uint32_t)LC_CHUNKS) {
                const uint32_t pre = inc - c;
                const uint32_t lo = DIR[2 * lane].x;
                DIR[2 * lane].y = pre;
                DIR[2 * lane + 1].y = pre + __popc(lo);
            }
            if (lane == 63) cnt[tile] = inc;
        }
        if constexpr (!W) {
            // in place and without barriers: a 32-bit entry always holds a
            // consistent (target, count) pair, so an older one only jumps less
            // far, and a wavefront stops when its own elements have reached
            // their starts (entries that point to themselves) or, on a cycle
            // inside the tile, counted more links than a tile has. An element
            // that has not moves at least one link a turn, so LC_T turns are
            // enough; on a cycle they are the end of counts that outgrow their
            // 16 bits. Bound by the LDS gathers (2^26 ids: 342 us with two
            // barriers a round, 275 without, 278 with the turns counted)
            for (uint32_t left = LC_T; left;) {
                uint32_t u[LC_PER];
                bool open = false;
#pragma unroll
                for (int j = 0; j < LC_PER; ++j)
                    u[j] = __hip_atomic_load(&PD[v[j] & LC_TGT], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
                for (int j = 0; j < LC_PER; ++j) {
                    const uint32_t q = u[j] & LC_TGT;
                    const bool move = q != (v[j] & LC_TGT) && (v[j] >> 16) < LC_T;
                    if (move) {
                        v[j] = q | (((v[j] >> 16) + (u[j] >> 16)) << 16);
                        __hip_atomic_store(&PD[j * LC_TPB + threadIdx.x], v[j], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                        open = true;
                    }
                }
                left = __any(open) ? left - 1u : 0u;
            }
            __syncthreads();  // DIR, and the starts' entries, before the next use
        } else {
            for (int round = 0; round < LC_ROUNDS; ++round) {
                int changed = 0;
                // target, count and weight live in two words: read all, then write all
                uint32_t nv[LC_PER];
                int64_t nw[LC_PER];
#pragma unroll
                for (int j = 0; j < LC_PER; ++j) {
                    const uint32_t i = j * LC_TPB + threadIdx.x;
                    const uint32_t p = v[j] & LC_TGT;
                    nv[j] = v[j];
                    nw[j] = ws[j];
                    if (i < len && p != i) {
                        const uint32_t u = PD[p];
                        const uint32_t q = u & LC_TGT;
                        if (q != p) {
                            nv[j] = q | (((v[j] >> 16) + (u >> 16)) << 16);
                            nw[j] = ws[j] + WS[p];
                        }
                    }
                }
                __syncthreads();
#pragma unroll
                for (int j = 0; j < LC_PER; ++j) {
                    const uint32_t i = j * LC_TPB + threadIdx.x;
                    if (nv[j] != v[j]) {
                        v[j] = nv[j];
                        ws[j] = nw[j];
                        PD[i] = v[j];
                        WS[i] = ws[j];
                        changed = 1;
                    }
                }
                if (!__syncthreads_or(changed)) break;
            }
        }
        if (threadIdx.x < (len + 31) / 32) dir[(b >> 5) + threadIdx.x] = DIR[threadIdx.x];
#pragma unroll
        for (int j = 0; j < LC_PER; ++j) {
            const uint32_t i = j * LC_TPB + threadIdx.x;
            if (i >= len) continue;
            const uint32_t x = b + i;
            const uint32_t p = v[j] & LC_TGT;
            const uint32_t dist = v[j] >> 16;
            // a start has no predecessor in the tile (its start bit); on a cycle inside
            // the tile the jumps never reach one, even where a target comes back to itself
            if (!((DIR[p >> 5].x >> (p & 31)) & 1u)) {
                pos[x] = NONE;
                atomicOr(&ctrl->err, 8u);
                continue;
            }
            const uint32_t lid = lc_below(DIR[p >> 5], p);
            pos[x] = (lid << 16) | dist;
            if constexpr (W) wd[x] = ws[j];
            const uint32_t s = sv[j];
            const uint32_t d = s - b;
            if (d < len && d != i) continue;  // the chain continues inside the tile
            Val val;
            uint32_t nxt;
            if (s == x || s >= n) {           // the chain ends at the terminal x
                val.c = dist;
                if constexpr (W) val.s = ws[j];
                nxt = TERM | x;
            } else {                          // the chain leaves the tile for the start s
                val.c = dist + 1;
                if constexpr (W) val.s = ws[j] + wv[j];
                nxt = s;
            }
            stage[(size_t)tile * LC_T + lid] = L::rec(nxt, val);
        }
        __syncthreads();  // LDS is reused by the next tile
    }
}

// Exclusive scan of the per-tile start counts (one workgroup); publishes the
// contracted list's size and the sizes of the ruling-set levels above it.

// forced: the contracted path runs alone and this kernel sets its mode. small: a
// list of at most that many elements (0: none) is not chased, its levels have
// the sizes of kss.
__global__ __launch_bounds__(1024) void k_lc_scan(uint32_t* __restrict__ cnt, uint32_t ntiles, Ctrl* ctrl,
                                                  uint32_t levels, LevelShifts ks, uint32_t cap, uint32_t forced,
                                                  uint32_t small, uint32_t slevels, LevelShifts kss, Gate gate) {
    if (gate.off()) return;
    __shared__ uint32_t sh[1024 / 64];
    const uint32_t total = wg_exscan_inplace(cnt, ntiles, sh);
    if (threadIdx.x == 0) {
        ctrl->hc_done = 0;  // the head-count kernels' workgroup counter
        if (forced) ctrl->mode = MODE_LOCAL;
        if (total > cap) {  // the guess was wrong: more than the contracted levels hold
            ctrl->mode = MODE_PLAIN;  // every later kernel of this path returns; the plain path runs
            return;
        }
        cnt[ntiles] = total;
        uint32_t m = total;
        ctrl->dm[0] = m;
        for (uint32_t l = 0; l < levels; ++l) {
            m = (m + (1u << ks.lg[l]) - 1u) >> ks.lg[l];
            ctrl->dm[l + 1] = m;
        }
        ctrl->single = 0;
        if (total <= small) {
            ctrl->mode = MODE_LOCAL_SMALL;
            m = total;
            ctrl->dms[0] = m;
            for (uint32_t l = 0; l < slevels; ++l) {
                m = (m + (1u << kss.lg[l]) - 1u) >> kss.lg[l];
                ctrl->dms[l + 1] = m;
            }
        }
    }
}

// Zero the first dm bytes of p (the contracted level's predecessor marks).
__global__ __launch_bounds__(TPB) void k_zero_dyn(uint32_t* __restrict__ p, const uint32_t* dm, Gate gate) {
    if (gate.off()) return;
    const uint32_t words = (dm[0] + 3) / 4;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride) p[i] = 0;
}

// One wave per tile: move the tile's staged records to their compact
// positions; an exit successor s (a chain start of another tile) becomes its
// compact id, whose record is marked as having a predecessor.
template <bool W>
__global__ __launch_bounds__(TPB) void k_lc_compact(const typename Lay<W>::Rec* __restrict__ stage,
                                                    const uint32_t* __restrict__ cnt, const uint2* __restrict__ dir,
                                                    uint32_t ntiles, uint32_t n, typename Lay<W>::Rec* __restrict__ lrec,
                                                    uint8_t* __restrict__ hp, Gate gate) {
    if (gate.off()) return;
    const uint32_t lane = lane_id();
    const uint32_t nwaves = (gridDim.x * blockDim.x) >> 6;
    for (uint32_t t = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; t < ntiles; t += nwaves) {
        const uint32_t base = cnt[t];
        const uint32_t c = cnt[t + 1] - base;
        for (uint32_t k = lane; k < c; k += 64) {
            typename Lay<W>::Rec r = stage[(size_t)t * LC_T + k];
            if (!(r.nxt & TERM)) {
                const uint32_t s = r.nxt < n ? r.nxt : n - 1;
                r.nxt = cnt[s >> LOCAL_SHIFT] + lc_below(dir[s >> 5], s);
                if (hp) hp[r.nxt] = 1;
            }
            lrec[base + k] = r;
        }
    }
}

// Pass 3: every element from its chain start's result (lane-strided wave
// tiles like the level expansion; the result gathers stay inside the tile's
// compact range).
template <bool W, class Out>
__global__ __launch_bounds__(TPB) void k_lc_expand(const uint32_t* __restrict__ pos, const int64_t* __restrict__ wd,
                                                   const uint32_t* __restrict__ cnt,
                                                   const typename Lay<W>::Res* __restrict__ res, uint32_t n,
                                                   Ctrl* ctrl, Out out, Gate gate) {
    if (gate.off()) return;
    using L = Lay<W>;
    const uint32_t mc = ctrl->dm[0];
    const uint32_t lane = lane_id();
    const uint32_t wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint32_t nwaves = (gridDim.x * blockDim.x) >> 6;
    const uint32_t ntile = (n + 64 * EXPAND_CH - 1) / (64 * EXPAND_CH);
    static_assert((64 * EXPAND_CH) <= LC_T && LC_T % (64 * EXPAND_CH) == 0, "a wave tile lies in one chain tile");
    bool bad = false;
    for (uint32_t tile = wave; tile < ntile; tile += nwaves) {
        const uint32_t base = tile * 64 * EXPAND_CH;
        // one chain tile per wave tile: its first compact id is one load
        const uint32_t cb = cnt[base >> LOCAL_SHIFT];
        if (base + lane >= n) continue;
        auto cur = out.begin(base + lane);
        uint32_t pv[EXPAND_CH];
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const uint32_t i = base + j * 64 + lane;
            pv[j] = (i < n) ? pos[i] : NONE;
        }
        // every gather issued before any store (see k_expand)
        uint32_t cv[EXPAND_CH];
        typename L::Res rv[EXPAND_CH];
        int64_t wv[EXPAND_CH];
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const uint32_t i = base + j * 64 + lane;
            cv[j] = (pv[j] == NONE) ? NONE : cb + (pv[j] >> 16);
            if (cv[j] < mc) rv[j] = res[cv[j]];
            wv[j] = 0;
            if constexpr (W) if (i < n) wv[j] = wd[i];
        }
        // all values first, then the stores: vector-memory counters also count
        // stores, so a store between two dependent gathers would make every
        // later gather wait for it
        typename L::Val ov[EXPAND_CH];
        uint32_t orr[EXPAND_CH];
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const bool ok = cv[j] < mc;
            bad |= !ok && (base + j * 64 + lane < n);
            typename L::Val v = L::val(rv[j]);
            v.c -= pv[j] & 0xffffu;
            if constexpr (W) v.s -= wv[j];
            ov[j] = ok ? v : L::junk();
            orr[j] = ok ? L::root(rv[j]) : NONE;
        }
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const uint32_t i = base + j * 64 + lane;
            if (i < n) out.store(cur, i, ov[j], orr[j]);
        }
    }
    if (__ballot(bad) && lane == 0) atomicOr(&ctrl->err, 4u);
}

// ------------------------------------------------------- ruler spawning --
// Section 2.2 on one GPU, in two chases with no atomics on the elements.
// Spawning exists to cut the long stretches between sampled rulers, whose
// walks decide how long a chase runs. Phase 1 is the ordinary chase from the
// sampled rulers and the heads, except that a walk stops after `cap` steps:
// it marks the next element, which no walk has reached, as its cap target
// (slot = SPF | walk, offset) and ends there. Between the phases every
// element whose slot is still free (reached by no walk) is known, and new
// rulers are spawned among exactly those: each cap target, and each free
// element that a hash picks at rate 1/k2. Phase 2 walks from the spawned
// rulers; its lanes tell a spawned ruler from a free element by one plain
// load of the slot, so every step is one round trip of plain loads. With
// phase 1 capped at c k steps only a fraction of about exp(-c) of the
// elements is left for phase 2, where walks are k2 long on average.
//
// Walk ids: [0, S0) sampled rulers (block b's ruler is walk b), [S0, T0)
// heads that are not sampled (start parked in the record), [T0, T0 + R2)
// spawned rulers (start parked in the record), numbered in tile order.
// Slots: all ones = free; (walk, offset) = reached; SPF | walk = a phase-1
// cap target (before the spawn pass) or a spawned ruler (after it).
constexpr uint32_t SPF = TERM;        // slot flag: cap target / spawned ruler
constexpr uint32_t LOG2_SPAWN_K2 = 31 - __builtin_clz((unsigned)LR_SPAWN_K2);  // second chase: mean walk 2^this
constexpr int SP_TPB = 256;

// Every slot free (all ones), and the control words of the path reset.
__global__ __launch_bounds__(TPB) void k_sp_prep(uint32_t* __restrict__ slotw, uint64_t words, Ctrl* ctrl,
                                                 Gate gate) {
    if (gate.off()) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctrl->spn = 0;
        ctrl->single = 0;
        ctrl->multi = 0;
        ctrl->mode = MODE_SPAWN;
    }
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t n4 = words / 4;
    const uint4 v = make_uint4(NONE, NONE, NONE, NONE);
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride)
        reinterpret_cast<uint4*>(slotw)[i] = v;
    for (uint64_t i = n4 * 4 + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride)
        slotw[i] = NONE;
}

// Phase 1: the chase of the sampled rulers' and heads' walks (one walk per
// lane, wavefront walk ranges as in k_chase), capped at `cap` steps. Unlike
// the levels' chase every walk is an element of the next list, so every walk
// that ends on a ruler marks that ruler as having a predecessor.
template <bool W, int WT>
__global__ __launch_bounds__(SP_TPB) void k_sp_chase1(SrcIn<W, WT> src, Sampler smp, Ctrl* ctrl,
                                                      typename Lay<W>::Slot* __restrict__ slot,
                                                      typename Lay<W>::Rec* __restrict__ lrec,
                                                      uint8_t* __restrict__ hp_c, uint32_t cap, Gate gate) {
    if (gate.off()) return;
    using L = Lay<W>;
    using Val = typename L::Val;
    const uint32_t m = smp.m;
    const uint32_t S0 = (m + (1u << smp.log2k) - 1u) >> smp.log2k;
    const uint32_t T0 = S0 + ctrl->lv[SPL].H;
    const uint32_t gwave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint32_t nwave = (gridDim.x * blockDim.x) >> 6;
    const uint32_t per = T0 / nwave + 1;
    uint32_t cursor = (uint32_t)min<uint64_t>((uint64_t)gwave * per, T0);
    const uint32_t whi = (uint32_t)min<uint64_t>((uint64_t)(gwave + 1) * per, T0);
    uint32_t w = NONE, x = 0, steps = 0;
    Val off = L::zero();
    for (;;) {
        const uint64_t idle = __ballot(w == NONE);
        if (idle == ~0ull && cursor >= whi) break;
        if (idle && cursor < whi) {
            const uint32_t my = cursor + mbcnt(idle);
            cursor = min(cursor + (uint32_t)__popcll(idle), whi);
            if (w == NONE && my < whi) {
                const uint32_t s0 = (my < S0) ? smp.start(my) : lrec[my].nxt;
                if (s0 < m) {
                    w = my;
                    x = s0;
                    off = L::zero();
                    steps = 0;
                } else {  // corrupt parked start (cannot happen for valid input)
                    lrec[my] = L::rec(TERM | IDX, L::zero());
                    atomicOr(&ctrl->err, 8u);
                }
            }
        }
        if (w == NONE) continue;
        uint32_t nxt;
        Val v;
        src.load(x, nxt, v);
        slot[x] = L::slot(w, off);
        if (nxt & TERM) {                           // x is a terminal: the walk ends on it
            lrec[w] = L::rec(nxt, L::add(off, v));
            w = NONE;
            continue;
        }
        off = L::add(off, v);
        if (smp.sampled(nxt)) {                     // reached the next sampled ruler
            const uint32_t c = nxt >> smp.log2k;
            lrec[w] = L::rec(c, off);
            hp_c[c] = 1;
            if (c == w) atomicOr(&ctrl->err, 8u);   // back at its own start: a cycle
            w = NONE;
        } else if (++steps >= cap) {                // capped: nxt becomes a spawned ruler
            slot[nxt] = L::slot(SPF | w, off);
            w = NONE;
        } else {
            x = nxt;
        }
    }
}

// Spawned rulers: per tile of TILE ids, lane j looks at ids tile*TILE + i*TPB
// + j (i < TILE / TPB), coalesced. A ruler is a cap target or a free element
// picked by the hash.
constexpr int SP_PER = TILE / TPB;

template <bool W>
__device__ __forceinline__ bool sp_ruler(const typename Lay<W>::Slot* slot, uint32_t z, uint32_t seed,
                                         uint32_t k2mask) {
    const uint32_t w = slot[z].w;
    if (w == NONE) return (hash32(seed, z) & k2mask) == 0u;
    return (w & SPF) != 0u;
}

template <bool W>
__global__ __launch_bounds__(TPB) void k_sp_count(const typename Lay<W>::Slot* __restrict__ slot, uint32_t n,
                                                  uint32_t seed, uint32_t k2mask, uint32_t* __restrict__ tilecnt,
                                                  uint32_t ntiles, Gate gate) {
    if (gate.off()) return;
    __shared__ uint32_t sh[TPB / 64];
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        uint32_t c = 0;
#pragma unroll
        for (int i = 0; i < SP_PER; ++i) {
            const uint32_t z = t * TILE + i * TPB + threadIdx.x;
            if (z < n) c += sp_ruler<W>(slot, z, seed, k2mask);
        }
        const uint32_t tot = block_sum(c, sh);
        if (threadIdx.x == 0) tilecnt[t] = tot;
        __syncthreads();
    }
}

// One workgroup: scan of the spawned-ruler counts; publishes their number.
__global__ __launch_bounds__(1024) void k_sp_scan(uint32_t* __restrict__ tilecnt, uint32_t ntiles, Ctrl* ctrl,
                                                  Gate gate) {
    if (gate.off()) return;
    __shared__ uint32_t sh[1024 / 64];
    const uint32_t total = wg_exscan_inplace(tilecnt, ntiles, sh);
    if (threadIdx.x == 0) ctrl->spn = total;
}

// Numbers the spawned rulers, parks each one's start in its record, flags its
// slot, and ends the capped walk whose target it is on it.
template <bool W>
__global__ __launch_bounds__(TPB) void k_sp_write(typename Lay<W>::Slot* __restrict__ slot, uint32_t n,
                                                  uint32_t seed, uint32_t k2mask,
                                                  const uint32_t* __restrict__ tileoff, uint32_t ntiles,
                                                  const Ctrl* ctrl, uint32_t S0, typename Lay<W>::Rec* __restrict__ lrec,
                                                  uint8_t* __restrict__ hp_c, Gate gate) {
    if (gate.off()) return;
    using L = Lay<W>;
    __shared__ uint32_t sh[TPB / 64];
    const uint32_t T0 = S0 + ctrl->lv[SPL].H;
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        uint32_t bits = 0;
#pragma unroll
        for (int i = 0; i < SP_PER; ++i) {
            const uint32_t z = t * TILE + i * TPB + threadIdx.x;
            if (z < n && sp_ruler<W>(slot, z, seed, k2mask)) bits |= 1u << i;
        }
        uint32_t total;
        uint32_t pos = T0 + tileoff[t] + block_exscan((uint32_t)__popc(bits), sh, &total);
        while (bits) {
            const int i = __ffs(bits) - 1;
            bits &= bits - 1;
            const uint32_t z = t * TILE + i * TPB + threadIdx.x;
            const typename L::Slot sv = slot[z];
            if (sv.w != NONE) {  // a cap target: its walk ends on this ruler
                lrec[sv.w & IDX] = L::rec(pos, L::val(sv));
                hp_c[pos] = 1;
            }
            slot[z] = L::slot(SPF | pos, L::zero());
            *reinterpret_cast<uint32_t*>(&lrec[pos]) = z;  // parked start
            ++pos;
        }
        __syncthreads();
    }
}

// Phase 2: the walks of the spawned rulers. A lane holds the record of x and
// the pending successor; each step loads the successor's slot and record
// together and then decides: a spawned ruler ends the walk, a free element is
// taken.
template <bool W, int WT>
__global__ __launch_bounds__(SP_TPB) void k_sp_chase2(SrcIn<W, WT> src, Sampler smp, Ctrl* ctrl,
                                                      typename Lay<W>::Slot* __restrict__ slot,
                                                      typename Lay<W>::Rec* __restrict__ lrec,
                                                      uint8_t* __restrict__ hp_c, Gate gate) {
    if (gate.off()) return;
    using L = Lay<W>;
    using Val = typename L::Val;
    const uint32_t m = smp.m;
    const uint32_t S0 = (m + (1u << smp.log2k) - 1u) >> smp.log2k;
    const uint32_t T0 = S0 + ctrl->lv[SPL].H;
    const uint32_t R2 = ctrl->spn;
    const uint32_t gwave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint32_t nwave = (gridDim.x * blockDim.x) >> 6;
    const uint32_t per = R2 / nwave + 1;
    uint32_t cursor = T0 + (uint32_t)min<uint64_t>((uint64_t)gwave * per, R2);
    const uint32_t whi = T0 + (uint32_t)min<uint64_t>((uint64_t)(gwave + 1) * per, R2);
    uint32_t w = NONE, x = 0, nxt = 0, steps = 0;
    Val v = L::zero(), off = L::zero();
    bool fresh = false;  // walk just started: the record of x is not loaded yet
    const uint32_t cap = walk_cap(m, LOG2_SPAWN_K2);
    for (;;) {
        const uint64_t idle = __ballot(w == NONE);
        if (idle == ~0ull && cursor >= whi) break;
        if (idle && cursor < whi) {
            const uint32_t my = cursor + mbcnt(idle);
            cursor = min(cursor + (uint32_t)__popcll(idle), whi);
            if (w == NONE && my < whi) {
                const uint32_t s0 = lrec[my].nxt;
                if (s0 < m) {
                    w = my;
                    x = s0;
                    off = L::zero();
                    fresh = true;
                    steps = 0;
                } else {
                    lrec[my] = L::rec(TERM | IDX, L::zero());
                    atomicOr(&ctrl->err, 8u);
                }
            }
        }
        if (w == NONE) continue;
        bool adv = false;
        Val o2 = off;
        if (!fresh) {
            o2 = L::add(off, v);
            if (nxt & TERM) {
                lrec[w] = L::rec(nxt, o2);
                w = NONE;
            } else if (smp.sampled(nxt)) {
                const uint32_t c = nxt >> smp.log2k;
                lrec[w] = L::rec(c, o2);
                hp_c[c] = 1;
                w = NONE;
            } else {
                adv = true;
            }
        }
        if (w == NONE) continue;
        const uint32_t q = fresh ? x : nxt;
        uint32_t sw = NONE, ln;
        Val lv;
        if (adv) sw = slot[q].w;
        src.load(q, ln, lv);
        if (fresh) {
            nxt = ln;
            v = lv;
            fresh = false;
        } else if (sw == NONE) {                    // a free element: the walk takes it
            slot[q] = L::slot(w, o2);
            x = q;
            off = o2;
            nxt = ln;
            v = lv;
            if (++steps >= cap) {                   // the bounded fallback takes over
                lrec[w] = L::rec(TERM | IDX, o2);
                ctrl->mode = MODE_FALLBACK;
                w = NONE;
            }
        } else if (sw & SPF) {                      // a spawned ruler: the walk ends on it
            const uint32_t c = sw & IDX;
            lrec[w] = L::rec(c, o2);
            hp_c[c] = 1;
            if (c == w) atomicOr(&ctrl->err, 8u);
            w = NONE;
        } else {                                    // reached twice: two predecessors
            lrec[w] = L::rec(TERM | IDX, o2);
            atomicOr(&ctrl->err, 2u);
            w = NONE;
        }
    }
}

// The walks' list: its size and the sizes of the levels above.
__global__ void k_sp_publish(Ctrl* ctrl, uint32_t S0, uint32_t cap, uint32_t levels, LevelShifts ks, Gate gate) {
    if (gate.off()) return;
    if (threadIdx.x == 0) {
        uint64_t t = (uint64_t)S0 + ctrl->lv[SPL].H + ctrl->spn;
        uint32_t m = (uint32_t)min<uint64_t>(t, cap);
        ctrl->dm[0] = m;
        for (uint32_t l = 0; l < levels; ++l) {
            m = (m + (1u << ks.lg[l]) - 1u) >> ks.lg[l];
            ctrl->dm[l + 1] = m;
        }
        ctrl->single = 0;
    }
}

// rank(x) = result(walk(x)) - offset(x), as k_expand, with the walk id taken
// from the slot without its spawned-ruler flag.
template <bool W, class Out>
__global__ __launch_bounds__(TPB) void k_sp_expand(const typename Lay<W>::Slot* __restrict__ slot, uint32_t n,
                                                   const typename Lay<W>::Res* __restrict__ res, Ctrl* ctrl,
                                                   Out out, Gate gate) {
    if (gate.off()) return;
    using L = Lay<W>;
    const uint32_t mc = ctrl->dm[0];
    const uint32_t lane = lane_id();
    const uint32_t wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint32_t nwaves = (gridDim.x * blockDim.x) >> 6;
    const uint32_t ntile = (n + 64 * EXPAND_CH - 1) / (64 * EXPAND_CH);
    bool bad = false;
    for (uint32_t tile = wave; tile < ntile; tile += nwaves) {
        const uint32_t base = tile * 64 * EXPAND_CH;
        if (base + lane >= n) continue;
        auto cur = out.begin(base + lane);
        typename L::Slot sv[EXPAND_CH];
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const uint32_t i = base + j * 64 + lane;
            if (i < n) sv[j] = slot[i];
        }
        typename L::Res rv[EXPAND_CH];
        uint32_t wv[EXPAND_CH];
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const uint32_t i = base + j * 64 + lane;
            wv[j] = (i < n) ? (sv[j].w & IDX) : NONE;
            if (wv[j] < mc) rv[j] = res[wv[j]];
        }
        typename L::Val ov[EXPAND_CH];
        uint32_t orr[EXPAND_CH];
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const bool ok = wv[j] < mc;
            bad |= !ok && (base + j * 64 + lane < n);
            ov[j] = ok ? L::sub(L::val(rv[j]), L::val(sv[j])) : L::junk();
            orr[j] = ok ? L::root(rv[j]) : NONE;
        }
#pragma unroll
        for (int j = 0; j < EXPAND_CH; ++j) {
            const uint32_t i = base + j * 64 + lane;
            if (i < n) out.store(cur, i, ov[j], orr[j]);
        }
    }
    if (__ballot(bad) && lane == 0) atomicOr(&ctrl->err, 4u);
}

// ============================================================== host side ==

// Device properties, looked up once (thread-safe initialisation of local
// statics) on the device current at the first call.
int device_cus() {
    static const int cus = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            return v;
        return 256;
    }();
    return cus;
}

size_t device_max_lds() {
    static const size_t lds = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && v > 0)
            return (size_t)v;
        return (size_t)65536;
    }();
    return lds;
}

static inline uint32_t grid_for(uint64_t work, uint32_t per_block, uint32_t cap_per_cu = 8) {
    uint64_t g = (work + per_block - 1) / per_block;
    const uint64_t cap = (uint64_t)device_cus() * cap_per_cu;
    if (g > cap) g = cap;
    if (g == 0) g = 1;
    return (uint32_t)g;
}

template <class K>
static uint32_t persistent_grid(K kernel, int tpb) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, tpb, 0) != hipSuccess || nb <= 0) nb = 4;
    return (uint32_t)nb * (uint32_t)device_cus();
}

static hipError_t fill(void* p, uint64_t bytes, uint32_t val, hipStream_t st, const Ctrl* skip_if_single = nullptr,
                       Gate gate = Gate{}) {
    const uint64_t words = (bytes + 3) / 4;
    if (!words) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3(grid_for(words, TPB * 4)), dim3(TPB), 0, st, (uint32_t*)p, words, val,
                       skip_if_single, gate);
    return hipGetLastError();
}

static inline void rec_ev(const RunArgs& a, int i) {
    if (a.ev) (void)hipEventRecord(a.ev[i], a.stream);
}

template <int COLS, bool W, class Src, class Out>
static hipError_t launch_base_cols(Src src, Out out, uint32_t m, uint32_t climit, Ctrl* ctrl, hipStream_t st,
                                   const uint32_t* dm, Gate gate) {
    constexpr size_t lds = (size_t)COLS * BASE_TPB * (W ? 16 : 8);
    void (*kern)(Src, Out, uint32_t, uint32_t, Ctrl*, const uint32_t*, Gate);
    if constexpr (W) kern = k_base_weighted<COLS, Src, Out>;
    else kern = k_base_unweighted<COLS, Src, Out>;
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(1), dim3(BASE_TPB), lds, st, src, out, m, climit, ctrl, dm, gate);
    return hipGetLastError();
}

// climit: elements of the input (no list has as many links).
template <bool W, class Src, class Out>
static hipError_t launch_base(Src src, Out out, uint32_t m, uint32_t climit, Ctrl* ctrl, hipStream_t st,
                              const uint32_t* dm, Gate gate) {
    if constexpr (!W) {
        if (m <= BASE_TPB) return launch_base_cols<1, false>(src, out, m, climit, ctrl, st, dm, gate);
        if (m <= 2 * BASE_TPB) return launch_base_cols<2, false>(src, out, m, climit, ctrl, st, dm, gate);
        if (m <= 4 * BASE_TPB) return launch_base_cols<4, false>(src, out, m, climit, ctrl, st, dm, gate);
        if (m <= 8 * BASE_TPB) return launch_base_cols<8, false>(src, out, m, climit, ctrl, st, dm, gate);
        return launch_base_cols<16, false>(src, out, m, climit, ctrl, st, dm, gate);
    } else {
        if (m <= BASE_TPB) return launch_base_cols<1, true>(src, out, m, climit, ctrl, st, dm, gate);
        if (m <= 2 * BASE_TPB) return launch_base_cols<2, true>(src, out, m, climit, ctrl, st, dm, gate);
        if (m <= 4 * BASE_TPB) return launch_base_cols<4, true>(src, out, m, climit, ctrl, st, dm, gate);
        if (m <= 8 * BASE_TPB) return launch_base_cols<8, true>(src, out, m, climit, ctrl, st, dm, gate);
        const size_t lds = base_lds_bytes(m, true);
        auto kern = k_base_weighted_large<Src, Out>;
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(1), dim3(BASE_TPB), lds, st, src, out, m, ctrl, dm, gate);
        return hipGetLastError();
    }
}

// The input by independent walks: levels 0 .. top - 1 walk, level top is
// doubled, then downward.
//
// Elements per lane of the downward pass: one is faster wherever it was timed
// (one / four, us a call: 262,144 elements 39.5 / 41.9, 300,007 43.5 / 46.9, 2^20
// 81.6 / 83.5; int64 sums of 262,144 68.7 / 73.6, of 500,003 103 / 108), but with it
// no more than 2^19 of a list's elements have a resident lane, and an order
// against the sampling is halved only among those. With four all 2^21 have one
// (60 registers, 8 waves a SIMD), weighted levels' 3 * 2^19 (74 registers, 6 waves; held to
// 64 registers the kernel spills).
constexpr int IW_PER = 4;
constexpr uint32_t IW_PER_MIN = 1u << 18;  // up to here one element a lane

template <bool W, class Src, class Out>
static hipError_t run_iw(const Plan& p, Src src, Out out, uint32_t n, Ctrl* ctrl, char* ws, hipStream_t st,
                         const uint32_t* dm, Gate gate) {
    uint64_t* nodes = reinterpret_cast<uint64_t*>(ws + p.off_nodes);
    const uint32_t T = p.top;
    uint32_t base[LR_MAX_LEVELS + 2] = {};
    for (uint32_t l = 0; l <= T; ++l) base[l + 1] = base[l] + (uint32_t)p.m[l];
    const uint32_t total = base[T + 1];
    auto smp = [&](uint32_t l) { return Sampler{(uint32_t)p.m[l], p.log2k[l], p.lseed[l]}; };
    auto dml = [&](uint32_t l) { return dm ? dm + l : nullptr; };
    auto grid = [](uint64_t m, uint32_t per) { return dim3((uint32_t)((m + per - 1) / per)); };
    const dim3 b(TPB), bd(IW_DBL_TPB);
    hipError_t e;
    if (T == 0) {
        hipLaunchKernelGGL((k_iw_first<W, false, Src>), grid(n, TPB), b, 0, st, src, Sampler{}, nodes, 0u, n,
                           IW_CAP_ALONE, ctrl, dm, gate);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL((k_iw_double<W, true, Out>), grid(n, IW_DBL_TPB), bd, 0, st, nodes, 0u, total, n, n, NONE,
                           ctrl, out, dm, gate);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_iw_first<W, true, Src>), grid(n, TPB), b, 0, st, src, smp(0), nodes, base[1], n,
                       (uint32_t)LR_IW_CAP, ctrl, dm, gate);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (uint32_t l = 1; l < T; ++l) {
        hipLaunchKernelGGL((k_iw_walk<W>), grid(p.m[l], TPB), b, 0, st, nodes, smp(l), base[l], base[l + 1], total,
                           (uint32_t)p.m[l], (uint32_t)LR_IW_CAP, dml(l), gate);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const OutLvl<W> none{};
    hipLaunchKernelGGL((k_iw_double<W, false, OutLvl<W>>), grid(p.m[T], IW_DBL_TPB), bd, 0, st, nodes, base[T], total,
                       (uint32_t)p.m[T], n, IW_TOP_CAP, ctrl, none, dml(T), gate);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (uint32_t l = T - 1; l > 0; --l) {
        hipLaunchKernelGGL((k_iw_down<W, false, 1, OutLvl<W>>), grid(p.m[l], TPB), b, 0, st, nodes, smp(l), base[l],
                           base[l + 1], total, (uint32_t)p.m[l], n, 0u, 0u, ctrl, none, dml(l), gate);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (n <= IW_PER_MIN)
        hipLaunchKernelGGL((k_iw_down<W, true, 1, Out>), grid(n, TPB), b, 0, st, nodes, smp(0), 0u, base[1], total, n, n,
                           1u, 1u, ctrl, out, dm, gate);
    else
        hipLaunchKernelGGL((k_iw_down<W, true, IW_PER, Out>), grid(n, TPB * IW_PER), b, 0, st, nodes, smp(0), 0u,
                           base[1], total, n, n, 1u, 1u, ctrl, out, dm, gate);
    return hipGetLastError();
}

// Levels' records, ranked in place: one list per path that the call enqueues
// (see IwArgs; unused ones have no plan). dm: the list's sizes on the device,
// level by level, or null.
template <bool W>
struct IwSet {
    const Plan* p = nullptr;
    typename Lay<W>::Rec* rec = nullptr;
    const uint32_t* dm = nullptr;
};

template <bool W>
static hipError_t run_iw_levels(const IwSet<W> (&set)[3], const uint32_t* mode, uint32_t climit, Ctrl* ctrl, char* ws,
                                hipStream_t st) {
    uint32_t depth = 0;  // most levels of walks
    for (const auto& q : set)
        if (q.p) depth = std::max(depth, q.p->top - q.p->run);
    // the launch on level run + j of every list that has one; top: its last
    auto args = [&](uint32_t j, bool top, bool rec, uint64_t* most) {
        IwArgs<W> s{};
        s.mode = mode;
        *most = 0;
        for (int k = 0; k < 3; ++k) {
            const Plan* p = set[k].p;
            if (!p) continue;
            const uint32_t d = p->top - p->run, i = top ? d : j;
            if (!top && i >= d && !(W && d == 0 && i == 0 && rec)) continue;  // a weighted list's nodes are always made
            IwArg<W>& a = s.a[k];
            uint32_t base = 0;
            for (uint32_t t = 0; t < i; ++t) base += (uint32_t)p->m[p->run + t];
            a.nodes = (!W && d == 0) ? reinterpret_cast<uint64_t*>(set[k].rec)
                                     : reinterpret_cast<uint64_t*>(ws + p->off_nodes);
            a.rec = (rec || d == 0) ? set[k].rec : nullptr;
            a.dm = set[k].dm ? set[k].dm + i : nullptr;
            a.m = (uint32_t)p->m[p->run + i];
            a.base = base;
            a.basen = base + a.m;
            a.total = base + a.m;
            for (uint32_t t = i + 1; t <= d; ++t) a.total += (uint32_t)p->m[p->run + t];
            a.log2k = i < d ? p->log2k[p->run + i] : 0u;
            a.seed = i < d ? p->lseed[p->run + i] : 0u;
            a.climit = climit;
            *most = std::max<uint64_t>(*most, a.m);
        }
        return s;
    };
    auto grid = [](uint64_t m, uint32_t per) { return dim3((uint32_t)((m + per - 1) / per)); };
    const dim3 b(TPB);
    uint64_t most;
    hipError_t e;
    IwArgs<W> s = args(0, false, true, &most);
    if (most) {
        hipLaunchKernelGGL(k_iwl_first<W>, grid(most, TPB), b, 0, st, s);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    for (uint32_t j = 1; j < depth; ++j) {
        s = args(j, false, false, &most);
        hipLaunchKernelGGL(k_iwl_walk<W>, grid(most, TPB), b, 0, st, s);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    s = args(0, true, false, &most);
    hipLaunchKernelGGL(k_iwl_double<W>, grid(most, IW_DBL_TPB), dim3(IW_DBL_TPB), 0, st, s, ctrl);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (uint32_t j = depth; j-- > 0;) {
        s = args(j, false, j == 0, &most);
        if constexpr (W) {
            for (int k = 0; k < 3; ++k)  // lists that the doubling took alone have nothing left
                if (set[k].p && set[k].p->top == set[k].p->run) s.a[k].m = 0;
        }
        if (most <= IW_PER_MIN) hipLaunchKernelGGL((k_iwl_down<W, 1>), grid(most, TPB), b, 0, st, s, ctrl);
        else hipLaunchKernelGGL((k_iwl_down<W, IW_PER>), grid(most, TPB * IW_PER), b, 0, st, s, ctrl);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool W>
static LogArrays<W> log_arrays(char* ws, const Plan& p) {
    LogArrays<W> a{};
    a.x = reinterpret_cast<uint32_t*>(ws + p.off_log[0]);
    a.w = reinterpret_cast<uint32_t*>(ws + p.off_log[1]);
    a.c = reinterpret_cast<uint32_t*>(ws + p.off_log[2]);
    a.s = W ? reinterpret_cast<int64_t*>(ws + p.off_log[3]) : nullptr;
    a.r = reinterpret_cast<uint64_t*>(ws + p.off_log[0]);  // packed: over the first two arrays
    if (p.pack) {
        a.cont = reinterpret_cast<uint2*>(ws + p.off_conts);
        a.ccap = p.ccap;
        a.bocap = p.bocap;
    }
    return a;
}

template <bool W, int LOG, int NW, class Src>
static hipError_t launch_chase(const Plan& p, int l, Src src, Sampler smp, Ctrl* ctrl, char* ws, hipStream_t st,
                               const uint32_t* dm = nullptr, Gate gate = Gate{}) {
    using L = Lay<W>;
    auto kern = k_chase<W, Src, LOG, NW>;
    static const uint32_t grid = [kern] {  // one per template instance, found once
        const uint32_t g = persistent_grid(kern, CHASE_TPB);
        return LOG != 0 ? std::min<uint32_t>(g, LOG_MAX_WAVES / (CHASE_TPB / 64)) : g;  // bounds the log slack
    }();
    const uint32_t S = (uint32_t)p.m[l + 1];
    auto* slot = reinterpret_cast<typename L::Slot*>(ws + p.off_slot[l]);
    auto* eb = reinterpret_cast<typename L::Rec*>(ws + p.off_eb[l]);
    uint8_t* hp_next = (l + 1 < (int)p.run) ? reinterpret_cast<uint8_t*>(ws + p.off_slot[l + 1]) : nullptr;
    LogArrays<W> lg = LOG != 0 ? log_arrays<W>(ws, p) : LogArrays<W>{};
    hipLaunchKernelGGL(kern, dim3(grid), dim3(CHASE_TPB), 0, st, src, smp, S, ctrl, l, slot, eb, hp_next,
                       p.refill, lg, p.max_chunks, dm, gate);
    return hipGetLastError();
}

// Level-0 chase into the visit log, in the plan's record format.
template <bool W, int NW, class Src>
static hipError_t launch_chase_log(const Plan& p, Src src, Sampler smp, Ctrl* ctrl, char* ws, hipStream_t st,
                                   const uint32_t* dm, Gate gate) {
    if (p.pack) return launch_chase<W, 2, NW>(p, 0, src, smp, ctrl, ws, st, dm, gate);
    return launch_chase<W, 1, NW>(p, 0, src, smp, ctrl, ws, st, dm, gate);
}

#define LR_TRY(x)                              \
    do {                                       \
        hipError_t e_ = (x);                   \
        if (e_ != hipSuccess) return e_;       \
    } while (0)

template <bool W>
static PlaceArrays<W> place_arrays(char* ws, const size_t* off) {
    PlaceArrays<W> a;
    a.x = reinterpret_cast<uint32_t*>(ws + off[0]);
    a.xr = reinterpret_cast<uint2*>(ws + off[0]);  // the first two arrays are adjacent
    a.t = reinterpret_cast<uint32_t*>(ws + off[2]);
    a.s = W ? reinterpret_cast<int64_t*>(ws + off[3]) : nullptr;
    return a;
}

template <class K>
static hipError_t allow_lds(K kern, size_t bytes) {
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Level-0 propagation in log mode: resolve + coarse grouping, fine grouping,
// placement. The fine-grouped records reuse the visit-log arrays.
template <bool W, bool ROOT, class Out0>
static hipError_t run_place_t(const RunArgs& a, const Plan& p, const typename Lay<W>::Res* res, uint32_t S,
                              Ctrl* ctrl, Out0 out0, const uint32_t* dm) {
    char* ws = a.ws;
    hipStream_t st = a.stream;
    const uint32_t n = (uint32_t)p.m[0];
    uint32_t* fill1 = reinterpret_cast<uint32_t*>(ws + p.off_fill);
    uint32_t* fill2 = fill1 + 2 * (size_t)p.nb1 * FILL_LINE;
    const PlaceArrays<W> P = place_arrays<W>(ws, p.off_p);
    const PlaceArrays<W> Q = place_arrays<W>(ws, p.off_log);
    constexpr uint32_t T = place_tile_records(W, ROOT);
    const dim3 tpb(place_tpb(W, ROOT));
    const size_t cap = (size_t)p.max_chunks * LOG_CHUNK;
    const size_t l1 = place_lds_bytes(W, ROOT, p.nb1);
    if (p.pack) {
        LR_TRY(allow_lds(k_place1<W, ROOT, true>, l1));
        hipLaunchKernelGGL((k_place1<W, ROOT, true>), dim3(grid_for(cap, T)), tpb, l1, st, log_arrays<W>(ws, p),
                           p.max_chunks, res, S, ctrl, n, p.s1, p.nb1, fill1, P, dm, a.gate);
    } else {
        LR_TRY(allow_lds(k_place1<W, ROOT, false>, l1));
        hipLaunchKernelGGL((k_place1<W, ROOT, false>), dim3(grid_for(cap, T)), tpb, l1, st, log_arrays<W>(ws, p),
                           p.max_chunks, res, S, ctrl, n, p.s1, p.nb1, fill1, P, dm, a.gate);
    }
    LR_TRY(hipGetLastError());
    rec_ev(a, EV_PART);
    const size_t l2 = place_lds_bytes(W, ROOT, 1u << (p.s1 - p.s2));
    LR_TRY(allow_lds(k_place2<W, ROOT>, l2));
    hipLaunchKernelGGL((k_place2<W, ROOT>), dim3(grid_for(n, T)), tpb, l2, st, P, ctrl, n, p.s1, p.s2, fill2,
                       Q, dm, fill1, a.gate);
    LR_TRY(hipGetLastError());
    const size_t l3 = ((size_t)1 << p.s2) * (4 + (ROOT ? 4 : 0) + (W ? 8 : 0));
    LR_TRY(allow_lds(k_place3<W, ROOT, Out0>, l3));
    hipLaunchKernelGGL((k_place3<W, ROOT, Out0>), dim3(std::min<uint32_t>(p.nb2, (uint32_t)device_cus() * 8)),
                       tpb, l3, st, Q, ctrl, n, p.s2, p.nb2, fill2, (int)a.validate, out0, dm, a.gate);
    return hipGetLastError();
}

template <bool W, class Out0>
static hipError_t run_place(const RunArgs& a, const Plan& p, const typename Lay<W>::Res* res, uint32_t S, Ctrl* ctrl,
                            Out0 out0, bool root, const uint32_t* dm) {
    if (root) return run_place_t<W, true>(a, p, res, S, ctrl, out0, dm);
    return run_place_t<W, false>(a, p, res, S, ctrl, out0, dm);
}


// Groups of the predecessor marks (k_mark1, k_mark_bits): 512 of them, two for
// each CU, of at most 2^19 ids (64 KB of LDS, so that two fit a CU); from 2^30
// ids on as many as the grouping can take, of up to 2^20.
struct MarkShape {
    uint32_t s1, nb1;
    explicit MarkShape(uint32_t n) {
        uint32_t lg = 0;
        while ((1ull << lg) < n) ++lg;
        s1 = std::min(19u, std::max(PLACE_FINE_SHIFT, lg > 9 ? lg - 9 : 0u));
        s1 = std::max(s1, lg > 11 ? lg - 11 : 0u);
        nb1 = (uint32_t)(((uint64_t)n + (1ull << s1) - 1) >> s1);
    }
    size_t lds() const { return (size_t)1 << (s1 - 3); }
    size_t fill_bytes() const { return 2 * (size_t)nb1 * FILL_LINE * 4; }
    dim3 grid() const { return dim3(std::min<uint32_t>(nb1, (uint32_t)device_cus() * 8)); }
};
static_assert(PLACE_MAX_RANGES >= 1u << 11, "groups of the largest input");

// Below, outside of log mode, one byte store per link (k_detect) and the heads'
// own kernels are as fast. Bytes -> groups, us a call, forests (int64 sums): (1.06 M
// 154 -> 149), 2.1 M 201 -> 194 (2.0 M 217 -> 207), 5 M 361 -> 324 (515 -> 479), 9 M
// 594 -> 523, 33 M 2096 -> 1807.
constexpr uint32_t MARKS_GROUPED_MIN = 1u << 20;

// Groups the targets (a successor array's, or with TGT a list of nin ids) into
// ids, with the groups' counters in fill1.
template <bool TGT>
static hipError_t mark_groups(const MarkShape& ms, const uint32_t* src, uint32_t n, uint32_t nin, void* ids,
                              uint32_t* fill1, Ctrl* ctrl, const uint32_t* dm, Gate g, hipStream_t st) {
    LR_TRY(fill(fill1, ms.fill_bytes(), 0u, st, nullptr, g));
    PlaceArrays<false> Q{};
    Q.x = static_cast<uint32_t*>(ids);
    const size_t l1 = 8 * (size_t)ms.nb1 + 4 * MARK_TILE;  // ids only
    LR_TRY(allow_lds(k_mark1<TGT>, l1));
    hipLaunchKernelGGL(k_mark1<TGT>, dim3(grid_for(TGT ? nin : n, MARK_TILE)), dim3(place_tpb(false, false)), l1, st,
                       src, n, ms.s1, ms.nb1, fill1, Q, ctrl, g, dm, nin);
    return hipGetLastError();
}

// Initial elements of level 0 (more than one list) from grouped predecessor
// marks. In log mode the log arrays and the second grouping array are free for the
// targets and the counters; otherwise both lie in the slot array, which the chase
// fills later.
static hipError_t run_marks(const RunArgs& a, const Plan& p, Ctrl* ctrl, const uint32_t* dm) {
    const uint32_t n = (uint32_t)p.m[0];
    const Gate mg{&ctrl->multi, 1u << 1};  // plain path taken and more than one list
    const MarkShape ms(n);
    const Sampler smp{n, p.log2k[0], p.lseed[0]};
    char* ids = a.ws + (p.log0 ? p.off_log[0] : p.off_slot[0]);
    uint32_t* fill1 = reinterpret_cast<uint32_t*>(
        p.log0 ? a.ws + p.off_p[1] : ids + (4 * (size_t)n + ALIGN - 1) / ALIGN * ALIGN);
    LR_TRY(mark_groups<false>(ms, a.succ, n, n, ids, fill1, ctrl, dm, mg, a.stream));
    LR_TRY(allow_lds(k_mark_bits<false>, ms.lds() + 1024));
    hipLaunchKernelGGL(k_mark_bits<false>, ms.grid(), dim3(MARK_TPB), ms.lds(), a.stream,
                       reinterpret_cast<const uint32_t*>(ids), n, ms.s1, ms.nb1, fill1, smp, a.ws + p.off_eb[0],
                       (uint32_t)p.m[1], (uint32_t)p.rec_bytes, (uint2*)nullptr, (uint32_t*)nullptr, ctrl, mg, dm);
    return hipGetLastError();
}

// Bitmap with running counts of the `count` positions below m in pos (each at
// most once), without a random store per position: they are grouped by range
// with the predecessor-mark passes. Uses the grouping arrays of the workspace
// of a rank call over m elements, free once that call has run; where its plan
// has none (no visit log at this size) position_dir_groups is false.
static bool position_dir_plan(uint32_t m, const lr_opts* opts, Plan* p) {
    return make_plan(m, false, opts, 0, p) == LR_OK && p->log0 && !p->local && !p->spawn;
}

bool position_dir_groups(uint32_t m, const lr_opts* opts) {
    Plan p;
    return position_dir_plan(m, opts, &p);
}

hipError_t position_dir(const uint32_t* pos, uint32_t count, uint32_t m, uint2* dir, uint32_t* cnt, void* ws,
                        const lr_opts* opts, hipStream_t st) {
    Plan p;
    if (!position_dir_plan(m, opts, &p)) return hipErrorInvalidValue;
    char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + ALIGN - 1) / ALIGN * ALIGN);
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(base + p.off_ctrl);
    const MarkShape ms(m);
    char* ids = base + p.off_log[0];
    uint32_t* fill1 = reinterpret_cast<uint32_t*>(base + p.off_p[1]);
    LR_TRY(mark_groups<true>(ms, pos, m, count, ids, fill1, ctrl, nullptr, Gate{}, st));
    LR_TRY(allow_lds(k_mark_bits<true>, ms.lds() + 1024));
    hipLaunchKernelGGL(k_mark_bits<true>, ms.grid(), dim3(MARK_TPB), ms.lds(), st,
                       reinterpret_cast<const uint32_t*>(ids), m, ms.s1, ms.nb1, fill1, Sampler{}, (char*)nullptr, 0u,
                       0u, dir, cnt, ctrl, Gate{}, nullptr);
    return hipGetLastError();
}

// Validation of the input (LR_VALIDATE): range and in-degree counts.
static hipError_t run_validate(const RunArgs& a, const Plan& p, uint32_t n) {
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(a.ws + p.off_ctrl);
    LR_TRY(fill(ctrl, sizeof(Ctrl), 0u, a.stream));
    uint32_t* counts = reinterpret_cast<uint32_t*>(a.ws + p.off_slot[0]);
    LR_TRY(fill(counts, (uint64_t)n * 4, 0u, a.stream));
    return run_validate_input(a.succ, n, counts, &ctrl->err, a.stream);
}

// One streaming pass over the input: terminal count, head sum (the one-list
// shortcut); the plain path's gate (mode 0) when the choice is automatic.
static hipError_t run_headsum(const RunArgs& a, const Plan& p, Gate g) {
    const uint32_t n = (uint32_t)p.m[0];
    hipStream_t st = a.stream;
    const bool vec = ((uintptr_t)a.succ % 16) == 0;
    const uint32_t gs = std::min<uint32_t>(grid_for(n, TPB * 16), HEADSUM_BLOCKS);
    uint32_t* part = reinterpret_cast<uint32_t*>(a.ws + p.off_hsum);
    if (vec) hipLaunchKernelGGL(k_headsum<true>, dim3(gs), dim3(TPB), 0, st, a.succ, n, part, g);
    else hipLaunchKernelGGL(k_headsum<false>, dim3(gs), dim3(TPB), 0, st, a.succ, n, part, g);
    LR_TRY(hipGetLastError());
    const Sampler smp0{n, p.log2k[0], p.lseed[0]};
    hipLaunchKernelGGL(k_headsum_final, dim3(1), dim3(TPB), 0, st, part, gs,
                       reinterpret_cast<Ctrl*>(a.ws + p.off_ctrl), smp0, a.ws + p.off_eb[0], (uint32_t)p.m[1],
                       (uint32_t)p.rec_bytes, 0, (uint32_t)MODE_PLAIN, g);
    return hipGetLastError();
}

// Batches, in place of the head-sum pass: the per-request head sums (from
// the gather pass) and, when every request is one list, their heads as the
// level-0 walks (see k_batch_heads); else the forest path.
static hipError_t run_batch_heads(const RunArgs& a, const Plan& p, Gate g) {
    hipStream_t st = a.stream;
    const uint2* part = reinterpret_cast<const uint2*>(a.ws + p.off_batch_part);
    uint2* sums = reinterpret_cast<uint2*>(a.ws + p.off_batch_sums);
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(a.ws + p.off_ctrl);
    const uint32_t grid = std::max(1u, std::min<uint32_t>(a.count, (uint32_t)device_cus() * 8));
    hipLaunchKernelGGL(k_batch_reduce, dim3(grid), dim3(TPB), 0, st, part, a.boff, a.bhdr, sums, g);
    LR_TRY(hipGetLastError());
    const Sampler smp0{(uint32_t)p.m[0], p.log2k[0], p.lseed[0]};
    hipLaunchKernelGGL(k_batch_heads, dim3(1), dim3(1024), 0, st, sums, a.bases, a.bhdr, ctrl, smp0,
                       a.ws + p.off_eb[0], (uint32_t)p.m[1], (uint32_t)p.rec_bytes,
                       a.dev_sizes ? (const uint32_t*)&ctrl->dm[0] : nullptr, g);
    return hipGetLastError();
}

// Automatic contraction, the device-side guess (sets Ctrl.mode).
static hipError_t run_guess(const RunArgs& a, const Plan& p, uint32_t thr) {
    const uint32_t n = (uint32_t)p.m[0];
    hipStream_t st = a.stream;
    const uint32_t ntiles = (n + LOCAL_TILE - 1) / LOCAL_TILE;
    const uint32_t nsamp = (ntiles + LOCAL_SAMPLE_STRIDE - 1) / LOCAL_SAMPLE_STRIDE;
    const uint32_t gs = std::max(1u, std::min<uint32_t>(nsamp, HEADSUM_BLOCKS));
    uint32_t* part = reinterpret_cast<uint32_t*>(a.ws + p.off_hsum);
    hipLaunchKernelGGL(k_lsample<true>, dim3(gs), dim3(TPB), 0, st, a.succ, n, part);
    LR_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_ldecide, dim3(1), dim3(TPB), 0, st, part, gs, n, thr,
                       reinterpret_cast<Ctrl*>(a.ws + p.off_ctrl));
    return hipGetLastError();
}

// The plain path up to the level above its chases. With a.prologue the call
// starts here (validation, head sum); otherwise the caller ran them and a.gate
// selects this path. *done: nothing is left (no level is chased).
template <bool W, int WT, class Out0>
static hipError_t run_srs_up(const RunArgs& a, Out0 out0, bool* done) {
    using L = Lay<W>;
    const Plan& p = *a.plan;
    char* ws = a.ws;
    hipStream_t st = a.stream;
    const Gate g = a.gate;
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws + p.off_ctrl);
    const uint32_t n = (uint32_t)p.m[0];
    // device-side sizes (a batch planned for a capacity): level l's actual
    // size and walk count are dm[l], dm[l + 1]; p.m[] are capacities
    auto dm_at = [&](uint32_t l) -> const uint32_t* { return a.dev_sizes ? &ctrl->dm[l] : nullptr; };
    SrcIn<W, WT> src0{a.succ, a.weight, n};
    if (a.prologue) {
        rec_ev(a, EV_START);
        if (a.validate) LR_TRY(run_validate(a, p, n));
    }
    if constexpr (std::is_same_v<Out0, OutBatch>) {
        if (batch_direct(p, a.validate)) {  // the requests were not copied together
            SrcBatch srcb{a.desc, a.bases, a.bhdr, n};
            if (p.iw) LR_TRY((run_iw<W>(p, srcb, out0, n, ctrl, ws, st, dm_at(0), g)));
            else LR_TRY((launch_base<W>(srcb, out0, n, n, ctrl, st, dm_at(0), g)));
            for (int i = EV_DETECT; i < EV_COUNT; ++i) rec_ev(a, i);
            *done = true;
            return hipSuccess;
        }
    }
    if (p.run == 0) {
        *done = true;
        if (p.iw) LR_TRY((run_iw<W>(p, src0, out0, n, ctrl, ws, st, dm_at(0), g)));
        else LR_TRY((launch_base<W>(src0, out0, n, n, ctrl, st, dm_at(0), g)));
        for (int i = EV_DETECT; i < EV_COUNT; ++i) rec_ev(a, i);
        return hipSuccess;
    }
    // level 0: initial elements. One list: its head from a streaming sum.
    // Otherwise: predecessor marks (the one-list case skips these kernels).
    const bool grouped = p.log0 || n >= MARKS_GROUPED_MIN;
    {
        if (a.prologue) LR_TRY(a.desc ? run_batch_heads(a, p, Gate{}) : run_headsum(a, p, Gate{}));
        if (grouped) {
            LR_TRY(run_marks(a, p, ctrl, dm_at(0)));
        } else {
            uint8_t* hp0 = reinterpret_cast<uint8_t*>(ws + p.off_slot[0]);
            LR_TRY(fill(hp0, n, 0u, st, ctrl, g));
            const bool vec = ((uintptr_t)a.succ % 16) == 0;
            const uint32_t gd = grid_for(n, TPB * 4 * 4);
            if (vec) hipLaunchKernelGGL(k_detect<true>, dim3(gd), dim3(TPB), 0, st, a.succ, n, hp0, ctrl, dm_at(0), g);
            else hipLaunchKernelGGL(k_detect<false>, dim3(gd), dim3(TPB), 0, st, a.succ, n, hp0, ctrl, dm_at(0), g);
            LR_TRY(hipGetLastError());
        }
    }
    rec_ev(a, EV_DETECT);
    for (uint32_t l = 0; l < p.run; ++l) {
        const uint32_t m = (uint32_t)p.m[l];
        const uint32_t S = (uint32_t)p.m[l + 1];
        const Sampler smp{m, p.log2k[l], p.lseed[l]};
        const uint8_t* hp = reinterpret_cast<const uint8_t*>(ws + p.off_slot[l]);
        uint32_t* tile = reinterpret_cast<uint32_t*>(ws + p.off_tile[l]);
        const bool more = l + 1 < p.run;
        uint32_t* zp = more ? reinterpret_cast<uint32_t*>(ws + p.off_slot[l + 1]) : nullptr;
        const uint32_t zw = more ? (S + 3) / 4 : 0;
        const uint32_t gt = std::min<uint32_t>(p.ntiles[l], (uint32_t)device_cus() * 8);
        const uint32_t last = p.ntiles[l] <= HEADS_SCAN_LAST_TILES;
        if (l == 0 && grouped) {  // the marks' pass found them
            if (zw) LR_TRY(fill(zp, 4 * (uint64_t)zw, 0u, st, nullptr, g));
        } else {
            hipLaunchKernelGGL(k_heads_count, dim3(gt), dim3(TPB), 0, st, hp, smp, tile, p.ntiles[l], zp, zw,
                               (uint32_t)(l == 0), last, ctrl, (int)l, dm_at(l), g);
            LR_TRY(hipGetLastError());
            if (!last) {
                hipLaunchKernelGGL(k_heads_scan, dim3(1), dim3(1024), 0, st, tile, p.ntiles[l], ctrl, (int)l,
                                   (uint32_t)(l == 0), g);
                LR_TRY(hipGetLastError());
            }
            hipLaunchKernelGGL(k_heads_write, dim3(gt), dim3(TPB), 0, st, hp, smp, tile, p.ntiles[l],
                               ws + p.off_eb[l], S, (uint32_t)p.rec_bytes, (l == 0) ? ctrl : nullptr, dm_at(l), g);
            LR_TRY(hipGetLastError());
        }
        if (a.validate && !(l == 0 && p.log0))
            LR_TRY(fill(ws + p.off_slot[l], (uint64_t)m * p.rec_bytes, 0xffffffffu, st, nullptr, g));
        if (l == 0) rec_ev(a, EV_HEADS);
        if (l == 0) {
            if (p.log0) {
                LR_TRY(fill(ws + p.off_fill, fill_words(p.nb1, p.nb2) * 4, 0u, st, nullptr, g));
                if constexpr (W && WT != 0) {
                    // weighted input: one record per element, interleaved into the
                    // grouping arrays after the first (free until the placement)
                    auto* pr = reinterpret_cast<PairRec<WT>*>(ws + p.off_p[1]);
                    hipLaunchKernelGGL(k_pair<WT>, dim3(grid_for(n, TPB * 4)), dim3(TPB), 0, st, a.succ, a.weight, n,
                                       pr, g);
                    LR_TRY(hipGetLastError());
                    SrcPair<WT> srcp{pr, n};
                    LR_TRY((launch_chase_log<W, 1>(p, srcp, smp, ctrl, ws, st, dm_at(0), g)));
                } else if (p.lane_walks == 2) {
                    LR_TRY((launch_chase_log<W, 2>(p, src0, smp, ctrl, ws, st, dm_at(0), g)));
                } else {
                    LR_TRY((launch_chase_log<W, 1>(p, src0, smp, ctrl, ws, st, dm_at(0), g)));
                }
            } else {
                if (p.lane_walks == 2) LR_TRY((launch_chase<W, 0, 2>(p, 0, src0, smp, ctrl, ws, st, dm_at(0), g)));
                else LR_TRY((launch_chase<W, 0, 1>(p, 0, src0, smp, ctrl, ws, st, dm_at(0), g)));
            }
            rec_ev(a, EV_CHASE0);
        } else {
            SrcLvl<W> src{reinterpret_cast<const typename L::Rec*>(ws + p.off_eb[l - 1]), m};
            LR_TRY((launch_chase<W, 0, 1>(p, (int)l, src, smp, ctrl, ws, st, dm_at(l), g)));
        }
    }
    return hipSuccess;
}

// From the solved level down to the outputs.
template <bool W, class Out0>
static hipError_t run_srs_down(const RunArgs& a, Out0 out0) {
    using L = Lay<W>;
    const Plan& p = *a.plan;
    char* ws = a.ws;
    hipStream_t st = a.stream;
    const Gate g = a.gate;
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws + p.off_ctrl);
    auto dm_at = [&](uint32_t l) -> const uint32_t* { return a.dev_sizes ? &ctrl->dm[l] : nullptr; };
    for (int l = (int)p.run - 1; l >= 0; --l) {
        const uint32_t m = (uint32_t)p.m[l];
        const uint32_t S = (uint32_t)p.m[l + 1];
        hipLaunchKernelGGL(k_resolve<W>, dim3(grid_for(m, TPB * 4, 4)), dim3(TPB), 0, st, ws + p.off_eb[l], S,
                           ctrl, l, dm_at((uint32_t)l), g);
        LR_TRY(hipGetLastError());
        const auto* slot = reinterpret_cast<const typename L::Slot*>(ws + p.off_slot[l]);
        const auto* res = reinterpret_cast<const typename L::Res*>(ws + p.off_eb[l]);
        const uint32_t ge = grid_for(m, TPB * EXPAND_CH);
        if (l == 0) {
            rec_ev(a, EV_UPPER);
            if (p.log0) {
                LR_TRY((run_place<W, Out0>(a, p, res, S, ctrl, out0, a.desc ? a.any_root : a.root != nullptr,
                                           dm_at(0))));
            } else {
                rec_ev(a, EV_PART);
                hipLaunchKernelGGL((k_expand<W, Out0>), dim3(ge), dim3(TPB), 0, st, slot, m, res, S, ctrl, 0, out0,
                                   dm_at(0), g);
            }
        } else {
            OutLvl<W> out{reinterpret_cast<typename L::Res*>(ws + p.off_eb[l - 1])};
            hipLaunchKernelGGL((k_expand<W, OutLvl<W>>), dim3(ge), dim3(TPB), 0, st, slot, m, res, S, ctrl, l,
                               out, dm_at((uint32_t)l), g);
        }
        LR_TRY(hipGetLastError());
    }
    rec_ev(a, EV_EXPAND);
    return hipSuccess;
}

// The chased levels over a contracted list (records at lrec, sizes in
// Ctrl.dm).
template <bool W>
static hipError_t run_clevels_up(const RunArgs& a, const Plan& p, typename Lay<W>::Rec* lrec, Ctrl* ctrl, Gate g,
                                 bool ev_chase0) {
    using L = Lay<W>;
    char* ws = a.ws;
    hipStream_t st = a.stream;
    const uint32_t Lv = p.run;
    for (uint32_t l = 0; l < Lv; ++l) {
        const uint32_t* dm = &ctrl->dm[l];
        const Sampler smp{(uint32_t)p.m[l], p.log2k[l], p.lseed[l]};
        const uint32_t S = (uint32_t)p.m[l + 1];
        const uint8_t* hp = reinterpret_cast<const uint8_t*>(ws + p.off_slot[l]);
        uint32_t* tile = reinterpret_cast<uint32_t*>(ws + p.off_tile[l]);
        const bool more = l + 1 < Lv;
        uint32_t* zp = more ? reinterpret_cast<uint32_t*>(ws + p.off_slot[l + 1]) : nullptr;
        const uint32_t zw = more ? (S + 3) / 4 : 0;
        const uint32_t gt = std::min<uint32_t>(p.ntiles[l], (uint32_t)device_cus() * 8);
        const uint32_t last = p.ntiles[l] <= HEADS_SCAN_LAST_TILES;
        hipLaunchKernelGGL(k_heads_count, dim3(gt), dim3(TPB), 0, st, hp, smp, tile, p.ntiles[l], zp, zw, 0u, last,
                           ctrl, (int)l, dm, g);
        LR_TRY(hipGetLastError());
        if (!last) {
            hipLaunchKernelGGL(k_heads_scan, dim3(1), dim3(1024), 0, st, tile, p.ntiles[l], ctrl, (int)l, 0u, g);
            LR_TRY(hipGetLastError());
        }
        hipLaunchKernelGGL(k_heads_write, dim3(gt), dim3(TPB), 0, st, hp, smp, tile, p.ntiles[l], ws + p.off_eb[l],
                           S, (uint32_t)p.rec_bytes, nullptr, dm, g);
        LR_TRY(hipGetLastError());
        if (a.validate && !(l == 0 && p.log0))
            LR_TRY(fill(ws + p.off_slot[l], (uint64_t)p.m[l] * p.rec_bytes, 0xffffffffu, st, nullptr, g));
        const auto* rec = (l == 0) ? lrec : reinterpret_cast<const typename L::Rec*>(ws + p.off_eb[l - 1]);
        SrcLvl<W> src{rec, (uint32_t)p.m[l]};
        if (l == 0 && p.log0) {  // a long contracted list: visit log and grouped placement, as the plain path
            LR_TRY(fill(ws + p.off_fill, fill_words(p.nb1, p.nb2) * 4, 0u, st, nullptr, g));
            LR_TRY((launch_chase_log<W, 1>(p, src, smp, ctrl, ws, st, dm, g)));
        } else {
            LR_TRY((launch_chase<W, 0, 1>(p, (int)l, src, smp, ctrl, ws, st, dm, g)));
        }
        if (l == 0 && ev_chase0) rec_ev(a, EV_CHASE0);
    }
    return hipSuccess;
}

// The records of the level above the chased ones (lrec: the contracted list).
template <bool W>
static typename Lay<W>::Rec* top_records(const Plan& p, char* ws, typename Lay<W>::Rec* lrec) {
    return p.run ? reinterpret_cast<typename Lay<W>::Rec*>(ws + p.off_eb[p.run - 1]) : lrec;
}

// That level by the base case (plans without independent walks).
template <bool W>
static hipError_t run_base_level(const Plan& p, typename Lay<W>::Rec* rec, uint32_t climit, Ctrl* ctrl,
                                 hipStream_t st, const uint32_t* dm, Gate g) {
    const uint32_t m = (uint32_t)p.m[p.run];
    return launch_base<W>(SrcLvl<W>{rec, m}, OutLvl<W>{rec}, m, climit, ctrl, st, dm, g);
}

// From the solved level down: on return lrec holds every contracted element's
// result.
template <bool W>
static hipError_t run_clevels_down(const RunArgs& a, const Plan& p, typename Lay<W>::Rec* lrec, Ctrl* ctrl, Gate g) {
    using L = Lay<W>;
    char* ws = a.ws;
    hipStream_t st = a.stream;
    for (int l = (int)p.run - 1; l >= 0; --l) {
        const uint32_t m = (uint32_t)p.m[l];
        const uint32_t S = (uint32_t)p.m[l + 1];
        const uint32_t* dm = &ctrl->dm[l];
        hipLaunchKernelGGL(k_resolve<W>, dim3(grid_for(m, TPB * 4, 4)), dim3(TPB), 0, st, ws + p.off_eb[l], S,
                           ctrl, l, dm, g);
        LR_TRY(hipGetLastError());
        const auto* slot = reinterpret_cast<const typename L::Slot*>(ws + p.off_slot[l]);
        const auto* res = reinterpret_cast<const typename L::Res*>(ws + p.off_eb[l]);
        auto* below = (l == 0) ? reinterpret_cast<typename L::Res*>(lrec)
                               : reinterpret_cast<typename L::Res*>(ws + p.off_eb[l - 1]);
        OutLvl<W> out{below};
        if (l == 0 && p.log0) {
            RunArgs b = a;
            b.gate = g;
            LR_TRY((run_place<W, OutLvl<W>>(b, p, res, S, ctrl, out, true, dm)));
        } else {
            hipLaunchKernelGGL((k_expand<W, OutLvl<W>>), dim3(grid_for(m, TPB * EXPAND_CH)), dim3(TPB), 0, st, slot,
                               m, res, S, ctrl, l, out, dm, g);
        }
        LR_TRY(hipGetLastError());
    }
    return hipSuccess;
}

// Tile-local contraction and the chased levels on the contracted list (sizes
// from the device). The plan sizes the levels for a contracted list of at most
// m[0] elements; lc_n is the input's length. Where the plan chases a level and
// the list turns out to have at most LOCAL_SMALL_MAX elements (a.splan), the
// scan turns the path to MODE_LOCAL_SMALL: its levels are not chased, the list
// itself goes to the independent walks.
struct LocalGates {
    Gate pre, levels, both;  // up to the scan; the chased levels; whatever the list's length
};
static LocalGates local_gates(const RunArgs& a, const Ctrl* ctrl) {
    // alone (forced), the path's mode is set by the scan: the kernels up to it
    // run ungated
    const Gate pre = a.prologue ? Gate{} : a.gate;
    if (!a.splan) return {pre, a.gate, a.gate};
    return {pre, Gate{&ctrl->mode, mode_bit(MODE_LOCAL)},
            Gate{&ctrl->mode, mode_bit(MODE_LOCAL) | mode_bit(MODE_LOCAL_SMALL)}};
}

template <bool W, int WT>
static hipError_t run_local_up(const RunArgs& a) {
    using L = Lay<W>;
    const Plan& p = *a.plan;
    char* ws = a.ws;
    hipStream_t st = a.stream;
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws + p.off_ctrl);
    const LocalGates g = local_gates(a, ctrl);
    const uint32_t n = (uint32_t)p.lc_n;
    if (a.prologue) {
        rec_ev(a, EV_START);
        if (a.validate) LR_TRY(run_validate(a, p, n));
    }
    uint32_t* cnt = reinterpret_cast<uint32_t*>(ws + p.off_lc_cnt);
    uint2* dir = reinterpret_cast<uint2*>(ws + p.off_lc_dir);
    uint32_t* pos = reinterpret_cast<uint32_t*>(ws + p.off_lc_pos);
    int64_t* wd = W ? reinterpret_cast<int64_t*>(ws + p.off_lc_wd) : nullptr;
    auto* lrec = reinterpret_cast<typename L::Rec*>(ws + p.off_lrec);
    auto* stage = reinterpret_cast<typename L::Rec*>(ws + p.off_lc_stage);
    uint8_t* hp0 = p.run ? reinterpret_cast<uint8_t*>(ws + p.off_slot[0]) : nullptr;
    const uint32_t gc = LR_LC_GRID_PER_CU ? std::min<uint32_t>(p.lc_ntiles, (uint32_t)device_cus() * LR_LC_GRID_PER_CU)
                                          : p.lc_ntiles;
    hipLaunchKernelGGL((k_lc_chain<W, WT>), dim3(gc), dim3(LC_TPB), 0, st, a.succ, a.weight, n, p.lc_ntiles, cnt, dir,
                       stage, pos, wd, ctrl, g.pre);
    LR_TRY(hipGetLastError());
    LevelShifts ks{}, kss{};
    for (uint32_t l = 0; l < p.levels; ++l) ks.lg[l] = (uint8_t)p.log2k[l];
    uint32_t small = 0, slevels = 0;
    if (a.splan) {
        small = (uint32_t)a.splan->m[0];
        slevels = a.splan->top;
        for (uint32_t l = 0; l < slevels; ++l) kss.lg[l] = (uint8_t)a.splan->log2k[l];
    }
    hipLaunchKernelGGL(k_lc_scan, dim3(1), dim3(1024), 0, st, cnt, p.lc_ntiles, ctrl, p.levels, ks, (uint32_t)p.m[0],
                       (uint32_t)a.prologue, small, slevels, kss, g.pre);
    LR_TRY(hipGetLastError());
    rec_ev(a, EV_DETECT);
    if (hp0) {
        hipLaunchKernelGGL(k_zero_dyn, dim3(grid_for(p.m[0] / 4 + 1, TPB * 4)), dim3(TPB), 0, st,
                           reinterpret_cast<uint32_t*>(hp0), (const uint32_t*)&ctrl->dm[0], g.levels);
        LR_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL((k_lc_compact<W>), dim3(grid_for((uint64_t)p.lc_ntiles * 64, TPB)), dim3(TPB), 0, st, stage,
                       cnt, dir, p.lc_ntiles, n, lrec, hp0, g.both);
    LR_TRY(hipGetLastError());
    rec_ev(a, EV_HEADS);
    return run_clevels_up<W>(a, p, lrec, ctrl, g.levels, true);
}

// Every element from its chain start.
template <bool W, class Out0>
static hipError_t run_local_down(const RunArgs& a, Out0 out0) {
    using L = Lay<W>;
    const Plan& p = *a.plan;
    char* ws = a.ws;
    hipStream_t st = a.stream;
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws + p.off_ctrl);
    const LocalGates g = local_gates(a, ctrl);
    const uint32_t n = (uint32_t)p.lc_n;
    auto* lrec = reinterpret_cast<typename L::Rec*>(ws + p.off_lrec);
    LR_TRY(run_clevels_down<W>(a, p, lrec, ctrl, g.levels));
    rec_ev(a, EV_UPPER);
    rec_ev(a, EV_PART);
    hipLaunchKernelGGL((k_lc_expand<W, Out0>), dim3(grid_for(n, TPB * EXPAND_CH)), dim3(TPB), 0, a.stream,
                       reinterpret_cast<const uint32_t*>(ws + p.off_lc_pos),
                       W ? reinterpret_cast<const int64_t*>(ws + p.off_lc_wd) : nullptr,
                       reinterpret_cast<const uint32_t*>(ws + p.off_lc_cnt),
                       reinterpret_cast<const typename L::Res*>(lrec), n, ctrl, out0, g.both);
    LR_TRY(hipGetLastError());
    rec_ev(a, EV_EXPAND);
    return hipSuccess;
}

// Ruler spawning: predecessor bytes and heads of the input, the capped chase,
// the spawned rulers, their chase (all walks form the contracted list, sized
// on the device), the ruling-set levels on that list, then every element
// from its walk.
template <bool W, int WT, class Out0>
static hipError_t run_spawn_t(const RunArgs& a, Out0 out0) {
    using L = Lay<W>;
    const Plan& p = *a.plan;
    char* ws = a.ws;
    hipStream_t st = a.stream;
    const Gate g = a.gate;
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws + p.off_ctrl);
    const uint32_t n = (uint32_t)p.sp_n;
    const uint32_t Lv = p.run;
    if (a.prologue) {
        rec_ev(a, EV_START);
        if (a.validate) LR_TRY(run_validate(a, p, n));
    }
    auto* slot = reinterpret_cast<typename L::Slot*>(ws + p.off_sp_slot);
    uint8_t* hp_in = reinterpret_cast<uint8_t*>(ws + p.off_sp_hp);
    uint32_t* tile = reinterpret_cast<uint32_t*>(ws + p.off_sp_tile);
    auto* lrec = reinterpret_cast<typename L::Rec*>(ws + p.off_lrec);
    uint8_t* hp_c = reinterpret_cast<uint8_t*>(ws + p.off_slot[0]);  // the walks' predecessor bytes
    const Sampler smp{n, p.sp_log2k, p.sp_seed};
    const uint32_t S0 = (n + (1u << p.sp_log2k) - 1u) >> p.sp_log2k;
    {
        const uint64_t words = (uint64_t)n * p.rec_bytes / 4;
        hipLaunchKernelGGL(k_sp_prep, dim3(grid_for(words, TPB * 4)), dim3(TPB), 0, st,
                           reinterpret_cast<uint32_t*>(slot), words, ctrl, Gate{});
        LR_TRY(hipGetLastError());
    }
    {  // one list: its head from the streaming sum, and no predecessor marks
        const bool vec = ((uintptr_t)a.succ % 16) == 0;
        const uint32_t gs = std::min<uint32_t>(grid_for(n, TPB * 16), HEADSUM_BLOCKS);
        uint32_t* part = reinterpret_cast<uint32_t*>(ws + p.off_hsum);
        if (vec) hipLaunchKernelGGL(k_headsum<true>, dim3(gs), dim3(TPB), 0, st, a.succ, n, part, g);
        else hipLaunchKernelGGL(k_headsum<false>, dim3(gs), dim3(TPB), 0, st, a.succ, n, part, g);
        LR_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_headsum_final, dim3(1), dim3(TPB), 0, st, part, gs, ctrl, smp,
                           reinterpret_cast<char*>(lrec), S0, (uint32_t)p.rec_bytes, SPL, NONE, g);
        LR_TRY(hipGetLastError());
    }
    LR_TRY(fill(hp_in, n, 0u, st, ctrl, g));
    {
        const bool vec = ((uintptr_t)a.succ % 16) == 0;
        const uint32_t gd = grid_for(n, TPB * 4 * 4);
        if (vec) hipLaunchKernelGGL(k_detect<true>, dim3(gd), dim3(TPB), 0, st, a.succ, n, hp_in, ctrl, nullptr, g);
        else hipLaunchKernelGGL(k_detect<false>, dim3(gd), dim3(TPB), 0, st, a.succ, n, hp_in, ctrl, nullptr, g);
        LR_TRY(hipGetLastError());
    }
    rec_ev(a, EV_DETECT);
    const uint32_t gt = std::min<uint32_t>(p.sp_ntiles, (uint32_t)device_cus() * 8);
    const uint32_t last = p.sp_ntiles <= HEADS_SCAN_LAST_TILES;
    hipLaunchKernelGGL(k_heads_count, dim3(gt), dim3(TPB), 0, st, hp_in, smp, tile, p.sp_ntiles,
                       reinterpret_cast<uint32_t*>(hp_c), (n + 3) / 4, 1u, last, ctrl, SPL, nullptr, g);
    LR_TRY(hipGetLastError());
    if (!last) {
        hipLaunchKernelGGL(k_heads_scan, dim3(1), dim3(1024), 0, st, tile, p.sp_ntiles, ctrl, SPL, 1u, g);
        LR_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(k_heads_write, dim3(gt), dim3(TPB), 0, st, hp_in, smp, tile, p.sp_ntiles,
                       reinterpret_cast<char*>(lrec), S0, (uint32_t)p.rec_bytes, ctrl, nullptr, g);
    LR_TRY(hipGetLastError());
    rec_ev(a, EV_HEADS);
    {
        SrcIn<W, WT> src{a.succ, a.weight, n};
        auto k1 = k_sp_chase1<W, WT>;
        auto k2 = k_sp_chase2<W, WT>;
        static const uint32_t g1 = persistent_grid(k1, SP_TPB);  // one per template instance, found once
        static const uint32_t g2 = persistent_grid(k2, SP_TPB);
        const uint32_t cap = (uint32_t)std::min<uint64_t>((uint64_t)LR_SPAWN_CAP << p.sp_log2k, n);
        hipLaunchKernelGGL(k1, dim3(g1), dim3(SP_TPB), 0, st, src, smp, ctrl, slot, lrec, hp_c, cap, g);
        LR_TRY(hipGetLastError());
        const uint32_t seed2 = p.sp_seed ^ 0x5bd1e995u, k2mask = LR_SPAWN_K2 - 1u;
        hipLaunchKernelGGL(k_sp_count<W>, dim3(gt), dim3(TPB), 0, st, slot, n, seed2, k2mask, tile, p.sp_ntiles, g);
        LR_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_sp_scan, dim3(1), dim3(1024), 0, st, tile, p.sp_ntiles, ctrl, g);
        LR_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_sp_write<W>, dim3(gt), dim3(TPB), 0, st, slot, n, seed2, k2mask, tile, p.sp_ntiles, ctrl,
                           S0, lrec, hp_c, g);
        LR_TRY(hipGetLastError());
        hipLaunchKernelGGL(k2, dim3(g2), dim3(SP_TPB), 0, st, src, smp, ctrl, slot, lrec, hp_c, g);
        LR_TRY(hipGetLastError());
    }
    LevelShifts ks{};
    for (uint32_t l = 0; l < p.levels; ++l) ks.lg[l] = (uint8_t)p.log2k[l];
    hipLaunchKernelGGL(k_sp_publish, dim3(1), dim3(64), 0, st, ctrl, S0, (uint32_t)p.m[0], p.levels, ks, g);
    LR_TRY(hipGetLastError());
    rec_ev(a, EV_CHASE0);
    LR_TRY(run_clevels_up<W>(a, p, lrec, ctrl, g, false));
    if (p.iw) {
        IwSet<W> set[3] = {{&p, top_records<W>(p, ws, lrec), &ctrl->dm[Lv]}, {}, {}};
        LR_TRY(run_iw_levels<W>(set, nullptr, n, ctrl, ws, st));
    } else {
        LR_TRY(run_base_level<W>(p, top_records<W>(p, ws, lrec), n, ctrl, st, &ctrl->dm[Lv], g));
    }
    LR_TRY(run_clevels_down<W>(a, p, lrec, ctrl, g));
    rec_ev(a, EV_UPPER);
    rec_ev(a, EV_PART);
    hipLaunchKernelGGL((k_sp_expand<W, Out0>), dim3(grid_for(n, TPB * EXPAND_CH)), dim3(TPB), 0, st, slot, n,
                       reinterpret_cast<const typename L::Res*>(lrec), ctrl, out0, g);
    LR_TRY(hipGetLastError());
    rec_ev(a, EV_EXPAND);
    return hipSuccess;
}

// Forced paths run alone. Automatic contraction: a sample of the tiles
// decides on the device, the contracted path's scan may still hand over to the
// plain path, and the plain path's head-sum pass runs only if that path is
// taken. Both paths are enqueued and the one not chosen returns from every
// kernel at once (no host synchronisation, so the call stays capturable).
template <bool W, int WT, class Out0>
static hipError_t run_path_t(const RunArgs& a, Out0 out0) {
    using L = Lay<W>;
    if (a.plan->spawn) return run_spawn_t<W, WT>(a, out0);
    char* ws = a.ws;
    hipStream_t st = a.stream;
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws + a.plan->off_ctrl);
    auto lrec_of = [&](const Plan& p) { return reinterpret_cast<typename L::Rec*>(ws + p.off_lrec); };
    // the contracted list's sets of the independent walks
    auto local_sets = [&](const RunArgs& la, IwSet<W>* set) {
        const Plan& q = *la.plan;
        if (q.iw) set[1] = {&q, top_records<W>(q, ws, lrec_of(q)), &ctrl->dm[q.run]};
        if (la.splan) set[2] = {la.splan, lrec_of(q), &ctrl->dms[0]};
    };
    IwSet<W> set[3];
    if (!a.lplan && a.plan->local) {
        const Plan& q = *a.plan;
        LR_TRY((run_local_up<W, WT>(a)));
        local_sets(a, set);
        if (!q.iw)
            LR_TRY(run_base_level<W>(q, top_records<W>(q, ws, lrec_of(q)), (uint32_t)q.lc_n, ctrl, st, &ctrl->dm[q.run],
                                     a.gate));
        if (q.iw) LR_TRY(run_iw_levels<W>(set, &ctrl->mode, (uint32_t)q.lc_n, ctrl, ws, st));
        return run_local_down<W>(a, out0);
    }
    const Plan& p = *a.plan;
    const uint32_t n = (uint32_t)p.m[0];
    const uint32_t* dm = a.dev_sizes ? &ctrl->dm[p.run] : nullptr;
    if (!a.lplan) {
        bool done = false;
        LR_TRY((run_srs_up<W, WT>(a, out0, &done)));
        if (done) return hipSuccess;
        auto* top = top_records<W>(p, ws, nullptr);
        if (p.iw) {
            set[0] = {&p, top, dm};
            LR_TRY(run_iw_levels<W>(set, nullptr, n, ctrl, ws, st));
        } else {
            LR_TRY(run_base_level<W>(p, top, n, ctrl, st, dm, a.gate));
        }
        return run_srs_down<W>(a, out0);
    }
    rec_ev(a, EV_START);
    if (a.validate) LR_TRY(run_validate(a, p, n));
    LR_TRY(run_guess(a, p, (uint32_t)local_guess_cap(p.m[0])));
    RunArgs la = a;
    la.plan = a.lplan;
    la.prologue = false;
    la.gate = Gate{&ctrl->mode, mode_bit(MODE_LOCAL)};
    LR_TRY((run_local_up<W, WT>(la)));  // its scan falls back to mode 0 if the list is too long
    RunArgs pa = a;
    pa.prologue = false;
    pa.gate = Gate{&ctrl->mode, mode_bit(MODE_PLAIN)};
    LR_TRY(a.desc ? run_batch_heads(pa, p, pa.gate) : run_headsum(pa, p, pa.gate));
    bool done = false;  // (an input of this size has a chased level)
    LR_TRY((run_srs_up<W, WT>(pa, out0, &done)));
    // both paths' lists share the launches of the independent walks
    const Plan& q = *la.plan;
    local_sets(la, set);
    if (p.iw) set[0] = {&p, top_records<W>(p, ws, nullptr), dm};
    if (!q.iw)
        LR_TRY(run_base_level<W>(q, top_records<W>(q, ws, lrec_of(q)), n, ctrl, st, &ctrl->dm[q.run], la.gate));
    if (!p.iw) LR_TRY(run_base_level<W>(p, top_records<W>(p, ws, nullptr), n, ctrl, st, dm, pa.gate));
    if (p.iw || q.iw) LR_TRY(run_iw_levels<W>(set, &ctrl->mode, n, ctrl, ws, st));
    LR_TRY((run_local_down<W>(la, out0)));
    return run_srs_down<W>(pa, out0);
}

// The bounded fallback over the input; both kernels return at once unless some
// walk reached its cap.
template <bool W, int WT, class Out0>
static hipError_t run_fallback_t(const RunArgs& a, Out0 out0) {
    using Src = SrcIn<W, WT>;
    const Plan& p = *a.plan;
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(a.ws + p.off_ctrl);
    const uint32_t n = (uint32_t)(p.spawn ? p.sp_n : (p.local ? p.lc_n : p.m[0]));
    const Gate g{&ctrl->mode, mode_bit(MODE_FALLBACK)};
    uint64_t* nodes = reinterpret_cast<uint64_t*>(a.ws + p.off_fb);
    const uint32_t* dm = a.dev_sizes ? &ctrl->dm[0] : nullptr;
    const Src src{a.succ, a.weight, n};
    hipLaunchKernelGGL((k_fb_first<W, Src>), dim3(grid_for(n, TPB)), dim3(TPB), 0, a.stream, src, nodes, n, dm, g);
    LR_TRY(hipGetLastError());
    auto kern = k_fb_double<W, Src, Out0>;
    static const uint32_t resident = persistent_grid(kern, TPB);  // one per template instance, found once
    hipLaunchKernelGGL(kern, dim3(std::min<uint32_t>(grid_for(n, TPB), resident)), dim3(TPB), 0, a.stream, src, nodes,
                       n, out0, a.validate ? &ctrl->err : nullptr, dm, g);
    return hipGetLastError();
}

// Every path's first kernels set Ctrl.mode and a capped walk turns it to
// MODE_FALLBACK; the fallback runs after the path and returns at once unless
// that happened. A path that runs alone has no gates (a gate costs every
// kernel a dependent load): after a cap it runs on to its end, bounded (every
// walk stops at its cap, every other kernel is bounded whatever its input),
// and the fallback then overwrites its outputs. Under automatic contraction
// both paths are gated on the mode anyway, so they stop at once. A plan
// without chased levels (the base case, or independent walks) has no fallback.
template <bool W, int WT, class Out0>
static hipError_t run_any_t(const RunArgs& a, Out0 out0) {
    const Plan& p = *a.plan;
    LR_TRY((run_path_t<W, WT>(a, out0)));
    return p.walks() ? run_fallback_t<W, WT>(a, out0) : hipSuccess;
}

template <int WT>
static hipError_t run_weighted(const RunArgs& a) {
    if (a.rank && a.root) return run_any_t<true, WT>(a, OutUser<true, true, true>{a.rank, a.root, a.sum});
    if (a.rank) return run_any_t<true, WT>(a, OutUser<true, true, false>{a.rank, nullptr, a.sum});
    if (a.root) return run_any_t<true, WT>(a, OutUser<true, false, true>{nullptr, a.root, a.sum});
    return run_any_t<true, WT>(a, OutUser<true, false, false>{nullptr, nullptr, a.sum});
}

hipError_t run_srs(const RunArgs& a) {
    const Plan& p = *a.plan;
    if (a.desc) {
        OutBatch out{a.desc, a.bases, a.bhdr};
        return run_any_t<false, 0>(a, out);
    }
    if (!p.weighted) {  // rank is required
        if (a.root) return run_any_t<false, 0>(a, OutUser<false, true, true>{a.rank, a.root, nullptr});
        return run_any_t<false, 0>(a, OutUser<false, true, false>{a.rank, nullptr, nullptr});
    }
    if (a.rec) {  // records for an internal caller
        OutLvl<true> out{reinterpret_cast<typename Lay<true>::Res*>(a.rec)};
        switch (a.wt) {
            case 1: return run_any_t<true, 1>(a, out);
            case 2: return run_any_t<true, 2>(a, out);
            case 3: return run_any_t<true, 3>(a, out);
            default: return run_any_t<true, 0>(a, out);
        }
    }
    switch (a.wt) {  // the sum is required; rank and root are optional
        case 1: return run_weighted<1>(a);
        case 2: return run_weighted<2>(a);
        default: return run_weighted<0>(a);
    }
}

template <bool W, int WT>
static hipError_t run_wyllie_t(const RunArgs& a, uint64_t n64) {
    using L = Lay<W>;
    const uint32_t n = (uint32_t)n64;
    auto* A = reinterpret_cast<typename L::Rec*>(a.ws);
    auto* B = reinterpret_cast<typename L::Rec*>(a.ws + ((n64 * sizeof(typename L::Rec) + ALIGN - 1) / ALIGN) * ALIGN);
    OutUser<W, true, true, true> out{a.rank, a.root, W ? a.sum : nullptr};
    const uint32_t g = grid_for(n, TPB * 4);
    SrcIn<W, WT> src{a.succ, a.weight, n};
    rec_ev(a, EV_START);
    hipLaunchKernelGGL((k_wy_init<W, SrcIn<W, WT>>), dim3(g), dim3(TPB), 0, a.stream, src, A, n);
    LR_TRY(hipGetLastError());
    uint32_t rounds = 0;
    while ((1ull << rounds) < n64) ++rounds;
    if (rounds == 0) {
        hipLaunchKernelGGL(k_wy_copy<W>, dim3(g), dim3(TPB), 0, a.stream, A, n, out);
        LR_TRY(hipGetLastError());
    }
    for (uint32_t r = 0; r < rounds; ++r) {
        if (r + 1 == rounds)
            hipLaunchKernelGGL((k_wy_round<W, true>), dim3(g), dim3(TPB), 0, a.stream, A, B, n, out);
        else
            hipLaunchKernelGGL((k_wy_round<W, false>), dim3(g), dim3(TPB), 0, a.stream, A, B, n, out);
        LR_TRY(hipGetLastError());
        std::swap(A, B);
    }
    for (int i = EV_DETECT; i < EV_COUNT; ++i) rec_ev(a, i);
    return hipSuccess;
}

hipError_t run_wyllie(const RunArgs& a, uint64_t n, bool weighted) {
    if (!weighted) return run_wyllie_t<false, 0>(a, n);
    switch (a.wt) {
        case 1: return run_wyllie_t<true, 1>(a, n);
        case 2: return run_wyllie_t<true, 2>(a, n);
        default: return run_wyllie_t<true, 0>(a, n);
    }
}

hipError_t run_batch_table(const lr_request* reqs, uint32_t count, const Plan& p, char* ws, bool dev_sizes,
                           uint32_t max_chunks, bool gather, hipStream_t st) {
    auto* desc = reinterpret_cast<BatchDesc*>(ws + p.off_batch_desc);
    auto* bases = reinterpret_cast<uint32_t*>(ws + p.off_batch_bases);
    uint32_t* boff = bases + p.batch_count + 1;
    auto* hdr = reinterpret_cast<BatchHdr*>(ws + p.off_batch_hdr);
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(ws + p.off_ctrl);
    LevelShifts ks{};
    for (uint32_t l = 0; l < p.levels; ++l) ks.lg[l] = (uint8_t)p.log2k[l];
    const uint32_t levels = dev_sizes ? p.levels : 0u;
    BatchDescArg arg{};
    arg.count = count;
    for (uint32_t first = 0; first < count || first == 0; first += BATCH_ARG_DESC) {
        arg.first = first;
        arg.cnt = std::min<uint32_t>(BATCH_ARG_DESC, count - first);
        for (uint32_t i = 0; i < arg.cnt; ++i) {
            const lr_request& r = reqs[first + i];
            arg.d[i] = BatchDesc{r.succ, r.rank, r.root, r.n};
        }
        if (count <= BATCH_ARG_DESC) {
            hipLaunchKernelGGL(k_batch_table, dim3(1), dim3(1024), 0, st, arg, desc, bases, boff, hdr, ctrl, levels, ks);
            LR_TRY(hipGetLastError());
            break;
        }
        hipLaunchKernelGGL(k_batch_desc, dim3(1), dim3(64), 0, st, arg, desc, hdr);
        LR_TRY(hipGetLastError());
    }
    if (count > BATCH_ARG_DESC) {
        hipLaunchKernelGGL(k_batch_index, dim3(1), dim3(1024), 0, st, desc, bases, boff, hdr, ctrl, levels, ks);
        LR_TRY(hipGetLastError());
    }
    if (!gather) return hipSuccess;
    const uint32_t grid = std::max(1u, std::min<uint32_t>(max_chunks, (uint32_t)device_cus() * 16));
    hipLaunchKernelGGL(k_batch_gather, dim3(grid), dim3(TPB), 0, st, desc, bases, boff, hdr,
                       reinterpret_cast<uint32_t*>(ws + p.off_batch_succ),
                       reinterpret_cast<uint2*>(ws + p.off_batch_part));
    return hipGetLastError();
}

hipError_t run_validate_input(const uint32_t* succ, uint32_t n, uint32_t* counts, uint32_t* err, hipStream_t st) {
    if (!n) return hipSuccess;
    hipLaunchKernelGGL(k_validate_in, dim3(grid_for(n, TPB * 4)), dim3(TPB), 0, st, succ, n, counts, err);
    return hipGetLastError();
}

hipError_t run_verify(const uint32_t* succ, const void* weight, int wt, const uint32_t* rank, const uint32_t* root,
                      const int64_t* sum, uint32_t n, uint32_t* err, hipStream_t st) {
    const dim3 g(grid_for(n, TPB * 4)), b(TPB);
    hipLaunchKernelGGL(k_fill, dim3(1), dim3(TPB), 0, st, err, 1ull, 0u, (const Ctrl*)nullptr, Gate{});
    if (wt == 1) hipLaunchKernelGGL(k_verify<1>, g, b, 0, st, succ, weight, rank, root, sum, n, err);
    else if (wt == 2) hipLaunchKernelGGL(k_verify<2>, g, b, 0, st, succ, weight, rank, root, sum, n, err);
    else hipLaunchKernelGGL(k_verify<0>, g, b, 0, st, succ, weight, rank, root, sum, n, err);
    return hipGetLastError();
}


// ----------------------------------------------------------- debug writes --
// Sets the counters of a call (null: count nothing) and clears them and the
// control block's debug bit (without validation nothing else clears it).
__global__ __launch_bounds__(TPB) void k_dbg_begin(DbgWrites d, uint32_t* __restrict__ base, uint64_t words,
                                                   Ctrl* ctrl) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
#if LR_DEBUG_WRITES
        g_dbg = d;
#endif
        ctrl->err &= ~ERR_DEBUG_WRITES;
    }
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride) base[i] = 0;
}

// Every slot of the levels from `slot_from` on written once, every mark at
// most once (only when the plain path ran to its end); then counting stops.
__global__ __launch_bounds__(TPB) void k_dbg_check(DbgWrites d, DbgSizes sz, uint32_t levels, uint32_t slot_from,
                                                   Ctrl* ctrl) {
#if LR_DEBUG_WRITES
    if (blockIdx.x == 0 && threadIdx.x == 0) g_dbg = DbgWrites{};
#endif
    if (ctrl->mode != MODE_PLAIN) return;
    const uint32_t stride = gridDim.x * blockDim.x;
    bool bad = false;
    for (uint32_t l = 0; l < levels; ++l) {
        for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < sz.m[l]; i += stride) {
            if (l >= slot_from && d.slot[l][i] != 1u) bad = true;
            if (d.mark[l][i] > 1u) bad = true;
        }
    }
    if (bad) atomicOr(&ctrl->err, ERR_DEBUG_WRITES);
}

hipError_t run_debug_begin(const RunArgs& a, const Plan& p) {
    if (!LR_DEBUG_WRITES) return hipSuccess;
    DbgWrites d{};
    uint64_t words = 0;
    const bool plain = !p.local && !p.spawn && !a.lplan;
    if (plain) {
        size_t off = p.off_dbg;
        for (uint32_t l = 0; l < p.levels; ++l) {
            d.slot[l] = reinterpret_cast<uint32_t*>(a.ws + off);
            d.mark[l] = d.slot[l] + p.m[l];
            off += (p.m[l] * 8 + ALIGN - 1) / ALIGN * ALIGN;
        }
        words = (off - p.off_dbg) / 4;
    }
    uint32_t* base = reinterpret_cast<uint32_t*>(a.ws + p.off_dbg);
    hipLaunchKernelGGL(k_dbg_begin, dim3(std::max<uint32_t>(1, grid_for(words, TPB * 4))), dim3(TPB), 0, a.stream, d,
                       base, words, reinterpret_cast<Ctrl*>(a.ws + p.off_ctrl));
    return hipGetLastError();
}

hipError_t run_debug_check(const RunArgs& a, const Plan& p) {
    if (!LR_DEBUG_WRITES) return hipSuccess;
    const bool plain = !p.local && !p.spawn && !a.lplan;
    DbgWrites d{};
    DbgSizes sz{};
    uint32_t levels = 0;
    if (plain) {
        size_t off = p.off_dbg;
        levels = p.run;
        for (uint32_t l = 0; l < p.run; ++l) {
            d.slot[l] = reinterpret_cast<uint32_t*>(a.ws + off);
            d.mark[l] = d.slot[l] + p.m[l];
            sz.m[l] = (uint32_t)p.m[l];
            off += (p.m[l] * 8 + ALIGN - 1) / ALIGN * ALIGN;
        }
    }
    Ctrl* ctrl = reinterpret_cast<Ctrl*>(a.ws + p.off_ctrl);
    // level 0 writes slots only when it is not chased through the visit log
    hipLaunchKernelGGL(k_dbg_check, dim3(std::max<uint32_t>(1, grid_for(p.m[0], TPB * 4))), dim3(TPB), 0, a.stream, d,
                       sz, levels, p.log0 ? 1u : 0u, ctrl);
    return hipGetLastError();
}

}  // namespace lr
