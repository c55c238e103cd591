// Device-side building blocks of the sparse ruling-set list ranker (gfx950).
//
// Data layout per recursion level l (m_l elements, S_l = m_{l+1} rulers):
//   slot_l[m_l]         walk id and offset of every element, written by the
//                       chase (the element's position inside its walk)
//   eb_l[S_l + m_l]     one record per walk. Entries [0, S_l) are the walks of
//                       the sampled rulers; after the chase they hold the
//                       elements of level l+1 (successor ruler + segment
//                       weight), after level l+1 is solved they hold its
//                       results (rank + root). Entries [S_l, ...) are the walks
//                       of initial elements that are not rulers; the compaction
//                       pass parks each such walk's start element in the entry's
//                       first word, the chase replaces it by the walk's end and
//                       weight, and the resolve pass by the walk's result.
//   hp_l[m_l] (bytes)   "has a predecessor" marks, aliased onto slot_l: they
//                       are read by the compaction pass before the chase of the
//                       same level overwrites slot_l.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace lr {

constexpr uint32_t TERM = 0x80000000u;      // record flag: element is a terminal
constexpr uint32_t IDX = 0x7fffffffu;       // payload bits (ids are < 2^31)
constexpr uint32_t NONE = 0xffffffffu;
constexpr int MAXL = 8;

struct Ctrl {
    struct Lv { uint32_t H, q; } lv[MAXL];  // per level: #initial-element walks, chase queue head
    uint32_t err;                           // validation error bits
    uint32_t chunks;                        // visit-log chunks handed out (level 0, log mode)
    uint32_t nterm;                         // level 0: number of terminals (= number of lists)
    uint32_t single;                        // level 0: one list, whose head is known from hsum
    uint64_t hsum;                          // level 0: sum of ids minus sum of successors of non-terminals
    uint32_t dm[MAXL + 1];                  // element count per level when sizes are known only on the
                                            // device (the contracted list of tile-local contraction)
    uint32_t mode;                          // the path that runs (MODE_*): set by each path's first
                                            // kernels, MODE_FALLBACK once a walk reached its cap
    uint32_t multi;                         // plain path with more than one list: predecessor marks needed
    uint32_t spn;                           // ruler spawning: number of spawned rulers
    uint32_t conts;                         // packed visit log: continuation ids handed out
    uint32_t hc_done;                       // workgroups of a head-count kernel that have finished
    uint32_t dms[4];                        // MODE_LOCAL_SMALL: element count per level
    uint32_t pad[24];
};
static_assert(sizeof(Ctrl) == 256, "Ctrl layout");

// Device-side choice between enqueued kernel sequences: a kernel whose gate
// is set runs only when the word it points to (Ctrl.mode) holds a value whose
// bit is in `want`, and otherwise returns before touching memory. A null gate
// always runs.
struct Gate {
    const uint32_t* p;
    uint32_t want;
    __device__ __forceinline__ bool off() const { return p && !((want >> *p) & 1u); }
};

// Values of Ctrl.mode: the path whose kernels run. Each path's first kernels
// set it (the automatic choice between plain and contracted path included),
// and a walk that reaches its step cap turns it to MODE_FALLBACK, so every
// later kernel of the path returns and only the fallback runs. MODE_LOCAL_SMALL:
// the contracted path with a list so short that it is not chased.
enum : uint32_t { MODE_PLAIN = 0, MODE_LOCAL = 1, MODE_FALLBACK = 2, MODE_SPAWN = 3, MODE_LOCAL_SMALL = 4 };
constexpr uint32_t mode_bit(uint32_t m) { return 1u << m; }

// Ctrl.err bits (LR_VALIDATE): the input check sets ERR_INPUT (an index out
// of range, two predecessors); the ranking path's consistency checks set
// others; the fallback sets ERR_FALLBACK_CYCLE for a path that never reaches
// a terminal. After a fallback only ERR_INPUT and ERR_FALLBACK_CYCLE count:
// a path stopped by a cap leaves inconsistent state behind.
constexpr uint32_t ERR_INPUT = 1u | 2u;
constexpr uint32_t ERR_FALLBACK_CYCLE = 256u;
constexpr uint32_t ERR_DEBUG_WRITES = 512u;  // debug builds: a slot or mark with another write count

// Walk step cap: a walk at level spacing k stops after WALK_CAP_MULT * k
// steps. On a list whose order is independent of the sampling, walk lengths
// are about geometric with mean k, so R walks exceed the cap with
// probability about R * e^-64 (never, in practice); only an order built
// against the sampling reaches it. The fallback then ranks the input by
// pointer doubling, whose rounds do not depend on the order.
// A walk that outgrows its level (a cycle: input that is not a forest) is
// stopped the same way; the fallback then reports it under LR_VALIDATE.
// Spacings are at most 2^12, so the cap fits 32 bits.
constexpr uint32_t WALK_CAP_MULT = 64;
__device__ __forceinline__ uint32_t walk_cap(uint32_t m, uint32_t log2k) { return min(m, WALK_CAP_MULT << log2k); }

// Visit log of the level-0 chase (log mode): one record (element, walk,
// offset) per visited element, in one of two formats.
//   wide:   three 32-bit arrays x, w, c.
//   packed: one 64-bit word r = x << (bw + bo) | walk << bo | offset, field
//           widths from LogFmt. A walk whose offset outgrows its bo bits goes
//           on under a continuation id nw + j (nw = walks of the level), whose
//           entry cont[j] = (walk, offset where the continuation starts); the
//           offset field then counts from there. Continuation ids are handed
//           out in blocks of CONT_GRAB per wavefront.
// Weighted levels add the 64-bit weight sum s in both formats.
template <bool W>
struct LogArrays {
    uint32_t* x;
    uint32_t* w;
    uint32_t* c;
    int64_t* s;  // weighted levels only
    uint64_t* r;     // packed records
    uint2* cont;     // packed: continuation entries (walk, base offset)
    uint32_t ccap;   // packed: continuation entries available
    uint32_t bocap;  // packed: most offset bits a record may use
};

constexpr uint32_t CONT_GRAB = 128;  // continuation ids a wavefront takes at a time (>= its lanes' walks)

// Field widths of the packed visit log for n elements and nw walks: 2^bx > n,
// so an all-ones record (chunk padding) names no element; 2^bw > nw + ccap
// (walks and continuations); bo gets the rest of the 64 bits, at most bocap
// and 31. Chase and grouping derive the same widths from the same numbers.
struct LogFmt {
    uint32_t bx, bw, bo;
    __device__ __forceinline__ LogFmt(uint32_t n, uint32_t nw, uint32_t ccap, uint32_t bocap) {
        bx = 32u - (uint32_t)__clz((int)n);
        bw = 32u - (uint32_t)__clz((int)(nw + ccap));
        bo = min(64u - bx - bw, min(bocap, 31u));
    }
    __device__ __forceinline__ uint64_t pack(uint32_t x, uint32_t w, uint32_t o) const {
        return ((uint64_t)x << (bw + bo)) | ((uint64_t)w << bo) | o;
    }
    __device__ __forceinline__ uint32_t x(uint64_t r) const { return (uint32_t)(r >> (bw + bo)); }
    __device__ __forceinline__ uint32_t w(uint64_t r) const { return (uint32_t)(r >> bo) & ((1u << bw) - 1u); }
    __device__ __forceinline__ uint32_t o(uint64_t r) const { return (uint32_t)r & ((1u << bo) - 1u); }
};

// ---------------------------------------------------------------- values --
// Unweighted levels carry a link count; weighted levels carry (count, sum).
// A result is a record whose list has been followed to its end, so an element
// that composes its record with a solved one is solved itself.
template <bool W> struct Lay;

template <> struct Lay<false> {
    struct Val { uint32_t c; };
    struct alignas(8) Slot { uint32_t w, c; };
    struct alignas(8) Rec { uint32_t nxt, c; };       // level element / walk end
    using Res = Rec;                                  // solved: nxt = TERM | terminal id, c = rank
    static __device__ __forceinline__ Val zero() { return {0u}; }
    static __device__ __forceinline__ Val one_link(int64_t) { return {1u}; }
    static __device__ __forceinline__ Val add(Val a, Val b) { return {a.c + b.c}; }
    static __device__ __forceinline__ Val sub(Val a, Val b) { return {a.c - b.c}; }
    static __device__ __forceinline__ Slot slot(uint32_t w, Val v) { return {w, v.c}; }
    static __device__ __forceinline__ Val val(Slot s) { return {s.c}; }
    static __device__ __forceinline__ Rec rec(uint32_t nxt, Val v) { return {nxt, v.c}; }
    static __device__ __forceinline__ Val val(Rec r) { return {r.c}; }
    static __device__ __forceinline__ Res res(Val v, uint32_t root) { return {TERM | root, v.c}; }
    static __device__ __forceinline__ uint32_t root(Res r) { return r.nxt & IDX; }
    static __device__ __forceinline__ Val junk() { return {NONE}; }
};

template <> struct Lay<true> {
    struct Val { uint32_t c; int64_t s; };
    struct alignas(16) Slot { uint32_t w, c; int64_t s; };
    struct alignas(16) Rec { uint32_t nxt, c; int64_t s; };
    using Res = Rec;
    static __device__ __forceinline__ Val zero() { return {0u, 0}; }
    static __device__ __forceinline__ Val one_link(int64_t w) { return {1u, w}; }
    static __device__ __forceinline__ Val add(Val a, Val b) { return {a.c + b.c, a.s + b.s}; }
    static __device__ __forceinline__ Val sub(Val a, Val b) { return {a.c - b.c, a.s - b.s}; }
    static __device__ __forceinline__ Slot slot(uint32_t w, Val v) { return {w, v.c, v.s}; }
    static __device__ __forceinline__ Val val(Slot s) { return {s.c, s.s}; }
    static __device__ __forceinline__ Rec rec(uint32_t nxt, Val v) { return {nxt, v.c, v.s}; }
    static __device__ __forceinline__ Val val(Rec r) { return {r.c, r.s}; }
    static __device__ __forceinline__ Res res(Val v, uint32_t root) { return {TERM | root, v.c, v.s}; }
    static __device__ __forceinline__ uint32_t root(Res r) { return r.nxt & IDX; }
    static __device__ __forceinline__ Val junk() { return {NONE, INT64_MIN}; }
};

// ------------------------------------------------------------ sampling --
// Ruler sampling by strata: level l cuts its index range into blocks of
// k = 2^log2k consecutive ids and makes exactly one element of every block a
// ruler, at a position drawn by a hash of (level seed, block). This is the
// per-PE quota of Section 2.1 (r/p rulers drawn locally) taken down to blocks
// of k ids, so the ruler count of every level is exactly ceil(m / k), known
// before the data is read, and the ruler of block c has compact id c.
// Hash: "lowbias32" integer finaliser (C. Wellons, hash-prospector).
__device__ __forceinline__ uint32_t hash32(uint32_t seed, uint32_t x) {
    uint32_t h = (x * 0x9e3779b9u) ^ seed;
    h ^= h >> 16;
    h *= 0x7feb352du;
    h ^= h >> 15;
    h *= 0x846ca68bu;
    h ^= h >> 16;
    return h;
}

struct Sampler {
    uint32_t m, log2k, seed;
    __device__ __forceinline__ uint32_t pos(uint32_t blk) const {
        const uint32_t base = blk << log2k;
        const uint32_t k = 1u << log2k;
        const uint32_t len = (m - base < k) ? (m - base) : k;
        const uint32_t h = hash32(seed, blk);
        return (len == k) ? (h & (k - 1u)) : (h % len);
    }
    __device__ __forceinline__ bool sampled(uint32_t y) const {
        const uint32_t blk = y >> log2k;
        return (y - (blk << log2k)) == pos(blk);
    }
    __device__ __forceinline__ uint32_t start(uint32_t c) const { return (c << log2k) + pos(c); }
};

// --------------------------------------------------------------- sources --
// A source yields, for element x of a level, its successor (TERM | terminal
// id when x is a terminal) and its value: the link weight for a non-terminal,
// the terminal's own weight for a terminal (0 on the input level).
// Out-of-range successors are read as terminals, so no walk leaves the array.
// fetch only reads, decode tells what was read: work between the two does not
// wait for the read.
template <bool W, int WT>  // WT: 0 = every link weighs 1, 1 = int32, 2 = int64, 3 = int8 weights (internal)
struct SrcIn {
    const uint32_t* succ;
    const void* weight;
    uint32_t m;
    using L = Lay<W>;
    __device__ __forceinline__ const SrcIn& bind(uint32_t) const { return *this; }
    static constexpr bool kLinks = true;  // every record is one link: a walk's count is its step count
    struct Raw { uint32_t s; std::conditional_t<WT == 2, int64_t, int32_t> w; };
    __device__ __forceinline__ Raw fetch(uint32_t x) const {
        Raw r;
        r.s = succ[x];
        r.w = 1;
        if constexpr (WT == 1) r.w = static_cast<const int32_t*>(weight)[x];
        if constexpr (WT == 3) r.w = static_cast<const int8_t*>(weight)[x];
        if constexpr (WT == 2) r.w = static_cast<const int64_t*>(weight)[x];
        return r;
    }
    __device__ __forceinline__ void decode(uint32_t x, const Raw& r, uint32_t& nxt, typename L::Val& v) const {
        const bool t = (r.s == x) | (r.s >= m);
        nxt = t ? (TERM | x) : r.s;
        v = t ? L::zero() : L::one_link((int64_t)r.w);
    }
    __device__ __forceinline__ void load(uint32_t x, uint32_t& nxt, typename L::Val& v) const {
        decode(x, fetch(x), nxt, v);
    }
};

// The input's successor and weight interleaved into one record, so a chase
// step gathers one line instead of two (int32 weights: 8 B, int64: 16 B).
template <int WT> struct PairRec;
template <> struct alignas(8) PairRec<1> { uint32_t s; int32_t w; };
template <> struct alignas(16) PairRec<2> { uint32_t s, pad; int64_t w; };
template <> struct alignas(8) PairRec<3> { uint32_t s; int32_t w; };  // int8 weights, widened

template <int WT>
struct SrcPair {
    const PairRec<WT>* r;
    uint32_t m;
    using L = Lay<true>;
    __device__ __forceinline__ const SrcPair& bind(uint32_t) const { return *this; }
    static constexpr bool kLinks = true;
    using Raw = PairRec<WT>;
    __device__ __forceinline__ Raw fetch(uint32_t x) const { return r[x]; }
    __device__ __forceinline__ void decode(uint32_t x, const Raw& p, uint32_t& nxt, typename L::Val& v) const {
        const bool t = (p.s == x) | (p.s >= m);
        nxt = t ? (TERM | x) : p.s;
        v = t ? L::zero() : L::one_link((int64_t)p.w);
    }
    __device__ __forceinline__ void load(uint32_t x, uint32_t& nxt, typename L::Val& v) const {
        decode(x, fetch(x), nxt, v);
    }
};

template <bool W>
struct SrcLvl {
    const typename Lay<W>::Rec* e;
    uint32_t m;
    using L = Lay<W>;
    __device__ __forceinline__ const SrcLvl& bind(uint32_t) const { return *this; }
    static constexpr bool kLinks = false;  // records are segments: counts exceed step counts
    using Raw = typename L::Rec;
    __device__ __forceinline__ Raw fetch(uint32_t x) const { return e[x]; }
    __device__ __forceinline__ void decode(uint32_t, const Raw& r, uint32_t& nxt, typename L::Val& v) const {
        nxt = r.nxt;
        v = L::val(r);
        if (!(nxt & TERM) && nxt >= m) { nxt = TERM | IDX; v = L::zero(); }
    }
    __device__ __forceinline__ void load(uint32_t x, uint32_t& nxt, typename L::Val& v) const {
        decode(x, fetch(x), nxt, v);
    }
};

// --------------------------------------------------------------- outputs --
// Outputs take (element, value, root). A cursor lets an output keep state
// between consecutive elements of one lane (the batch output walks its
// request table forward instead of searching it per element).
// The caller's outputs. RK / RT say at compile time whether rank and root are
// written (the ranking kernels are instantiated per combination, so their
// store loops carry no branches); DYN checks the pointers at run time instead.
template <bool W, bool RK = true, bool RT = true, bool DYN = false>
struct OutUser {
    uint32_t* rank;
    uint32_t* root;
    int64_t* sum;
    using L = Lay<W>;
    struct Cur {};
    __device__ __forceinline__ Cur begin(uint32_t) const { return {}; }
    __device__ __forceinline__ void store(Cur&, uint32_t i, typename L::Val v, uint32_t r) const {
        if constexpr (DYN) {
            if (rank) rank[i] = v.c;
            if (root) root[i] = r;
            if constexpr (W) { if (sum) sum[i] = v.s; }
        } else {
            if constexpr (RK) rank[i] = v.c;
            if constexpr (RT) root[i] = r;
            if constexpr (W) sum[i] = v.s;
        }
    }
};

template <bool W>
struct OutLvl {
    typename Lay<W>::Res* e;
    using L = Lay<W>;
    struct Cur {};
    __device__ __forceinline__ Cur begin(uint32_t) const { return {}; }
    __device__ __forceinline__ void store(Cur&, uint32_t i, typename L::Val v, uint32_t r) const {
        e[i] = L::res(v, r);
    }
};

// Batch request table in device memory: bases[q] is the first global id of
// request q, bases[count] the total. The table is written on the device from
// descriptors passed by value as kernel arguments (no host staging, nothing
// for a graph replay to read from host memory); the header holds the sizes.
struct BatchDesc {
    const uint32_t* succ;
    uint32_t* rank;
    uint32_t* root;
    uint64_t n;
};
struct BatchHdr {
    uint32_t count;    // requests
    uint32_t nchunks;  // BATCH_CHUNK-id chunks over all requests (none crosses a request)
    uint32_t total;    // elements (= bases[count])
    uint32_t pad;
};

__device__ __forceinline__ uint32_t batch_find(const uint32_t* bases, uint32_t count, uint32_t g) {
    uint32_t lo = 0, hi = count;  // invariant: bases[lo] <= g < bases[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (bases[mid] <= g) lo = mid; else hi = mid;
    }
    return lo;
}

// A batch's requests as one source over the concatenated ids, without copying
// them together: bind finds the request of an element, whose list never leaves
// it.
struct SrcBatch {
    const BatchDesc* d;
    const uint32_t* bases;
    const BatchHdr* hdr;
    uint32_t m;
    struct Req {
        const uint32_t* succ;
        uint32_t lo, n;
        __device__ __forceinline__ void load(uint32_t x, uint32_t& nxt, Lay<false>::Val& v) const {
            const uint32_t s = succ[x - lo];
            const bool t = (s == x - lo) | (s >= n);
            nxt = t ? (TERM | x) : lo + s;
            v.c = t ? 0u : 1u;
        }
    };
    __device__ __forceinline__ Req bind(uint32_t x) const {
        const uint32_t q = batch_find(bases, hdr->count, x);
        const uint32_t lo = bases[q];
        return {d[q].succ, lo, bases[q + 1] - lo};
    }
};

struct OutBatch {
    const BatchDesc* d;
    const uint32_t* bases;
    const BatchHdr* hdr;
    using L = Lay<false>;
    // the request holding the current element, with its output arrays
    struct Cur { uint32_t q, lo, hi, count; uint32_t* rank; uint32_t* root; };
    __device__ __forceinline__ Cur begin(uint32_t g) const {
        const uint32_t count = hdr->count;
        const uint32_t q = batch_find(bases, count, g);
        return {q, bases[q], bases[q + 1], count, d[q].rank, d[q].root};
    }
    __device__ __forceinline__ void store(Cur& c, uint32_t g, L::Val v, uint32_t r) const {
        if (g >= c.hi && c.q + 1 < c.count) {
            while (g >= c.hi && c.q + 1 < c.count) { c.q++; c.lo = c.hi; c.hi = bases[c.q + 1]; }
            c.rank = d[c.q].rank;
            c.root = d[c.q].root;
        }
        if (g >= c.hi) return;  // past the last request (cannot happen for ids below the total)
        const uint32_t l = g - c.lo;
        c.rank[l] = v.c;
        if (c.root) c.root[l] = r - c.lo;
    }
};

// ------------------------------------------------------------ wave utils --
__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

__device__ __forceinline__ uint32_t mbcnt(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// Exclusive block scan (all lanes get their prefix; *total = block sum).
__device__ __forceinline__ uint32_t block_exscan(uint32_t v, uint32_t* sh, uint32_t* total) {
    const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o);
        if (lane >= (uint32_t)o) inc += y;
    }
    if (lane == 63) sh[wv] = inc;
    __syncthreads();
    uint32_t before = 0, all = 0;
    const uint32_t nw = blockDim.x / 64;
    for (uint32_t i = 0; i < nw; ++i) {
        const uint32_t s = sh[i];
        if (i < wv) before += s;
        all += s;
    }
    *total = all;
    return before + inc - v;
}

// In-place exclusive scan of a[0, n) by one workgroup of 1024 lanes; returns
// the total to every lane. Each lane owns a contiguous run of a multiple of 4
// entries, read and written as 16-byte vectors, so both passes issue all of a
// lane's loads at once (a must be 16-byte aligned).
__device__ __forceinline__ uint32_t wg_exscan_inplace(uint32_t* __restrict__ a, uint32_t n, uint32_t* sh) {
    const uint32_t per = (((n + blockDim.x - 1u) / blockDim.x) + 3u) & ~3u;
    const uint32_t lo = min(threadIdx.x * per, n);
    const uint32_t hi = min(lo + per, n);
    const uint32_t nv = (hi - lo) >> 2;  // whole vectors; the rest one by one
    uint4* av = reinterpret_cast<uint4*>(a + lo);
    uint32_t s = 0;
    for (uint32_t k = 0; k < nv; ++k) {
        const uint4 v = av[k];
        s += v.x + v.y + v.z + v.w;
    }
    for (uint32_t i = lo + 4 * nv; i < hi; ++i) s += a[i];
    uint32_t total;
    uint32_t run = block_exscan(s, sh, &total);
    for (uint32_t k = 0; k < nv; ++k) {
        const uint4 v = av[k];
        uint4 o;
        o.x = run;
        o.y = o.x + v.x;
        o.z = o.y + v.y;
        o.w = o.z + v.z;
        run = o.w + v.w;
        av[k] = o;
    }
    for (uint32_t i = lo + 4 * nv; i < hi; ++i) {
        const uint32_t v = a[i];
        a[i] = run;
        run += v;
    }
    return total;
}

// 32 mark bytes (0 or 1, two vectors in id order) -> 32 bits.
__device__ __forceinline__ uint32_t mark_bits(uint4 a, uint4 b) {
    const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t bits = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) bits |= ((w[k] * 0x10204080u) >> 28) << (4 * k);  // the four bytes' low bits
    return bits;
}

}  // namespace lr
