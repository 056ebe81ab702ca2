// Device preprocessing: clean, orient and lay out the graph, then bin its vertices.
//
//  1. canonicalise: each sample (a, b) becomes the key (min << nb) | max;
//     self-loops and out-of-range ids become a sentinel that sorts last
//     (cleaning rules of the paper, Section 2.6: duplicates and self-loops
//     removed, directed pairs read as undirected); single graphs form the
//     keys as the first sort pass reads its input;
//  2. radix passes (tc_sort.h) over the top bits of the keys: all but at most 16 low bits of the upper
//     id, so that equal keys meet in groups of equal top bits; k_dedup and, for groups of many tiles,
//     k_dedup_long find the first of each distinct key in its group (a bit per sample; duplicates stay in
//     place and are skipped downstream) and count the degrees of the lower ids (runs of equal ids);
//  3. degrees of the upper ids: one partition pass by their top bits, then counters in LDS (k_upper_count);
//     the rank in (degree, id) order from a radix sort of (degree, id);
//  4. orientation by rank-by-degree (Section 2.2): the edge runs from the
//     lower-ranked to the higher-ranked endpoint, and every id is replaced by
//     its rank, so out-neighbour lists hold ranks and hashing the low bits of
//     a rank spreads neighbours of similar degree over consecutive buckets
//     (the reordering idea of Section 4.1; other orders are optional);
//  5. CSR: radix passes of the oriented keys by row; lists and offsets from the runs of equal rows.  A list's
//     order is unspecified and differs between builds of the same samples (the keys of a group are in no
//     order, and the first row pass and the partition by upper id do not keep any); the rows that
//     global-memory tables probe are put in rank order (k_sort_rows);
//  5c (optional): the record layout: rank r's record at p(r) holds d+(r) and then the record id
//     rec_id(p(v)) of each out-neighbour v; records go in rank order, a short one moved to the next
//     128-byte line where it would straddle one (placed first, written by k_work, which reads d+(v)
//     anyway);
//  6. scheduling (Section 4.3): out-degree d+ and collective work
//     W(u) = sum of d+(v) over out-neighbours v (the collective degree of
//     Equation 2); vertices with d+ < 2 or W = 0 are skipped, the rest go by
//     d+ to a global-memory-table bin, a large-LDS bin, a workgroup bin, a
//     wavefront bin or (light vertices, when they dominate) a packed bin, and
//     each bin is ordered by decreasing W (largest work first);
//  7. the core path's block words and the schedule of the lists cut before the core (tc_core.hip).
//
// Every histogram of digits is counted by the kernel that makes the keys, and a pass forms its keys as it
// loads them, so the sorts add nothing but their passes.
#include <algorithm>
#include <cstring>

#include <rocprim/rocprim.hpp>

#include "tc_internal.h"
#include "tc_sort.h"

namespace tc {
namespace {

constexpr int kThreads = 256;

inline uint32_t grid_for(uint64_t items) {
    uint64_t g = (items + kThreads - 1) / kThreads;
    if (g > 65536) g = 65536;
    if (g == 0) g = 1;
    return (uint32_t)g;
}

inline uint32_t id_bits(uint32_t n) {  // bits to hold any id < n (at least 1)
    uint32_t b = 1;
    while (b < 32 && (1ull << b) < (uint64_t)n) ++b;
    return b;
}

// Bits of any vertex degree: at most min(n - 1, 2 m_in).
uint32_t degree_bits(uint32_t n, uint64_t m_in) {
    const uint64_t dmax = (uint64_t)n - 1 < 2 * m_in ? (uint64_t)n - 1 : 2 * m_in;
    uint32_t b = 1;
    while (b < 32 && (1ull << b) <= dmax) ++b;
    return b;
}

// Canonical keys: passes over all but at most kGroupBits low bits (k_dedup tells the keys of a group of
// equal top bits apart by those): R-MAT 22 takes four passes instead of five, 2^25 ids four instead of six.
constexpr uint32_t kGroupBits = 16;
inline uint32_t canon_passes(uint32_t nb) {
    const uint32_t bits = 2 * nb > kGroupBits ? 2 * nb - kGroupBits : 1;
    return (bits + kDigit - 1) / kDigit;
}
inline uint32_t canon_low(uint32_t nb) {  // low bits that the passes leave out
    const uint32_t bits = canon_passes(nb) * kDigit;
    return 2 * nb > bits ? 2 * nb - bits : 0;
}
inline uint32_t row_passes(uint32_t nb) { return (nb + kDigit - 1) / kDigit; }

// Upper ids: partitioned by their top bits (a digit of 9 or 10 bits) so that a partition's counters,
// 2^15 at most at a time, fit in LDS.  No partition up to 15 bits; from 28 bits on one atomic per edge.
constexpr uint32_t kCounterBits = 15;
inline uint32_t upper_digit(uint32_t nb) { return nb <= kCounterBits ? 0u : nb <= 24 ? 9u : nb <= 27 ? 10u : 0u; }
inline bool upper_atomics(uint32_t nb) { return nb > 27; }

// Orientation.  The rank of an edge's lower id comes with the sorted order; the upper id's is a gather from
// anywhere, 128 bytes moved for 4 (2^25 vertices, 537 M edges: 10.7 ms of 66).  From 2^21 vertices on the
// edges take one more pass, partitioned by upper id with the lower id's rank in place, and the gather goes to
// a partition's ranks in LDS: 5.2 ms.  Whole one-shot counts without / with it, 8 samples a vertex, ids at
// random: 3 M vertices 3.10 / 3.04 ms, 2^22 3.98 / 3.80, 2^23 7.92 / 7.36, 2^25 32.4 / 29.5; R-MAT (16 samples),
// whose hubs' ranks stay in the caches: 2^22 12.49 / 12.51, 2^23 29.00 / 29.09, 2^24 72.0 / 71.3.  Up to 25
// bits (2^15 ranks per partition: the LDS); not for batches, whose gathers stay within a small graph.
inline bool attach_ranks(uint32_t nb) { return nb >= 22 && nb <= 25; }
// Its ranks and the counters of the rows' top digit (three row passes).
inline uint32_t orient_lds(uint32_t nb) { return (4u << (nb - upper_digit(nb))) + (64u << (nb - 2 * kDigit)); }

// Digit histograms of the build's passes (512 words each; the upper ids' has 1024) and their tickets.
constexpr uint32_t kMaxPasses = 6 + 4 + 4 + 2;
constexpr uint32_t kHistWords = kMaxPasses * 512 + 1024 + 2 * kRestClasses;
constexpr uint32_t kTicketWords = 64;

// Canonical key of sample i (a self-loop or out-of-range id gives the sentinel).
struct CanonKey {
    typedef uint2 Raw;
    const uint32_t* src;
    const uint32_t* dst;
    uint32_t n, nb;
    unsigned long long sentinel;
    __device__ Raw raw(uint64_t i) const { return make_uint2(src[i], dst[i]); }
    __device__ bool make(Raw r, uint32_t, unsigned long long& key) const {
        const uint32_t lo = r.x < r.y ? r.x : r.y, hi = r.x < r.y ? r.y : r.x;
        key = (hi >= n || lo == hi) ? sentinel : ((unsigned long long)lo << nb) | hi;
        return true;
    }
};

struct LoadKey {
    typedef unsigned long long Raw;
    const unsigned long long* keys;
    __device__ Raw raw(uint64_t i) const { return keys[i]; }
    __device__ bool make(Raw r, uint32_t, unsigned long long& key) const {
        key = r;
        return true;
    }
};

struct StoreKey {
    unsigned long long* keys;
    __device__ void operator()(uint64_t i, unsigned long long key) const { keys[i] = key; }
};

// Distinct edges are marked by one bit per sample of the sorted keys.
__device__ __forceinline__ bool is_first(const unsigned long long* first, uint64_t i) {
    return (first[i >> 6] >> (i & 63u)) & 1ull;
}

struct KeyBits {
    unsigned long long key, bits;
};
struct LoadFirst {  // the distinct edges' keys (sorted or, at the same places, oriented)
    typedef KeyBits Raw;
    const unsigned long long* keys;
    const unsigned long long* first;
    __device__ Raw raw(uint64_t i) const { return {keys[i], first[i >> 6]}; }
    __device__ bool make(const Raw& r, uint32_t lane, unsigned long long& key) const {
        key = r.key;
        return (r.bits >> lane) & 1ull;
    }
};

struct LoadRanked {  // the same with the lower id's rank in place of the lower id
    typedef KeyBits Raw;
    const unsigned long long* keys;
    const unsigned long long* first;
    const uint32_t* rank;
    uint32_t n, nb;
    unsigned long long mask;
    __device__ Raw raw(uint64_t i) const { return {keys[i], first[i >> 6]}; }
    __device__ bool make(const Raw& r, uint32_t lane, unsigned long long& key) const {
        const bool on = (r.bits >> lane) & 1ull;
        const uint32_t lo = (uint32_t)(r.key >> nb);  // (past the last sample a lane has another's bit: any key)
        key = ((unsigned long long)rank[on && lo < n ? lo : 0u] << nb) | (r.key & mask);
        return on;
    }
};

struct LoadUpper {  // their upper ids
    typedef KeyBits Raw;
    const unsigned long long* keys;
    const unsigned long long* first;
    unsigned long long mask;
    __device__ Raw raw(uint64_t i) const { return {keys[i], first[i >> 6]}; }
    __device__ bool make(const Raw& r, uint32_t lane, uint32_t& id) const {
        id = (uint32_t)(r.key & mask);
        return (r.bits >> lane) & 1ull;
    }
};

struct StoreId {
    uint32_t* ids;
    __device__ void operator()(uint64_t i, uint32_t id) const { ids[i] = id; }
};

// Vertices by degree: elements degree << 32 | id; the last pass also writes the inverse (rank of every
// id) and, in a batch, the graph of every rank.
struct LoadDegree {
    typedef unsigned long long Raw;
    const uint32_t* deg;
    __device__ Raw raw(uint64_t i) const { return ((unsigned long long)deg[i] << 32) | (uint32_t)i; }
    __device__ bool make(Raw r, uint32_t, unsigned long long& e) const {
        e = r;
        return true;
    }
};
__device__ __forceinline__ uint32_t owner(const unsigned long long* off, uint32_t k, unsigned long long x);
struct StoreRank {
    unsigned long long* order;
    uint32_t* rank;
    const unsigned long long* voff;
    uint32_t k;
    uint32_t* gid;
    __device__ void operator()(uint64_t r, unsigned long long e) const;
};

struct StoreItem {  // schedule elements: key << 32 | rank
    uint32_t* items;
    __device__ void operator()(uint64_t i, unsigned long long e) const { items[i] = (uint32_t)e; }
};

// Record placement (kPlaceChunk ranks per thread, in rank order): the start of a record of s words
// at cursor c, moved to the next 32-word line boundary when s <= 32 and the record would straddle one.
__device__ __forceinline__ uint32_t place_at(uint32_t c, uint32_t s) {
    return (s <= 32u && (c & 31u) + s > 32u) ? ((c + 31u) & ~31u) : c;
}

// Words of each chunk of records, rounded up to a line (chunks start on line boundaries); entry
// `chunks` is 0, so that an exclusive scan gives the chunk bases and, last, the extent.
__global__ void k_place_size(const uint32_t* __restrict__ off32, uint32_t n, unsigned long long* __restrict__ csz) {
    const uint32_t chunks = (uint32_t)place_chunks(n);
    for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c <= chunks; c += gridDim.x * blockDim.x) {
        if (c == chunks) { csz[c] = 0; continue; }
        const uint32_t r0 = c * kPlaceChunk, r1 = r0 + kPlaceChunk < n ? r0 + kPlaceChunk : n;
        uint32_t cur = 0;
        for (uint32_t r = r0; r < r1; ++r) {
            const uint32_t sz = off32[r + 1] - off32[r] + 1u;
            cur = place_at(cur, sz) + sz;
        }
        csz[c] = (cur + 31u) & ~31u;
    }
}

// {p(r), d+(r)} of every rank from the chunk bases; entry n gets {extent, 0}.
__global__ void k_place_write(const uint32_t* __restrict__ off32, uint32_t n,
                              const unsigned long long* __restrict__ cbase, uint2* __restrict__ place) {
    const uint32_t chunks = (uint32_t)place_chunks(n);
    for (uint32_t c = blockIdx.x * blockDim.x + threadIdx.x; c <= chunks; c += gridDim.x * blockDim.x) {
        if (c == chunks) { place[n] = make_uint2((uint32_t)cbase[chunks], 0u); continue; }
        const uint32_t r0 = c * kPlaceChunk, r1 = r0 + kPlaceChunk < n ? r0 + kPlaceChunk : n;
        uint32_t cur = (uint32_t)cbase[c];
        for (uint32_t r = r0; r < r1; ++r) {
            const uint32_t d = off32[r + 1] - off32[r];
            cur = place_at(cur, d + 1u);
            place[r] = make_uint2(cur, d);
            cur += d + 1u;
        }
    }
}

// Zeroes the record layout's per-vertex staging where the count adds to it: at every record's start
// (the ids the count handles are record ids), in rank order.
__global__ void k_clear_record_starts(unsigned long long* __restrict__ tv, const uint32_t* __restrict__ place,
                                      uint32_t n) {
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x)
        tv[rec_id(place[2 * (uint64_t)r])] = 0ull;
}

// The CSR offsets narrowed to 32 bits for the count kernels (m_in < 2^31): at 2^25 vertices the
// 64-bit array (268 MB) no longer fits the Infinity Cache, the 32-bit one (134 MB) does.
__global__ void k_narrow(const int64_t* __restrict__ off, uint64_t n1, uint32_t* __restrict__ off32) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n1; i += (uint64_t)gridDim.x * blockDim.x)
        off32[i] = (uint32_t)off[i];
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v, size_t words) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < words; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_clear_ranges(Ranges r) {
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
#pragma unroll
    for (int q = 0; q < 3; ++q)
        if (r.p[q])
            for (size_t i = t; i < r.words[q]; i += step) r.p[q][i] = 0;
}

// Largest g in [0, k) with off[g] <= x (off is non-decreasing, off[0] = 0).
__device__ __forceinline__ uint32_t owner(const unsigned long long* off, uint32_t k, unsigned long long x) {
    uint32_t lo = 0, hi = k - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (off[mid] <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__device__ void StoreRank::operator()(uint64_t r, unsigned long long e) const {
    order[r] = e;
    rank[(uint32_t)e] = (uint32_t)r;
    if (gid) gid[r] = owner(voff, k, (uint32_t)e);
}

constexpr uint32_t kMaxCanonPasses = 6;

// Digit histograms of the canonical keys of a single graph; an out-of-range id raises the range error.
__global__ void __launch_bounds__(1024) k_canon_hist(CanonKey canon, uint64_t m_in, uint32_t low, uint32_t passes,
                                                     uint32_t* __restrict__ hist, GraphMeta* meta) {
    __shared__ uint32_t s_h[kMaxCanonPasses][512];
    for (uint32_t i = threadIdx.x; i < passes * 512; i += blockDim.x) (&s_h[0][0])[i] = 0;
    __syncthreads();
    uint32_t bad = 0;
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < m_in; base += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = base + threadIdx.x;
        const bool act = i < m_in;
        unsigned long long key = 0;
        if (act) {
            const uint2 s = canon.raw(i);
            canon.make(s, 0, key);
            if (s.x >= canon.n || s.y >= canon.n) bad = 1;
        }
        for (uint32_t p = 0; p < passes; ++p) count_digit(s_h[p], (uint32_t)(key >> (low + kDigit * p)) & 511u, act);
    }
    if (bad) atomicOr(&meta->err, 1u);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < passes * 512; i += blockDim.x)
        if (const uint32_t c = (&s_h[0][0])[i]) atomicAdd(&hist[i], c);
}

// Batch form: sample e belongs to graph g with eoff[g] <= e < eoff[g+1]; its
// local ids are shifted by voff[g].  Local ids >= n_g, and union ids >= n
// (malformed offsets), are range errors.  Writes the keys and their digit histograms.
__global__ void __launch_bounds__(1024) k_canon_batch(const uint32_t* __restrict__ src,
                                                      const uint32_t* __restrict__ dst, uint64_t m_in, uint32_t n,
                                                      uint32_t nb, unsigned long long sentinel,
                                                      const unsigned long long* __restrict__ voff,
                                                      const unsigned long long* __restrict__ eoff, uint32_t k,
                                                      uint32_t low, uint32_t passes,
                                                      unsigned long long* __restrict__ keys,
                                                      uint32_t* __restrict__ hist, GraphMeta* meta) {
    __shared__ uint32_t s_h[kMaxCanonPasses][512];
    for (uint32_t i = threadIdx.x; i < passes * 512; i += blockDim.x) (&s_h[0][0])[i] = 0;
    uint32_t bad = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0 &&
        (voff[0] != 0 || eoff[0] != 0 || voff[k] != n || eoff[k] != m_in))
        bad = 1;
    // The graph of sample i: one binary search per block and step (its first sample), then each
    // thread moves forward over the few graphs a run of blockDim samples can span.
    __shared__ uint32_t s_g;
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < m_in; base += (uint64_t)gridDim.x * blockDim.x) {
        if (threadIdx.x == 0) s_g = owner(eoff, k, base);
        __syncthreads();
        const uint64_t i = base + threadIdx.x;
        uint32_t g = s_g;
        __syncthreads();
        const bool act = i < m_in;
        unsigned long long key = sentinel;
        if (act) {
            while (g + 1 < k && eoff[g + 1] <= i) ++g;
            const unsigned long long v0 = voff[g], ng = voff[g + 1] - v0;
            const unsigned long long a = (unsigned long long)src[i] + v0, b = (unsigned long long)dst[i] + v0;
            if (src[i] >= ng || dst[i] >= ng || a >= n || b >= n) bad = 1;
            else if (a != b) {
                const unsigned long long lo = a < b ? a : b, hi = a < b ? b : a;
                key = (lo << nb) | hi;
            }
            keys[i] = key;
        }
        for (uint32_t p = 0; p < passes; ++p) count_digit(s_h[p], (uint32_t)(key >> (low + kDigit * p)) & 511u, act);
    }
    if (bad) atomicOr(&meta->err, 1u);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < passes * 512; i += blockDim.x)
        if (const uint32_t c = (&s_h[0][0])[i]) atomicAdd(&hist[i], c);
}

// Distinct edges.  The keys are sorted by all but their `low` lowest bits; the keys of a group (equal top
// bits) come in any order.  The first of each distinct key gets its bit in `first` (cleared beforehand).
// k_dedup: a workgroup handles the groups that start in its tile of kDedupTile keys, other than long ones: the
// keys of groups of one are first by themselves, the others go into an LDS hash set (group number in the
// tile << low | low bits: 28 bits name a key exactly), and the group that runs on into the next tiles is
// read to its end with a bit set over its low bits (words of `first` that two tiles share are ORed).
// k_dedup_long: long groups hold the first keys of kLongTiles tiles or more (dense neighbourhoods, samples
// that repeat), and every tile marks its own keys of them: a bit set over the low bits in LDS, merged word
// by word into the group's bit set in memory (`bits`, cleared beforehand); what the merge finds clear is
// first.  The first boundary of tiles in the group names its set: those of long groups are at least
// kLongTiles apart.  (One workgroup reading every group to its end took 25 ms for 2^24 samples of one pair, whole
// calls of 0.5 to 0.9 ms now, and 0.65 ms for the 4 M edges between 2000 and 2000 vertices, calls of 0.41.)
//
// Its lower id gets one degree: a wavefront walks 256 consecutive keys 64 at a time; equal lower ids are
// contiguous lanes (groups, found by ballot), the last lane of each group adds the group's distinct
// edges, and the group reaching the wavefront's last lane carries over to the next step, so a long run (a
// hub's row) costs one atomic per 256 keys.  Upper ids: their digit histogram for the partition pass, or
// (atomics) one degree atomic each.  m = the number of distinct edges.
constexpr uint32_t kDedupThreads = 1024, kDedupItems = 4, kDedupTile = kDedupThreads * kDedupItems;
constexpr uint32_t kDedupSlots = 2 * kDedupTile;  // 2^13
constexpr uint32_t kDedupWords = kDedupTile / 64;
constexpr uint32_t kLongTiles = 4;

// Words of a long group's bit set, and of those that m_in samples can need.
__host__ __device__ inline uint32_t long_words(uint32_t low) { return low > 5 ? 1u << (low - 5) : 1u; }
inline uint64_t long_set_words(uint32_t low, uint64_t m_in) {
    return (uint64_t)long_words(low) * ((m_in + kDedupTile - 1) / kDedupTile / kLongTiles + 1);
}

struct Dedup {
    const unsigned long long* keys;
    uint64_t cap;
    unsigned long long sentinel;
    unsigned long long* first;
    uint32_t* bits;
    uint32_t* deg;
    uint32_t* uhist;
    GraphMeta* meta;
    uint32_t* any_long;  // set when there is a long group
    uint32_t nb, low, ubins, ushift;
    bool uatomics;
};

// Degrees and the upper digit histogram of a tile's distinct edges: k its keys, s_first their bits.
__device__ __forceinline__ void count_firsts(const Dedup& a, const unsigned long long (&k)[kDedupItems],
                                             const unsigned long long* s_first, uint32_t* s_hist, uint32_t wave,
                                             uint32_t lane) {
    const unsigned long long mask = (a.nb >= 32) ? 0xFFFFFFFFull : ((1ull << a.nb) - 1);
    const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1);  // lanes 0..lane
    uint32_t clo = 0xFFFFFFFFu, cc = 0;  // carried group (uniform)
#pragma unroll
    for (int i = 0; i < (int)kDedupItems; ++i) {
        const unsigned long long F = s_first[wave * kDedupItems + i];
        const uint32_t lo = (uint32_t)(k[i] >> a.nb);
        const bool mine = (F >> lane) & 1ull;
        if (mine) {
            const uint32_t hi = (uint32_t)(k[i] & mask);
            if (a.ubins) atomicAdd(&s_hist[hi >> a.ushift], 1u);
            if (a.uatomics) atomicAdd(&a.deg[hi], 1u);
        }
        const uint32_t lo_prev = (uint32_t)__shfl_up((int)lo, 1, 64);
        const unsigned long long H = __ballot(lane == 0 || lo != lo_prev);  // group starts
        const uint32_t s = 63u - (uint32_t)__builtin_clzll(H & upto);      // this lane's group start
        const uint32_t c = (uint32_t)__popcll((F & upto) >> s);            // its firsts up to this lane
        const bool merge = __builtin_amdgcn_readfirstlane(lo) == clo;     // first group continues the carry
        const uint32_t tail = 63u - (uint32_t)__builtin_clzll(H);          // start of lane 63's group
        if (lane != 63 && ((H >> (lane + 1)) & 1ull)) {                    // last lane of an inner group
            const uint32_t cnt = c + ((s == 0 && merge) ? cc : 0u);
            if (cnt) atomicAdd(&a.deg[lo], cnt);
        }
        const uint32_t c63 = (uint32_t)__builtin_amdgcn_readlane((int)c, 63);
        const uint32_t lo63 = (uint32_t)__builtin_amdgcn_readlane((int)lo, 63);
        if (tail == 0 && merge) {
            cc += c63;
        } else {
            if (!merge && cc && lane == 0) atomicAdd(&a.deg[clo], cc);
            clo = lo63;
            cc = c63;
        }
    }
    if (cc && lane == 0) atomicAdd(&a.deg[clo], cc);
}

// A tile's view of long groups, by the groups at its boundary and those of three tiles before and four after (a
// wavefront's lanes 0..7): bit 0, the group of the tile's first key is long; bit 1, that of the next tile's
// first key, and begins in this tile or there.
__device__ __forceinline__ uint32_t long_groups(const Dedup& a, uint64_t base, uint32_t lane) {
    static_assert(kLongTiles == 4, "boundaries looked at");
    const int64_t x = (int64_t)base + ((int64_t)lane - 3) * kDedupTile;
    const bool on = lane < 8 && x >= 0 && x < (int64_t)a.cap;
    const unsigned long long top = on ? a.keys[x] >> a.low : ~0ull;
    // (samples without an edge come last; where the top bits hold the whole lower id their group holds
    // nothing else and is left alone)
    const bool edges = on && (a.low > a.nb || top != a.sentinel >> a.low);
    const uint32_t here = (uint32_t)__ballot(edges && top == __shfl(top, 3, 64));  // consecutive, lane 3 among them
    const uint32_t next = (uint32_t)__ballot(edges && top == __shfl(top, 4, 64));
    return ((uint32_t)__popc(here) >= kLongTiles ? 1u : 0u) | ((next >> 4) == 15u ? 2u : 0u);
}

__global__ void __launch_bounds__(kDedupThreads) __attribute__((amdgpu_waves_per_eu(8))) k_dedup(Dedup a) {
    __shared__ __align__(16) uint32_t s_set[kDedupSlots];  // hash set, then the bits of the crossing group
    __shared__ unsigned long long s_start[kDedupWords], s_first[kDedupWords];
    __shared__ uint32_t s_pre[kDedupWords];
    __shared__ uint32_t s_hist[1024];
    __shared__ unsigned long long s_m;
    const unsigned long long* const keys = a.keys;
    const uint64_t cap = a.cap;
    const unsigned long long sentinel = a.sentinel;
    const uint32_t nb = a.nb, low = a.low;
    constexpr uint32_t kEmptySlot = 0xFFFFFFFFu;
    for (uint32_t i = threadIdx.x; i < a.ubins; i += kDedupThreads) s_hist[i] = 0;
    if (threadIdx.x == 0) s_m = 0;
    unsigned long long found = 0;
    for (uint64_t base = blockIdx.x * (uint64_t)kDedupTile; base < cap; base += (uint64_t)gridDim.x * kDedupTile) {
        // (What follows from the thread's number is worked out anew for every tile: kept across tiles it takes
        // the registers that the tile needs.)
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const uint32_t lane = tid & 63u, wave = tid >> 6;
        const unsigned long long mask = (nb >= 32) ? 0xFFFFFFFFull : ((1ull << nb) - 1);
        const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1);  // lanes 0..lane
        const uint64_t end = base + kDedupTile < cap ? base + kDedupTile : cap;
        unsigned long long k[kDedupItems];
#pragma unroll
        for (int i = 0; i < (int)kDedupItems; ++i) {
            const uint64_t x = base + wave * (64u * kDedupItems) + i * 64u + lane;
            k[i] = x < cap ? keys[x] : ~0ull;
        }
#pragma unroll
        for (int i = 0; i < (int)kDedupItems; ++i) {
            const uint64_t x = base + wave * (64u * kDedupItems) + i * 64u + lane;
            unsigned long long before = ((unsigned long long)(uint32_t)__shfl_up((int)(uint32_t)(k[i] >> 32), 1, 64) << 32) |
                                        (uint32_t)__shfl_up((int)(uint32_t)k[i], 1, 64);
            if (lane == 0 && x > 0 && x < cap) before = keys[x - 1];
            const bool start = x < cap && (x == 0 || (before >> low) != (k[i] >> low));
            const unsigned long long s = __ballot(start);
            if (lane == 0) s_start[wave * kDedupItems + i] = s;
        }
        __syncthreads();
        const unsigned long long starts = lane < kDedupWords ? s_start[lane] : 0ull;
        if (wave == 0) {  // starts before each word, and clear bits
            const uint32_t c = (uint32_t)__popcll(starts);
            const uint32_t pre = wave_incl_scan(c) - c;
            if (lane < kDedupWords) {
                s_pre[lane] = pre;
                s_first[lane] = 0;
            }
        }
        const unsigned long long has = __ballot(starts != 0);  // words with a start
        __syncthreads();
        if (!has) continue;  // uniform: the whole tile belongs to another tile's group
        const uint32_t w0 = (uint32_t)__builtin_ctzll(has), w1 = 63u - (uint32_t)__builtin_clzll(has);
        const uint32_t p0 = w0 * 64u + (uint32_t)__builtin_ctzll(s_start[w0]);         // first start
        const uint32_t p1 = w1 * 64u + 63u - (uint32_t)__builtin_clzll(s_start[w1]);   // last start
        const bool cross = end < cap && (keys[end] >> low) == (keys[end - 1] >> low) &&
                           !(low <= nb && (keys[end] >> low) == (sentinel >> low));
        const uint32_t stop = cross ? p1 : (uint32_t)(end - base);  // keys [p0, stop) are in closed groups
        // groups of one, and whether there are others
        uint32_t many = 0, one = 0;
#pragma unroll
        for (int i = 0; i < (int)kDedupItems; ++i) {
            const uint32_t p = wave * (64u * kDedupItems) + i * 64u + lane;
            if (p < p0 || p >= stop || k[i] == sentinel) continue;
            const bool here = (s_start[p >> 6] >> (p & 63u)) & 1ull;
            const uint32_t q = p + 1;
            const bool next = q == stop || ((s_start[q >> 6] >> (q & 63u)) & 1ull);
            if (here && next) one |= 1u << i;
            else many |= 1u << i;
        }
        if (__syncthreads_or(many != 0)) {
            for (uint32_t i = tid; i < kDedupSlots / 4; i += kDedupThreads)
                reinterpret_cast<uint4*>(s_set)[i] = make_uint4(kEmptySlot, kEmptySlot, kEmptySlot, kEmptySlot);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < (int)kDedupItems; ++i) {
                if (!((many >> i) & 1u)) continue;
                const uint32_t p = wave * (64u * kDedupItems) + i * 64u + lane;
                const uint32_t g = s_pre[p >> 6] + (uint32_t)__popcll(s_start[p >> 6] & upto) - 1u;
                const uint32_t name = (g << low) | ((uint32_t)k[i] & ((1u << low) - 1u));
                uint32_t at = (name * 0x9E3779B1u) >> 19;  // 13 bits: kDedupSlots
                for (;;) {
                    const uint32_t old = atomicCAS(&s_set[at], kEmptySlot, name);
                    if (old == kEmptySlot) one |= 1u << i;
                    if (old == kEmptySlot || old == name) break;
                    at = (at + 1) & (kDedupSlots - 1);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < (int)kDedupItems; ++i) {
            const unsigned long long f = __ballot((one >> i) & 1u);
            if (lane == 0) s_first[wave * kDedupItems + i] = f;
        }
        __syncthreads();
        // (long: the group holds the boundary kLongTiles - 1 past its first one)
        const uint64_t far = base + (p1 ? kLongTiles : kLongTiles - 1) * kDedupTile;
        if (cross && far < cap && (keys[far] >> low) == (keys[end] >> low)) {
            if (tid == 0) *a.any_long = 1;
        } else if (cross) {
            for (uint32_t i = tid; i < long_words(low); i += kDedupThreads) s_set[i] = 0;
            __syncthreads();
            uint32_t beyond = 0;  // distinct keys past this tile
            uint32_t lo = 0;
            const unsigned long long group = keys[base + p1] >> low;
            for (uint64_t x0 = base + (p1 & ~63u);; x0 += kDedupThreads) {
                const uint64_t x = x0 + tid;
                const unsigned long long key = x < cap ? keys[x] : ~0ull;
                const bool in = x < cap && (key >> low) == group;
                bool win = false;
                if (in && x >= base + p1 && key != sentinel) {
                    const uint32_t b = (uint32_t)key & ((1u << low) - 1u);
                    win = !((atomicOr(&s_set[b >> 5], 1u << (b & 31u)) >> (b & 31u)) & 1u);
                    if (win && x >= end) {
                        const uint32_t hi = (uint32_t)(key & mask);
                        if (a.ubins) atomicAdd(&s_hist[hi >> a.ushift], 1u);
                        if (a.uatomics) atomicAdd(&a.deg[hi], 1u);
                        const uint32_t l = (uint32_t)(key >> nb);
                        if (beyond && l != lo) {
                            atomicAdd(&a.deg[lo], beyond);
                            beyond = 0;
                        }
                        lo = l;
                        ++beyond;
                        ++found;
                    }
                }
                const unsigned long long f = __ballot(win);  // (x of lane 0 is a multiple of 64, as is end)
                if (lane == 0 && f) {
                    if (x < end) s_first[(x - base) >> 6] |= f;
                    else atomicOr(&a.first[x >> 6], f);
                }
                if (!__syncthreads_and(in || x < base + p1)) break;
            }
            // lower-id degrees of the keys past the tile (one id, or few where the group holds several)
            const uint32_t lead = __builtin_amdgcn_readfirstlane(lo);
            const unsigned long long differ = __ballot(beyond && lo != lead);
            if (!differ) {
                const uint32_t t = wave_sum(beyond);
                if (lane == 0 && t) atomicAdd(&a.deg[lead], t);
            } else if (beyond) {
                atomicAdd(&a.deg[lo], beyond);
            }
        }
        // bits, lower-id degrees and the upper digit histogram of this tile's distinct edges
        if (lane < kDedupItems) {
            const uint32_t word = wave * kDedupItems + lane;
            const unsigned long long F = s_first[word];
            if (word * 64u >= p0) {
                if (base + word * 64u < cap) a.first[(base >> 6) + word] = F;
            } else if (F) {
                atomicOr(&a.first[(base >> 6) + word], F);
            }
            found += (unsigned long long)__popcll(F);
        }
        count_firsts(a, k, s_first, s_hist, wave, lane);
        __syncthreads();  // the LDS is reused by the next tile
    }
    if (found) atomicAdd(&s_m, found);
    __syncthreads();
    if (threadIdx.x == 0 && s_m) atomicAdd(&a.meta->m, s_m);
    for (uint32_t i = threadIdx.x; i < a.ubins; i += kDedupThreads)
        if (s_hist[i]) atomicAdd(&a.uhist[i], s_hist[i]);
}

// The first of the boundaries (first keys of tiles) of group `top`, of which boundary t is one.
__device__ __forceinline__ uint32_t first_boundary(const unsigned long long* keys, uint32_t low, unsigned long long top,
                                                   uint32_t t, uint32_t lane) {
    uint32_t lo = 0, hi = t;  // boundaries below lo are not in the group, hi is
    uint32_t from = t > 64 ? t - 64 : 0u;  // most groups begin near
    while (lo < hi) {
        const uint32_t step = (hi - from + 63) / 64, b = from + lane * step;
        const unsigned long long in =
            __ballot(b < hi && (keys[(uint64_t)(b < hi ? b : hi) * kDedupTile] >> low) == top);
        if (!in) {
            lo = from + (hi - from - 1) / step * step + 1;  // past the last one looked at
        } else {
            const uint32_t i = (uint32_t)__builtin_ctzll(in);
            hi = from + i * step;
            if (i) lo = from + (i - 1) * step + 1;
            else if (from <= lo) lo = hi;
        }
        from = lo;
    }
    return hi;
}

// The long groups, tile by tile (see above).
__global__ void __launch_bounds__(kDedupThreads) k_dedup_long(Dedup a) {
    __shared__ uint32_t s_set[1u << (kGroupBits - 5)];
    __shared__ unsigned long long s_first[kDedupWords];
    __shared__ uint32_t s_hist[1024];
    __shared__ unsigned long long s_m;
    if (!*a.any_long) return;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t low_mask = (1u << a.low) - 1u, set_words = long_words(a.low);
    for (uint32_t i = tid; i < a.ubins; i += kDedupThreads) s_hist[i] = 0;
    if (tid == 0) s_m = 0;
    unsigned long long found = 0;
    for (uint64_t base = blockIdx.x * (uint64_t)kDedupTile; base < a.cap; base += (uint64_t)gridDim.x * kDedupTile) {
        const uint32_t len = a.cap - base < kDedupTile ? (uint32_t)(a.cap - base) : kDedupTile;
        const uint32_t longs = long_groups(a, base, lane);
        if (!longs) continue;  // uniform in the workgroup
        unsigned long long k[kDedupItems];
        unsigned long long F[kDedupItems];
        const unsigned long long head = a.keys[base] >> a.low;
        const unsigned long long next = base + len < a.cap ? a.keys[base + len] >> a.low : ~0ull;
#pragma unroll
        for (int i = 0; i < (int)kDedupItems; ++i) {
            const uint64_t x = base + wave * (64u * kDedupItems) + i * 64u + lane;
            k[i] = x < a.cap ? a.keys[x] : ~0ull;
            F[i] = 0;
        }
        // the group of the tile's first key, then the one that is cut at its end
        for (uint32_t part = 0; part < 2; ++part) {
            if (!(longs & (1u << part)) || (part == 1 && next == head)) continue;
            const unsigned long long top = part ? next : head;
            const uint32_t tile = (uint32_t)(base / kDedupTile);
            const uint32_t name = part ? tile + 1 : tile ? first_boundary(a.keys, a.low, top, tile, lane) : 0u;
            uint32_t* const set = a.bits + (uint64_t)(name / kLongTiles) * set_words;
            __syncthreads();
            for (uint32_t i = tid; i < set_words; i += kDedupThreads) s_set[i] = 0;
            __syncthreads();
            uint32_t mine = 0;  // keys that set their bit in this tile's set
#pragma unroll
            for (int i = 0; i < (int)kDedupItems; ++i) {
                const uint64_t x = base + wave * (64u * kDedupItems) + i * 64u + lane;
                if (x >= a.cap || (k[i] >> a.low) != top || k[i] == a.sentinel) continue;
                const uint32_t b = (uint32_t)k[i] & low_mask, bit = 1u << (b & 31u);
                if (__hip_atomic_load(&s_set[b >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & bit) continue;
                if (!(atomicOr(&s_set[b >> 5], bit) & bit)) mine |= 1u << i;
            }
            __syncthreads();
            for (uint32_t i = tid; i < set_words; i += kDedupThreads) {
                const uint32_t v = s_set[i];
                if (!v) continue;
                uint32_t old = __hip_atomic_load(&set[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (v & ~old) old = atomicOr(&set[i], v);
                s_set[i] = v & ~old;
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < (int)kDedupItems; ++i) {
                const uint32_t b = (uint32_t)k[i] & low_mask;
                F[i] |= __ballot(((mine >> i) & 1u) && ((s_set[b >> 5] >> (b & 31u)) & 1u));
            }
        }
#pragma unroll
        for (int i = 0; i < (int)kDedupItems; ++i) {
            const uint32_t word = wave * kDedupItems + i;
            if (lane == 0) {
                s_first[word] = F[i];
                if (F[i]) a.first[(base >> 6) + word] |= F[i];
                found += (unsigned long long)__popcll(F[i]);
            }
        }
        wave_sync();  // a wavefront reads its own words
        count_firsts(a, k, s_first, s_hist, wave, lane);
    }
    __syncthreads();
    if (found) atomicAdd(&s_m, found);
    __syncthreads();
    if (tid == 0 && s_m) atomicAdd(&a.meta->m, s_m);
    for (uint32_t i = tid; i < a.ubins; i += kDedupThreads)
        if (s_hist[i]) atomicAdd(&a.uhist[i], s_hist[i]);
}

// Upper ids' degrees.  The ids are partitioned by hi >> sub (bins partitions, sizes in uhist; with one
// partition they are read from the sorted keys).  A work unit is up to kUpperUnit ids of one partition;
// its counters live in LDS (2^kCounterBits at a time) and are added to deg, by atomics only where a
// partition has several units.
constexpr uint32_t kUpperUnit = 1u << 20;

// The partition of unit u, given the 1024 partitions' first units (empty ones repeat the next value).
__device__ __forceinline__ uint32_t partition_of(const uint32_t* s_unit, uint32_t u) {
    uint32_t l = 0, r = 1023;
    while (l < r) {
        const uint32_t mid = (l + r + 1) >> 1;
        if (s_unit[mid] <= u) l = mid; else r = mid - 1;
    }
    return l;
}

__global__ void __launch_bounds__(1024) k_upper_count(const uint32_t* __restrict__ ids, LoadUpper direct, uint64_t cap,
                                                      uint32_t bins, uint32_t sub, uint32_t n,
                                                      const uint32_t* __restrict__ uhist, uint32_t unit_size,
                                                      uint32_t* __restrict__ deg) {
    extern __shared__ __align__(16) uint32_t s_cnt[];
    __shared__ uint32_t s_unit[1025], s_at[1025], s_scan[16];
    const uint32_t tid = threadIdx.x;
    const uint32_t size = ids ? (tid < bins ? uhist[tid] : 0u) : (tid == 0 ? (uint32_t)cap : 0u);
    const uint32_t units = (size + unit_size - 1) / unit_size;
    const uint32_t u0 = block_excl_scan<16>(units, s_scan), a0 = block_excl_scan<16>(size, s_scan);
    s_unit[tid] = u0;
    s_at[tid] = a0;
    if (tid == 1023) s_unit[1024] = u0 + units;
    __syncthreads();
    const uint32_t total = s_unit[1024];
    const uint32_t span = sub < kCounterBits ? 1u << sub : 1u << kCounterBits;  // counters at a time
    for (uint32_t u = blockIdx.x; u < total; u += gridDim.x) {
        const uint32_t l = partition_of(s_unit, u);
        const uint32_t parts = s_unit[l + 1] - s_unit[l], part = u - s_unit[l];
        const uint32_t len = ids ? uhist[l] : (uint32_t)cap;
        const uint64_t x0 = s_at[l] + (uint64_t)part * unit_size;
        const uint64_t x1 = part + 1 < parts ? x0 + unit_size : (uint64_t)s_at[l] + len;
        for (uint32_t c0 = 0; c0 < (1u << sub); c0 += span) {
            for (uint32_t i = tid; i < span; i += 1024) s_cnt[i] = 0;
            __syncthreads();
            for (uint64_t x = x0 + tid; x < x1; x += 1024) {
                uint32_t id;
                if (ids) id = ids[x];
                else if (!direct.make(direct.raw(x), (uint32_t)(x & 63u), id)) continue;
                const uint32_t c = (id & ((1u << sub) - 1u)) - c0;
                if (c < span) atomicAdd(&s_cnt[c], 1u);
            }
            __syncthreads();
            const uint64_t v0 = ((uint64_t)l << sub) + c0;
            for (uint32_t i = tid; i < span && v0 + i < n; i += 1024) {
                const uint32_t c = s_cnt[i];
                if (c) {
                    if (parts == 1) deg[v0 + i] += c;
                    else atomicAdd(&deg[v0 + i], c);
                }
            }
            __syncthreads();
        }
    }
}

// Digit histograms of the degrees.
__global__ void __launch_bounds__(1024) k_degree_hist(const uint32_t* __restrict__ deg, uint32_t n, uint32_t passes,
                                                      uint32_t* __restrict__ hist) {
    __shared__ uint32_t s_h[4][512];
    for (uint32_t i = threadIdx.x; i < passes * 512; i += blockDim.x) (&s_h[0][0])[i] = 0;
    __syncthreads();
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < n; base += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = base + threadIdx.x;
        const bool act = i < n;
        const uint32_t d = act ? deg[i] : 0u;
        for (uint32_t p = 0; p < passes; ++p) count_digit(s_h[p], (d >> (kDigit * p)) & 511u, act);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < passes * 512; i += blockDim.x)
        if (const uint32_t c = (&s_h[0][0])[i]) atomicAdd(&hist[i], c);
}

__global__ void k_orient_count(const unsigned long long* __restrict__ keys, uint32_t nb, uint64_t cap,
                               const unsigned long long* __restrict__ first, const uint32_t* __restrict__ rank,
                               uint32_t* __restrict__ dplus) {
    const unsigned long long mask = (nb >= 32) ? 0xFFFFFFFFull : ((1ull << nb) - 1);
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < cap; i += (uint64_t)gridDim.x * blockDim.x) {
        if (!is_first(first, i)) continue;
        const unsigned long long k = keys[i];
        const uint32_t ra = rank[(uint32_t)(k >> nb)], rb = rank[(uint32_t)(k & mask)];
        atomicAdd(&dplus[ra < rb ? ra : rb], 1u);
    }
}

__global__ void k_orient_fill(const unsigned long long* __restrict__ keys, uint32_t nb, uint64_t cap,
                              const unsigned long long* __restrict__ first, const uint32_t* __restrict__ rank,
                              const int64_t* __restrict__ off, uint32_t* __restrict__ cursor,
                              uint32_t* __restrict__ col) {
    const unsigned long long mask = (nb >= 32) ? 0xFFFFFFFFull : ((1ull << nb) - 1);
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < cap; i += (uint64_t)gridDim.x * blockDim.x) {
        if (!is_first(first, i)) continue;
        const unsigned long long k = keys[i];
        const uint32_t ra = rank[(uint32_t)(k >> nb)], rb = rank[(uint32_t)(k & mask)];
        const uint32_t s = ra < rb ? ra : rb, d = ra < rb ? rb : ra;
        const uint32_t pos = atomicAdd(&cursor[s], 1u);
        col[off[s] + pos] = d;
    }
}

// Oriented keys (rank_lo << nb | rank_hi) of the distinct edges, at the places of the sorted keys, and
// the digit histograms of their rows.  Bound by the gathers of rank[hi] (see attach_ranks for large graphs).
__global__ void __launch_bounds__(1024) k_orient_keys(const unsigned long long* __restrict__ keys, uint32_t nb,
                                                      uint64_t cap, const unsigned long long* __restrict__ first,
                                                      const uint32_t* __restrict__ rank, uint32_t passes,
                                                      unsigned long long* __restrict__ okeys,
                                                      uint32_t* __restrict__ hist) {
    // The top digit has few values and on skewed graphs most rows share one: 16 copies of its counters.
    __shared__ uint32_t s_h[3][512], s_top[512 * 16];
    const uint32_t top = passes - 1, tops = 1u << (nb - kDigit * top);
    for (uint32_t i = threadIdx.x; i < top * 512; i += blockDim.x) (&s_h[0][0])[i] = 0;
    for (uint32_t i = threadIdx.x; i < tops * 16; i += blockDim.x) s_top[i] = 0;
    __syncthreads();
    const unsigned long long mask = (nb >= 32) ? 0xFFFFFFFFull : ((1ull << nb) - 1);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < cap; base += 2 * stride) {
        bool act[2];
        uint32_t ra[2] = {0, 0}, rb[2] = {0, 0};
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint64_t i = base + j * stride + threadIdx.x;
            act[j] = i < cap && is_first(first, i);
            if (act[j]) {
                const unsigned long long k = keys[i];
                ra[j] = rank[(uint32_t)(k >> nb)];
                rb[j] = rank[(uint32_t)(k & mask)];
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t row = ra[j] < rb[j] ? ra[j] : rb[j], head = ra[j] < rb[j] ? rb[j] : ra[j];
            if (act[j]) okeys[base + j * stride + threadIdx.x] = ((unsigned long long)row << nb) | head;
            for (uint32_t p = 0; p < top; ++p) count_digit(s_h[p], (row >> (kDigit * p)) & 511u, act[j]);
            if (act[j]) atomicAdd(&s_top[(row >> (kDigit * top)) * 16u + (threadIdx.x & 15u)], 1u);
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < top * 512; i += blockDim.x)
        if (const uint32_t c = (&s_h[0][0])[i]) atomicAdd(&hist[i], c);
    for (uint32_t i = threadIdx.x; i < tops; i += blockDim.x) {
        uint32_t c = 0;
        for (uint32_t j = 0; j < 16; ++j) c += s_top[i * 16 + j];
        if (c) atomicAdd(&hist[top * 512 + i], c);
    }
}

// The same from the distinct edges with the lower ids' ranks in place, partitioned by their upper ids
// (LoadRanked): a work unit is a share of one partition, and gathers from the ranks of the partition's ids in
// LDS (2^15 at most: one workgroup per CU then, two at 2^14).  2^25 vertices, 537 M edges: 2.2 ms (bytes 1.8 at
// the copy rate), after a pass of 3.0; the lookups past the L1 instead, in partitions of 2^16 ids: 6.3.
__global__ void __launch_bounds__(1024) k_orient_parts(const unsigned long long* __restrict__ keys, uint32_t nb,
                                                       uint32_t bins, uint32_t sub, uint32_t n,
                                                       const uint32_t* __restrict__ uhist,
                                                       uint32_t unit, const uint32_t* __restrict__ rank, uint32_t passes,
                                                       unsigned long long* __restrict__ okeys,
                                                       uint32_t* __restrict__ hist) {
    constexpr int kItems = 4;
    extern __shared__ __align__(16) uint32_t s_rank[];  // [1 << sub], then the top digit's counters (16 copies)
    __shared__ uint32_t s_h[2][512];
    __shared__ uint32_t s_unit[1025], s_at[1025], s_scan[16];
    const uint32_t tid = threadIdx.x;
    const uint32_t top = passes - 1, tops = 1u << (nb - kDigit * top);
    uint32_t* const s_top = s_rank + (1u << sub);
    for (uint32_t i = tid; i < top * 512; i += 1024) (&s_h[0][0])[i] = 0;
    for (uint32_t i = tid; i < tops * 16; i += 1024) s_top[i] = 0;
    const uint32_t size = tid < bins ? uhist[tid] : 0u;
    const uint32_t units = (size + unit - 1) / unit;
    const uint32_t u0 = block_excl_scan<16>(units, s_scan), a0 = block_excl_scan<16>(size, s_scan);
    s_unit[tid] = u0;
    s_at[tid] = a0;
    if (tid == 1023) {
        s_unit[1024] = u0 + units;
        s_at[1024] = a0 + size;
    }
    __syncthreads();
    const unsigned long long mask = (1ull << nb) - 1;
    const uint32_t total = s_unit[1024], ids = (1u << sub) - 1u;
    for (uint32_t u = blockIdx.x; u < total; u += gridDim.x) {
        const uint32_t l = partition_of(s_unit, u);
        const uint32_t parts = s_unit[l + 1] - s_unit[l], part = u - s_unit[l];
        const uint32_t len = s_at[l + 1] - s_at[l], share = (len + parts - 1) / parts;
        const uint32_t x0 = s_at[l] + part * share, x1 = part + 1 < parts ? x0 + share : s_at[l] + len;
        const uint32_t v0 = l << sub, have = n - v0 < ids + 1 ? n - v0 : ids + 1;
        for (uint32_t i = tid; i < have; i += 1024) s_rank[i] = rank[v0 + i];
        __syncthreads();
        for (uint32_t base = x0; base < x1; base += kItems * 1024) {
            unsigned long long k[kItems];
#pragma unroll
            for (int j = 0; j < kItems; ++j) {
                const uint32_t x = base + j * 1024 + tid;
                k[j] = keys[x < x1 ? x : x1 - 1];
            }
#pragma unroll
            for (int j = 0; j < kItems; ++j) {
                const uint32_t x = base + j * 1024 + tid;
                const bool act = x < x1;
                const uint32_t ra = (uint32_t)(k[j] >> nb), rb = s_rank[(uint32_t)(k[j] & mask) & ids];
                const uint32_t row = ra < rb ? ra : rb, head = ra < rb ? rb : ra;
                if (act) okeys[x] = ((unsigned long long)row << nb) | head;
                for (uint32_t p = 0; p < top; ++p) count_digit(s_h[p], (row >> (kDigit * p)) & 511u, act);
                if (act) atomicAdd(&s_top[(row >> (kDigit * top)) * 16u + (tid & 15u)], 1u);
            }
        }
        __syncthreads();
    }
    for (uint32_t i = tid; i < top * 512; i += 1024)
        if (const uint32_t c = (&s_h[0][0])[i]) atomicAdd(&hist[i], c);
    for (uint32_t i = tid; i < tops; i += 1024) {
        uint32_t c = 0;
        for (uint32_t j = 0; j < 16; ++j) c += s_top[i * 16 + j];
        if (c) atomicAdd(&hist[top * 512 + i], c);
    }
}

// From the m oriented keys sorted by row: the lists, and the offsets of every row (64 and 32 bits: the
// count kernels read the latter, m_in < 2^31).  Edge e of a row unlike its predecessor's gives the offset
// e to its row and to the empty rows before it; the rows before the first edge's and after the last
// edge's are filled by the whole grid, long gaps in between by the wavefront.  work (W of every row, summed
// next) is cleared here.
__global__ void __launch_bounds__(256) k_csr(const unsigned long long* __restrict__ okeys, uint32_t nb,
                                             const GraphMeta* meta, uint32_t n, int64_t* __restrict__ off,
                                             uint32_t* __restrict__ off32, uint32_t* __restrict__ col,
                                             unsigned long long* __restrict__ work) {
    const uint64_t m = meta->m;
    const unsigned long long mask = (nb >= 32) ? 0xFFFFFFFFull : ((1ull << nb) - 1);
    const uint64_t t0 = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x, step = (uint64_t)gridDim.x * blockDim.x;
    const uint32_t lane = threadIdx.x & 63u;
    auto put = [&](uint64_t r, uint32_t v) {
        off[r] = v;
        off32[r] = v;
    };
    const uint64_t head = m ? (uint32_t)(okeys[0] >> nb) : n;  // rows [0, head] start at 0
    const uint64_t tail = m ? (uint32_t)(okeys[m - 1] >> nb) + 1ull : n + 1ull;
    for (uint64_t r = t0; r < n; r += step) work[r] = 0;
    for (uint64_t r = t0; r <= head; r += step) put(r, 0u);
    for (uint64_t r = tail + t0; r <= n; r += step) put(r, (uint32_t)m);
    for (uint64_t base = t0 - lane; base < m; base += step) {
        const uint64_t e = base + lane;
        uint32_t r = 0, prev = 0;
        if (e < m) {
            const unsigned long long k = okeys[e];
            col[e] = (uint32_t)(k & mask);
            r = prev = (uint32_t)(k >> nb);
            if (e) prev = (uint32_t)(okeys[e - 1] >> nb);
        }
        const uint32_t gap = r - prev;  // rows (prev, r] start at e
        const bool far = gap > 32;
        if (gap && !far)
            for (uint32_t q = prev + 1; q <= r; ++q) put(q, (uint32_t)e);
        for (unsigned long long left = __ballot(far); left; left &= left - 1) {
            const int src = __builtin_ctzll(left);
            const uint32_t a = __builtin_amdgcn_readlane(prev, src), b = __builtin_amdgcn_readlane(r, src);
            const uint32_t at = (uint32_t)(base + (uint32_t)src);
            for (uint64_t q = (uint64_t)a + 1 + lane; q <= b; q += 64) put(q, at);
        }
    }
}

// Collective work W(r) = sum of d+(v) over r's out-neighbours v, from the oriented keys sorted by row.  A
// wavefront walks a range of consecutive edges, 256 at a time with their gathers (v's offsets) issued
// together, and sums the runs of equal rows: runs that begin and end inside are stored, the first and the
// last are added to work (cleared beforehand; with ranges of 256 edges those atomics cost 2 of 13 ms).  Bound
// by the gathers: one 128-byte line per edge at 2^25 vertices (10.6 ms for 537 M edges), 0.36 ms for the 64 M of
// R-MAT 22, 0.09 ms for the 16 M of R-MAT 20 (16 lanes per row took 0.47 and 0.39, waiting for the longest
// rows).  Record layout: d+(v) comes with v's placement {p(v), d+(v)}, and edge e writes v's record id into its
// row's record; the row's first edge also writes the header d+(r).  On light graphs the bounds of
// v's list are kept per edge as well: 8 coalesced bytes that spare the count its own gather of them.
constexpr uint32_t kWorkItems = 4;

template <bool REC>
__global__ void __launch_bounds__(256) k_work(const unsigned long long* __restrict__ okeys, uint32_t nb,
                                              const uint32_t* __restrict__ off, const uint2* __restrict__ place,
                                              uint32_t* __restrict__ rec, const GraphMeta* meta,
                                              unsigned long long* __restrict__ work, uint2* __restrict__ elist) {
    const uint64_t m = meta->m;
    if (!light_on(*meta)) elist = nullptr;
    const unsigned long long mask = (nb >= 32) ? 0xFFFFFFFFull : ((1ull << nb) - 1);
    const uint32_t lane = threadIdx.x & 63u;
    const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1);  // lanes 0..lane
    constexpr uint64_t kSpan = 64 * kWorkItems;
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    const uint64_t per = ((m + waves - 1) / waves + kSpan - 1) / kSpan * kSpan;  // this wavefront's edges
    const uint64_t lo = (blockIdx.x * (uint64_t)(blockDim.x >> 6) + (threadIdx.x >> 6)) * per;
    const uint64_t hi = lo + per < m ? lo + per : m;
    // carried run (uniform): row, sum so far, and whether it may have begun before these edges
    uint32_t crow = 0;
    unsigned long long csum = 0;
    bool open = true;
    for (uint64_t base = lo; base < hi; base += kSpan) {
        uint32_t row[kWorkItems], v[kWorkItems], len[kWorkItems];
#pragma unroll
        for (uint32_t i = 0; i < kWorkItems; ++i) {
            const uint64_t e = base + i * 64u + lane;
            const unsigned long long k = okeys[e < m ? e : m - 1];
            row[i] = (uint32_t)(k >> nb);
            v[i] = (uint32_t)(k & mask);
        }
#pragma unroll
        for (uint32_t i = 0; i < kWorkItems; ++i) {
            const uint64_t e = base + i * 64u + lane;
            if constexpr (REC) {
                const uint2 pv = place[v[i]], pr = place[row[i]];
                len[i] = pv.y;
                if (e < m) {
                    const uint32_t j = (uint32_t)e - off[row[i]];
                    rec[pr.x + 1u + j] = rec_id(pv.x);
                    if (j == 0) rec[pr.x] = pr.y;
                    if (elist) elist[e] = make_uint2(pv.x + 1u, pv.y);
                }
            } else {
                struct __attribute__((packed, aligned(4))) Pair { uint32_t a, b; };  // one 8-byte load
                const Pair o = *reinterpret_cast<const Pair*>(off + v[i]);
                len[i] = o.b - o.a;
                if (elist && e < m) elist[e] = make_uint2(o.a, len[i]);
            }
            if (e >= m) len[i] = 0;
        }
        if (base == lo) crow = __builtin_amdgcn_readfirstlane(row[0]);
#pragma unroll
        for (uint32_t i = 0; i < kWorkItems; ++i) {
            const uint32_t prev = (uint32_t)__shfl_up((int)row[i], 1, 64);
            const unsigned long long H = __ballot(lane == 0 ? row[i] != crow : row[i] != prev);  // run starts
            const uint32_t incl = wave_incl_scan(len[i]);  // out-degrees are below 2^17 (m < 2^31): no overflow
            const unsigned long long mine = H & upto;
            const uint32_t s = mine ? 63u - (uint32_t)__builtin_clzll(mine) : 0u;  // this lane's run start
            const uint32_t from = (uint32_t)__shfl((int)incl, (int)((s + 63u) & 63u), 64);  // every lane takes part
            const uint32_t sum = incl - (s ? from : 0u);
            const bool last = lane != 63 && ((H >> (lane + 1)) & 1ull);  // the next lane starts another run
            if (last) {
                if (mine) {
                    work[row[i]] = sum;  // begins and ends in this step
                } else {
                    const unsigned long long t = csum + sum;
                    if (open) atomicAdd(&work[row[i]], t);
                    else work[row[i]] = t;
                }
            }
            if (H & 1ull) {  // the carried run ended with the previous step
                if (lane == 0) {
                    if (open) atomicAdd(&work[crow], csum);
                    else work[crow] = csum;
                }
            }
            const uint32_t sum63 = (uint32_t)__builtin_amdgcn_readlane((int)sum, 63);
            csum = H ? sum63 : csum + sum63;
            open = H ? false : open;
            crow = (uint32_t)__builtin_amdgcn_readlane((int)row[i], 63);
        }
    }
    if (lane == 0 && csum) atomicAdd(&work[crow], csum);  // may go on in the next wavefront's edges
}

// The same from lists (relabelled graphs and counting-sort builds, which have no sorted keys): 16 lanes per row.
constexpr uint32_t kWorkLanes = 16;

__global__ void __launch_bounds__(256) k_work_rows(const uint32_t* __restrict__ off, const uint32_t* __restrict__ col,
                                                   uint32_t n, unsigned long long* __restrict__ work) {
    const uint32_t sub = threadIdx.x % kWorkLanes, per = blockDim.x / kWorkLanes;
    for (uint64_t r = blockIdx.x * (uint64_t)per + threadIdx.x / kWorkLanes; r < n; r += (uint64_t)gridDim.x * per) {
        const uint32_t b = off[r], d = off[r + 1] - b;
        unsigned long long w = 0;
        for (uint32_t p = sub; p < d; p += kWorkLanes) {
            const uint32_t v = col[b + p];
            w += off[v + 1] - off[v];
        }
#pragma unroll
        for (uint32_t o = 1; o < kWorkLanes; o <<= 1) w += __shfl_xor(w, o);  // lanes of a row run together
        if (sub == 0) work[r] = w;
    }
}

// The headers of rows without edges (record layout; the others: k_work).
__global__ void k_record_empty(const uint2* __restrict__ place, uint32_t n, uint32_t* __restrict__ rec) {
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x) {
        const uint2 p = place[r];
        if (p.y == 0) rec[p.x] = 0;
    }
}

// W+ = sum over v of (in-degree) d+(v), and the owners, before any W(u) is known (light_on); the ranks from
// the first one with more than big_cap out-neighbours.
__global__ void __launch_bounds__(1024) k_owners(const uint32_t* __restrict__ off,
                                                 const unsigned long long* __restrict__ order, uint32_t n,
                                                 uint32_t big_cap, GraphMeta* meta) {
    __shared__ unsigned long long s_w, s_o;
    if (threadIdx.x == 0) s_w = s_o = 0;
    __syncthreads();
    unsigned long long w = 0, o = 0;
    uint32_t span = 0;
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t d = off[r + 1] - off[r], deg = (uint32_t)(order[r] >> 32);  // degree << 32 | id
        w += (unsigned long long)(deg - d) * d;
        o += d >= 2;
        if (d > big_cap && n - (uint32_t)r > span) span = n - (uint32_t)r;
    }
    if (span) atomicMax(&meta->hub_span, span);
    for (int k = 32; k > 0; k >>= 1) {
        w += __shfl_xor(w, k);
        o += __shfl_xor(o, k);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&s_w, w);
        atomicAdd(&s_o, o);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_o) {
        atomicAdd(&meta->pre_work, s_w);
        atomicAdd(&meta->pre_owners, s_o);
    }
}

// Rows of the ranks that owners of global-memory tables (more than big_cap out-neighbours) probe, in rank
// order: where neighbours share their ranks' neighbourhood, the lanes of a wavefront then look up
// neighbouring buckets, and a line of the table in memory serves several of them (a complete graph of 8000
// vertices, samples in any order: per-vertex count 10.2 -> 7.1 s, total 410 -> 358 ms; 20 of 5000 vertices
// 29.5 -> 18.3 s, 1532 -> 1196 ms).  Such owners' neighbours have larger ranks and degrees above big_cap, so
// there are at most 2 m / big_cap of them: a bit set in LDS takes a row's ids and gives them back in order.
// Keys and lists both (the edges' list bounds are laid out by the keys).
constexpr uint32_t kSortWords = 32768, kSortMin = 64;  // shorter rows are left as they are

__global__ void __launch_bounds__(1024) k_sort_rows(const GraphMeta* meta, const uint32_t* __restrict__ off, uint32_t n,
                                                    uint32_t nb, uint32_t* __restrict__ col,
                                                    unsigned long long* __restrict__ okeys) {
    extern __shared__ __align__(16) uint32_t s_bits[];  // ranks from the row's own on, in words
    __shared__ uint32_t s_scan[16];
    const uint32_t span = meta->hub_span, tid = threadIdx.x;
    for (uint64_t r = (uint64_t)n - span + blockIdx.x; r < n; r += gridDim.x) {  // (none where span is 0)
        const uint32_t b = off[r], d = off[r + 1] - b;
        if (d < kSortMin) continue;
        const uint32_t words = (uint32_t)((n - r + 31) / 32);
        for (uint32_t i = tid; i < words; i += 1024) s_bits[i] = 0;
        __syncthreads();
        for (uint32_t i = tid; i < d; i += 1024) {
            const uint32_t x = col[b + i] - (uint32_t)r;
            atomicOr(&s_bits[x >> 5], 1u << (x & 31u));
        }
        __syncthreads();
        const uint32_t per = (words + 1023) / 1024, i0 = tid * per, i1 = i0 + per < words ? i0 + per : words;
        uint32_t c = 0;
        for (uint32_t i = i0; i < i1; ++i) c += (uint32_t)__popc(s_bits[i]);
        uint32_t at = b + block_excl_scan<16>(c, s_scan);
        for (uint32_t i = i0; i < i1; ++i)
            for (uint32_t x = s_bits[i]; x; x &= x - 1u, ++at) {
                const uint32_t v = (uint32_t)r + 32u * i + (uint32_t)__builtin_ctz(x);
                col[at] = v;
                okeys[at] = (r << nb) | v;
            }
        __syncthreads();
    }
}

// Census for the packed bin: vertices that would get a wavefront-size table, and how many of them
// are light enough to pack (out-degree <= pack_cap, W(u) <= kPackMaxWork).  Packing pays when light
// vertices dominate (their per-vertex fixed work is what it shares); the schedule packs only then.
__global__ void __launch_bounds__(1024) k_pack_census(const uint32_t* __restrict__ off,
                                                      const unsigned long long* __restrict__ work, uint32_t n,
                                                      BinCaps caps, GraphMeta* meta) {
    __shared__ uint32_t s_w, s_p;
    if (threadIdx.x == 0) s_w = s_p = 0;
    __syncthreads();
    uint32_t wc = 0, pc = 0;
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t d = off[r + 1] - off[r];
        const unsigned long long w = work[r];
        if (d < 2 || w == 0 || d > caps.wave_cap) continue;
        ++wc;
        pc += (d <= caps.pack_cap && w <= kPackMaxWork) ? 1u : 0u;
    }
    if (wc) atomicAdd(&s_w, wc);
    if (pc) atomicAdd(&s_p, pc);
    __syncthreads();
    if (threadIdx.x == 0 && s_w) {
        atomicAdd(&meta->wave_cands, s_w);
        atomicAdd(&meta->pack_cands, s_p);
    }
}

// Largest-work-first code of 15 bits, smaller for more work: exponent and 10 bits below the leading one
// (exact below 2048, to 0.1% above: ties there only loosen the order, and kCoreMinWork = 2^10 divides it).
__device__ __forceinline__ uint32_t work_code(unsigned long long w) {
    const uint32_t x = w > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)w;
    if (x == 0) return 32767u;
    const uint32_t e = 31u - (uint32_t)__builtin_clz(x);
    const uint32_t f = (e >= 10 ? x >> (e - 10) : x << (10 - e)) & 1023u;
    return 32767u - ((e << 10) | f);
}
static_assert(kCoreMinWork == 1024, "the core path's owners of the wavefront bin are a prefix of its order");

// One thread per vertex: bin and schedule element (group of the bin << 15 | work code) << 32 | rank, which
// replaces the rank's (degree << 32 | id), and the digit histograms of the keys.  Bins: 0 global-memory
// table (too large for any LDS table), 1 large LDS table (whole LDS of a workgroup, one per CU),
// 2 workgroup LDS table, 3 wavefront LDS slice, 4 light vertices packed
// several to a wavefront, 5 skipped.  Bin 1 is split in two groups, each by decreasing work: first
// the vertices whose tables need more than half a CU's LDS (counted by one workgroup per CU), then
// those up to caps.mid_cap (two workgroups per CU).
__global__ void __launch_bounds__(1024) k_schedule(const uint32_t* __restrict__ off,
                                                  const unsigned long long* __restrict__ work, uint32_t n, BinCaps caps,
                                                  GraphMeta* meta, unsigned long long* elem,
                                                  uint32_t* __restrict__ hist) {
    __shared__ uint32_t s_h[2][512];
    for (uint32_t i = threadIdx.x; i < 1024; i += blockDim.x) (&s_h[0][0])[i] = 0;
    __shared__ unsigned long long s_hw, s_ce;
    __shared__ unsigned int s_h3;
    __shared__ unsigned long long s_w;
    __shared__ unsigned int s_max, s_bins[6], s_full;
    __shared__ unsigned long long s_bw[6];
    if (threadIdx.x < 6) {
        s_bins[threadIdx.x] = 0;
        s_bw[threadIdx.x] = 0;
    }
    if (threadIdx.x == 0) { s_w = 0; s_max = 0; s_full = 0; s_hw = 0; s_ce = 0; s_h3 = 0; }
    __syncthreads();
    const uint32_t pack_cap = (caps.pack_cap && 2ull * meta->pack_cands >= meta->wave_cands) ? caps.pack_cap : 0u;
    // Per-thread partials, reduced across the wave, then one LDS atomic per wave.
    unsigned long long wsum = 0;
    uint32_t dmax = 0, nb0 = 0, nb1 = 0, nb2 = 0, nb3 = 0, nb4 = 0, nb5 = 0, nfull = 0;
    unsigned long long bw[6] = {0, 0, 0, 0, 0, 0};
    unsigned long long hw = 0, ce = 0;
    uint32_t h3 = 0;
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < n; base += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t r = base + threadIdx.x;
        const bool act = r < n;
        const uint32_t d = act ? off[r + 1] - off[r] : 0u;
        const unsigned long long w = act ? work[r] : 0ull;
        uint32_t bin = 5, group = 6;
        if (act) {
            if (d < 2 || w == 0) bin = 5;
            else if (caps.force_hub || d > caps.big_cap) bin = 0;
            else if (caps.force_big || d > caps.wg_cap) bin = 1;
            else if (caps.force_wg || d > caps.wave_cap) bin = 2;
            else if (d <= pack_cap && w <= kPackMaxWork) bin = 4;
            else bin = 3;
            if (caps.core_bits) {  // elem[r] still holds r's degree: deg - d+ edges end in r
                if (r >= caps.core_first) ce += (uint32_t)(elem[r] >> 32) - d;
                const bool h = bin == 3 && w >= kCoreMinWork;
                h3 += h;
                if (h || bin == 2 || (bin == 1 && (caps.core_big_all || d <= caps.mid_cap))) hw += w;
            }
            const bool full = bin == 1 && d > caps.mid_cap;
            nfull += full;
            group = bin + ((bin > 1 || (bin == 1 && !full)) ? 1u : 0u);
        }
        const uint32_t key = (group << 15) | (caps.lpt ? work_code(w) : 0u);
        if (act) elem[r] = ((unsigned long long)key << 32) | r;
        count_digit(s_h[0], key & 511u, act);
        count_digit(s_h[1], key >> kDigit, act);
        if (!act) continue;
        wsum += w;
#pragma unroll
        for (int q = 0; q < 6; ++q) bw[q] += (bin == (uint32_t)q) ? w : 0ull;
        dmax = d > dmax ? d : dmax;
        nb0 += bin == 0;
        nb1 += bin == 1;
        nb2 += bin == 2;
        nb3 += bin == 3;
        nb4 += bin == 4;
        nb5 += bin == 5;
    }
    for (int o = 32; o > 0; o >>= 1) {
        wsum += __shfl_xor(wsum, o);
#pragma unroll
        for (int q = 0; q < 6; ++q) bw[q] += __shfl_xor(bw[q], o);
        const uint32_t dm = __shfl_xor(dmax, o);
        dmax = dm > dmax ? dm : dmax;
        nb0 += __shfl_xor(nb0, o);
        nb1 += __shfl_xor(nb1, o);
        nb2 += __shfl_xor(nb2, o);
        nb3 += __shfl_xor(nb3, o);
        nb4 += __shfl_xor(nb4, o);
        nb5 += __shfl_xor(nb5, o);
        nfull += __shfl_xor(nfull, o);
        if (caps.core_bits) {
            hw += __shfl_xor(hw, o);
            ce += __shfl_xor(ce, o);
            h3 += __shfl_xor(h3, o);
        }
    }
    if ((threadIdx.x & 63) == 0) {
        if (hw) atomicAdd(&s_hw, hw);
        if (ce) atomicAdd(&s_ce, ce);
        if (h3) atomicAdd(&s_h3, h3);
        atomicAdd(&s_w, wsum);
        atomicMax(&s_max, dmax);
        atomicAdd(&s_bins[0], nb0);
        atomicAdd(&s_bins[1], nb1);
        atomicAdd(&s_bins[2], nb2);
        atomicAdd(&s_bins[3], nb3);
        atomicAdd(&s_bins[4], nb4);
        atomicAdd(&s_bins[5], nb5);
        if (nfull) atomicAdd(&s_full, nfull);
#pragma unroll
        for (int q = 0; q < 6; ++q)
            if (bw[q]) atomicAdd(&s_bw[q], bw[q]);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicAdd(&meta->wplus, s_w);
        atomicMax(&meta->max_dplus, s_max);
        if (s_full) atomicAdd(&meta->big_full, s_full);
        if (s_hw) atomicAdd(&meta->heavy_work, s_hw);
        if (s_ce) atomicAdd(&meta->core_edges, s_ce);
        if (s_h3) atomicAdd(&meta->heavy3, s_h3);
        for (int i = 0; i < 6; ++i) atomicAdd(&meta->bins[i], s_bins[i]);
        for (int i = 0; i < 6; ++i)
            if (s_bw[i]) atomicAdd(&meta->bin_work[i], s_bw[i]);
    }
    for (uint32_t i = threadIdx.x; i < 1024; i += blockDim.x)
        if (const uint32_t c = (&s_h[0][0])[i]) atomicAdd(&hist[i], c);
}

__global__ void k_rank(const uint32_t* __restrict__ order, uint32_t n, uint32_t* __restrict__ rank) {
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x)
        rank[order[r]] = r;
}

// Out-degrees from the offsets (entry n: 0), for the relabelling.
__global__ void k_dplus(const uint32_t* __restrict__ off, uint32_t n, uint32_t* __restrict__ dplus) {
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r <= n; r += (uint64_t)gridDim.x * blockDim.x)
        dplus[r] = r < n ? off[r + 1] - off[r] : 0u;
}

// ---- vertex orders for the hash ids (Section 4.1, reordering)

// In-degree order: larger oriented in-degree d-(r) = deg(r) - d+(r) first, ties by rank.
__global__ void k_key_indegree(const unsigned long long* __restrict__ order, const uint32_t* __restrict__ dplus,
                               uint32_t n, unsigned long long* __restrict__ key) {
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t din = (uint32_t)(order[r] >> 32) - dplus[r];  // order[r] = degree << 32 | id
        key[r] = ((unsigned long long)(0xFFFFFFFFu - din) << 32) | r;
    }
}

// Collective degree W(r), larger first, ties by rank.
__global__ void k_key_collective(const unsigned long long* __restrict__ work, uint32_t n,
                                 unsigned long long* __restrict__ key) {
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x) {
        const unsigned long long w = work[r] > 0xFFFFFFFFull ? 0xFFFFFFFFull : work[r];
        key[r] = ((0xFFFFFFFFull - w) << 32) | r;
    }
}

// Greedy numbering of the collective order, in parallel: vertices taken in W order hand the next ids
// to their not-yet-numbered out-neighbours in the order of those' input ids, so v's id follows its first
// claim, the smallest (position of u in W order, input id of v) over its in-edges u -> v.  (Not the place
// in u's list, which differs from build to build.)  order: degree << 32 | input id of every rank.  One
// wavefront per row.
__global__ void k_claim(const int64_t* __restrict__ off, const uint32_t* __restrict__ col,
                        const uint32_t* __restrict__ posw, const unsigned long long* __restrict__ order, uint32_t n,
                        unsigned long long* __restrict__ claim) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t nwv = (gridDim.x * blockDim.x) >> 6;
    for (uint64_t r = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; r < n; r += nwv) {
        const int64_t b = off[r];
        const uint32_t d = (uint32_t)(off[r + 1] - b);
        const unsigned long long hi = (unsigned long long)posw[r] << 32;
        for (uint32_t j = lane; j < d; j += 64) {
            const uint32_t v = col[b + j];
            atomicMin(&claim[v], hi | (uint32_t)order[v]);
        }
    }
}

// Unclaimed vertices (no in-edges) follow every claimed one, by rank.
__global__ void k_key_claimed(uint32_t n, unsigned long long* __restrict__ claim) {
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x)
        if (claim[r] == ~0ull) claim[r] = (0xFFFFFFFFull << 32) | r;
}

__global__ void k_perm_dplus(const uint32_t* __restrict__ dplus, const uint32_t* __restrict__ pi, uint32_t n,
                             uint32_t* __restrict__ nd) {
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x) {
        nd[pi[r]] = dplus[r];
        if (r == 0) nd[n] = 0;
    }
}

// Row r of the CSR becomes row pi[r] with every entry v mapped to pi[v].  One wavefront per row.
__global__ void k_relabel_rows(const int64_t* __restrict__ off, const uint32_t* __restrict__ col,
                               const uint32_t* __restrict__ pi, const int64_t* __restrict__ off2, uint32_t n,
                               uint32_t* __restrict__ col2) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t nwv = (gridDim.x * blockDim.x) >> 6;
    for (uint64_t r = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; r < n; r += nwv) {
        const int64_t b = off[r];
        const uint32_t d = (uint32_t)(off[r + 1] - b);
        const int64_t b2 = off2[pi[r]];
        for (uint32_t j = lane; j < d; j += 64) col2[b2 + j] = pi[col[b + j]];
    }
}

__global__ void k_compose(uint32_t* __restrict__ rank, const uint32_t* __restrict__ pi, uint32_t n) {
    for (uint64_t x = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; x < n; x += (uint64_t)gridDim.x * blockDim.x) rank[x] = pi[rank[x]];
}

__global__ void k_scatter_u32(const uint32_t* __restrict__ in, const uint32_t* __restrict__ pi, uint32_t n,
                              uint32_t* __restrict__ out) {
    for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r < n; r += (uint64_t)gridDim.x * blockDim.x) out[pi[r]] = in[r];
}

__global__ void k_gather(const unsigned long long* __restrict__ tv, const uint32_t* __restrict__ rank, uint32_t n,
                         const uint32_t* __restrict__ place, unsigned long long* __restrict__ out) {
    for (uint64_t x = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; x < n; x += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t r = rank[x];
        out[x] = tv[place ? rec_id(place[2 * (uint64_t)r]) : r];
    }
}

#define TC_TRY(expr)                        \
    do {                                    \
        hipError_t e_ = (expr);             \
        if (e_ != hipSuccess) return e_;    \
    } while (0)

}  // namespace

hipError_t fill_u32(void* p, uint32_t value, size_t words, hipStream_t stream) {
    if (words == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(words)), dim3(kThreads), 0, stream, (uint32_t*)p, value, words);
    return hipGetLastError();
}

hipError_t clear_ranges(const Ranges& r, hipStream_t stream) {
    size_t most = 0;
    for (int q = 0; q < 3; ++q)
        if (r.p[q]) most = std::max(most, r.words[q]);
    if (most == 0) return hipSuccess;
    hipLaunchKernelGGL(k_clear_ranges, dim3(grid_for(most)), dim3(kThreads), 0, stream, r);
    return hipGetLastError();
}

hipError_t gather_per_vertex(const unsigned long long* tv, const uint32_t* rank, uint32_t n, const uint32_t* place,
                             unsigned long long* out, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather, dim3(grid_for(n)), dim3(kThreads), 0, stream, tv, rank, n, place, out);
    return hipGetLastError();
}

hipError_t clear_record_staging(unsigned long long* tv, const uint32_t* place, uint32_t n, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_clear_record_starts, dim3(grid_for(n)), dim3(kThreads), 0, stream, tv, place, n);
    return hipGetLastError();
}

size_t prep_sort_tmp_bytes(uint32_t n, bool relabel, bool scatter) {
    size_t best = 0, sz = 0;
    unsigned long long* k64 = nullptr;
    uint32_t* u32p = nullptr;
    int64_t* i64p = nullptr;
    if ((relabel || scatter) &&
        rocprim::exclusive_scan(nullptr, sz, u32p, i64p, (unsigned long long)0, (size_t)n + 1,
                                rocprim::plus<unsigned long long>()) == hipSuccess && sz > best) best = sz;
    sz = 0;
    if (rocprim::exclusive_scan(nullptr, sz, k64, k64, (unsigned long long)0, (size_t)place_chunks(n) + 1,
                                rocprim::plus<unsigned long long>()) == hipSuccess && sz > best) best = sz;
    sz = 0;
    if (relabel && rocprim::radix_sort_pairs(nullptr, sz, k64, k64, rocprim::counting_iterator<uint32_t>(0), u32p,
                                             (size_t)n, 0, 64) == hipSuccess && sz > best) best = sz;
    return best;
}

PrepZero prep_zero(uint32_t n, uint64_t m_in) {
    PrepZero z{};
    const uint32_t nb = id_bits(n);
    size_t w = kTicketWords + kHistWords;
    z.deg = w;     w += ((size_t)n + 1 + 3) & ~(size_t)3;
    z.first = w;   w += 2 * (((size_t)m_in + 63) / 64 + 1);
    z.bits = w;    w += (size_t)long_set_words(canon_low(nb), m_in);
    w = (w + 3) & ~(size_t)3;
    z.status = w;
    const uint64_t tm = pass_tiles(m_in, 8), tu = pass_tiles(m_in, 4), tn = pass_tiles(n, 8);
    const uint64_t words = std::max<uint64_t>({attach_ranks(nb) ? tm << upper_digit(nb) : tm * 512, upper_digit(nb) ? tu << upper_digit(nb) : 0, tn * 512});
    w += 2 * (size_t)words;
    z.words = w;
    return z;
}

hipError_t prep_init() {  // opt-in LDS: 2^15 counters of k_upper_count, as many ranks of k_orient_parts, k_sort_rows's bits
    TC_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(k_sort_rows), hipFuncAttributeMaxDynamicSharedMemorySize,
                               4 * kSortWords));
    TC_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(k_orient_parts),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)orient_lds(25)));
    return hipFuncSetAttribute(reinterpret_cast<const void*>(k_upper_count),
                               hipFuncAttributeMaxDynamicSharedMemorySize, 4 << kCounterBits);
}

inline uint32_t work_grid(uint32_t n) {
    return std::min(grid_for((uint64_t)n * kWorkLanes), 16384u);
}

// Relabel the oriented rank-space CSR into another order of hash ids (the orientation stays).
hipError_t relabel(uint32_t n, const GraphDev& g, const BuildTemp& t, const BatchIn* batch, uint32_t order,
                   uint64_t m_in, hipStream_t stream) {
    size_t tmp;
    const uint32_t wave_grid = std::min<uint32_t>(grid_for((uint64_t)n * 64), 8192u);
    hipLaunchKernelGGL(k_dplus, dim3(grid_for((uint64_t)n + 1)), dim3(kThreads), 0, stream, g.off32, n, t.dplus);
    TC_TRY(hipGetLastError());
    if (order == 1) {
        hipLaunchKernelGGL(k_key_indegree, dim3(grid_for(n)), dim3(kThreads), 0, stream, t.skey_a, t.dplus, n, t.rk_a);
        TC_TRY(hipGetLastError());
    } else {
        unsigned long long* work = t.skey_b;
        hipLaunchKernelGGL(k_work_rows, dim3(work_grid(n)), dim3(kThreads), 0, stream, g.off32, g.col, n, work);
        TC_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_key_collective, dim3(grid_for(n)), dim3(kThreads), 0, stream, work, n, t.rk_a);
        TC_TRY(hipGetLastError());
        tmp = t.sort_tmp_bytes;
        TC_TRY(rocprim::radix_sort_pairs(t.sort_tmp, tmp, t.rk_a, t.rk_b, rocprim::counting_iterator<uint32_t>(0),
                                         t.order, (size_t)n, 0, 64, stream));
        uint32_t* posw = reinterpret_cast<uint32_t*>(t.skey_b);
        hipLaunchKernelGGL(k_rank, dim3(grid_for(n)), dim3(kThreads), 0, stream, t.order, n, posw);
        TC_TRY(hipGetLastError());
        TC_TRY(fill_u32(t.rk_a, 0xFFFFFFFFu, 2 * (size_t)n, stream));
        hipLaunchKernelGGL(k_claim, dim3(wave_grid), dim3(kThreads), 0, stream, g.off, g.col, posw, t.skey_a, n,
                           t.rk_a);
        TC_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_key_claimed, dim3(grid_for(n)), dim3(kThreads), 0, stream, n, t.rk_a);
        TC_TRY(hipGetLastError());
    }
    tmp = t.sort_tmp_bytes;
    TC_TRY(rocprim::radix_sort_pairs(t.sort_tmp, tmp, t.rk_a, t.rk_b, rocprim::counting_iterator<uint32_t>(0),
                                     t.order, (size_t)n, 0, 64, stream));
    uint32_t* pi = t.deg;  // new id of every rank
    hipLaunchKernelGGL(k_rank, dim3(grid_for(n)), dim3(kThreads), 0, stream, t.order, n, pi);
    TC_TRY(hipGetLastError());
    uint32_t* nd = reinterpret_cast<uint32_t*>(t.skey_b);  // out-degrees by new id, [n + 1]
    hipLaunchKernelGGL(k_perm_dplus, dim3(grid_for(n)), dim3(kThreads), 0, stream, t.dplus, pi, n, nd);
    TC_TRY(hipGetLastError());
    tmp = t.sort_tmp_bytes;
    TC_TRY(rocprim::exclusive_scan(t.sort_tmp, tmp, nd, t.off2, (unsigned long long)0, (size_t)n + 1,
                                   rocprim::plus<unsigned long long>(), stream));
    uint32_t* col2 = reinterpret_cast<uint32_t*>(t.keys_b);
    hipLaunchKernelGGL(k_relabel_rows, dim3(wave_grid), dim3(kThreads), 0, stream, g.off, g.col, pi, t.off2, n, col2);
    TC_TRY(hipGetLastError());
    TC_TRY(hipMemcpyAsync(g.col, col2, 4 * (size_t)m_in, hipMemcpyDeviceToDevice, stream));
    TC_TRY(hipMemcpyAsync(g.off, t.off2, 8 * ((size_t)n + 1), hipMemcpyDeviceToDevice, stream));
    TC_TRY(hipMemcpyAsync(t.dplus, nd, 4 * ((size_t)n + 1), hipMemcpyDeviceToDevice, stream));
    hipLaunchKernelGGL(k_compose, dim3(grid_for(n)), dim3(kThreads), 0, stream, g.rank, pi, n);
    TC_TRY(hipGetLastError());
    if (batch) {
        TC_TRY(hipMemcpyAsync(t.order, g.gid, 4 * (size_t)n, hipMemcpyDeviceToDevice, stream));
        hipLaunchKernelGGL(k_scatter_u32, dim3(grid_for(n)), dim3(kThreads), 0, stream, t.order, pi, n, g.gid);
        TC_TRY(hipGetLastError());
    }
    return hipSuccess;
}

hipError_t prep_build(uint32_t n, uint64_t m_in, const uint32_t* src, const uint32_t* dst, const GraphDev& g,
                      const BuildTemp& t, const BinCaps& caps, const BatchIn* batch, int cu_count,
                      hipStream_t stream) {
    const uint32_t nb = id_bits(n);
    const unsigned long long sentinel = (2 * nb >= 64) ? ~0ull : ((1ull << (2 * nb)) - 1);
    const unsigned long long mask = (nb >= 32) ? 0xFFFFFFFFull : ((1ull << nb) - 1);
    size_t tmp = t.sort_tmp_bytes;

    // Zeroed memory: tickets and digit histograms, degrees, first bits, look-back words.
    uint32_t* next_ticket = t.zero;
    uint32_t* next_hist = t.zero + kTicketWords;
    uint32_t epoch = 0;
    auto take_hist = [&](uint32_t words) {
        uint32_t* h = next_hist;
        next_hist += words;
        return h;
    };
    TC_TRY(clear_ranges({{t.zero, reinterpret_cast<uint32_t*>(g.meta), caps.core_bits ? reinterpret_cast<uint32_t*>(g.rest_meta) : nullptr},
                         {t.zero_words, sizeof(GraphMeta) / 4, sizeof(GraphMeta) / 4}}, stream));
    // two workgroups of 1024 threads per CU: each ends with an atomic per digit
    const uint32_t hist_grid = (uint32_t)std::min<uint64_t>((m_in + 4095) / 4096, 2 * (uint64_t)cu_count);

    // 1-2: canonical keys (sorted into keys_b by all but their `low` lowest bits; batches form the keys
    // first: each sample's graph is searched for).
    const uint32_t cp = canon_passes(nb), low = canon_low(nb);
    {
        uint32_t* hist = take_hist(512 * cp);
        auto buf = [&](uint32_t writes_left) { return writes_left % 2 ? t.keys_b : t.keys_a; };  // the last write: keys_b
        const CanonKey canon{src, dst, n, nb, sentinel};
        unsigned long long* in = nullptr;
        if (batch) {
            in = buf(cp + 1);
            hipLaunchKernelGGL(k_canon_batch, dim3(hist_grid), dim3(1024), 0, stream, src, dst, m_in, n, nb, sentinel,
                               batch->voff, batch->eoff, batch->k, low, cp, in, hist, g.meta);
        } else {
            hipLaunchKernelGGL(k_canon_hist, dim3(hist_grid), dim3(1024), 0, stream, canon, m_in, low, cp, hist, g.meta);
        }
        TC_TRY(hipGetLastError());
        for (uint32_t p = 0; p < cp; ++p) {
            unsigned long long* out = buf(cp - p);
            const uint32_t shift = low + kDigit * p;
            if (p > 0)
                TC_TRY((radix_pass<kDigit, true, unsigned long long>(LoadKey{in}, StoreKey{out}, m_in, nullptr, shift,
                                                               hist + 512 * p, t.status, ++epoch, next_ticket++, stream)));
            else if (batch)
                TC_TRY((radix_pass<kDigit, false, unsigned long long>(LoadKey{in}, StoreKey{out}, m_in, nullptr, shift,
                                                               hist + 512 * p, t.status, ++epoch, next_ticket++, stream)));
            else
                TC_TRY((radix_pass<kDigit, false, unsigned long long>(canon, StoreKey{out}, m_in, nullptr, shift,
                                                               hist + 512 * p, t.status, ++epoch, next_ticket++, stream)));
            in = out;
        }
    }

    uint32_t* uhist = take_hist(1024);
    // 2-3: distinct edges and degrees, rank in (degree, id) order (the sort is stable).
    {
        const uint32_t ud = upper_digit(nb), sub = ud ? nb - ud : nb;
        const uint64_t tiles = (m_in + kDedupTile - 1) / kDedupTile;
        const uint32_t grid = (uint32_t)std::min<uint64_t>(tiles, 2 * (uint64_t)cu_count);
        const Dedup d{t.keys_b, m_in, sentinel, t.first, t.bits, t.deg, uhist, g.meta, t.zero + kTicketWords - 1, nb, low,
                      ud ? 1u << ud : 0u, sub, upper_atomics(nb)};
        hipLaunchKernelGGL(k_dedup, dim3(grid), dim3(kDedupThreads), 0, stream, d);
        TC_TRY(hipGetLastError());
        if (tiles >= kLongTiles) {
            hipLaunchKernelGGL(k_dedup_long, dim3(grid), dim3(kDedupThreads), 0, stream, d);
            TC_TRY(hipGetLastError());
        }
        const LoadUpper upper{t.keys_b, t.first, mask};
        uint32_t* ids = nullptr;
        if (ud) {
            ids = t.aux;
            if (ud == 9)
                TC_TRY((radix_pass<9, false, uint32_t>(upper, StoreId{ids}, m_in, nullptr, sub, uhist, t.status, ++epoch,
                                                next_ticket++, stream)));
            else
                TC_TRY((radix_pass<10, false, uint32_t>(upper, StoreId{ids}, m_in, nullptr, sub, uhist, t.status, ++epoch,
                                                 next_ticket++, stream)));
        }
        if (!upper_atomics(nb)) {
            const uint32_t unit = (uint32_t)std::max<uint64_t>(4096, std::min<uint64_t>(kUpperUnit, m_in / 512));
            const uint64_t units = (m_in + unit - 1) / unit + (ud ? 1u << ud : 1u);
            hipLaunchKernelGGL(k_upper_count, dim3((uint32_t)std::min<uint64_t>(units, 2 * (uint32_t)cu_count)), dim3(1024),
                               4u << std::min(sub, kCounterBits), stream, ids, upper, m_in, ud ? 1u << ud : 1u, sub, n,
                               uhist, unit, t.deg);
            TC_TRY(hipGetLastError());
        }
    }
    {
        const uint32_t passes = (degree_bits(n, m_in) + kDigit - 1) / kDigit;
        uint32_t* hist = take_hist(512 * passes);
        hipLaunchKernelGGL(k_degree_hist, dim3(std::min(((n - 1) / 4096) + 1, 512u)), dim3(1024), 0, stream, t.deg, n,
                           passes, hist);
        TC_TRY(hipGetLastError());
        auto buf = [&](uint32_t writes_left) { return writes_left % 2 ? t.skey_a : t.skey_b; };  // the last write: skey_a
        const StoreRank last{t.skey_a, g.rank, batch ? batch->voff : nullptr, batch ? batch->k : 0u, g.gid};
        for (uint32_t p = 0; p < passes; ++p) {
            const uint32_t* h = hist + 512 * p;
            const uint32_t shift = 32 + kDigit * p;
            unsigned long long* in = buf(passes - p + 1);
            unsigned long long* out = buf(passes - p);
            const bool end = p + 1 == passes;
            const LoadDegree deg{t.deg};
            if (p == 0 && end)
                TC_TRY((radix_pass<kDigit, true, unsigned long long>(deg, last, n, nullptr, shift, h, t.status, ++epoch,
                                                               next_ticket++, stream)));
            else if (p == 0)
                TC_TRY((radix_pass<kDigit, true, unsigned long long>(deg, StoreKey{out}, n, nullptr, shift, h, t.status, ++epoch,
                                                               next_ticket++, stream)));
            else if (end)
                TC_TRY((radix_pass<kDigit, true, unsigned long long>(LoadKey{in}, last, n, nullptr, shift, h, t.status, ++epoch,
                                                               next_ticket++, stream)));
            else
                TC_TRY((radix_pass<kDigit, true, unsigned long long>(LoadKey{in}, StoreKey{out}, n, nullptr, shift, h, t.status,
                                                               ++epoch, next_ticket++, stream)));
        }
    }

    // 4-5: orientation and CSR in rank space.
    unsigned long long* const osorted = reinterpret_cast<unsigned long long*>(t.aux);
    if (!caps.scatter_csr) {
        // Sort the oriented keys by row only (the high nb bits; lists need no order for hashing, so the first
        // pass keeps none): rows come out contiguous, in aux.
        const uint32_t passes = row_passes(nb);
        auto buf = [&](uint32_t writes_left) { return writes_left % 2 ? osorted : t.keys_a; };
        uint32_t* hist = take_hist(512 * passes);
        unsigned long long* in = buf(passes + 1);
        const bool attach = !batch && attach_ranks(nb);
        if (attach) {
            const uint32_t ud = upper_digit(nb), sub = nb - ud;
            unsigned long long* ranked = buf(passes);
            const LoadRanked load{t.keys_b, t.first, g.rank, n, nb, mask};
            if (ud == 9)
                TC_TRY((radix_pass<9, false, unsigned long long>(load, StoreKey{ranked}, m_in, nullptr, sub, uhist, t.status,
                                                          ++epoch, next_ticket++, stream)));
            else
                TC_TRY((radix_pass<10, false, unsigned long long>(load, StoreKey{ranked}, m_in, nullptr, sub, uhist, t.status,
                                                           ++epoch, next_ticket++, stream)));
            // four units per CU or more (R-MAT 22 in units of 2^19: half the CUs idle), large enough to load ranks for
            const uint32_t unit = (uint32_t)std::max<uint64_t>(1u << 15, m_in / (4 * (uint64_t)cu_count));
            hipLaunchKernelGGL(k_orient_parts, dim3(2 * (uint32_t)cu_count), dim3(1024), orient_lds(nb), stream, ranked, nb,
                               1u << ud, sub, n, uhist, unit, g.rank, passes, in, hist);
        } else {
            hipLaunchKernelGGL(k_orient_keys, dim3(hist_grid), dim3(1024), 0, stream, t.keys_b, nb, m_in,
                               t.first, g.rank, passes, in, hist);
        }
        TC_TRY(hipGetLastError());
        for (uint32_t p = 0; p < passes; ++p) {
            unsigned long long* out = buf(passes - p);
            const uint32_t shift = nb + kDigit * p;
            if (p == 0 && !attach)
                TC_TRY((radix_pass<kDigit, false, unsigned long long>(LoadFirst{in, t.first}, StoreKey{out}, m_in, nullptr, shift,
                                                               hist, t.status, ++epoch, next_ticket++, stream)));
            else
                TC_TRY((radix_pass<kDigit, true, unsigned long long>(LoadKey{in}, StoreKey{out}, m_in, &g.meta->m, shift,
                                                               hist + 512 * p, t.status, ++epoch, next_ticket++, stream)));
            in = out;
        }
        hipLaunchKernelGGL(k_csr, dim3(std::min(grid_for(std::max<uint64_t>(m_in, n)), 16384u)), dim3(kThreads), 0, stream,
                           osorted, nb, g.meta, n, g.off, g.off32, g.col, t.skey_b);
        TC_TRY(hipGetLastError());
    } else {
        // Counting sort: out-degrees, offsets, then an atomic scatter (list order unspecified).
        TC_TRY(fill_u32(t.dplus, 0, (size_t)n + 1, stream));
        hipLaunchKernelGGL(k_orient_count, dim3(grid_for(m_in)), dim3(kThreads), 0, stream, t.keys_b, nb, m_in,
                           t.first, g.rank, t.dplus);
        TC_TRY(hipGetLastError());
        tmp = t.sort_tmp_bytes;
        TC_TRY(rocprim::exclusive_scan(t.sort_tmp, tmp, t.dplus, g.off, (unsigned long long)0, (size_t)n + 1,
                                       rocprim::plus<unsigned long long>(), stream));
        TC_TRY(fill_u32(t.deg, 0, (size_t)n + 1, stream));
        hipLaunchKernelGGL(k_orient_fill, dim3(grid_for(m_in)), dim3(kThreads), 0, stream, t.keys_b, nb, m_in,
                           t.first, g.rank, g.off, t.deg, g.col);
        TC_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_narrow, dim3(grid_for((uint64_t)n + 1)), dim3(kThreads), 0, stream, g.off, (uint64_t)n + 1,
                           g.off32);
        TC_TRY(hipGetLastError());
    }

    // 5b (optional): hash ids in another vertex order.
    if (caps.order) {
        TC_TRY(relabel(n, g, t, batch, caps.order, m_in, stream));
        hipLaunchKernelGGL(k_narrow, dim3(grid_for((uint64_t)n + 1)), dim3(kThreads), 0, stream, g.off, (uint64_t)n + 1,
                           g.off32);
        TC_TRY(hipGetLastError());
    }

    // 6: W(u), bins and largest-work-first order.  5c with it: records are placed first ({p(r), d+(r)} per
    // rank), then k_work reads v's placement for d+(v) and writes p(v) into the records.
    uint32_t* rec = (caps.records && !caps.order && !caps.scatter_csr) ? g.rec : nullptr;
    unsigned long long* const work = t.skey_b;
    if (!caps.order && !caps.scatter_csr) {
        hipLaunchKernelGGL(k_owners, dim3(std::min((n - 1) / 1024 + 1, 2 * (uint32_t)cu_count)), dim3(1024), 0, stream,
                           g.off32, t.skey_a, n, caps.big_cap, g.meta);
        TC_TRY(hipGetLastError());
        // (out-degrees are at most sqrt(2 m); record ids follow record sizes, not ranks)
        const uint64_t words = (std::min<uint64_t>(n, 2 * m_in / (caps.big_cap + 1) + 1) + 31) / 32;
        if (!rec && 2 * m_in > (uint64_t)caps.big_cap * caps.big_cap && words <= kSortWords) {
            hipLaunchKernelGGL(k_sort_rows, dim3(2 * (uint32_t)cu_count), dim3(1024), 4 * (uint32_t)words, stream, g.meta,
                               g.off32, n, nb, g.col, osorted);
            TC_TRY(hipGetLastError());
        }
    }
    if (rec) {
        const uint64_t chunks = place_chunks(n);
        hipLaunchKernelGGL(k_place_size, dim3(grid_for(chunks + 1)), dim3(kThreads), 0, stream, g.off32, n,
                           t.place_sz);
        TC_TRY(hipGetLastError());
        tmp = t.sort_tmp_bytes;
        unsigned long long* cbase = t.place_sz + chunks + 1;
        TC_TRY(rocprim::exclusive_scan(t.sort_tmp, tmp, t.place_sz, cbase, (unsigned long long)0,
                                       (size_t)chunks + 1, rocprim::plus<unsigned long long>(), stream));
        uint2* place = reinterpret_cast<uint2*>(g.place);
        hipLaunchKernelGGL(k_place_write, dim3(grid_for(chunks + 1)), dim3(kThreads), 0, stream, g.off32, n,
                           cbase, place);
        TC_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_record_empty, dim3(grid_for(n)), dim3(kThreads), 0, stream, place, n, rec);
        TC_TRY(hipGetLastError());
    }
    if (caps.order || caps.scatter_csr) {
        hipLaunchKernelGGL(k_work_rows, dim3(work_grid(n)), dim3(kThreads), 0, stream, g.off32, g.col, n, work);
    } else {
        const uint32_t grid = (uint32_t)std::min<uint64_t>((m_in + 1023) / 1024, 32 * (uint64_t)cu_count);
        if (rec)
            hipLaunchKernelGGL(k_work<true>, dim3(grid), dim3(kThreads), 0, stream, osorted, nb, g.off32,
                               reinterpret_cast<const uint2*>(g.place), rec, g.meta, work, g.elist);
        else
            hipLaunchKernelGGL(k_work<false>, dim3(grid), dim3(kThreads), 0, stream, osorted, nb, g.off32, nullptr, nullptr,
                               g.meta, work, g.elist);
    }
    TC_TRY(hipGetLastError());
    if (caps.pack_cap && !(caps.force_hub || caps.force_big || caps.force_wg)) {
        hipLaunchKernelGGL(k_pack_census, dim3(std::min((n - 1) / 1024 + 1, 2 * (uint32_t)cu_count)), dim3(1024), 0, stream,
                           g.off32, work, n, caps, g.meta);
        TC_TRY(hipGetLastError());
    }
    // one block of 1024 threads per CU: each ends with some 20 atomics on the same summary words (R-MAT 20:
    // 1024 blocks of 256 threads spent 0.1 ms on them)
    {
        uint32_t* hist = take_hist(1024);
        hipLaunchKernelGGL(k_schedule, dim3(std::min((n - 1) / 1024 + 1, (uint32_t)cu_count)), dim3(1024), 0, stream, g.off32, work, n,
                           caps, g.meta, t.skey_a, hist);
        TC_TRY(hipGetLastError());
        TC_TRY((radix_pass<kDigit, true, unsigned long long>(LoadKey{t.skey_a}, StoreKey{t.skey_b}, n, nullptr, 32, hist,
                                                       t.status, ++epoch, next_ticket++, stream)));
        TC_TRY((radix_pass<kDigit, true, unsigned long long>(LoadKey{t.skey_b}, StoreItem{g.items}, n, nullptr, 32 + kDigit,
                                                       hist + 512, t.status, ++epoch, next_ticket++, stream)));
    }
    // 7: block words of the core path and the schedule of the lists cut before the core.
    if (caps.core_bits) {
        CoreBuild c{};
        c.meta = g.meta;
        c.off = g.off32;
        c.okeys = osorted;
        c.mask = mask;
        c.nb = nb;
        c.col = g.col;
        c.blk = reinterpret_cast<uint32_t*>(g.blk);
        c.bl = g.bl;
        c.rend = g.rend;
        c.items = g.items;
        c.rest_meta = g.rest_meta;
        c.rest_items = g.rest_items;
        c.cls = t.order;
        c.hist = take_hist(2 * kRestClasses);
        c.n = n;
        c.m_in = m_in;
        c.S = caps.core_bits;
        c.c0 = caps.core_first;
        c.magic = core_magic(c.S);
        c.big_all = caps.core_big_all;
        c.caps = caps;
        TC_TRY(core_build(c, cu_count, stream));
    }
    return hipSuccess;
}

}  // namespace tc
