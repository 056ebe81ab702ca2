// The core path: owners with much 2-hop work probe their out-neighbours' lists 20-22 ids at a time.
//
// Ranks follow degree, so on skewed graphs nearly every 2-hop id is one of the last K ranks (the core;
// R-MAT scale 22: 99% of the probes end in the last 43,008 of 4.2 M ranks), and a list's core ids crowd
// together.  Each list's core ids are stored as block words: block index << S | S-bit mask of the
// block's ids, S = 20..22 (core_shape), one word per block that holds any (R-MAT 22: 2.8 ids per word;
// every list padded to whole 16-byte quads).  An owner u keeps its own words in an LDS table indexed by
// the block (2^(32-S) words: no hashing, no chains, no filter), and a probe is
//     hits += popcount(table[word >> S] & word),
// three vector instructions and one 4-byte LDS read for up to S ids, where the bucket path takes about
// 15-20 instructions per id; a wavefront reads 1 KB of a list per load.
//
// A triangle (u, v, w), ranks ascending, is counted here when w is in the core.  When w is not, v and
// w are both outside, so those triangles are the ones of the graph with every list cut before its core
// ids: the bucket kernels count them over the same owners with the cut lists (rest_meta, rest_items;
// lists keep their ids outside the core first, end at rend).  Owners with little work (W(u) below
// kCoreMinWork) stay on the bucket kernels with their whole lists: the packed and wavefront paths have
// less fixed work per owner.
//
// Whether a graph takes this path is decided on the device (core_on): the owners with enough work must
// hold at least half of W+, and the path must find enough 2-hop ids per edge in the core.
#include <algorithm>

#include "tc_fetch.h"
#include "tc_internal.h"
#include "tc_wave.h"

namespace tc {
namespace {

// ---------------------------------------------------------------- build: block words

__device__ __forceinline__ uint32_t block_of(uint32_t x, uint32_t magic) { return __umulhi(x, magic); }

// Rows that lie within a tile of 2048 consecutive edges: an LDS hash table of (row in the tile, block)
// collects the block masks, and the edge that brought a block writes its word once the masks are
// complete; positions in the row come from prefix counts over one bit per edge.  No row waits for another:
// one wavefront per row, each with a table of its own, took 0.96 ms at R-MAT 22 (4.2 M rows, a chain of LDS
// accesses each) against 0.60 ms here with the rows that cross tiles.
constexpr uint32_t kTileThreads = 512, kTileItems = 4, kTileEdges = kTileThreads * kTileItems;
constexpr uint32_t kTileWords = kTileEdges / 64, kTileSlots = 2 * kTileEdges;  // 2^12

// Set bits of a tile's bit set before position p (pre: set bits before each word).
__device__ __forceinline__ uint32_t bits_before(const unsigned long long* w, const uint32_t* pre, uint32_t p) {
    if (p == kTileEdges) return pre[kTileWords];
    return pre[p >> 6] + (uint32_t)__popcll(w[p >> 6] & ((1ull << (p & 63u)) - 1ull));
}

__global__ void __launch_bounds__(kTileThreads) k_core_tiles(CoreBuild a) {
    __shared__ uint32_t s_key[kTileSlots], s_mask[kTileSlots];
    __shared__ unsigned long long s_start[kTileWords], s_rest[kTileWords], s_new[kTileWords];
    __shared__ uint32_t s_row[kTileWords + 1], s_prer[kTileWords + 1], s_pren[kTileWords + 1];
    if (!core_on(*a.meta)) return;
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint64_t m = a.meta->m;
    const uint32_t S = a.S;
    for (uint64_t base = blockIdx.x * (uint64_t)kTileEdges; base < m; base += (uint64_t)gridDim.x * kTileEdges) {
        const uint32_t len = m - base < kTileEdges ? (uint32_t)(m - base) : kTileEdges;
        uint32_t row[kTileItems], id[kTileItems];
#pragma unroll
        for (uint32_t i = 0; i < kTileItems; ++i) {
            const uint32_t p = wave * (64u * kTileItems) + i * 64u + lane;
            const unsigned long long k = a.okeys[base + (p < len ? p : len - 1)];
            row[i] = (uint32_t)(k >> a.nb);
            id[i] = (uint32_t)(k & a.mask);
        }
        for (uint32_t i = tid; i < kTileSlots; i += kTileThreads) {
            s_key[i] = kNone;
            s_mask[i] = 0;
        }
#pragma unroll
        for (uint32_t i = 0; i < kTileItems; ++i) {
            const uint32_t p = wave * (64u * kTileItems) + i * 64u + lane;
            uint32_t prev = (uint32_t)__shfl_up((int)row[i], 1, 64);
            if (lane == 0 && base + p > 0 && p < len) prev = (uint32_t)(a.okeys[base + p - 1] >> a.nb);
            const bool start = p < len && (base + p == 0 || prev != row[i]);
            const unsigned long long st = __ballot(start), rs = __ballot(p < len && id[i] < a.c0);
            if (lane == 0) {
                s_start[wave * kTileItems + i] = st;
                s_rest[wave * kTileItems + i] = rs;
                s_new[wave * kTileItems + i] = 0;
            }
        }
        // the tile's last row is closed when the next edge is another row's (or there is none)
        const bool open = base + len < m &&
                          (uint32_t)(a.okeys[base + len] >> a.nb) == (uint32_t)(a.okeys[base + len - 1] >> a.nb);
        __syncthreads();
        const unsigned long long starts = lane < kTileWords ? s_start[lane] : 0ull;
        const unsigned long long has = __ballot(starts != 0);
        if (wave == 0) {
            const uint32_t c = (uint32_t)__popcll(starts), r = lane < kTileWords ? (uint32_t)__popcll(s_rest[lane]) : 0u;
            const uint32_t ic = wave_incl_scan(c), ir = wave_incl_scan(r);
            if (lane <= kTileWords) {
                s_row[lane] = ic - c;
                s_prer[lane] = ir - r;
            }
        }
        __syncthreads();
        if (!has) continue;  // uniform: the whole tile lies inside one row
        const uint32_t w0 = (uint32_t)__builtin_ctzll(has), w1 = 63u - (uint32_t)__builtin_clzll(has);
        const uint32_t p0 = w0 * 64u + (uint32_t)__builtin_ctzll(s_start[w0]);
        const uint32_t stop = open ? w1 * 64u + 63u - (uint32_t)__builtin_clzll(s_start[w1]) : len;
        // blocks: which edges bring one
        uint32_t slot[kTileItems], first = 0;
#pragma unroll
        for (uint32_t i = 0; i < kTileItems; ++i) {
            const uint32_t p = wave * (64u * kTileItems) + i * 64u + lane;
            slot[i] = 0;
            if (p < p0 || p >= stop || id[i] < a.c0) continue;
            const uint32_t g = bits_before(s_start, s_row, p) + ((s_start[p >> 6] >> (p & 63u)) & 1ull ? 1u : 0u);
            const uint32_t x = id[i] - a.c0, idx = block_of(x, a.magic);
            const uint32_t name = (g << (32 - S)) | idx;  // 12 bits of row, 12 at most of block
            uint32_t at = (name * 0x9E3779B1u) >> 20;
            for (;;) {
                const uint32_t old = atomicCAS(&s_key[at], kNone, name);
                if (old == kNone) first |= 1u << i;
                if (old == kNone || old == name) break;
                at = (at + 1) & (kTileSlots - 1);
            }
            slot[i] = at;
            atomicOr(&s_mask[at], 1u << (x - idx * S));
        }
#pragma unroll
        for (uint32_t i = 0; i < kTileItems; ++i) {
            const unsigned long long f = __ballot((first >> i) & 1u);
            if (lane == 0) s_new[wave * kTileItems + i] = f;
        }
        __syncthreads();
        if (wave == 0) {
            const uint32_t c = lane < kTileWords ? (uint32_t)__popcll(s_new[lane]) : 0u;
            const uint32_t ic = wave_incl_scan(c);
            if (lane <= kTileWords) s_pren[lane] = ic - c;
        }
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < kTileItems; ++i) {
            const uint32_t p = wave * (64u * kTileItems) + i * 64u + lane;
            if (p < p0 || p >= stop) continue;
            // the row's edges [rs, re): the last start at or before p, the first after it
            uint32_t w = p >> 6;
            unsigned long long b = s_start[w] & ((2ull << (p & 63u)) - 1ull);
            while (!b) b = s_start[--w];
            const uint32_t rs = w * 64u + 63u - (uint32_t)__builtin_clzll(b);
            uint32_t re = stop;
            w = p >> 6;
            b = (p & 63u) == 63u ? 0ull : s_start[w] & ~((2ull << (p & 63u)) - 1ull);
            while (!b && ++w < kTileWords) b = s_start[w];
            if (b) {
                const uint32_t q = w * 64u + (uint32_t)__builtin_ctzll(b);
                re = q < stop ? q : stop;
            }
            const uint32_t r0 = bits_before(s_rest, s_prer, rs), rests = bits_before(s_rest, s_prer, re) - r0;
            const uint32_t rest_at = bits_before(s_rest, s_prer, p) - r0;
            const bool rest = id[i] < a.c0;
            const uint32_t off = (uint32_t)base + rs;
            a.col[off + (rest ? rest_at : rests + (p - rs - rest_at))] = id[i];
            const uint32_t n0 = bits_before(s_new, s_pren, rs);
            uint32_t* const out = a.blk + 4 * core_start(off, row[i]);
            if ((first >> i) & 1u) {
                const uint32_t name = s_key[slot[i]];
                out[bits_before(s_new, s_pren, p) - n0] = (name << S) | s_mask[slot[i]];  // the row's bits shift out
            }
            if (p == rs) {
                const uint32_t nw = bits_before(s_new, s_pren, re) - n0;
                for (uint32_t z = nw; z < ((nw + 3u) & ~3u); ++z) out[z] = 0;
                a.bl[row[i]] = make_uint2((uint32_t)core_start(off, row[i]), (nw + 3u) / 4u);
                a.rend[row[i]] = off + rests;
            }
        }
        __syncthreads();  // the LDS is reused by the next tile
    }
}

// The other rows: those that cross a tile's end, one wavefront each (the wavefront of the tile where the row
// begins), and those without edges.  The row's core ids are ORed into the wavefront's LDS table of block
// masks (2^(32-S) words); the first lane to take a block's mask back (an exchange with zero, which also
// clears the table) writes its word.  The row's ids go to col, those outside the core first.
__global__ void __launch_bounds__(64) k_core_rows(CoreBuild a) {
    extern __shared__ __align__(16) uint32_t T[];
    if (!core_on(*a.meta)) return;
    const uint32_t lane = threadIdx.x, S = a.S, words = 1u << (32 - S);
    for (uint64_t r = blockIdx.x * 64ull + lane; r < a.n; r += gridDim.x * 64ull) {
        const uint32_t b = a.off[r];
        if (a.off[r + 1] == b) {
            a.bl[r] = make_uint2((uint32_t)core_start(b, (uint32_t)r), 0u);
            a.rend[r] = b;
        }
    }
    for (uint32_t i = lane; i < words; i += 64) T[i] = 0;
    wave_sync();
    const uint64_t m = a.meta->m;
    auto key = [&](uint64_t at) { return (uint32_t)(a.okeys[at] & a.mask); };
    for (uint64_t e = (blockIdx.x + 1ull) * kTileEdges; e < m; e += (uint64_t)gridDim.x * kTileEdges) {
        const uint32_t r = __builtin_amdgcn_readfirstlane((uint32_t)(a.okeys[e] >> a.nb));
        const uint32_t beg = __builtin_amdgcn_readfirstlane(a.off[r]);
        if (beg >= e || beg < e - kTileEdges) continue;  // begins here, or belongs to an earlier tile's end
        const uint32_t d = __builtin_amdgcn_readfirstlane(a.off[r + 1]) - beg;
        uint32_t* const out = a.blk + 4 * core_start(beg, r);
        uint32_t rest = 0, cores = 0, nb = 0;
        for (uint32_t c = 0; c < d; c += 64) {  // masks, and the ids outside the core
            const bool act = c + lane < d;
            const uint32_t id = act ? key((uint64_t)beg + c + lane) : 0u;
            const bool core = act && id >= a.c0;
            if (core) {
                const uint32_t x = id - a.c0, idx = block_of(x, a.magic);
                atomicOr(&T[idx], 1u << (x - idx * S));
            }
            const unsigned long long rm = __ballot(act && !core);
            if (act && !core) a.col[beg + rest + lanes_below(rm)] = id;
            rest += (uint32_t)__popcll(rm);
        }
        wave_sync();
        for (uint32_t c = 0; c < d; c += 64) {  // block words, and the core ids
            const bool act = c + lane < d;
            const uint32_t id = act ? key((uint64_t)beg + c + lane) : 0u;
            const bool core = act && id >= a.c0;
            uint32_t word = 0;
            if (core) {
                const uint32_t idx = block_of(id - a.c0, a.magic);
                const uint32_t mk = atomicExch(&T[idx], 0u);
                if (mk) word = (idx << S) | mk;
            }
            const unsigned long long cm = __ballot(core), fm = __ballot(word != 0);
            if (core) a.col[beg + rest + cores + lanes_below(cm)] = id;
            if (word) out[nb + lanes_below(fm)] = word;
            cores += (uint32_t)__popcll(cm);
            nb += (uint32_t)__popcll(fm);
        }
        wave_sync();
        if (lane < ((0u - nb) & 3u)) out[nb + lane] = 0;
        if (lane == 0) {
            a.bl[r] = make_uint2((uint32_t)core_start(beg, r), (nb + 3u) / 4u);
            a.rend[r] = beg + rest;
        }
    }
}

// ---------------------------------------------------------------- build: the cut lists' schedule

// Owners of the core path that have triangles outside the core: cut lists of at least two ids with 2-hop
// work, in the bins of the bucket kernels by cut out-degree, each bin by the power of two of its work
// (largest first).  Five groups: the global-table bin, the two parts of the large-LDS bin, the workgroup
// and the wavefront bin.
constexpr uint32_t kRestLanes = 8;  // lanes per owner

__device__ __forceinline__ uint32_t heavy_items(const GraphMeta& m, uint32_t big_lo, uint32_t& base) {
    base = m.bins[0] + big_lo;
    return m.bins[1] - big_lo + m.bins[2] + m.heavy3;
}

__global__ void __launch_bounds__(256) k_rest_classes(CoreBuild a) {
    __shared__ uint32_t s_h[kRestClasses];
    const GraphMeta& m = *a.meta;
    if (!core_on(m)) return;
    for (uint32_t i = threadIdx.x; i < kRestClasses; i += blockDim.x) s_h[i] = 0;
    __syncthreads();
    uint32_t base;
    const uint32_t cnt = heavy_items(m, a.big_all ? 0u : m.big_full, base);
    const uint32_t sub = threadIdx.x % kRestLanes, per = blockDim.x / kRestLanes;
    for (uint32_t j0 = blockIdx.x * per; j0 < cnt; j0 += gridDim.x * per) {
        const uint32_t j = j0 + threadIdx.x / kRestLanes;
        uint32_t d = 0, w = 0;
        if (j < cnt) {
            const uint32_t u = a.items[base + j], b = a.off[u];
            d = a.rend[u] - b;
            if (d >= 2)
                for (uint32_t p = sub; p < d; p += kRestLanes) {
                    const uint32_t v = a.col[b + p];
                    w += a.rend[v] - a.off[v];
                }
        }
        for (uint32_t o = 1; o < kRestLanes; o <<= 1) w += __shfl_xor(w, o);
        if (sub == 0 && j < cnt) {
            uint32_t cls = 0xFFFFFFFFu;
            if (d >= 2 && w) {
                const uint32_t g = d > a.caps.big_cap ? 0u
                                   : d > a.caps.wg_cap ? (d <= a.caps.mid_cap ? 2u : 1u)
                                                       : d > a.caps.wave_cap ? 3u : 4u;
                cls = g * 32u + (uint32_t)__builtin_clz(w);
                atomicAdd(&s_h[cls], 1u);
            }
            a.cls[j] = cls;
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kRestClasses; i += blockDim.x)
        if (s_h[i]) atomicAdd(&a.hist[i], s_h[i]);
}

__global__ void __launch_bounds__(256) k_rest_place(CoreBuild a) {
    __shared__ uint32_t s_start[kRestClasses + 1], s_n[kRestClasses], s_at[kRestClasses];
    const GraphMeta& m = *a.meta;
    if (!core_on(m)) return;
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (uint32_t i = 0; i < kRestClasses; ++i) {
            s_start[i] = t;
            t += a.hist[i];
        }
        s_start[kRestClasses] = t;
    }
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        GraphMeta* r = a.rest_meta;
        r->bins[0] = s_start[32];
        r->bins[1] = s_start[96] - s_start[32];
        r->big_full = s_start[64] - s_start[32];
        r->bins[2] = s_start[128] - s_start[96];
        r->bins[3] = s_start[160] - s_start[128];
    }
    uint32_t base;
    const uint32_t cnt = heavy_items(m, a.big_all ? 0u : m.big_full, base);
    for (uint32_t j0 = blockIdx.x * blockDim.x; j0 < cnt; j0 += gridDim.x * blockDim.x) {
        for (uint32_t i = threadIdx.x; i < kRestClasses; i += blockDim.x) s_n[i] = 0;
        __syncthreads();
        const uint32_t j = j0 + threadIdx.x;
        const uint32_t cls = j < cnt ? a.cls[j] : 0xFFFFFFFFu;
        uint32_t at = 0;
        if (cls != 0xFFFFFFFFu) at = atomicAdd(&s_n[cls], 1u);
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < kRestClasses; i += blockDim.x)
            if (s_n[i]) s_at[i] = s_start[i] + atomicAdd(&a.hist[kRestClasses + i], s_n[i]);
        __syncthreads();
        if (cls != 0xFFFFFFFFu) a.rest_items[s_at[cls] + at] = a.items[base + j];
        __syncthreads();
    }
}

// ---------------------------------------------------------------- count

constexpr uint32_t kCoreQueue = 128;  // entries of a wavefront's hit queue

// Per-vertex counts of the last kHotRanks ranks (by PART; what the LDS has room for) are summed in LDS by each workgroup and added to the
// staging when it ends: the last ranks are members of nearly every owner's list, and global atomics on
// one address run at about 1.5e8/s (R-MAT 16: 2e4 adds to the last rank alone).  One owner adds at most
// twice its out-degree (8192) to a rank, so kHotOwners owners fit 32 bits.
constexpr uint32_t kHotRanks[3] = {512, 1024, 1024}, kHotOwners = 1u << 17;

// The probe of one wavefront over quads [lo, hi) of the owner's flattened lists.  As in the bucket
// kernels each lane keeps a forward-only cursor (k, cur, end), here in units of 16-byte quads.
//
// Per-vertex mode: words with hits go to the wavefront's queue as {block << S | hit mask, k}; with 64
// of them queued, the last 64 are taken together: their hit counts are added to tally[k] once per run of
// equal k (neighbouring entries come from the same list), and their two lowest hit bits each to the tally
// of its member, whose index is the block's first member (kept above the mask in the table) plus the
// members below it.  Entries with more bits go back to the queue (k = kTallied): most words have one hit
// and a few many, and taking all bits at once made 64 entries wait for the fullest.
constexpr uint32_t kTallied = 0xFFFFFFFFu;

template <bool PV>
struct CoreProbe {
    const uint4* __restrict__ blk;
    const uint32_t* T;
    const u32x2* P;
    uint32_t* tally;   // hits by out-neighbour k (the triangle's v)
    uint32_t* member;  // hits by core member of the owner's list, in block order (the triangle's w)
    u32x2* queue;
    uint32_t S, mask;
    int lane;
    uint32_t hits = 0, qn = 0;

    __device__ __forceinline__ void take(uint32_t cnt) {  // the last cnt <= 64 queue entries
        wave_sync();
        const bool act = (uint32_t)lane < cnt;
        u32x2 e = u32x2{0u, 0u};
        if (act) e = queue[qn - cnt + (uint32_t)lane];
        qn -= cnt;
        uint32_t h = e.x & mask;
        const uint32_t c = e.y == kTallied ? 0u : (uint32_t)__popc(h);
        const uint32_t incl = wave_incl_scan(c);
        const uint32_t kprev = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)e.y, 0x138, 0xf, 0xf, false);
        const uint32_t knext = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)e.y, 0x130, 0xf, 0xf, false);
        if (c && ((uint32_t)lane + 1u == cnt || knext != e.y)) atomicAdd(&tally[e.y], incl);
        if (c && lane != 0 && kprev != e.y) atomicSub(&tally[e.y], incl - c);
        const uint32_t r = T[e.x >> S];
        const uint32_t members = r & mask, at = r >> S;
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (h) {
                const uint32_t bit = h & (0u - h);
                h ^= bit;
                atomicAdd(&member[at + (uint32_t)__popc(members & (bit - 1u))], 1u);
            }
        const unsigned long long more = __ballot(h != 0);
        if (more) {
            wave_sync();
            if (h) queue[qn + lanes_below(more)] = u32x2{(e.x & ~mask) | h, kTallied};
            qn += (uint32_t)__popcll(more);
        }
        wave_sync();
    }

    __device__ __forceinline__ void word(uint32_t x, uint32_t k) {
        const uint32_t t = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(T) + ((x >> (S - 2)) & ~3u));
        if constexpr (!PV) {
            hits += (uint32_t)__popc(t & x);
        } else {
            const uint32_t h = t & x & mask;
            hits += (uint32_t)__popc(h);
            const unsigned long long m = __ballot(h != 0);
            if (h) queue[qn + lanes_below(m)] = u32x2{(x & ~mask) | h, k};
            qn += (uint32_t)__popcll(m);
            while (qn >= 64u) take(64u);  // (what a take puts back may keep it there)
        }
    }

    __device__ __forceinline__ void range(uint32_t d, uint32_t lo, uint32_t hi) {
        if (lo >= hi) return;
        uint32_t k, cur, end, base;
        {
            const uint32_t i0 = lo + (uint32_t)lane;
            k = vc_owner(d, i0 < hi ? i0 : hi - 1u, [&](uint32_t j) { return P[j].x; });
            const u32x2 rec = P[k];
            base = rec.y;
            cur = base + i0;
            end = base + rec.x;
        }
        auto fetch = [&](uint4& x, uint32_t& kk) {
            if (cur >= end) {
                const uint32_t i = cur - base;
                uint32_t e;
                do {
                    ++k;
                    const u32x2 rec = P[k];
                    e = rec.x;
                    base = rec.y;
                } while (i >= e);
                cur = base + i;
                end = base + e;
            }
            x = blk[cur];
            kk = k;
            cur += 64u;
        };
        auto quad = [&](const uint4& x, uint32_t kk) {
            word(x.x, kk);
            word(x.y, kk);
            word(x.z, kk);
            word(x.w, kk);
        };
        constexpr int U = 2;
        const uint32_t nfull = (hi - lo) >> 6;
        uint32_t c = 0;
        if (nfull >= 2u * U) {
            uint4 xa[U], xb[U];
            uint32_t ka[U], kb[U];
#pragma unroll
            for (int j = 0; j < U; ++j) fetch(xa[j], ka[j]);
            c = U;
            while (c + 2u * U <= nfull) {
#pragma unroll
                for (int j = 0; j < U; ++j) fetch(xb[j], kb[j]);
#pragma unroll
                for (int j = 0; j < U; ++j) quad(xa[j], ka[j]);
#pragma unroll
                for (int j = 0; j < U; ++j) fetch(xa[j], ka[j]);
#pragma unroll
                for (int j = 0; j < U; ++j) quad(xb[j], kb[j]);
                c += 2u * U;
            }
#pragma unroll
            for (int j = 0; j < U; ++j) quad(xa[j], ka[j]);
        }
        // the remaining chunks in pairs, the ragged last one with the lanes past hi idle
        const uint32_t last = lo + (nfull << 6) + (uint32_t)lane;
        while (true) {
            uint4 x[U];
            uint32_t kk[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                x[j] = make_uint4(0u, 0u, 0u, 0u);
                kk[j] = k;
                if (c + j < nfull || (c + j == nfull && last < hi)) fetch(x[j], kk[j]);
            }
#pragma unroll
            for (int j = 0; j < U; ++j)
                if (c + j <= nfull) quad(x[j], kk[j]);
            c += U;
            if (c > nfull) break;
        }
    }
};

// Sum of v over the workgroup up to and including this thread, and the workgroup's total.  `s` is a
// buffer of NW words that no other scan between the surrounding barriers uses; one barrier inside.
template <int NW>
__device__ __forceinline__ uint32_t group_scan(uint32_t v, uint32_t* s, int wave, int lane, uint32_t& total) {
    const uint32_t incl = wave_incl_scan(v);
    if (lane == 63) s[wave] = incl;
    __syncthreads();
    uint32_t before = 0, t = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const uint32_t x = s[w];
        before += w < wave ? x : 0u;
        t += x;
    }
    total = t;
    return before + incl;
}

// One workgroup of NW wavefronts per owner.  PART 0: the wavefront bin's owners with enough work
// (out-degree at most 64 NW, one list element and one own block word per thread; the next owner's are
// loaded while this one is probed), PART 1: the workgroup bin, PART 2: the large-LDS bin.
template <bool PV, int NW, int PART>
__global__ void __launch_bounds__(64 * NW) tc_core_kernel(CoreArgs a) {
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ uint32_t s_scan[2][NW];
    __shared__ uint32_t s_next;
    __shared__ unsigned long long s_acc[NW];
    constexpr bool ONE = PART == 0;
    constexpr uint32_t NT = 64 * NW;
    const GraphMeta& m = *a.meta;
    if (!core_on(m)) return;
    const uint32_t tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t S = a.S, mask = (1u << S) - 1u, words = 1u << (32 - S);
    uint32_t* const T = lds;
    u32x2* const P = reinterpret_cast<u32x2*>(lds + words);
    uint32_t* const tally = lds + words + 2 * a.dcap;
    uint32_t* const member = tally + a.dcap;
    u32x2* const queue = reinterpret_cast<u32x2*>(lds + words + (PV ? 4u : 2u) * a.dcap) + (uint32_t)wave * kCoreQueue;
    uint32_t* const hot = lds + words + 4u * a.dcap + 2u * kCoreQueue * NW;  // per-vertex mode
    constexpr uint32_t HR = kHotRanks[PART];
    const uint32_t hot0 = a.n > HR ? a.n - HR : 0u;
    uint32_t owners = 0;  // since the hot counts were last added to the staging
    auto flush_hot = [&]() {  // every thread, between barriers
        for (uint32_t i = tid; i < HR && hot0 + i < a.n; i += NT) {
            const uint32_t t = hot[i];
            if (t) atomicAdd(&a.tv[hot0 + i], (unsigned long long)t);
            hot[i] = 0;
        }
    };
    const uint32_t big_lo = a.big_all ? 0u : m.big_full;
    const uint32_t base = PART == 2 ? m.bins[0] + big_lo
                          : PART == 1 ? m.bins[0] + m.bins[1] : m.bins[0] + m.bins[1] + m.bins[2];
    const uint32_t n = PART == 2 ? m.bins[1] - big_lo : PART == 1 ? m.bins[2] : m.heavy3;
    const Guided guided(n, gridDim.x, 1u, ONE ? 16u : 1u);
    const uint32_t fetches = guided.fetches();
    if (blockIdx.x >= fetches) return;
    for (uint32_t i = tid; i < words; i += NT) T[i] = 0;
    if constexpr (PV) {
        for (uint32_t i = tid; i < 2 * a.dcap; i += NT) tally[i] = 0;
        for (uint32_t i = tid; i < HR; i += NT) hot[i] = 0;
    }
    unsigned long long acc = 0;
    uint32_t q = blockIdx.x % kWaveQueues;
    uint32_t* const heads = a.heads + 3u * kHeadStride + 8u * (PART + 1u);

    for (uint32_t f = blockIdx.x; f < fetches;) {
        uint32_t j0, j1;
        guided.range(f, j0, j1);
        const uint32_t cnt = j1 - j0;
        uint32_t ticket = 0;
        if (tid == 0 && fetches > gridDim.x) ticket = atomicAdd(&heads[q * kHeadStride], 1u);
        // the fetch's owners (lane i of every wavefront holds the i-th)
        uint32_t vu = 0, vb = 0, vd = 0, vs = 0, vq = 0;
        if ((uint32_t)lane < cnt) {
            vu = a.items[base + j0 + lane];
            if (a.shards <= 1 || vu % a.shards == a.shard) {
                vb = a.off[vu];
                vd = a.off[vu + 1] - vb;
                const uint2 o = a.bl[vu];
                vs = o.x;
                vq = o.y;
            }
        }
        uint32_t xw = 0, xs = 0, xn = 0, xb = 0;  // ONE: this thread's list element, its list, and own word
        auto element = [&](uint32_t i, uint32_t& w, uint32_t& b) {
            const uint32_t beg = __builtin_amdgcn_readlane(vb, i), d = __builtin_amdgcn_readlane(vd, i);
            const uint32_t s = __builtin_amdgcn_readlane(vs, i), own = __builtin_amdgcn_readlane(vq, i);
            w = b = 0;
            if (tid < d) w = a.col[beg + tid];
            if (tid < 4 * own) b = reinterpret_cast<const uint32_t*>(a.blk)[4 * (uint64_t)s + tid];
        };
        auto list = [&](uint32_t i, uint32_t w, uint32_t& s, uint32_t& len) {
            s = len = 0;
            if (tid < __builtin_amdgcn_readlane(vd, i)) {
                const uint2 l = a.bl[w];
                s = l.x;
                len = l.y;
            }
        };
        if constexpr (ONE) {
            element(0, xw, xb);
            list(0, xw, xs, xn);
        }
        for (uint32_t i = 0; i < cnt; ++i) {
            const uint32_t u = __builtin_amdgcn_readlane(vu, i), beg = __builtin_amdgcn_readlane(vb, i);
            const uint32_t d = __builtin_amdgcn_readlane(vd, i);
            const uint32_t own = 4u * __builtin_amdgcn_readlane(vq, i);
            const uint32_t* const mine =
                reinterpret_cast<const uint32_t*>(a.blk) + 4 * (uint64_t)__builtin_amdgcn_readlane(vs, i);
            uint32_t W = 0;
            uint32_t nw = 0, nb = 0, ns = 0, nn = 0;
            if constexpr (ONE) {
                if (i + 1 < cnt) element(i + 1, nw, nb);
                uint32_t incl = wave_incl_scan(xn), members = 0;
                if constexpr (PV) members = wave_incl_scan((uint32_t)__popc(xb & mask));
                if (lane == 63) {
                    s_scan[0][wave] = incl;
                    if constexpr (PV) s_scan[1][wave] = members;
                }
                __syncthreads();
                uint32_t first = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const uint32_t x = s_scan[0][w];
                    incl += w < wave ? x : 0u;
                    W += x;
                    if constexpr (PV) first += w < wave ? s_scan[1][w] : 0u;
                }
                if (tid < d) P[tid] = u32x2{incl, xs - (incl - xn)};
                if (xb) T[xb >> S] = PV ? ((first + members - (uint32_t)__popc(xb & mask)) << S) | (xb & mask) : xb & mask;
            } else {
                if (d == 0) continue;
                uint32_t t;
                for (uint32_t p0 = 0; p0 < d; p0 += NT) {
                    const uint32_t p = p0 + tid;
                    uint2 l = make_uint2(0u, 0u);
                    if (p < d) l = a.bl[a.col[beg + p]];
                    const uint32_t e = W + group_scan<NW>(l.y, s_scan[(p0 / NT) & 1], wave, lane, t);
                    if (p < d) P[p] = u32x2{e, l.x - (e - l.y)};
                    W += t;
                }
                __syncthreads();
                uint32_t first = 0;
                for (uint32_t p0 = 0; p0 < own; p0 += NT) {
                    const uint32_t p = p0 + tid;
                    const uint32_t b = p < own ? mine[p] : 0u;
                    if constexpr (PV) {
                        const uint32_t c = (uint32_t)__popc(b & mask);
                        const uint32_t e = first + group_scan<NW>(c, s_scan[(p0 / NT) & 1], wave, lane, t);
                        if (b) T[b >> S] = ((e - c) << S) | (b & mask);
                        first += t;
                    } else {
                        if (b) T[b >> S] = b & mask;
                    }
                }
            }
            __syncthreads();
            if constexpr (ONE)
                if (i + 1 < cnt) list(i + 1, nw, ns, nn);
            W = __builtin_amdgcn_readfirstlane(W);
            CoreProbe<PV> pr{a.blk, T, P, tally, member, queue, S, mask, lane};
            pr.range(d, __builtin_amdgcn_readfirstlane((uint32_t)(((uint64_t)W * (uint32_t)wave) / NW)),
                     __builtin_amdgcn_readfirstlane((uint32_t)(((uint64_t)W * (uint32_t)(wave + 1)) / NW)));
            if constexpr (PV) {
                while (pr.qn) pr.take(pr.qn < 64u ? pr.qn : 64u);
                const uint32_t mine_hits = wave_sum(pr.hits);
                acc += mine_hits;
                if (lane == 0 && mine_hits) atomicAdd(&a.tv[u], (unsigned long long)mine_hits);
            } else {
                acc += pr.hits;
            }
            __syncthreads();
            if constexpr (PV) {
                // out-neighbour p's triangles: as v (tally[p]) and, for a core member, as w (its member tally)
                for (uint32_t p = tid; p < d; p += NT) {
                    const uint32_t w = ONE ? xw : a.col[beg + p];
                    uint32_t t = tally[p];
                    if (t) tally[p] = 0;
                    if (w >= a.c0) {
                        const uint32_t x = w - a.c0, idx = block_of(x, a.magic);
                        const uint32_t r = T[idx];
                        const uint32_t at = (r >> S) + (uint32_t)__popc(r & ((1u << (x - idx * S)) - 1u));
                        const uint32_t c = member[at];
                        if (c) member[at] = 0;
                        t += c;
                    }
                    if (t) {
                        if (w >= hot0) atomicAdd(&hot[w - hot0], t);
                        else atomicAdd(&a.tv[w], (unsigned long long)t);
                    }
                }
                __syncthreads();
                if (++owners == kHotOwners) {
                    owners = 0;
                    flush_hot();
                }
            }
            if constexpr (ONE) {
                if (xb) T[xb >> S] = 0;
                xw = nw;
                xb = nb;
                xs = ns;
                xn = nn;
            } else {
                for (uint32_t p = tid; p < own; p += NT) {
                    const uint32_t b = mine[p];
                    if (b) T[b >> S] = 0;
                }
            }
        }
        if (fetches <= gridDim.x) break;
        if (wave == 0) {  // the next fetch, from another sub-queue once this one is drained
            uint32_t next = 0xFFFFFFFFu;
            for (;;) {
                const uint32_t g = gridDim.x + __builtin_amdgcn_readfirstlane(ticket) * kWaveQueues + q;
                if (g < fetches) {
                    next = g;
                    break;
                }
                uint32_t seen = 0;
                if (lane < (int)kWaveQueues)
                    seen = __hip_atomic_load(&heads[(uint32_t)lane * kHeadStride], __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
                const uint32_t left = (uint32_t)__ballot(
                    lane < (int)kWaveQueues && gridDim.x + (uint64_t)seen * kWaveQueues + (uint32_t)lane < fetches);
                if (!left) break;
                const uint32_t above = left >> q;
                q = above ? q + (uint32_t)__builtin_ctz(above) : (uint32_t)__builtin_ctz(left);
                ticket = 0;
                if (lane == 0) ticket = atomicAdd(&heads[q * kHeadStride], 1u);
            }
            if (lane == 0) s_next = next;
        }
        __syncthreads();
        f = s_next;
        __syncthreads();
    }
    if constexpr (PV) {
        flush_hot();  // (every path here is behind a barrier)
        if (lane == 0) s_acc[wave] = acc;
    } else {
        for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
        if (lane == 0) s_acc[wave] = acc;
    }
    __syncthreads();
    if (tid == 0) {
        unsigned long long sum = 0;
        for (int w = 0; w < NW; ++w) sum += s_acc[w];
        if (sum) atomicAdd(a.total, sum);
    }
}

typedef void (*CoreFn)(CoreArgs);
constexpr uint32_t kCoreDcap[3] = {128, 1024, 4096};

CoreFn pick_core(int part, bool pv, uint32_t S) {
    switch (part) {
        case 0:
            if (core_waves(0, S) == 4) return pv ? tc_core_kernel<true, 4, 0> : tc_core_kernel<false, 4, 0>;
            return pv ? tc_core_kernel<true, 2, 0> : tc_core_kernel<false, 2, 0>;
        case 1: return pv ? tc_core_kernel<true, 8, 1> : tc_core_kernel<false, 8, 1>;
        default: return pv ? tc_core_kernel<true, 16, 2> : tc_core_kernel<false, 16, 2>;
    }
}

uint32_t core_lds(int part, bool pv, uint32_t S) {
    return 4u * ((1u << (32 - S)) + (pv ? 4u : 2u) * kCoreDcap[part] + (pv ? 2u * kCoreQueue * core_waves(part, S) + kHotRanks[part] : 0u));
}

#define TC_TRY(expr)                        \
    do {                                    \
        hipError_t e_ = (expr);             \
        if (e_ != hipSuccess) return e_;    \
    } while (0)

}  // namespace

// Wavefronts per owner.  Part 0: two (R-MAT 22, 8 KB tables: 3.0 ms against 3.2 with four, per-vertex 3.65
// against 4.3), but four beside a 16 KB table, of which a CU holds few (R-MAT 26 per-vertex 94.8 ms against 98.0;
// whole counts, total / per-vertex, of 80,000 vertices of degree 200: uniform 0.56 / 0.70 ms against 0.59 / 0.76,
// power law 0.21 / 0.34 against 0.24 / 0.36).  Part 1: eight (2.7 ms; per-vertex 4.8 against 5.7 with four and
// 8.0 with sixteen).
uint32_t core_waves(int part, uint32_t S) { return part == 0 ? (S > 20 ? 2u : 4u) : part == 1 ? 8u : 16u; }

hipError_t core_build(const CoreBuild& a, int cu_count, hipStream_t stream) {
    const uint32_t lds = 4u << (32 - a.S);
    const uint32_t cus = (uint32_t)(cu_count > 0 ? cu_count : 1);
    const uint32_t per_cu = 163840u / lds < 32u ? 163840u / lds : 32u;
    const uint64_t tiles = (a.m_in + kTileEdges - 1) / kTileEdges;
    hipLaunchKernelGGL(k_core_tiles, dim3((uint32_t)(tiles < 4ull * cus ? tiles : 4ull * cus)), dim3(kTileThreads), 0, stream, a);
    TC_TRY(hipGetLastError());
    const uint64_t rows = std::max<uint64_t>(tiles, ((uint64_t)a.n + 63) / 64);
    hipLaunchKernelGGL(k_core_rows, dim3((uint32_t)(rows < cus * per_cu ? rows : cus * per_cu)), dim3(64), lds, stream, a);
    TC_TRY(hipGetLastError());
    if (a.c0 == 0) return hipSuccess;  // every rank is in the core: no cut lists
    const uint32_t per = 256 / kRestLanes, want = (a.n + per - 1) / per;
    hipLaunchKernelGGL(k_rest_classes, dim3(want < 8 * cus ? want : 8 * cus), dim3(256), 0, stream, a);
    TC_TRY(hipGetLastError());
    const uint32_t want2 = (a.n + 255) / 256;
    hipLaunchKernelGGL(k_rest_place, dim3(want2 < 4 * cus ? want2 : 4 * cus), dim3(256), 0, stream, a);
    return hipGetLastError();
}

hipError_t core_info(int part, bool pv, uint32_t S, int* blocks_per_cu) {
    const void* f = reinterpret_cast<const void*>(pick_core(part, pv, S));
    const uint32_t lds = core_lds(part, pv, S);
    if (lds > 65536)
        TC_TRY(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)core_lds(part, pv, kCoreMinBits)));
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, f, 64 * core_waves(part, S), lds);
}

hipError_t core_launch(int part, bool pv, uint32_t grid, CoreArgs a, hipStream_t stream) {
    a.dcap = kCoreDcap[part];
    hipLaunchKernelGGL(pick_core(part, pv, a.S), dim3(grid), dim3(64 * core_waves(part, a.S)), core_lds(part, pv, a.S), stream, a);
    return hipGetLastError();
}

}  // namespace tc
