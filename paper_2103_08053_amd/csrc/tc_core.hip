// The core path: owners with much 2-hop work probe their out-neighbours' lists 20-22 ids at a time.
//
// Ranks follow degree, so on skewed graphs nearly every 2-hop id is one of the last K ranks (the core;
// R-MAT scale 22: 99% of the probes end in the last 43,008 of 4.2 M ranks), and a list's core ids crowd
// together.  Each list's core ids are stored as block words: block index << S | S-bit mask of the
// block's ids, S = 20..22 (CoreShape), one word per block that holds any (R-MAT 22: 2.8 ids per word;
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
// hold at least half of W+, and a quarter of the edges must end in the core.
#include "tc_fetch.h"
#include "tc_internal.h"
#include "tc_wave.h"

namespace tc {
namespace {

// ---------------------------------------------------------------- build: block words

__device__ __forceinline__ uint32_t block_of(uint32_t x, uint32_t magic) { return __umulhi(x, magic); }

constexpr uint32_t kBlockRows = 32;  // consecutive rows a wavefront takes at a time

template <int R>
__device__ __forceinline__ void group_or_step(uint32_t idx, uint32_t own, uint32_t& all, bool& first, uint32_t at) {
    if constexpr (R < 16) {  // row_ror:R: lane at receives from lane (at - R) mod 16
        const uint32_t i = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)idx, 0x120 + R, 0xf, 0xf, false);
        const uint32_t b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own, 0x120 + R, 0xf, 0xf, false);
        if (i == idx) {
            all |= b;
            first = first && at < (uint32_t)R;  // a sender at - R >= 0 is below this lane
        }
        group_or_step<R + 1>(idx, own, all, first, at);
    }
}
// Within rows of 16 lanes: bits |= the bits of every lane with the same idx; first: no lane below has it.
template <int R>
__device__ __forceinline__ void group_or(uint32_t idx, uint32_t& bits, bool& first, uint32_t at) {
    const uint32_t own = bits;
    uint32_t all = own;
    bool f = first;
    group_or_step<R>(idx, own, all, f, at);
    bits = all;
    first = f;
}

// One wavefront per row: the row's core ids are ORed into the wavefront's LDS table of block masks; the
// first lane to take a block's mask back (an exchange with zero, which also clears the table) writes its
// word.  The row's ids go to col, those outside the core first.  Rows are short and the work per row is a
// chain of LDS accesses, so the kernel lives from the number of wavefronts the tables (2^(32-S) words
// each) leave room for.  Long rows are those of the last ranks: they go first.
__global__ void __launch_bounds__(64) k_core_blocks(CoreBuild a) {
    extern __shared__ __align__(16) uint32_t T[];
    if (!core_on(*a.meta)) return;
    const uint32_t lane = threadIdx.x, S = a.S, words = 1u << (32 - S);
    for (uint32_t i = lane; i < words; i += 64) T[i] = 0;
    wave_sync();
    const uint32_t batches = (a.n + kBlockRows - 1) / kBlockRows;
    for (uint32_t t = blockIdx.x; t < batches; t += gridDim.x) {
        const uint32_t r0 = (batches - 1 - t) * kBlockRows;
        const uint32_t rows = a.n - r0 < kBlockRows ? a.n - r0 : kBlockRows;
        uint32_t vb = 0, vd = 0, vq = 0, vr = 0;
        if (lane < rows) {
            vb = a.off[r0 + lane];
            vd = a.off[r0 + lane + 1] - vb;
        }
        auto key = [&](uint32_t at) { return (uint32_t)(a.okeys[at] & a.mask); };
        uint32_t ahead = 0;  // the next row's first 64 ids
        {
            const uint32_t b = __builtin_amdgcn_readlane(vb, 0), d = __builtin_amdgcn_readlane(vd, 0);
            if (lane < d) ahead = key(b + lane);
        }
        for (uint32_t i = 0; i < rows; ++i) {
            const uint32_t beg = __builtin_amdgcn_readlane(vb, i), d = __builtin_amdgcn_readlane(vd, i);
            const uint32_t first = ahead;
            if (i + 1 < rows) {
                const uint32_t b = __builtin_amdgcn_readlane(vb, i + 1), dn = __builtin_amdgcn_readlane(vd, i + 1);
                if (lane < dn) ahead = key(b + lane);
            }
            if (d <= 16) continue;
            uint32_t* const out = a.blk + 4 * core_start(beg, r0 + i);
            uint32_t rest = 0, cores = 0, nb = 0;
            for (uint32_t c = 0; c < d; c += 64) {  // masks, and the ids outside the core
                const bool act = c + lane < d;
                const uint32_t id = c ? (act ? key(beg + c + lane) : 0u) : first;
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
                const uint32_t id = c ? (act ? key(beg + c + lane) : 0u) : first;
                const bool core = act && id >= a.c0;
                uint32_t word = 0;
                if (core) {
                    const uint32_t idx = block_of(id - a.c0, a.magic);
                    const uint32_t m = atomicExch(&T[idx], 0u);
                    if (m) word = (idx << S) | m;
                }
                const unsigned long long cm = __ballot(core), fm = __ballot(word != 0);
                if (core) a.col[beg + rest + cores + lanes_below(cm)] = id;
                if (word) out[nb + lanes_below(fm)] = word;
                cores += (uint32_t)__popcll(cm);
                nb += (uint32_t)__popcll(fm);
            }
            wave_sync();
            const uint32_t pad = (0u - nb) & 3u;
            if (lane < pad) out[nb + lane] = 0;
            if (lane == i) {
                vq = (nb + 3u) / 4u;
                vr = rest;
            }
        }
        // Rows of at most 16 ids, four at a time: 16 lanes hold a row, and a lane learns the ids of its block
        // from the others' by row rotations; the lowest lane of a block writes its word.
        const unsigned long long small = __ballot(vd > 0 && vd <= 16);
        for (unsigned long long left = small; left;) {
            uint32_t pick = 64;  // the row this lane's group takes
#pragma unroll
            for (uint32_t g = 0; g < 4; ++g)
                if (left) {
                    if ((lane >> 4) == g) pick = (uint32_t)__builtin_ctzll(left);
                    left &= left - 1;
                }
            const uint32_t at = lane & 15u;
            const uint32_t beg = (uint32_t)__shfl((int)vb, (int)(pick & 63u), 64);
            const uint32_t dr = (uint32_t)__shfl((int)vd, (int)(pick & 63u), 64);  // every lane takes part
            const uint32_t d = pick < 64 ? dr : 0u;
            const bool act = at < d;
            const uint32_t id = act ? key(beg + at) : 0u;
            const bool core = act && id >= a.c0;
            const uint32_t x = id - a.c0, idx = core ? block_of(x, a.magic) : 0xFFFFFFFFu - at;
            uint32_t bits = core ? 1u << (x - idx * S) : 0u;
            bool first = core;
            group_or<1>(idx, bits, first, at);
            const unsigned long long rm = __ballot(act && !core), cm = __ballot(core), fm = __ballot(first);
            const uint32_t sh = lane & 48u;
            const uint32_t r16 = (uint32_t)(rm >> sh) & 0xFFFFu, c16 = (uint32_t)(cm >> sh) & 0xFFFFu;
            const uint32_t f16 = (uint32_t)(fm >> sh) & 0xFFFFu, below = (1u << at) - 1u;
            const uint32_t rest = (uint32_t)__popc(r16), nb = (uint32_t)__popc(f16);
            if (act) a.col[beg + (core ? rest + (uint32_t)__popc(c16 & below) : (uint32_t)__popc(r16 & below))] = id;
            uint32_t* const out = a.blk + 4 * core_start(beg, r0 + pick);
            if (first) out[__popc(f16 & below)] = (idx << S) | bits;
            if (d && at >= nb && at < ((nb + 3u) & ~3u)) out[at] = 0;
            // back to the lane that holds the row
            unsigned long long todo = __ballot(at == 0 && d != 0);
            for (; todo; todo &= todo - 1) {
                const int src = __builtin_ctzll(todo);
                const uint32_t row = __builtin_amdgcn_readlane(pick, src);
                const uint32_t q = (__builtin_amdgcn_readlane(nb, src) + 3u) / 4u, rr = __builtin_amdgcn_readlane(rest, src);
                if (lane == row) {
                    vq = q;
                    vr = rr;
                }
            }
        }
        if (lane < rows) {
            a.bl[r0 + lane] = make_uint2((uint32_t)core_start(vb, r0 + lane), vq);
            a.rend[r0 + lane] = vb + vr;
        }
    }
}

// ---------------------------------------------------------------- build: the cut lists' schedule

// Owners of the core path that have triangles outside the core: cut lists of at least two ids with 2-hop
// work, in the bins of the bucket kernels by cut out-degree, each bin by the power of two of its work
// (largest first).  Five groups: the global-table bin, the two parts of the large-LDS bin, the workgroup
// and the wavefront bin.
constexpr uint32_t kRestClasses = 5 * 32;
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

// Wavefronts per owner.  Part 0: two (R-MAT 22, 8 KB tables: 3.0 ms against 3.2 with four, per-vertex 3.65
// against 4.3), but four beside a 16 KB table, of which a CU holds few (R-MAT 26 per-vertex 94.8 ms against 98.0).  Part 1:
// eight (2.7 ms; per-vertex 4.8 against 5.7 with four and 8.0 with sixteen).
int core_waves(int part, uint32_t S) { return part == 0 ? (S > 20 ? 2 : 4) : part == 1 ? 8 : 16; }

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

hipError_t core_build(const CoreBuild& a, int cu_count, hipStream_t stream) {
    const uint32_t lds = 4u << (32 - a.S);
    const uint32_t cus = (uint32_t)(cu_count > 0 ? cu_count : 1);
    const uint32_t per_cu = 163840u / lds < 32u ? 163840u / lds : 32u;
    const uint32_t batches = (a.n + kBlockRows - 1) / kBlockRows;
    TC_TRY(fill_u32(a.hist, 0, 2 * kRestClasses, stream));
    TC_TRY(fill_u32(a.rest_meta, 0, sizeof(GraphMeta) / 4, stream));
    hipLaunchKernelGGL(k_core_blocks, dim3(batches < cus * per_cu ? batches : cus * per_cu), dim3(64), lds, stream, a);
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
