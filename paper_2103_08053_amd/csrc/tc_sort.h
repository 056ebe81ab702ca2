// Stable radix partition passes (device code and launch templates), used by the build's sorts.
//
// One pass moves `count` elements to the order of one digit (D bits at `shift`), reading and writing each
// element once: a tile of 1024 x ITEMS elements is ranked in the workgroup, the number of elements with
// the same digit in earlier tiles comes from a decoupled look-back over the tiles' published counts, and
// the tile is written out from LDS, digit after digit, so that the elements of a digit leave in runs.
// The digits' totals (`hist`) are counted beforehand, by whichever kernel makes the elements.
// (The published method is single-pass radix sorting: A. Adinets and D. Merrill, "Onesweep: A Faster Least
// Significant Digit Radix Sort for GPUs", on the look-back of D. Merrill and M. Garland, "Single-pass Parallel
// Prefix Scan with Decoupled Look-back".)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "tc_wave.h"

namespace tc {

constexpr uint32_t kPassThreads = 1024;
constexpr uint32_t kPassWaves = kPassThreads / 64;
constexpr uint32_t kDigit = 9;              // bits per pass (a pass of 8 bits costs the same)
// Look-back words: flag (1 count of this tile, 2 count up to and including it) << 62 | epoch << 54 | count.
// Words of an earlier pass carry another epoch, so the array is cleared once per build.
constexpr uint32_t kEpochShift = 54, kFlagShift = 62;

// Elements per thread.  What a pass pays per tile is the look-back: every digit's words of the tiles in
// flight, read past the L2.  So a large input takes the largest tile that one workgroup per CU can stage
// in LDS (147 KB of 64-bit elements): 2^26 keys in 0.32 ms against 0.42 with two workgroups of 57 KB per CU
// (half the tiles, half of them in flight) and 0.74 with 28 KB; the library's 9-bit pass takes 0.36 ms.
// Inputs too small to fill the device that way take small tiles.
constexpr uint32_t pass_items(uint64_t count, uint32_t bytes) {
    return count >= 3500000 ? (bytes == 8 ? 18u : 28u) : count >= (1ull << 19) ? 4u : 2u;
}
constexpr uint64_t pass_tiles(uint64_t count, uint32_t bytes) {
    const uint64_t tile = (uint64_t)kPassThreads * pass_items(count, bytes);
    return (count + tile - 1) / tile;
}

// Lanes of the wavefront whose D-bit value equals this lane's.
template <int D>
__device__ __forceinline__ unsigned long long same_value(uint32_t v) {
    uint32_t lo = ~0u, hi = ~0u;
#pragma unroll
    for (int b = 0; b < D; ++b) {
        const uint32_t mine = (uint32_t)((int32_t)(v << (31 - b)) >> 31);  // all ones where the bit is set
        const unsigned long long set = __ballot(mine != 0);
        // m & ~(set ^ mine), one instruction per half (truth table of a & ~(b ^ c))
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)set, mine, 0x90);
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(set >> 32), mine, 0x90);
    }
    return ((unsigned long long)hi << 32) | lo;
}

// hist[d] += lanes with digit d: one add when the whole wavefront agrees (sorted or constant input).
__device__ __forceinline__ void count_digit(uint32_t* hist, uint32_t d, bool act) {
    const uint32_t first = __builtin_amdgcn_readfirstlane(d);
    const unsigned long long on = __ballot(act);
    if (!__ballot(act && d != first) && (on & 1ull)) {
        if (lanes_below(~0ull) == 0) atomicAdd(&hist[first], (uint32_t)__popcll(on));
    } else if (act) {
        atomicAdd(&hist[d], 1u);
    }
}

// Exclusive sum over the workgroup's threads of v (s: one word per wavefront, WAVES of them; two barriers).
template <uint32_t WAVES = kPassWaves>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* s) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t incl = wave_incl_scan(v);
    if (lane == 63) s[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (uint32_t w = 0; w < WAVES; ++w) before += w < wave ? s[w] : 0u;
    __syncthreads();
    return before + incl - v;
}

// `load.raw(i)` reads what element i is made of, and `load.make(raw, lane, &e)` gives the element and whether
// it takes part (others are dropped); all reads of a tile are issued before the first is used.  (i of lane 0
// is a multiple of 64.)  `store(pos, e)` takes the element at position pos of the pass's order.  `live` (or null): the number of elements, if fewer than count.
// STABLE: elements of a digit keep their order (a pass over the lowest digit, or a lone partition, need not:
// its ranks are LDS atomics on one counter per digit instead of matches within each wavefront).
template <int D, int ITEMS, bool STABLE, typename E, typename Load, typename Store>
__global__ void __launch_bounds__(kPassThreads) __attribute__((amdgpu_waves_per_eu(4)))
k_pass(Load load, Store store, uint64_t count, const unsigned long long* live, uint32_t shift, const uint32_t* hist,
       unsigned long long* status, uint32_t epoch, uint32_t* ticket) {
    constexpr uint32_t BINS = 1u << D, TILE = kPassThreads * ITEMS, W = STABLE ? kPassWaves : 1u;
    constexpr uint32_t BPT = BINS > kPassThreads ? BINS / kPassThreads : 1u;  // bins per thread
    constexpr size_t kStage = sizeof(E) * TILE, kCnt = 4 * (size_t)W * BINS;
    extern __shared__ __align__(16) unsigned char lds[];
    E* const stage = reinterpret_cast<E*>(lds);              // after the ranks are known
    uint32_t* const cnt = reinterpret_cast<uint32_t*>(lds);  // [W][BINS], before
    uint32_t* const gbase = reinterpret_cast<uint32_t*>(lds + (kStage > kCnt ? kStage : kCnt));  // [BINS]
    __shared__ uint32_t s_scan[kPassWaves];
    __shared__ uint32_t s_tile, s_valid;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (live && *live < count) count = *live;
    if (tid == 0) s_tile = atomicAdd(ticket, 1u);
    for (uint32_t b = tid; b < W * BINS; b += kPassThreads) cnt[b] = 0;
    __syncthreads();
    const uint32_t tile = s_tile;
    const uint64_t base = (uint64_t)tile * TILE;
    if (base >= count) return;

    E e[ITEMS];
    uint32_t at[ITEMS];  // rank among the wavefront's (or, unstable, the tile's) elements of the digit
    uint32_t act = 0;
    const uint64_t at0 = base + wave * (64u * ITEMS);  // this wavefront's first element
    {
        typename Load::Raw raw[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint64_t x = at0 + i * 64u + lane;
            raw[i] = load.raw(x < count ? x : count - 1);
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            e[i] = 0;
            if (load.make(raw[i], lane, e[i]) && at0 + i * 64u + lane < count) act |= 1u << i;
        }
    }
    uint32_t* const mine = cnt + (STABLE ? wave * BINS : 0u);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint32_t d = (uint32_t)(e[i] >> shift) & (BINS - 1u);
        const bool on = (act >> i) & 1u;
        if constexpr (STABLE) {
            const unsigned long long m = same_value<D>(d) & __ballot(on);
            const uint32_t below = lanes_below(m);
            at[i] = mine[d] + below;  // (the wavefront's LDS accesses are in order)
            wave_sync();
            if (on && below == 0) mine[d] = at[i] + (uint32_t)__popcll(m);
            wave_sync();
        } else {
            at[i] = on ? atomicAdd(&mine[d], 1u) : 0u;
        }
    }
    __syncthreads();
    // totals of the tile, and their positions in it
    uint32_t tot[BPT], lead[BPT], gl[BPT], run = 0, grun = 0;
#pragma unroll
    for (uint32_t j = 0; j < BPT; ++j) {
        const uint32_t b = tid * BPT + j;
        tot[j] = gl[j] = 0;
        if (b < BINS) {
#pragma unroll
            for (uint32_t w = 0; w < W; ++w) tot[j] += cnt[w * BINS + b];
            gl[j] = hist[b];
            __hip_atomic_store(&status[(uint64_t)tile * BINS + b],
                               ((unsigned long long)(tile ? 1u : 2u) << kFlagShift) |
                                   ((unsigned long long)epoch << kEpochShift) | tot[j],
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        lead[j] = run;
        run += tot[j];
        const uint32_t g = gl[j];
        gl[j] = grun;
        grun += g;
    }
    const uint32_t first = block_excl_scan(run, s_scan), gfirst = block_excl_scan(grun, s_scan);
#pragma unroll
    for (uint32_t j = 0; j < BPT; ++j) {
        const uint32_t b = tid * BPT + j;
        lead[j] += first;
        gl[j] += gfirst;
        if (b < BINS) {
            uint32_t p = lead[j];
#pragma unroll
            for (uint32_t w = 0; w < W; ++w) {
                const uint32_t c = cnt[w * BINS + b];
                cnt[w * BINS + b] = p;
                p += c;
            }
            if (b == BINS - 1) s_valid = p;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) at[i] += mine[(uint32_t)(e[i] >> shift) & (BINS - 1u)];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if ((act >> i) & 1u) stage[at[i]] = e[i];
    // elements of the digit in earlier tiles: tickets are handed out in order, so every earlier tile is
    // running or done, and publishes without waiting for a later one
#pragma unroll
    for (uint32_t j = 0; j < BPT; ++j) {
        const uint32_t b = tid * BPT + j;
        if (b >= BINS) continue;
        unsigned long long before = 0;
        constexpr unsigned long long kCount = (1ull << kEpochShift) - 1;
        constexpr int kBack = 2;  // words read at a time (more read past what is needed: 4 cost 2%, 8 10%)
        for (int64_t t = (int64_t)tile - 1; t >= 0;) {
            unsigned long long v[kBack];
#pragma unroll
            for (int q = 0; q < kBack; ++q)
                v[q] = t >= q ? __hip_atomic_load(&status[(uint64_t)(t - q) * BINS + b], __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT)
                              : 0ull;
            bool open = true, done = false;  // open: every word so far was there
#pragma unroll
            for (int q = 0; q < kBack; ++q) {
                open = open && !done && ((v[q] >> kEpochShift) & 0xFFull) == epoch && (v[q] >> kFlagShift) != 0;
                if (open) {
                    before += v[q] & kCount;
                    done = (v[q] >> kFlagShift) == 2u;
                    --t;
                }
            }
            if (done) break;
        }
        if (tile)
            __hip_atomic_store(&status[(uint64_t)tile * BINS + b],
                               (2ull << kFlagShift) | ((unsigned long long)epoch << kEpochShift) | (before + tot[j]),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        gbase[b] = gl[j] + (uint32_t)before - lead[j];
    }
    __syncthreads();
    const uint32_t valid = s_valid;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const uint32_t p = tid + i * kPassThreads;
        if (p < valid) {
            const E x = stage[p];
            store(gbase[(uint32_t)(x >> shift) & (BINS - 1u)] + p, x);
        }
    }
}

template <int D, int ITEMS, bool STABLE, typename E>
constexpr uint32_t pass_lds() {
    const uint32_t stage = sizeof(E) * kPassThreads * ITEMS, cnt = 4 * (STABLE ? kPassWaves : 1u) * (1u << D);
    return (stage > cnt ? stage : cnt) + 4u * (1u << D);
}

template <int D, int ITEMS, bool STABLE, typename E, typename Load, typename Store>
hipError_t launch_pass(Load load, Store store, uint64_t count, const unsigned long long* live, uint32_t shift,
                       const uint32_t* hist, unsigned long long* status, uint32_t epoch, uint32_t* ticket,
                       hipStream_t stream) {
    constexpr uint32_t lds = pass_lds<D, ITEMS, STABLE, E>();
    if constexpr (lds > 65536) {  // opt-in LDS, once per device
        static std::atomic<uint64_t> done{0};
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev >= 64 || !((done.load(std::memory_order_relaxed) >> dev) & 1ull)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_pass<D, ITEMS, STABLE, E, Load, Store>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            if (dev < 64) done.fetch_or(1ull << dev, std::memory_order_relaxed);
        }
    }
    const uint64_t tile = (uint64_t)kPassThreads * ITEMS;
    hipLaunchKernelGGL((k_pass<D, ITEMS, STABLE, E, Load, Store>), dim3((uint32_t)((count + tile - 1) / tile)),
                       dim3(kPassThreads), lds, stream, load, store, count, live, shift, hist, status, epoch, ticket);
    return hipGetLastError();
}

template <int D, bool STABLE, typename E, typename Load, typename Store>
hipError_t radix_pass(Load load, Store store, uint64_t count, const unsigned long long* live, uint32_t shift,
                      const uint32_t* hist, unsigned long long* status, uint32_t epoch, uint32_t* ticket,
                      hipStream_t stream) {
    if (count == 0) return hipSuccess;
    constexpr int big = sizeof(E) == 8 ? 18 : 28;
    const uint32_t items = pass_items(count, sizeof(E));
    if (items == (uint32_t)big)
        return launch_pass<D, big, STABLE, E>(load, store, count, live, shift, hist, status, epoch, ticket, stream);
    if (items == 4)
        return launch_pass<D, 4, STABLE, E>(load, store, count, live, shift, hist, status, epoch, ticket, stream);
    return launch_pass<D, 2, STABLE, E>(load, store, count, live, shift, hist, status, epoch, ticket, stream);
}

}  // namespace tc
