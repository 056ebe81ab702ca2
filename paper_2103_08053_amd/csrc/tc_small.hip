// One-shot counts of small graphs: the adjacency as a bit matrix.
//
// A graph of a few thousand vertices has no work to speak of; what its count costs is the chain of some
// twenty launches that clean, sort and schedule it (1000 vertices: 0.11 ms of kernels, 0.17 ms per call).
// Its adjacency matrix is small instead: n rows of n bits, 128 KB at 1000 vertices and 8 MB at 8192, which
// the L2s hold.  Setting bits removes duplicates and directions by itself, and an edge (a, b) closes
// popcount(row a & row b) triangles, so three launches do: clear, set (which also marks the first sample of
// every distinct edge, a bit per sample), count.  A row takes one 16-byte load per lane and 128 vertices: a
// group of lanes per edge, as many as the row has quads.
//
// Every triangle is found by its three edges, and by two of them for each of its vertices: the last
// workgroup to finish divides.
#include "tc_internal.h"
#include "tc_wave.h"

namespace tc {
namespace {

constexpr uint32_t kThreads = 256;

__global__ void __launch_bounds__(1024) k_small_clear(SmallArgs a) {
    const uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x, step = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t quads = (uint64_t)a.n * a.quads;
    for (uint64_t i = t; i < quads; i += step) a.rows[i] = make_uint4(0u, 0u, 0u, 0u);
    if (a.out)
        for (uint64_t i = t; i < a.n; i += step) a.out[i] = 0;
    if (t == 0) *a.result = SmallResult{0ull, 0u, 0u};
}

// Atomics on a word that many samples name are the whole time of an input of repeated samples (one address takes
// 9e7 a second: 2^24 samples of one pair 190 ms).  So a sample goes to memory only if its workgroup has not just
// sent the same pair there (s_seen, by hash; whoever replaces an entry goes), and where most of the wavefront's
// last ones found their bits set, only if the word, read past the caches, has it clear.  2^24 samples of one pair
// 0.14 ms, of 100 pairs of 16 vertices 0.2 ms.  Large workgroups, because each sends every pair once (2^20 samples
// of 120 pairs 0.25 ms against 0.93 with 256 threads); small ones up to 2^18 samples, which are too few for many of
// them, and no table up to 4096, which one address takes in 45 us (1000 vertices and 4000 samples 35.5 us a call;
// with the table 36.4, with large workgroups 37.8).
constexpr uint32_t kSetThreads = 1024;
constexpr uint64_t kSetFew = 1u << 18, kSetTiny = 4096;

__global__ void __launch_bounds__(kSetThreads) k_small_set(SmallArgs a) {
    __shared__ uint32_t s_seen[4 * kSetThreads];
    const uint32_t seen_shift = 30u - (31u - (uint32_t)__builtin_clz(blockDim.x));  // four entries per thread
    const bool table = a.m_in > kSetTiny;
    if (table) {
        for (uint32_t i = threadIdx.x; i < 4 * blockDim.x; i += blockDim.x) s_seen[i] = 0xFFFFFFFFu;  // no pair's name
        __syncthreads();
    }
    uint32_t* const rows = reinterpret_cast<uint32_t*>(a.rows);
    const uint64_t words = 4ull * a.quads;
    uint32_t bad = 0;
    bool look = false;  // uniform in the wavefront
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x; base < a.m_in; base += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = base + threadIdx.x;
        bool go = false, first = false;
        if (i < a.m_in) {
            const uint32_t x = a.src[i], y = a.dst[i];
            if (x >= a.n || y >= a.n) {
                bad = 1;
            } else if (x != y) {
                const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
                const uint32_t bit = 1u << (hi & 31u), pair = lo * kSmallMaxN + hi;
                uint32_t* const word = &rows[lo * words + (hi >> 5)];
                go = !table || atomicExch(&s_seen[(pair * 0x9E3779B1u) >> seen_shift], pair) != pair;
                if (go && (!look || !(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit)))
                    first = !(atomicOr(word, bit) & bit);
                if (first) atomicOr(&rows[hi * words + (lo >> 5)], 1u << (lo & 31u));
            }
        }
        const unsigned long long f = __ballot(first), g = __ballot(go);
        if ((threadIdx.x & 63u) == 0 && i < a.m_in) a.first[i >> 6] = f;
        if (g) look = 2 * __popcll(f) < __popcll(g);
    }
    if (bad) atomicOr(&a.result->err, 1u);
}

// G lanes per edge.
template <uint32_t G, bool PV>
__global__ void __launch_bounds__(kThreads) k_small_count(SmallArgs a) {
    __shared__ unsigned long long s_sum;
    __shared__ uint32_t s_last;
    if (threadIdx.x == 0) s_sum = 0;
    __syncthreads();
    constexpr uint32_t P = 64 / G, U = 4;  // edges at a time; rounds whose rows are loaded together
    const uint32_t lane = threadIdx.x & 63u, gi = lane / G, gl = lane % G;
    const uint64_t wave = blockIdx.x * (uint64_t)(blockDim.x >> 6) + (threadIdx.x >> 6);
    const uint64_t step = (uint64_t)gridDim.x * (blockDim.x >> 6) * P * U;
    unsigned long long sum = 0;
    for (uint64_t base = wave * P * U; base < a.m_in; base += step) {
        uint32_t x[U], y[U];
        bool on[U];
        uint4 r[U], s[U];
#pragma unroll
        for (uint32_t j = 0; j < U; ++j) {
            const uint64_t i = base + j * P + gi;
            on[j] = i < a.m_in && ((a.first[i >> 6] >> (i & 63u)) & 1ull);
            x[j] = on[j] ? a.src[i] : 0u;
            y[j] = on[j] ? a.dst[i] : 0u;
        }
#pragma unroll
        for (uint32_t j = 0; j < U; ++j) {
            r[j] = s[j] = make_uint4(0u, 0u, 0u, 0u);
            if (on[j] && gl < a.quads) {
                r[j] = a.rows[(uint64_t)x[j] * a.quads + gl];
                s[j] = a.rows[(uint64_t)y[j] * a.quads + gl];
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < U; ++j) {
            uint32_t c = (uint32_t)__popc(r[j].x & s[j].x) + (uint32_t)__popc(r[j].y & s[j].y) +
                         (uint32_t)__popc(r[j].z & s[j].z) + (uint32_t)__popc(r[j].w & s[j].w);
            if constexpr (PV) {
#pragma unroll
                for (uint32_t o = 1; o < G; o <<= 1) c += (uint32_t)__shfl_xor((int)c, (int)o, 64);
                if (gl == 0 && c) {
                    atomicAdd(&a.out[x[j]], (unsigned long long)c);
                    atomicAdd(&a.out[y[j]], (unsigned long long)c);
                    sum += c;
                }
            } else {
                sum += c;
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if (lane == 0 && sum) atomicAdd(&s_sum, sum);
    // Every wavefront's adds to `out` are done before this workgroup counts as finished: the barrier waits for
    // LDS only, and thread 0's fence below for its own wavefront's adds.  A wait is enough: what the adds leave in
    // the XCD's L2 is written back by that fence (8192 vertices and 2^19 samples 469 us, as without the wait;
    // 4096 and 2^16 125 -> 130; with a fence per wavefront 606 and 174).
    if constexpr (PV) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_sum) atomicAdd(&a.result->total, s_sum);
        __threadfence();
        s_last = atomicAdd(&a.result->done, 1u) + 1u == gridDim.x;
    }
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    if (threadIdx.x == 0)
        a.result->total = __hip_atomic_load(&a.result->total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) / 3ull;
    if constexpr (PV)
        for (uint32_t i = threadIdx.x; i < a.n; i += blockDim.x)
            a.out[i] = __hip_atomic_load(&a.out[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) / 2ull;
}

template <bool PV>
void launch_count(const SmallArgs& a, uint32_t cus, hipStream_t stream) {
    uint32_t G = 1;
    while (G < a.quads) G <<= 1;
    const uint64_t waves = (a.m_in + 4ull * (64 / G) - 1) / (4ull * (64 / G));
    const uint64_t want = (waves + kThreads / 64 - 1) / (kThreads / 64);
    const dim3 grid((uint32_t)(want < 8ull * cus ? want : 8ull * cus)), block(kThreads);
    switch (G) {
        case 1: hipLaunchKernelGGL((k_small_count<1, PV>), grid, block, 0, stream, a); break;
        case 2: hipLaunchKernelGGL((k_small_count<2, PV>), grid, block, 0, stream, a); break;
        case 4: hipLaunchKernelGGL((k_small_count<4, PV>), grid, block, 0, stream, a); break;
        case 8: hipLaunchKernelGGL((k_small_count<8, PV>), grid, block, 0, stream, a); break;
        case 16: hipLaunchKernelGGL((k_small_count<16, PV>), grid, block, 0, stream, a); break;
        case 32: hipLaunchKernelGGL((k_small_count<32, PV>), grid, block, 0, stream, a); break;
        default: hipLaunchKernelGGL((k_small_count<64, PV>), grid, block, 0, stream, a); break;
    }
}

}  // namespace

SmallLayout small_layout(uint32_t n, uint64_t m_in) {
    SmallLayout L{};
    const uint64_t quads = (n + 127) / 128;
    uint64_t o = 256;  // the result
    L.rows = o;  o += 16 * quads * n;
    L.first = o; o += 8 * ((m_in + 63) / 64);
    L.bytes = (o + 255) & ~255ull;
    return L;
}

hipError_t small_set(const SmallArgs& a, int cu_count, hipStream_t stream) {
    const uint64_t cus = (uint64_t)(cu_count > 0 ? cu_count : 1);
    const uint64_t q = ((uint64_t)a.n * a.quads + 1023) / 1024, threads = a.m_in > kSetFew ? kSetThreads : kThreads;
    const uint64_t s = (a.m_in + threads - 1) / threads, most = 2 * cus * (kSetThreads / threads);
    hipLaunchKernelGGL(k_small_clear, dim3((uint32_t)(q < 2 * cus ? q : 2 * cus)), dim3(1024), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_small_set, dim3((uint32_t)(s < most ? s : most)), dim3((uint32_t)threads), 0, stream, a);
    return hipGetLastError();
}

hipError_t small_count(const SmallArgs& a, int cu_count, hipStream_t stream) {
    const uint32_t cus = (uint32_t)(cu_count > 0 ? cu_count : 1);
    if (a.out) launch_count<true>(a, cus, stream);
    else launch_count<false>(a, cus, stream);
    return hipGetLastError();
}

}  // namespace tc
