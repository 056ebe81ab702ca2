// Division of an ordered item list into queue fetches (device code).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tc {

// Guided fetches of a bin in largest-work-first order by `waves` workers (wavefronts or workgroups): the
// first `waves` fetches take `unit` items each, the next `waves` twice as many, and so on up to `cap` items per fetch.  With `cap` from the start
// one wavefront took the 16 (packed: 64) heaviest vertices of the bin one after another: R-MAT scale 16
// spent 1.57 ms in a chain of 16 vertices of 3e4 probes, Barabasi-Albert with 1000 vertices ran on 16
// wavefronts.
struct Guided {
    uint32_t n, waves, unit, cap, levels, level0;  // level0: items the doubling levels take
    __device__ __forceinline__ Guided(uint32_t n_, uint32_t waves_, uint32_t unit_, uint32_t cap_)
        : n(n_), waves(waves_ < 65536u ? waves_ : 65536u), unit(unit_), cap(cap_), levels(0) {
        while ((unit << levels) < cap) ++levels;  // sizes unit << l below cap
        level0 = unit * waves * ((1u << levels) - 1u);
    }
    __device__ __forceinline__ Guided(uint32_t n_, uint32_t waves_, uint32_t unit_, uint32_t cap_, uint32_t levels_)
        : n(n_), waves(waves_ < 65536u ? waves_ : 65536u), unit(unit_), cap(cap_), levels(levels_) {
        level0 = unit * waves * ((1u << levels) - 1u);
    }
    __device__ __forceinline__ uint32_t fetches() const {
        if (n > level0) return levels * waves + (n - level0 + cap - 1) / cap;
        uint32_t f = 0, left = n;
        for (uint32_t l = 0; left; ++l) {
            const uint32_t size = unit << l, most = (left + size - 1) / size;
            const uint32_t take = most < waves ? most : waves;
            f += take;
            left = most <= waves ? 0u : left - waves * size;
        }
        return f;
    }
    __device__ __forceinline__ void range(uint32_t f, uint32_t& j0, uint32_t& j1) const {
        const uint32_t l = f / waves;
        uint32_t size = cap;
        if (l < levels) {
            size = unit << l;
            j0 = unit * waves * ((1u << l) - 1u) + (f - l * waves) * size;
        } else {
            j0 = level0 + (f - levels * waves) * cap;
        }
        j1 = j0 + size < n ? j0 + size : n;
    }
};

}  // namespace tc
