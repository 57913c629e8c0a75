// The steering sum of one 16-byte slice of a row (internal) of the fused probe
// + steering pass, which adds in the order of the steering kernel: acc (the
// slice, widened to fp64) += alpha[s] * v_s for every set bit s of sel,
// ascending, one fp64 FMA per element.  N vectors at a time: which ones,
// with their alphas (steer_pick), their slices (steer_fetch), the adds
// (steer_add_group).
#pragma once

#include "common.hpp"

namespace xmix {

// Up to N vectors of the steering sum with their alphas.
template <int N>
struct SteerGroup {
    uint4 v[N];
    float a[N];
    int s[N], n;
};

// The next set bits of `rest` (ascending; they are cleared from it) and their
// alphas, of n_steer in the row; the last one's stand in where there are fewer.
// Vector loads: scalar ones return out of order, so the first use of one would
// wait for all of them.
template <int N>
__device__ __forceinline__ void steer_pick(SteerGroup<N>& g, uint32_t& rest,
                                           const float* __restrict__ a_row, int32_t n_steer) {
    g.n = min(__popc(rest), N);
    int zero = 0;
    asm("" : "+v"(zero));
#pragma unroll
    for (int j = 0; j < N; ++j) {
        g.s[j] = min(__builtin_ctz(rest | 0x80000000u), n_steer - 1);
        rest &= rest - 1;  // 0 stays 0
        g.a[j] = a_row[g.s[j] + zero];
    }
}

// The group's slices: `count` slices of a row at V (the vectors nvec apart).
template <int N>
__device__ __forceinline__ void steer_fetch(SteerGroup<N>& g, const uint4* __restrict__ V,
                                            int32_t nvec, int32_t count, uint32_t off) {
#pragma unroll
    for (int j = 0; j < N; ++j)
        g.v[j] = slice_load(V + static_cast<int64_t>(g.s[j]) * nvec, j < g.n ? count : 0, off);
}

// acc += a[j] * v_j for the group's vectors in order, one fp64 FMA per element.
template <bool BF16, int N>
__device__ __forceinline__ void steer_add_group(double (&acc)[BF16 ? 8 : 4],
                                                const SteerGroup<N>& g) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (j >= g.n) break;
        const uint32_t vw[4] = {g.v[j].x, g.v[j].y, g.v[j].z, g.v[j].w};
        // opaque here, so that its conversion is not moved up (and its load
        // waited for) before the slices are requested
        float af = g.a[j];
        asm volatile("" : "+v"(af));
        const double a = af;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (BF16) {
                acc[2 * e] = fma(a, static_cast<double>(lo_bf16(vw[e])), acc[2 * e]);
                acc[2 * e + 1] = fma(a, static_cast<double>(hi_bf16(vw[e])), acc[2 * e + 1]);
            } else {
                acc[e] = fma(a, static_cast<double>(__uint_as_float(vw[e])), acc[e]);
            }
        }
    }
}

}  // namespace xmix
