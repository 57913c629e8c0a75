// SAE clamp-decode: h[t] += sum_q (c_q - z_q) * W_dec[id_q] for the tokens of
// one app, or of several apps in their order, fp32 accumulation and one RNE
// rounding per app.  Only the n_clamp decoder rows are read; the dense m x d
// decode is never formed.
//
// One workgroup takes kClampTok tokens: the coefficients c - z of every
// (app, clamp, token) are worked out in LDS first, then a thread owns a
// 16-byte column slice of the group's rows, so that each decoder slice is
// fetched and widened once for the group and the rows are in flight together.
// HBM bounds a chunk of many tokens (each selected row read and written once);
// with one token per workgroup the chain mask -> clamp table -> encoded values
// -> decoder rows bounded it (8192 tokens of width 4096, two apps of four
// clamps, half of the tokens each: 48 us).
#include <stddef.h>
#include <string.h>

#include "common.hpp"
#include "kernels.hpp"
#include "launch.hpp"

namespace xmix {

constexpr int kClampThreads = 256;
constexpr int kClampMax = 16;
constexpr int kClampTok = 4;  // tokens per workgroup

struct ClampApps {
    ClampAppIn a[kMultiMax];
    int32_t n;
};

// LIST: the tokens are slots of one app's token list (apps.n == 1), slots past
// its count left alone; otherwise token slots whose masks select the apps.
template <bool LIST>
__global__ void __launch_bounds__(kClampThreads)
clamp_kernel(uint16_t* __restrict__ h, int32_t d, int32_t T_max,
             const uint32_t* __restrict__ tok_mask, const int32_t* __restrict__ app_count,
             const int32_t* __restrict__ tok_list, ClampApps apps) {
    __shared__ __align__(16) float coef[kMultiMax][kClampMax][kClampTok];
    __shared__ int32_t cid[kMultiMax][kClampMax];  // the row read for each clamp (0 if invalid)
    __shared__ int32_t rid[kMultiMax][kClampMax];  // the id a selected latent must match (-1: none)
    __shared__ float cval[kMultiMax][kClampMax];
    const int32_t n0 = static_cast<int32_t>(blockIdx.x) * kClampTok;
    const int tid = threadIdx.x, threads = blockDim.x;
    int32_t tok[kClampTok];
    uint32_t sel[kClampTok], any = 0;  // apps that clamp the token
    const int32_t cnt = LIST ? min(max(*app_count, 0), T_max) : T_max;
#pragma unroll
    for (int j = 0; j < kClampTok; ++j) {
        const bool in = n0 + j < cnt;
        tok[j] = LIST ? (in ? tok_list[n0 + j] : 0) : n0 + j;
        uint32_t m = 0;
        if (in) {
            if constexpr (LIST) {
                m = 1u;
            } else {
                const uint32_t mask = tok_mask[n0 + j];
                for (int a = 0; a < apps.n; ++a) m |= ((mask >> apps.a[a].bit) & 1u) << a;
            }
        }
        sel[j] = m;
        any |= m;
    }
    if (any == 0) return;  // uniform

    const int32_t nvec = d / 8;
    const int32_t step = static_cast<int32_t>(gridDim.y) * threads;
    int32_t i = static_cast<int32_t>(blockIdx.y) * threads + tid;
    uint4 hv[kClampTok];
    auto load_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kClampTok; ++j)
            hv[j] = sel[j] && i < nvec
                        ? reinterpret_cast<const uint4*>(h)[static_cast<int64_t>(tok[j]) * nvec + i]
                        : make_uint4(0u, 0u, 0u, 0u);
    };
    load_rows();  // the first slices are on their way while the tables are made
    for (int e = tid; e < apps.n * kClampMax; e += threads) {
        const int a = e / kClampMax, q = e % kClampMax;
        const ClampAppIn& p = apps.a[a];
        if (((any >> a) & 1u) && q < p.n_clamp) {
            const int32_t id = p.clamp_ids[q];
            const bool ok = id >= 0 && id < p.m;  // an id outside [0, m) clamps nothing
            const float c = p.clamp_vals[q];
            cid[a][q] = ok ? id : 0;
            rid[a][q] = ok ? id : -1;
            cval[a][q] = c;
#pragma unroll
            for (int j = 0; j < kClampTok; ++j) coef[a][q][j] = ok ? c : 0.0f;
        }
    }
    __syncthreads();
    // z of a clamped feature = its encoded value if selected: one wave per
    // (token, app), one lane per encoded latent (k <= 64)
    const int lane = lane_id(), waves = threads / kWave;
    for (int w = tid / kWave; w < apps.n * kClampTok; w += waves) {
        const int a = w / kClampTok, j = w % kClampTok;
        const ClampAppIn& p = apps.a[a];
        int32_t t = tok[0];
        uint32_t sj = sel[0];
#pragma unroll
        for (int u = 1; u < kClampTok; ++u) {
            t = j == u ? tok[u] : t;
            sj = j == u ? sel[u] : sj;
        }
        if (((sj >> a) & 1u) && lane < p.k) {
            const int64_t o = static_cast<int64_t>(t) * p.k + lane;
            const int32_t id = p.idx[o];
            const float z = bf16_to_f32(p.val[o]);
            for (int q = 0; q < p.n_clamp; ++q)
                if (id >= 0 && id == rid[a][q]) coef[a][q][j] = cval[a][q] - z;
        }
    }
    __syncthreads();

    for (;;) {
        if (i < nvec) {
#pragma unroll 1
            for (int a = 0; a < apps.n; ++a) {
                if (!((any >> a) & 1u)) continue;  // uniform
                const ClampAppIn& p = apps.a[a];
                float delta[kClampTok][8];
#pragma unroll
                for (int j = 0; j < kClampTok; ++j)
#pragma unroll
                    for (int e = 0; e < 8; ++e) delta[j][e] = 0.0f;
                const uint4* W = reinterpret_cast<const uint4*>(p.W_dec) + i;
#pragma unroll 4
                for (int q = 0; q < p.n_clamp; ++q) {
                    const uint4 wv = W[static_cast<int64_t>(cid[a][q]) * nvec];
                    const float4 c4 = *reinterpret_cast<const float4*>(coef[a][q]);
                    const float c[kClampTok] = {c4.x, c4.y, c4.z, c4.w};
                    const uint32_t ww[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
                    for (int j = 0; j < kClampTok; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            delta[j][2 * e] = fmaf(c[j], lo_bf16(ww[e]), delta[j][2 * e]);
                            delta[j][2 * e + 1] = fmaf(c[j], hi_bf16(ww[e]), delta[j][2 * e + 1]);
                        }
                }
#pragma unroll
                for (int j = 0; j < kClampTok; ++j) {
                    if (!((sel[j] >> a) & 1u)) continue;  // uniform
                    uint32_t hw[4] = {hv[j].x, hv[j].y, hv[j].z, hv[j].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        hw[e] = pack_bf16(lo_bf16(hw[e]) + delta[j][2 * e],
                                          hi_bf16(hw[e]) + delta[j][2 * e + 1]);
                    hv[j] = make_uint4(hw[0], hw[1], hw[2], hw[3]);
                    if (p.delta_out) {
                        float4* dp = reinterpret_cast<float4*>(
                                         p.delta_out + static_cast<int64_t>(tok[j]) * d) + 2 * i;
                        dp[0] = make_float4(delta[j][0], delta[j][1], delta[j][2], delta[j][3]);
                        dp[1] = make_float4(delta[j][4], delta[j][5], delta[j][6], delta[j][7]);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < kClampTok; ++j)
                if (sel[j])
                    reinterpret_cast<uint4*>(h)[static_cast<int64_t>(tok[j]) * nvec + i] = hv[j];
        }
        i += step;
        if (i - tid >= nvec) break;  // uniform
        load_rows();
    }
}

// Workgroups: the token groups, and while these alone do not fill the chip
// several times the column slices beside them (each repeats the small table
// work of its group).
static void clamp_grid(int32_t T_max, int32_t d, dim3* grid, dim3* block) {
    const int32_t nvec = d / 8, groups = (T_max + kClampTok - 1) / kClampTok;
    // also for a narrow row: the waves share the table work of (app, token) pairs
    // (340 tokens of width 512, three apps of 16 clamps: 22.7 us with one wave)
    const int32_t threads = kClampThreads;
    *block = dim3(threads);
    *grid = dim3(groups, groups >= 1024 ? 1 : (nvec + threads - 1) / threads);
}

hipError_t launch_clamp_multi(uint16_t* h, int32_t d, int32_t T_max, const uint32_t* tok_mask,
                              int32_t n, const ClampAppIn* apps, hipStream_t stream) {
    dim3 grid, block;
    clamp_grid(T_max, d, &grid, &block);
    for (int32_t c0 = 0; c0 < n; c0 += kMultiMax) {
        ClampApps ca;
        memset(&ca, 0, sizeof(ca));
        ca.n = n - c0 < kMultiMax ? n - c0 : kMultiMax;
        for (int32_t i = 0; i < ca.n; ++i) ca.a[i] = apps[c0 + i];
        hipLaunchKernelGGL(clamp_kernel<false>, grid, block, 0, stream, h, d, T_max, tok_mask,
                           static_cast<const int32_t*>(nullptr),
                           static_cast<const int32_t*>(nullptr), ca);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_clamp_decode(uint16_t* h, int32_t d, const int32_t* app_count,
                               const int32_t* tok_list, int32_t T_max, const int32_t* idx,
                               const uint16_t* val, int32_t k, const uint16_t* W_dec, int32_t m,
                               const int32_t* clamp_ids, const float* clamp_vals,
                               int32_t n_clamp, float* delta_out, hipStream_t stream) {
    dim3 grid, block;
    clamp_grid(T_max, d, &grid, &block);
    ClampApps ca;
    memset(&ca, 0, sizeof(ca));
    ca.n = 1;
    ca.a[0].idx = idx;
    ca.a[0].val = val;
    ca.a[0].W_dec = W_dec;
    ca.a[0].clamp_ids = clamp_ids;
    ca.a[0].clamp_vals = clamp_vals;
    ca.a[0].delta_out = delta_out;
    ca.a[0].k = k;
    ca.a[0].m = m;
    ca.a[0].n_clamp = n_clamp;
    hipLaunchKernelGGL(clamp_kernel<true>, grid, block, 0, stream, h, d, T_max,
                       static_cast<const uint32_t*>(nullptr), app_count, tok_list, ca);
    return hipGetLastError();
}

// Where the batched descriptor holds device pointers (for the graph
// executor's redirection).
template <>
struct ArgPointers<ClampApps> {
    static std::vector<uint16_t> offsets() {
        std::vector<uint16_t> o;
        for (int i = 0; i < kMultiMax; ++i)
            for (const size_t f : {offsetof(ClampAppIn, idx), offsetof(ClampAppIn, val),
                                   offsetof(ClampAppIn, W_dec), offsetof(ClampAppIn, clamp_ids),
                                   offsetof(ClampAppIn, clamp_vals),
                                   offsetof(ClampAppIn, delta_out)})
                o.push_back(
                    static_cast<uint16_t>(offsetof(ClampApps, a) + i * sizeof(ClampAppIn) + f));
        return o;
    }
};

void add_clamp_kernels(std::vector<KernelInfo>& t) {
    t.push_back(kernel_info(clamp_kernel<true>));
    t.push_back(kernel_info(clamp_kernel<false>));
}

}  // namespace xmix
