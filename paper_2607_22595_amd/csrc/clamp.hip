// SAE clamp-decode: h[t] += sum_q (c_q - z_q) * W_dec[id_q] for the tokens of
// one app, or of several apps in their order, fp32 accumulation and one RNE
// rounding per app.  Only the n_clamp decoder rows are read; the dense m x d
// decode is never formed.
//
// A workgroup takes one token, or four of a large launch: the coefficients
// c - z of every (app, clamp, token) are worked out in LDS first, then a thread
// owns a 16-byte column slice of the group's rows.  A launch of few tokens is the
// chain mask -> clamp table and encoded values -> decoder rows, and one token per
// workgroup keeps it short: 140 tokens of width 512, three apps of six clamps,
// 30 % of the tokens each, take 5.6 us, and 9.3 in groups of four.  With many
// subscribed tokens the decoder slices, read again for each token, bound it, and
// a group fetches and widens each once for its four: 8192 tokens of width 4096,
// four apps of twelve clamps, every token, take 90 us, and 142 one by one.
#include <stddef.h>
#include <string.h>

#include "common.hpp"
#include "kernels.hpp"
#include "launch.hpp"

namespace xmix {

constexpr int kClampThreads = 256;
constexpr int kClampMax = 16;
struct ClampApps {
    ClampAppIn a[kMultiMax];
    int32_t n;
};

// LIST: the tokens are slots of one app's token list (apps.n == 1), slots past
// its count left alone; otherwise token slots whose masks select the apps.
template <bool LIST, int TOK>
__global__ void __launch_bounds__(kClampThreads)
clamp_kernel(uint16_t* __restrict__ h, int32_t d, int32_t T_max,
             const uint32_t* __restrict__ tok_mask, const int32_t* __restrict__ app_count,
             const int32_t* __restrict__ tok_list, int32_t fours, ClampApps apps) {
    __shared__ __align__(16) float coef[kMultiMax][kClampMax][TOK];
    __shared__ int32_t cid[kMultiMax][kClampMax];  // the row read for each clamp (0 if invalid)
    int32_t n0 = static_cast<int32_t>(blockIdx.x) * TOK;
    if (TOK == 1 && fours > 0) {  // token 4 x + j where workgroup x of fours per column runs
        const int32_t x = n0 / 32 * 8 + ((n0 - static_cast<int32_t>(blockIdx.y) * fours) & 7);
        n0 = 4 * x + (n0 / 8 & 3);
    }
    const int tid = threadIdx.x;
    int32_t tok[TOK];
    uint32_t sel[TOK], any = 0;  // apps that clamp the token
    const int32_t cnt = LIST ? min(max(*app_count, 0), T_max) : T_max;
#pragma unroll
    for (int j = 0; j < TOK; ++j) {
        const int32_t n = min(n0 + j, T_max - 1);
        const bool in = n0 + j < cnt;
        if constexpr (LIST) {
            const int32_t t = tok_list[n];
            tok[j] = in ? t : 0;
            sel[j] = in ? 1u : 0u;
        } else {
            const uint32_t mask = tok_mask[n];
            uint32_t m = 0;
#pragma unroll
            for (int a = 0; a < kMultiMax; ++a)
                if (a < apps.n) m |= ((mask >> apps.a[a].bit) & 1u) << a;
            tok[j] = n;
            sel[j] = in ? m : 0u;
        }
        any |= sel[j];
    }
    if (any == 0) return;  // uniform

    // z of a clamped feature = its encoded value if selected: one wave per
    // (app, token), a lane per clamp and per encoded latent (k <= 64).  The
    // clamp table and the encoded values of kTurn pairs, and behind them the
    // first slices of the rows, are asked for together and behind no branch.
    constexpr int kWaves = kClampThreads / kWave;
    constexpr int kTurn = LIST ? 1 : TOK == 1 ? kMultiMax / kWaves : 4;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int pairs = (LIST ? 1 : apps.n) * TOK;
    int32_t id[kTurn], li[kTurn];
    float cv[kTurn], lv[kTurn];
    bool on[kTurn];
    auto ask = [&](const int w0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
            const int w = min(w0 + u * kWaves, pairs - 1), a = w / TOK, j = w % TOK;
            const ClampAppIn& p = apps.a[a];
            int32_t t = tok[0];
            uint32_t sj = sel[0];
#pragma unroll
            for (int v = 1; v < TOK; ++v) {
                t = j == v ? tok[v] : t;
                sj = j == v ? sel[v] : sj;
            }
            on[u] = w0 + u * kWaves < pairs && ((sj >> a) & 1u);
            const int64_t o = static_cast<int64_t>(t) * p.k;
            const int32_t nc = on[u] ? p.n_clamp : 0, nk = on[u] ? p.k : 0;
            id[u] = lane_load(p.clamp_ids, nc, lane);
            cv[u] = __int_as_float(lane_load(p.clamp_vals, nc, lane));
            li[u] = lane_load(p.idx + o, nk, lane);
            lv[u] = bf16_to_f32(lane_load(p.val + o, nk, lane));
        }
    };
    ask(wave);
    __builtin_amdgcn_sched_barrier(0);
    const int32_t nvec = d / 8;
    const int32_t step = static_cast<int32_t>(gridDim.y) * kClampThreads;
    int32_t i = static_cast<int32_t>(blockIdx.y) * kClampThreads + tid;
    uint4 hv[TOK];
    auto load_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TOK; ++j)
            hv[j] = sel[j] && i < nvec
                        ? reinterpret_cast<const uint4*>(h)[static_cast<int64_t>(tok[j]) * nvec + i]
                        : make_uint4(0u, 0u, 0u, 0u);
    };
    load_rows();
    __builtin_amdgcn_sched_barrier(0);
    for (int w0 = wave; w0 < pairs;) {
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
            if (!on[u]) continue;  // uniform
            const int w = w0 + u * kWaves, a = w / TOK, j = w % TOK;
            const ClampAppIn& p = apps.a[a];
            const bool ok = id[u] >= 0 && id[u] < p.m;  // an id outside [0, m) clamps nothing
            const int32_t have = lane < p.k ? li[u] : -1;
            float c = cv[u];
            for (int q0 = 0; q0 < p.n_clamp; q0 += 4) {  // kClampMax is a multiple of 4
                uint64_t hit[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    hit[e] = wave_ballot(have == __builtin_amdgcn_readlane(id[u], q0 + e));
                if ((hit[0] | hit[1] | hit[2] | hit[3]) == 0) continue;  // uniform
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (hit[e] != 0 && lane == q0 + e)
                        c = cv[u] - readlane_f(lv[u], 63 - __builtin_clzll(hit[e]));
            }
            if (lane < p.n_clamp) {
                cid[a][lane] = ok ? id[u] : 0;
                coef[a][lane][j] = ok ? c : 0.0f;
            }
        }
        w0 += kTurn * kWaves;
        if (w0 >= pairs) break;
        ask(w0);
    }
    __syncthreads();

    for (;;) {
        if (i < nvec) {
#pragma unroll 1
            for (int a = 0; a < apps.n; ++a) {
                if (!((any >> a) & 1u)) continue;  // uniform
                const ClampAppIn& p = apps.a[a];
                float delta[TOK][8];
#pragma unroll
                for (int j = 0; j < TOK; ++j)
#pragma unroll
                    for (int e = 0; e < 8; ++e) delta[j][e] = 0.0f;
                const uint4* W = reinterpret_cast<const uint4*>(p.W_dec) + i;
#pragma unroll 4
                for (int q = 0; q < p.n_clamp; ++q) {
                    const uint4 wv = W[static_cast<int64_t>(cid[a][q]) * nvec];
                    float c[TOK];
                    if constexpr (TOK == 4) {
                        const float4 c4 = *reinterpret_cast<const float4*>(coef[a][q]);
                        c[0] = c4.x, c[1] = c4.y, c[2] = c4.z, c[3] = c4.w;
                    } else {
#pragma unroll
                        for (int j = 0; j < TOK; ++j) c[j] = coef[a][q][j];
                    }
                    const uint32_t ww[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
                    for (int j = 0; j < TOK; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            delta[j][2 * e] = fmaf(c[j], lo_bf16(ww[e]), delta[j][2 * e]);
                            delta[j][2 * e + 1] = fmaf(c[j], hi_bf16(ww[e]), delta[j][2 * e + 1]);
                        }
                }
#pragma unroll
                for (int j = 0; j < TOK; ++j) {
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
            for (int j = 0; j < TOK; ++j)
                if (sel[j])
                    reinterpret_cast<uint4*>(h)[static_cast<int64_t>(tok[j]) * nvec + i] = hv[j];
        }
        i += step;
        if (i - tid >= nvec) break;  // uniform
        load_rows();
    }
}

// Workgroups: the token groups, and while these alone do not fill the chip
// several times the column slices beside them (each repeats the table work of
// its group).  A list launch holds fewer groups than its slots allow (4096 slots
// of width 8192, 30 % of them listed, two clamps: 12.5 us with column slices,
// 16.7 without).
template <bool LIST, int TOK>
static hipError_t launch_clamp_t(uint16_t* h, int32_t d, int32_t T_max, const uint32_t* tok_mask,
                                 const int32_t* app_count, const int32_t* tok_list,
                                 const ClampApps& ca, hipStream_t stream) {
    const int32_t nvec = d / 8, slices = (nvec + kClampThreads - 1) / kClampThreads;
    // also for a narrow row: the waves share the table work of (app, token) pairs
    // (340 tokens of width 512, three apps of 16 clamps: 22.7 us with one wave)
    const int32_t cols = T_max >= (LIST ? 8192 : 4096) ? 1 : min(slices, kGridCols);
    // Tokens taken one by one where the steering kernel groups its rows: the same
    // rows on the same XCDs, whose L2 holds what a steering call before this one
    // wrote (1100 rows of 8192, two steering vectors and two clamps, every token:
    // 25 us for both in that order, 32 without)
    int32_t groups = (T_max + TOK - 1) / TOK, fours = 0;
    if (TOK == 1 && rows_grouped(T_max, slices)) {
        fours = (T_max + 3) / 4;
        groups = (fours + 7) / 8 * 32;
    }
    hipLaunchKernelGGL((clamp_kernel<LIST, TOK>), dim3(groups, cols), dim3(kClampThreads), 0,
                       stream, h, d, T_max, tok_mask, app_count, tok_list, fours, ca);
    return hipGetLastError();
}

template <bool LIST>
static hipError_t launch_clamp(uint16_t* h, int32_t d, int32_t T_max, const uint32_t* tok_mask,
                               const int32_t* app_count, const int32_t* tok_list,
                               const ClampApps& ca, hipStream_t stream) {
    int32_t clamps = 0;
    for (int32_t i = 0; i < ca.n; ++i) clamps += ca.a[i].n_clamp;
    // Groups of four pay where the decoder slices shared by a group outweigh its
    // longer chain.  How many tokens subscribe is not known here, so the line is
    // drawn where a fully subscribed launch gains little (one token against four:
    // 1024 rows of 4096, four apps of twelve clamps 22.2 and 20.4 us with every
    // token, three of six 11.1 and 11.9 with 30 %), and further out for few
    // clamps, which leave little to share (4096 rows of 4096, two apps of three:
    // 25.5 and 23.2 us with every token, 9.4 and 12.3 with 10 %).  Beyond it a
    // sparse launch would still do better one by one (4096 rows of 8192, four
    // apps of two, 10 %: 19 and 30 us), a full one far worse (2048 rows of 8192,
    // four of twelve: 70 and 52).
    const int64_t work = static_cast<int64_t>(T_max) * d;
    const bool one = work <= (4 << 20) || (clamps <= 6 && work <= (16 << 20));
    return (one ? launch_clamp_t<LIST, 1> : launch_clamp_t<LIST, 4>)(
        h, d, T_max, tok_mask, app_count, tok_list, ca, stream);
}

hipError_t launch_clamp_multi(uint16_t* h, int32_t d, int32_t T_max, const uint32_t* tok_mask,
                              int32_t n, const ClampAppIn* apps, hipStream_t stream) {
    for (int32_t c0 = 0; c0 < n; c0 += kMultiMax) {
        ClampApps ca;
        memset(&ca, 0, sizeof(ca));
        ca.n = n - c0 < kMultiMax ? n - c0 : kMultiMax;
        for (int32_t i = 0; i < ca.n; ++i) ca.a[i] = apps[c0 + i];
        const hipError_t e =
            launch_clamp<false>(h, d, T_max, tok_mask, nullptr, nullptr, ca, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_clamp_decode(uint16_t* h, int32_t d, const int32_t* app_count,
                               const int32_t* tok_list, int32_t T_max, const int32_t* idx,
                               const uint16_t* val, int32_t k, const uint16_t* W_dec, int32_t m,
                               const int32_t* clamp_ids, const float* clamp_vals,
                               int32_t n_clamp, float* delta_out, hipStream_t stream) {
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
    return launch_clamp<true>(h, d, T_max, nullptr, app_count, tok_list, ca, stream);
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
    t.push_back(kernel_info(clamp_kernel<true, 1>));
    t.push_back(kernel_info(clamp_kernel<true, 4>));
    t.push_back(kernel_info(clamp_kernel<false, 1>));
    t.push_back(kernel_info(clamp_kernel<false, 4>));
}

}  // namespace xmix
