// Linear probes: per-token logit/sigmoid, and mean-pooled per request.
//
// Token pass: a workgroup of 512 threads takes TT token slots (one in a small
// launch, for the shortest chain; four in a large one).  Each thread reads
// 16-byte slices of the rows, the group's rows in flight together, and
// accumulates one partial dot product per (token, probe) in registers, the
// probe weights fetched and widened once for the group; partials are reduced
// with fixed DPP moves inside each wave and a fixed-order sum over the waves
// (bit-reproducible, no atomics, and the same for either TT).  HBM bounds a
// large launch; with one token per workgroup 8192 tokens of width 4096 and
// four probes took 28 us, most of it the chain mask -> row -> reduction of
// eight rounds of workgroups.
//
// Mean pooling is a segmented reduction in two launches: the token pass
// writes each token's dot products (without bias) to the workspace, then one
// workgroup per request sums its contiguous span in a fixed order.  Whether
// a request is pooled is decided at the first token of its span, so in this
// mode the token pass finds each token's span and takes the subscription of
// the span's first token: every token of a pooled span gets its dots, also
// where its own mask lacks the bit (a conditional filter narrowed it, or the
// span runs past T_valid).
//
// Last-token mode runs the token pass with one workgroup per request on the
// last token of its span, writing [n_probe][R_max].
//
// A small launch is a chain of round trips; EARLY (one row per workgroup, see
// early_rows) requests the row before the mask is known, and no load of a slice
// stands behind a branch.  Three calls over 8192 tokens (per-token, pooled, last
// token) 43.3 -> 41.4 us.
#include "common.hpp"
#include "kernels.hpp"
#include "launch.hpp"

namespace xmix {

constexpr int kProbeThreads = 512;  // the fused probe + steering pass slices rows the same way
constexpr int kProbeWaves = kProbeThreads / kWave;

// The requests whose spans [cu[r], cu[r+1]) hold tokens t0 .. t0 + TT - 1, or
// -1: with cu non-decreasing, r + 1 is the number of entries cu[0..R] that
// are <= t.  Each wave counts for itself (no barrier); the results are uniform.
template <int TT>
__device__ __forceinline__ void span_of_tokens(const int32_t* __restrict__ cu, int32_t R,
                                               int32_t t0, int32_t (&r)[TT]) {
#pragma unroll
    for (int j = 0; j < TT; ++j) r[j] = -1;
    for (int32_t i0 = 0; i0 <= R; i0 += kWave) {
        const int32_t i = i0 + lane_id();
        const int32_t c = i <= R ? cu[i] : 0x7FFFFFFF;
#pragma unroll
        for (int j = 0; j < TT; ++j) r[j] += __popcll(wave_ballot(c <= t0 + j));
    }
}

template <bool BF16, int MAXP, int TT, bool EARLY>
__global__ void __launch_bounds__(kProbeThreads)
probe_token_kernel(const void* __restrict__ h, int32_t d, int32_t T_max,
                   const uint32_t* __restrict__ tok_mask, const void* __restrict__ w,
                   const float* __restrict__ b, int32_t n_probe,
                   const int32_t* __restrict__ cu, int32_t R, int32_t mode, int32_t slots,
                   float* __restrict__ logit, float* __restrict__ score,
                   float* __restrict__ dots, BitList bits) {
    __shared__ float red[kProbeWaves][TT * MAXP];
    // token mode: slot = token; last-token mode: slot = request, reading the
    // last token of its span (subscription of its first token); mean mode:
    // slot = token, subscription of the first token of its span
    const int32_t s0 = static_cast<int32_t>(blockIdx.x) * TT;
    constexpr int EPV = BF16 ? 8 : 4;
    const int32_t nvec = d / EPV;
    const uint4* H = reinterpret_cast<const uint4*>(h);
    const uint32_t off = threadIdx.x * 16u;
    const int32_t count0 = min(nvec, kProbeThreads);
    // EARLY: the row's first slice, on its way before the mask is known
    // (last-token mode: once its token is)
    uint4 first = make_uint4(0u, 0u, 0u, 0u);
    if constexpr (EARLY) {
        if (mode != 2) {
            first = slice_load(H + static_cast<int64_t>(s0) * nvec, count0, off);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    int32_t tok[TT];
    uint32_t sel[TT], any = 0;  // probes of each slot, of the group
    int32_t span[TT];
    if (mode == 1) span_of_tokens<TT>(cu, R, s0, span);
#pragma unroll
    for (int j = 0; j < TT; ++j) {
        tok[j] = s0 + j;
        sel[j] = 0;
        if (s0 + j >= slots) continue;  // uniform
        int32_t at = s0 + j;            // the token whose mask decides (< 0: none)
        if (mode == 2) {
            const int32_t lo = cu[s0 + j], hi = cu[s0 + j + 1];
            at = hi <= lo || lo < 0 || hi > T_max ? -1 : lo;
            tok[j] = hi - 1;
        } else if (mode == 1) {
            const int32_t r = span[j];
            at = -1;
            if (r >= 0 && r < R) {
                const int32_t lo = cu[r], hi = cu[r + 1];
                // a token past its span's end lies in none; the pooling skips
                // a span outside the slots too
                if (s0 + j < hi && lo >= 0 && hi <= T_max) at = lo;
            }
        }
        if (at < 0) continue;
        if constexpr (EARLY) {
            if (mode == 2) {
                first = slice_load(H + static_cast<int64_t>(tok[j]) * nvec, count0, off);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const uint32_t mask = tok_mask[at];
        XMIX_ARGS_NOW("s"(w), "s"(b), "s"(dots), "s"(bits.first));
        sel[j] = __builtin_amdgcn_readfirstlane(select_bits(mask, bits, n_probe));
        any |= sel[j];
    }
    if (any == 0) return;  // uniform

    // what this thread may finish at the end: probe p of slot s0 + j
    const int p = threadIdx.x / TT, j_out = threadIdx.x % TT;
    const float bias = b[min(p, n_probe - 1)];
    const uint4* W = reinterpret_cast<const uint4*>(w);
    float part[TT][MAXP];
#pragma unroll
    for (int j = 0; j < TT; ++j)
#pragma unroll
        for (int p = 0; p < MAXP; ++p) part[j][p] = 0.0f;

    // weights fetched together with the rows (the rest, for more than eight
    // probes, when used)
    constexpr int AP = MAXP < 8 ? MAXP : 8;
    // words of a row widened at a time: one where that brings the kernel from 70
    // registers under 64 (four workgroups per CU, not three: four token and four
    // pooled probes of 8192 tokens of width 4096, 46.5 -> 43.5 us for the pass of
    // all reads), else all (eight probes stay above 80 and were 3 % slower)
    constexpr int EW = BF16 && MAXP == 4 ? 1 : 4;
    auto slice = [&](const int32_t i0, const uint4* fetched) __attribute__((always_inline)) {
        const int32_t count = min(nvec - i0, kProbeThreads);  // slices of this turn
        // a wave past the row has nothing to add
        const int32_t i = i0 + static_cast<int32_t>(threadIdx.x);
        if (static_cast<int32_t>(__builtin_amdgcn_readfirstlane(i)) >= nvec) return;
        // the rows and the weights of the group's probes, all loaded before the
        // first use, so that the slice waits for one memory round trip
        uint4 hv[TT], wv[AP];
#pragma unroll
        for (int j = 0; j < TT; ++j)
            hv[j] = fetched ? fetched[j]
                            : slice_load(H + static_cast<int64_t>(tok[j]) * nvec + i0,
                                         sel[j] ? count : 0, off);
#pragma unroll
        for (int p = 0; p < AP; ++p)
            wv[p] = slice_load(W + static_cast<int64_t>(p) * nvec + i0,
                               ((any >> p) & 1u) ? count : 0, off);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e0 = 0; e0 < 4; e0 += EW) {
            float x[TT][EW * EPV / 4];
#pragma unroll
            for (int j = 0; j < TT; ++j) {
                const uint32_t hw[4] = {hv[j].x, hv[j].y, hv[j].z, hv[j].w};
#pragma unroll
                for (int e = 0; e < EW; ++e) {
                    if constexpr (BF16) {
                        x[j][2 * e] = lo_bf16(hw[e0 + e]);
                        x[j][2 * e + 1] = hi_bf16(hw[e0 + e]);
                    } else {
                        x[j][e] = __uint_as_float(hw[e0 + e]);
                    }
                }
            }
#pragma unroll
            for (int p = 0; p < MAXP; ++p) {
                if (!((any >> p) & 1u)) continue;  // uniform
                const uint4 w4 = p < AP ? wv[p < AP ? p : 0]
                                        : slice_load(W + static_cast<int64_t>(p) * nvec + i0,
                                                     count, off);
                const uint32_t ww[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                for (int e = 0; e < EW; ++e) {
#pragma unroll
                    for (int j = 0; j < TT; ++j) {
                        if constexpr (BF16) {
                            part[j][p] = fmaf(lo_bf16(ww[e0 + e]), x[j][2 * e], part[j][p]);
                            part[j][p] = fmaf(hi_bf16(ww[e0 + e]), x[j][2 * e + 1], part[j][p]);
                        } else {
                            part[j][p] = fmaf(__uint_as_float(ww[e0 + e]), x[j][e], part[j][p]);
                        }
                    }
                }
            }
        }
    };
    if constexpr (EARLY) slice(0, &first);
    for (int32_t i0 = EARLY ? kProbeThreads : 0; i0 < nvec; i0 += kProbeThreads)
        slice(i0, nullptr);

    const int wave = threadIdx.x / kWave;
#pragma unroll
    for (int p = 0; p < MAXP; ++p) {
        if (!((any >> p) & 1u)) continue;
#pragma unroll
        for (int j = 0; j < TT; ++j) {
            const float s = wave_sum(part[j][p]);
            if (lane_id() == 0) red[wave][p * TT + j] = s;
        }
    }
    __syncthreads();
    const int j = j_out;
    uint32_t sj = sel[0];
#pragma unroll
    for (int u = 1; u < TT; ++u) sj = j == u ? sel[u] : sj;
    if (p < n_probe && ((sj >> p) & 1u)) {
        float dot = 0.0f;
#pragma unroll
        for (int wv = 0; wv < kProbeWaves; ++wv) dot += red[wv][p * TT + j];
        const int64_t o = static_cast<int64_t>(p) * slots + s0 + j;
        if (dots) {
            dots[o] = dot;
        } else {
            const float l = bias + dot;
            logit[o] = l;
            score[o] = logistic(l);
        }
    }
}

// One workgroup per (request, probe): the pooled logit where the request
// carries the probe's bit.  Threads sum strided tokens of the span in order,
// then a fixed DPP pattern and a fixed-order sum over the waves combine them.
__global__ void __launch_bounds__(kProbeThreads)
probe_pool_kernel(const float* __restrict__ dots, int32_t T_max,
                  const uint32_t* __restrict__ tok_mask, const int32_t* __restrict__ cu,
                  const float* __restrict__ b, BitList bits, int32_t n_probe, int32_t R_max,
                  float* __restrict__ logit, float* __restrict__ score) {
    __shared__ float red[kProbeWaves];
    const int32_t r = blockIdx.x, p = blockIdx.y;
    const int32_t lo = cu[r], hi = cu[r + 1];
    if (hi <= lo || lo < 0 || hi > T_max) return;
    const uint32_t mask = tok_mask[lo];
    if (!((mask >> bits.bit(p)) & 1u)) return;  // uniform over the block
    const float* dp = dots + static_cast<int64_t>(p) * T_max;
    float s = 0.0f;
    for (int32_t t = lo + threadIdx.x; t < hi; t += kProbeThreads) s += dp[t];
    s = wave_sum(s);
    if (lane_id() == 0) red[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        float tot = 0.0f;
#pragma unroll
        for (int wv = 0; wv < kProbeWaves; ++wv) tot += red[wv];
        const float l = b[p] + tot / static_cast<float>(hi - lo);
        const int64_t o = static_cast<int64_t>(p) * R_max + r;
        logit[o] = l;
        score[o] = logistic(l);
    }
}

// Slots from which a workgroup takes four: the groups still fill the chip
// twice over.
constexpr int kProbeGroupMin = 2048;

template <bool BF16, int MAXP>
static void launch_probe_p(const void* h, int32_t d, int32_t T_max, const uint32_t* tok_mask,
                           const void* w, const float* b, const BitList& bits, int32_t n_probe,
                           const int32_t* cu, int32_t R, int32_t mode, int32_t slots,
                           float* logit, float* score, float* dots, hipStream_t stream) {
    if constexpr (MAXP <= 8) {
        if (slots >= kProbeGroupMin) {
            hipLaunchKernelGGL((probe_token_kernel<BF16, MAXP, 4, false>), dim3((slots + 3) / 4),
                               dim3(kProbeThreads), 0, stream, h, d, T_max, tok_mask, w, b,
                               n_probe, cu, R, mode, slots, logit, score, dots, bits);
            return;
        }
    }
    constexpr bool kCanEarly = MAXP <= 8;  // more are bound by their weights
    const auto kernel = kCanEarly && early_rows(slots, d / (BF16 ? 8 : 4))
                            ? probe_token_kernel<BF16, MAXP, 1, kCanEarly>
                            : probe_token_kernel<BF16, MAXP, 1, false>;
    hipLaunchKernelGGL(kernel, dim3(slots), dim3(kProbeThreads), 0,
                       stream, h, d, T_max, tok_mask, w, b, n_probe, cu, R, mode, slots, logit,
                       score, dots, bits);
}

template <bool BF16>
static hipError_t launch_probe_t(const void* h, int32_t d, int32_t T_max,
                                 const uint32_t* tok_mask, const void* w, const float* b,
                                 const BitList& bits, int32_t n_probe, const int32_t* cu,
                                 int32_t R, int32_t mode, int32_t slots, float* logit,
                                 float* score, float* dots, hipStream_t stream) {
    const auto launch = n_probe <= 4    ? launch_probe_p<BF16, 4>
                        : n_probe <= 8  ? launch_probe_p<BF16, 8>
                        : n_probe <= 16 ? launch_probe_p<BF16, 16>
                                        : launch_probe_p<BF16, 32>;
    launch(h, d, T_max, tok_mask, w, b, bits, n_probe, cu, R, mode, slots, logit, score, dots,
           stream);
    return hipGetLastError();
}

hipError_t launch_probe(const void* h, bool bf16, int32_t d, int32_t T_max,
                        const uint32_t* tok_mask, const void* w, const float* b,
                        const BitList& bits, int32_t n_probe, int32_t mode,
                        const int32_t* cu_seqlens, int32_t R_max, float* logit, float* score,
                        float* ws, hipStream_t stream) {
    float* dots = mode == 1 ? ws : nullptr;
    const int32_t* cu = mode == 0 ? nullptr : cu_seqlens;
    const int32_t slots = mode == 2 ? R_max : T_max;
    hipError_t e = bf16 ? launch_probe_t<true>(h, d, T_max, tok_mask, w, b, bits, n_probe, cu,
                                               R_max, mode, slots, logit, score, dots, stream)
                        : launch_probe_t<false>(h, d, T_max, tok_mask, w, b, bits, n_probe, cu,
                                                R_max, mode, slots, logit, score, dots, stream);
    if (e != hipSuccess || mode != 1) return e;
    hipLaunchKernelGGL(probe_pool_kernel, dim3(R_max, n_probe), dim3(kProbeThreads), 0, stream,
                       ws, T_max, tok_mask, cu_seqlens, b, bits, n_probe, R_max, logit, score);
    return hipGetLastError();
}

void add_probe_kernels(std::vector<KernelInfo>& t) {
    t.push_back(kernel_info(probe_token_kernel<true, 4, 1, true>));
    t.push_back(kernel_info(probe_token_kernel<true, 4, 1, false>));
    t.push_back(kernel_info(probe_token_kernel<true, 4, 4, false>));
    t.push_back(kernel_info(probe_token_kernel<true, 8, 1, true>));
    t.push_back(kernel_info(probe_token_kernel<true, 8, 1, false>));
    t.push_back(kernel_info(probe_token_kernel<true, 8, 4, false>));
    t.push_back(kernel_info(probe_token_kernel<true, 16, 1, false>));
    t.push_back(kernel_info(probe_token_kernel<true, 32, 1, false>));
    t.push_back(kernel_info(probe_token_kernel<false, 4, 1, true>));
    t.push_back(kernel_info(probe_token_kernel<false, 4, 1, false>));
    t.push_back(kernel_info(probe_token_kernel<false, 4, 4, false>));
    t.push_back(kernel_info(probe_token_kernel<false, 8, 1, true>));
    t.push_back(kernel_info(probe_token_kernel<false, 8, 1, false>));
    t.push_back(kernel_info(probe_token_kernel<false, 8, 4, false>));
    t.push_back(kernel_info(probe_token_kernel<false, 16, 1, false>));
    t.push_back(kernel_info(probe_token_kernel<false, 32, 1, false>));
    t.push_back(kernel_info(probe_pool_kernel));
}

}  // namespace xmix
