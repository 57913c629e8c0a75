// Per-token probes and the steering add in one pass over each row: a hook
// where apps read and write (probes and steering vectors composed at one
// layer).  The row is read once in 16-byte slices; the probes take their
// dot products from the values as read (the activation as the model
// produced it), the steering sum is added in fp64 and the row written back
// rounded once.  The arithmetic and its order are those of the separate
// probe and steering kernels (same slicing, same per-thread accumulation,
// same reductions), so the results are bit-identical to a token-mode probe
// call followed by a steering call.  One workgroup of 512 threads per
// token slot (a 4096-wide bf16 row is one slice per thread, so every load
// of the pass goes out at once); a row with neither kind of bit returns
// after reading its mask word (EARLY: and asking for its first slices).
//
// With r_tvalid given, the kernel also builds the step's routing (in place
// of a route-build launch): n_apps more workgroups, dispatched first, each
// build one app's token list from the routing inputs staged in LDS and
// publish it with its count (the first also the error word), and each token
// workgroup computes its token's mask itself and writes it.
#include "common.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "route_list.hpp"
#include "steer_add.hpp"

namespace xmix {

constexpr int kFuseThreads = 512;  // a 4096-wide bf16 row is one 16-byte slice per thread
constexpr int kFuseWaves = kFuseThreads / kWave;

// MAXP: at most this many probes; NS: steering vectors fetched together.
template <bool BF16, int MAXP, int NS, bool EARLY>
__global__ void __launch_bounds__(kFuseThreads)
steer_probe_kernel(void* __restrict__ h, int32_t d, int32_t T_max,
                   const uint32_t* __restrict__ tok_mask, const int32_t* __restrict__ req,
                   const int32_t* __restrict__ r_tvalid, const uint32_t* __restrict__ r_sub,
                   int32_t r_Rmax, int32_t r_napps, const void* __restrict__ vecs,
                   const float* __restrict__ alpha, int32_t n_steer, const void* __restrict__ w,
                   const float* __restrict__ b, int32_t n_probe, float* __restrict__ logit,
                   float* __restrict__ score, uint32_t* __restrict__ r_mask,
                   int32_t* __restrict__ r_count, int32_t* __restrict__ r_lists,
                   uint32_t* __restrict__ r_err, BitList sbits, BitList pbits) {
    __shared__ float red[kFuseWaves][MAXP];
    const int n_list = r_tvalid ? r_napps : 0;  // route-list workgroups
    if (static_cast<int>(blockIdx.x) < n_list) {  // uniform
        __shared__ int32_t list_s[kRouteMaxT];
        __shared__ int32_t rtot_s[kFuseWaves];
        __shared__ int32_t req_s[kRouteMaxT];
        __shared__ uint32_t sub_s[kStageSubMax];
        const int a = blockIdx.x;
        stage_route<kFuseThreads>(req, T_max, r_sub, r_Rmax, req_s, sub_s);
        uint32_t err = 0;
        const int32_t tv = clamp_t_valid(*r_tvalid, T_max, err);
        const uint32_t keep = r_napps >= 32 ? 0xFFFFFFFFu : ((1u << r_napps) - 1u);
        __syncthreads();  // the staged inputs
        const int32_t n = build_token_list<kFuseThreads>(req_s, tv, sub_s, r_sub, r_Rmax, keep, a,
                                                         T_max, list_s, rtot_s, nullptr, err);
        publish_token_list<kFuseThreads>(list_s, n, T_max,
                                         r_lists + static_cast<int64_t>(a) * T_max, r_count + a);
        if (a == 0) publish_error(err, r_err);  // its pass saw every slot
        return;
    }
    const int32_t t = static_cast<int32_t>(blockIdx.x) - n_list;
    constexpr int EPV = BF16 ? 8 : 4;  // elements per 16-byte vector
    const int32_t nvec = d / EPV;
    uint4* row = reinterpret_cast<uint4*>(h) + static_cast<int64_t>(t) * nvec;
    const uint32_t off = threadIdx.x * 16u;
    uint4 first;  // the row's first slice, on its way before the mask is known
    if constexpr (EARLY) {
        first = slice_load(row, min(nvec, kFuseThreads), off);
        __builtin_amdgcn_sched_barrier(0);
    }
    const int32_t rq = req[t];  // loaded beside the mask (alpha's row depends on it)
    uint32_t mask = tok_mask[t];  // (not the step's when the routing is built here)
    XMIX_ARGS_NOW("s"(rq), "s"(mask), "s"(vecs), "s"(alpha), "s"(n_steer), "s"(w), "s"(b),
                  "s"(n_probe), "s"(sbits.first), "s"(pbits.first));
    const float bias = b[min(static_cast<int32_t>(threadIdx.x), n_probe - 1)];
    if (r_tvalid) {  // uniform
        uint32_t unused = 0;
        const int32_t tv = clamp_t_valid(*r_tvalid, T_max, unused);
        const uint32_t keep = r_napps >= 32 ? 0xFFFFFFFFu : ((1u << r_napps) - 1u);
        mask = request_mask(rq, t, tv, r_sub, r_Rmax, keep, unused);
        if (threadIdx.x == 0) r_mask[t] = mask;
    }
    const uint32_t ss = __builtin_amdgcn_readfirstlane(select_bits(mask, sbits, n_steer));
    const uint32_t sp = __builtin_amdgcn_readfirstlane(select_bits(mask, pbits, n_probe));
    if ((ss | sp) == 0) return;
    const float* a_row = ss ? alpha + static_cast<int64_t>(rq) * n_steer : alpha;
    const uint4* V = reinterpret_cast<const uint4*>(vecs);
    const uint4* W = reinterpret_cast<const uint4*>(w);
    float part[MAXP];
#pragma unroll
    for (int p = 0; p < MAXP; ++p) part[p] = 0.0f;
    SteerGroup<NS> g0;  // the token's first NS steering vectors
    uint32_t rest0 = ss;
    steer_pick(g0, rest0, a_row, n_steer);

    // probe weights fetched together with the row (the rest, for more than
    // eight probes, when used)
    constexpr int AP = MAXP < 8 ? MAXP : 8;
    auto slice = [&](const int32_t i0, const uint4* fetched) __attribute__((always_inline)) {
        const int32_t count = min(nvec - i0, kFuseThreads);  // slices of this turn
        const int32_t i = i0 + static_cast<int32_t>(threadIdx.x);
        // a wave past the row has nothing to add (340 rows of width 512: 6.6 us
        // with it, 4.9 without)
        if (static_cast<int32_t>(__builtin_amdgcn_readfirstlane(i)) >= nvec) return;
        // Every load of the slice before its first use, and none behind a
        // branch: the row, the weights of the token's probes and its first NS
        // steering vectors, so that the slice waits for one memory round trip,
        // not one per operand.
        const uint4 hv = fetched ? *fetched : slice_load(row + i0, count, off);
        uint4 wv[AP];
#pragma unroll
        for (int p = 0; p < AP; ++p)
            wv[p] = slice_load(W + static_cast<int64_t>(p) * nvec + i0,
                               ((sp >> p) & 1u) ? count : 0, off);
        steer_fetch(g0, V + i0, nvec, count, off);
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t hw[4] = {hv.x, hv.y, hv.z, hv.w};
        // probes, on the row as read
        float x[EPV];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (BF16) {
                x[2 * e] = lo_bf16(hw[e]);
                x[2 * e + 1] = hi_bf16(hw[e]);
            } else {
                x[e] = __uint_as_float(hw[e]);
            }
        }
#pragma unroll
        for (int p = 0; p < MAXP; ++p) {
            if (!((sp >> p) & 1u)) continue;
            const uint4 w4 = p < AP ? wv[p < AP ? p : 0]
                                    : slice_load(W + static_cast<int64_t>(p) * nvec + i0, count, off);
            const uint32_t ww[4] = {w4.x, w4.y, w4.z, w4.w};
            float acc = part[p];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (BF16) {
                    acc = fmaf(lo_bf16(ww[e]), x[2 * e], acc);
                    acc = fmaf(hi_bf16(ww[e]), x[2 * e + 1], acc);
                } else {
                    acc = fmaf(__uint_as_float(ww[e]), x[e], acc);
                }
            }
            part[p] = acc;
        }
        // steering, written back: the first NS vectors as fetched, then the
        // rest NS at a time
        if (ss) {
            double acc[EPV];
#pragma unroll
            for (int e = 0; e < EPV; ++e) acc[e] = x[e];
            steer_add_group<BF16>(acc, g0);
            for (uint32_t rest = rest0; rest != 0;) {
                SteerGroup<NS> g;
                steer_pick(g, rest, a_row, n_steer);
                steer_fetch(g, V + i0, nvec, count, off);
                steer_add_group<BF16>(acc, g);
            }
            uint4 out;
            if constexpr (BF16) {
                out.x = pack_bf16_from_f64(acc[0], acc[1]);
                out.y = pack_bf16_from_f64(acc[2], acc[3]);
                out.z = pack_bf16_from_f64(acc[4], acc[5]);
                out.w = pack_bf16_from_f64(acc[6], acc[7]);
            } else {
                out.x = __float_as_uint(static_cast<float>(acc[0]));
                out.y = __float_as_uint(static_cast<float>(acc[1]));
                out.z = __float_as_uint(static_cast<float>(acc[2]));
                out.w = __float_as_uint(static_cast<float>(acc[3]));
            }
            if (i < nvec) row[i] = out;
        }
    };
    if constexpr (EARLY) slice(0, &first);
    for (int32_t i0 = EARLY ? kFuseThreads : 0; i0 < nvec; i0 += kFuseThreads) slice(i0, nullptr);
    if (sp == 0) return;  // uniform over the block

    const int wave = threadIdx.x / kWave;
#pragma unroll
    for (int p = 0; p < MAXP; ++p) {
        if (!((sp >> p) & 1u)) continue;
        const float s = wave_sum(part[p]);
        if (lane_id() == 0) red[wave][p] = s;
    }
    __syncthreads();
    const int p = threadIdx.x;
    if (p < n_probe && ((sp >> p) & 1u)) {
        float dot = 0.0f;
#pragma unroll
        for (int wv = 0; wv < kFuseWaves; ++wv) dot += red[wv][p];
        const int64_t o = static_cast<int64_t>(p) * T_max + t;
        const float l = bias + dot;
        logit[o] = l;
        score[o] = logistic(l);
    }
}

template <bool BF16, int MAXP>
static auto pick_kernel(bool two, bool early) {
    return two ? (early ? steer_probe_kernel<BF16, MAXP, 2, true>
                        : steer_probe_kernel<BF16, MAXP, 2, false>)
               : (early ? steer_probe_kernel<BF16, MAXP, 4, true>
                        : steer_probe_kernel<BF16, MAXP, 4, false>);
}

template <bool BF16>
static hipError_t launch_steer_probe_t(void* h, int32_t d, int32_t T_max,
                                       const uint32_t* tok_mask, const int32_t* req,
                                       const void* vecs, const BitList& sbits,
                                       const float* alpha, int32_t n_steer, const void* w,
                                       const float* b, const BitList& pbits, int32_t n_probe,
                                       float* logit, float* score, const RouteIn& r,
                                       hipStream_t stream) {
    // A load that finds nothing to fetch still has to be issued: with two probes
    // and two steering vectors at most no more are asked for (16 layers of 512 fp32
    // rows of 16 KB, two of each, 5 % of the bits set: 79.5 us with room for four
    // of each, 67.0 without).
    const bool two = n_steer <= 2;
    // more than eight probes leave a pass bound by its weights, not by the chain
    const bool early = early_rows(T_max, d / (BF16 ? 8 : 4));
    const auto kernel =
        n_probe <= 2    ? pick_kernel<BF16, 2>(two, early)
        : n_probe <= 4  ? pick_kernel<BF16, 4>(two, early)
        : n_probe <= 8  ? (early ? steer_probe_kernel<BF16, 8, 4, true>
                                 : steer_probe_kernel<BF16, 8, 4, false>)
        : n_probe <= 16 ? steer_probe_kernel<BF16, 16, 4, false>
                        : steer_probe_kernel<BF16, 32, 4, false>;
    hipLaunchKernelGGL(kernel, dim3(T_max + (r.T_valid ? r.n_apps : 0)), dim3(kFuseThreads), 0,
                       stream, h, d, T_max, tok_mask, req, r.T_valid, r.sub, r.R_max, r.n_apps,
                       vecs, alpha, n_steer, w, b, n_probe, logit, score, r.tok_mask, r.app_count,
                       r.app_tokens, r.err_word, sbits, pbits);
    return hipGetLastError();
}

hipError_t launch_steer_probe(void* h, bool bf16, int32_t d, int32_t T_max,
                              const uint32_t* tok_mask, const int32_t* req, const void* vecs,
                              const BitList& sbits, const float* alpha, int32_t n_steer,
                              const void* w, const float* b, const BitList& pbits,
                              int32_t n_probe, float* logit, float* score, hipStream_t stream,
                              const RouteIn* route) {
    RouteIn r{};
    if (route) {
        if (T_max > kRouteMaxT || T_max < route->n_apps) {
            // the kernel cannot route this batch: the route-build launch first
            const hipError_t e = launch_route_build(route->req, route->T_valid, route->sub,
                                                    route->R_max, T_max, route->n_apps,
                                                    route->tok_mask, route->app_count,
                                                    route->app_tokens, route->err_word, stream);
            if (e != hipSuccess) return e;
        } else {
            r = *route;
        }
    }
    return bf16 ? launch_steer_probe_t<true>(h, d, T_max, tok_mask, req, vecs, sbits, alpha,
                                             n_steer, w, b, pbits, n_probe, logit, score, r,
                                             stream)
                : launch_steer_probe_t<false>(h, d, T_max, tok_mask, req, vecs, sbits, alpha,
                                              n_steer, w, b, pbits, n_probe, logit, score, r,
                                              stream);
}

template <bool BF16>
static void add_steer_probe_t(std::vector<KernelInfo>& t) {
    for (const bool two : {false, true})
        for (const bool early : {false, true}) {
            t.push_back(kernel_info(pick_kernel<BF16, 2>(two, early)));
            t.push_back(kernel_info(pick_kernel<BF16, 4>(two, early)));
        }
    t.push_back(kernel_info(steer_probe_kernel<BF16, 8, 4, true>));
    t.push_back(kernel_info(steer_probe_kernel<BF16, 8, 4, false>));
    t.push_back(kernel_info(steer_probe_kernel<BF16, 16, 4, false>));
    t.push_back(kernel_info(steer_probe_kernel<BF16, 32, 4, false>));
}

void add_steer_probe_kernels(std::vector<KernelInfo>& t) {
    add_steer_probe_t<true>(t);
    add_steer_probe_t<false>(t);
}

}  // namespace xmix
