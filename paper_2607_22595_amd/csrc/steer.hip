// Steering add: h[t] += sum over the token's steering bits of alpha * v,
// accumulated in fp64 and rounded once.  The products alpha (fp32) x v
// (bf16/fp32) are exact in fp64 and the few-term sum carries ~1e-16
// relative error, so the single rounding to the storage type is correct even
// when h and the steering terms nearly cancel (fp32 accumulation can be off
// by an ulp of the small result there).
//
// A thread owns one 16-byte column slice of TT token rows: every access is a
// coalesced 16-byte load or store, the rows of the group are in flight
// together, and a steering vector is fetched and widened once for the group.
// HBM bounds a chunk of many tokens, but only just: the fp64 adds run at the
// fp32 rate, while each widening and the rounding back cost several times as
// much (pack_bf16_from_f64 rounds on 32-bit words for that reason).  Rows
// without a steering bit are not read; a group without one returns after
// reading its mask words.  The group's masks and requests come in one round trip,
// and its alphas with the vectors they multiply: loaded at their adds they were
// waited for one by one (steering and clamps of 8192 tokens 60 -> 57 us).
#include "common.hpp"
#include "kernels.hpp"
#include "launch.hpp"

namespace xmix {

constexpr int kSteerThreads = 256;
constexpr int kSteerGroup = 4;  // token rows per workgroup in a large launch

template <bool BF16, int TT>
__global__ void __launch_bounds__(kSteerThreads)
steer_kernel(void* __restrict__ h, int32_t d, int32_t T_max,
             const uint32_t* __restrict__ tok_mask, const int32_t* __restrict__ req,
             const void* __restrict__ vecs, const float* __restrict__ alpha, int32_t n_steer,
             BitList bits) {
    constexpr int EPV = BF16 ? 8 : 4;  // elements per 16-byte vector
    const int32_t t0 = static_cast<int32_t>(blockIdx.x) * TT;
    const int32_t nvec = d / EPV;
    const int32_t i = static_cast<int32_t>(
        (blockIdx.z * kGridCols + blockIdx.y) * kSteerThreads + threadIdx.x);
    // masks and requests of the group in one round trip
    uint32_t sel[TT], any = 0;
    int32_t rq[TT];
#pragma unroll
    for (int j = 0; j < TT; ++j) {
        const int32_t t = min(t0 + j, T_max - 1);
        sel[j] = tok_mask[t];
        rq[j] = req[t];
    }
    XMIX_ARGS_NOW("s"(sel[0]), "s"(rq[0]), "s"(sel[TT / 4]), "s"(rq[TT / 4]), "s"(sel[TT / 2]),
                  "s"(rq[TT / 2]), "s"(sel[TT - 1]), "s"(rq[TT - 1]), "s"(vecs), "s"(alpha),
                  "s"(n_steer), "s"(bits.first));
    const float* a_row[TT];
#pragma unroll
    for (int j = 0; j < TT; ++j) {
        sel[j] = select_bits(t0 + j < T_max ? sel[j] : 0u, bits, n_steer);
        any |= sel[j];
        a_row[j] = sel[j] ? alpha + static_cast<int64_t>(rq[j]) * n_steer : alpha;
    }
    if (any == 0 || i >= nvec) return;

    uint4* row = reinterpret_cast<uint4*>(h) + static_cast<int64_t>(t0) * nvec + i;
    const uint4* V = reinterpret_cast<const uint4*>(vecs) + i;
    uint4 hv[TT];
#pragma unroll
    for (int j = 0; j < TT; ++j)
        hv[j] = sel[j] ? row[static_cast<int64_t>(j) * nvec] : make_uint4(0u, 0u, 0u, 0u);
    double acc[TT][EPV];
    bool widened = false;
    for (uint32_t rest = any; rest != 0;) {
        // up to four vectors (ascending bits), fetched together
        uint4 v[4];
        float al[4][TT];  // their alphas (entry 0 for a vector or row without one)
        int sv[4], n = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = make_uint4(0u, 0u, 0u, 0u);
            sv[q] = 0;
            if (rest != 0) {
                sv[q] = __builtin_ctz(rest);
                rest &= rest - 1;
                v[q] = V[static_cast<int64_t>(sv[q]) * nvec];
                n = q + 1;
            }
#pragma unroll
            for (int j = 0; j < TT; ++j) al[q][j] = a_row[j][sv[q]];
        }
        if (!widened) {  // the rows, once the first vectors are on their way
            widened = true;
#pragma unroll
            for (int j = 0; j < TT; ++j) {
                const uint32_t hw[4] = {hv[j].x, hv[j].y, hv[j].z, hv[j].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (BF16) {
                        acc[j][2 * e] = lo_bf16(hw[e]);
                        acc[j][2 * e + 1] = hi_bf16(hw[e]);
                    } else {
                        acc[j][e] = __uint_as_float(hw[e]);
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q >= n) break;  // uniform
            const uint32_t vw[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
            double x[EPV];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (BF16) {
                    x[2 * e] = lo_bf16(vw[e]);
                    x[2 * e + 1] = hi_bf16(vw[e]);
                } else {
                    x[e] = __uint_as_float(vw[e]);
                }
            }
#pragma unroll
            for (int j = 0; j < TT; ++j) {
                if (!((sel[j] >> sv[q]) & 1u)) continue;  // uniform
                const double a = al[q][j];
#pragma unroll
                for (int e = 0; e < EPV; ++e) acc[j][e] = fma(a, x[e], acc[j][e]);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < TT; ++j) {
        if (!sel[j]) continue;  // uniform
        uint4 out;
        if constexpr (BF16) {
            out.x = pack_bf16_from_f64(acc[j][0], acc[j][1]);
            out.y = pack_bf16_from_f64(acc[j][2], acc[j][3]);
            out.z = pack_bf16_from_f64(acc[j][4], acc[j][5]);
            out.w = pack_bf16_from_f64(acc[j][6], acc[j][7]);
        } else {
            out.x = __float_as_uint(static_cast<float>(acc[j][0]));
            out.y = __float_as_uint(static_cast<float>(acc[j][1]));
            out.z = __float_as_uint(static_cast<float>(acc[j][2]));
            out.w = __float_as_uint(static_cast<float>(acc[j][3]));
        }
        row[static_cast<int64_t>(j) * nvec] = out;
    }
}

template <bool BF16>
static hipError_t launch_steer_t(void* h, int32_t d, int32_t T_max, const uint32_t* tok_mask,
                                 const int32_t* req, const void* vecs, const BitList& bits,
                                 const float* alpha, int32_t n_steer, hipStream_t stream) {
    const int32_t nvec = d / (BF16 ? 8 : 4);
    const int32_t threads = nvec < kSteerThreads ? (nvec + kWave - 1) / kWave * kWave : kSteerThreads;
    const int32_t cols = (nvec + threads - 1) / threads;
    const int32_t z = (cols - 1) / kGridCols + 1, y = z > 1 ? kGridCols : cols;
    if (rows_grouped(T_max, cols))
        hipLaunchKernelGGL((steer_kernel<BF16, kSteerGroup>),
                           dim3((T_max + kSteerGroup - 1) / kSteerGroup, y, z), dim3(threads), 0,
                           stream, h, d, T_max, tok_mask, req, vecs, alpha, n_steer, bits);
    else
        hipLaunchKernelGGL((steer_kernel<BF16, 1>), dim3(T_max, y, z), dim3(threads), 0, stream, h,
                           d, T_max, tok_mask, req, vecs, alpha, n_steer, bits);
    return hipGetLastError();
}

hipError_t launch_steer(void* h, bool bf16, int32_t d, int32_t T_max, const uint32_t* tok_mask,
                        const int32_t* req, const void* vecs, const BitList& bits,
                        const float* alpha, int32_t n_steer, hipStream_t stream) {
    return bf16 ? launch_steer_t<true>(h, d, T_max, tok_mask, req, vecs, bits, alpha, n_steer,
                                       stream)
                : launch_steer_t<false>(h, d, T_max, tok_mask, req, vecs, bits, alpha, n_steer,
                                        stream);
}

void add_steer_kernels(std::vector<KernelInfo>& t) {
    t.push_back(kernel_info(steer_kernel<true, 1>));
    t.push_back(kernel_info(steer_kernel<true, kSteerGroup>));
    t.push_back(kernel_info(steer_kernel<false, 1>));
    t.push_back(kernel_info(steer_kernel<false, kSteerGroup>));
}

}  // namespace xmix
