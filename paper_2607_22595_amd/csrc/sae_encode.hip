// SAE encode with TopK: pre = W_enc . h + c_fold for the tokens subscribed
// to one app, then the k largest pre-activations per token.
//
// Stage 1 (sae_stream_kernel) is an MFMA bf16 GEMM with fp32 accumulation, in
// three kinds of tiles by the live tokens and the size of the dictionary
// (tile_kind).  In the basic one a workgroup (8 waves, two per SIMD so one wave's waits overlap the other's
// MFMAs) owns 256 latents x 128 subscribed tokens and walks K = d in chunks
// of 64:
//   - the dictionary (operand A) streams from HBM straight into registers
//     from the tiled layout below (each wave-wide load is 1 KB contiguous,
//     each workgroup reads its 2 MiB slice front to back; nontemporal
//     loads, as nothing reads it again), each wave owning 32 latents,
//     through a four-deep register ring (three chunks in flight);
//   - the token rows (operand B) are gathered through the app's token list
//     into LDS (double buffered; the 16-byte chunk c of row n is stored at
//     c ^ ((n >> 1) & 7), so the 16 rows one MFMA-layout read touches per
//     LDS cycle land in 16 distinct bank groups) and shared by the 8 waves.
// Epilogue, per token of the tile: a threshold tau is chosen so that the
// number of latents with pre >= tau lies in a small window (first guess
// mean + z * stdev of the tile's 256 values, then bisection on the value if
// needed); every latent with pre >= tau is emitted as a candidate, and the
// count and the tile's bound are recorded: a value that every latent left
// out lies below (the decode kernels: the next value above the largest one
// left out; the prefill GEMM: tau, or the next value above the tile's
// maximum when nothing is emitted).  This costs O(1) work per value.
// The decode kernel writes the tile to LDS token-major, and eight lanes of
// one wave select for each token with no barrier or LDS atomic between the
// waves.  The prefill kernel (one wave per SIMD, values in accumulator
// registers) runs the four token groups of a wave through each phase
// together; a wave alone on its SIMD has no other wave to hide its
// latencies, and the LDS path measured slower there.
//
// Stage 2 (sae_merge_kernel): one workgroup per subscribed token gathers the
// candidates of all tiles and selects the exact top-k of that pool (a radix
// select over (value, latent) composites, ties to the lower latent).  The result is the exact top-k of
// all m latents whenever the k-th selected value is >= every tile's bound,
// because a latent that was not emitted lies below its tile's bound.  When
// that certificate fails (only for inputs whose best latents crowd into a
// few tiles or tie across whole tiles), the workgroup recomputes tiles'
// 256 pre-activations, in descending order of
// their bounds, until no tile left can hold a winner.  Every path, the recompute
// among them, sums a pre-activation with the same instruction in the same order, so
// a token's result depends on its row and the dictionary alone: not on the batch
// it is in, the tiles that are chosen or the other apps of the launch.  The
// decode kernel's first threshold guess leaves a tile's outlying values
// out of the statistics (beyond mean +- 5 stdev), so that a few strong
// latents, such as features clamped high by a steering app, or rows of a
// much larger norm than the others, do not lift it: with a decode
// dictionary's ratio of k to m the certificate has little slack.  The
// prefill kernel keeps the plain statistics (a GEMM epilogue
// pays for every extra pass, and the repair covers the rare failure).
//
// The workgroup-to-tile maps are XCD-aware (unit_tile, sae_gemm_kernel): launch
// slots are dealt round-robin to the 8 XCDs, so consecutive tiles of one XCD share
// a dictionary slice in that XCD's L2.
#include <math.h>
#include <stddef.h>
#include <string.h>

#include <atomic>
#include <type_traits>

#include "common.hpp"
#include "emit_plan.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "route_list.hpp"

namespace xmix {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

constexpr int kBM = 256;  // latents per workgroup
constexpr int kBN = 128;  // tokens per workgroup
constexpr int kBK = 64;   // K chunk
constexpr int kEncWaves = 8;
constexpr int kEncThreads = kEncWaves * kWave;
constexpr int kRefineIters = 24;
// Values beyond mean +- kTrimZ * stdev of a tile's 256 pre-activations are
// left out of the statistics behind the decode kernel's first threshold
// guess (one strong latent, or one of a large norm on either side, would
// otherwise raise the guess for its whole tile).
constexpr float kTrimZ = 5.0f;

// mean + z * stdev of n values with sum s1 and sum of squares s2
__device__ __forceinline__ float trimmed_guess(float s1, float s2, int n, float z) {
    const float inv = 1.0f / static_cast<float>(n > 0 ? n : 1);
    const float mu = s1 * inv;
    return mu + z * sqrtf(fmaxf(s2 * inv - mu * mu, 0.0f));
}

// Step of the threshold search away from a count outside the window, from a
// tenth of |tau| doubling from round to round.  A tile that keeps a few values
// too many is usually inside the window one such step on, still well below
// the token's k-th value; a step of |tau| / 4 + 1 went past its maximum, and
// a tile that keeps none of its ten best sends the token to the repair.
__device__ __forceinline__ float refine_step(float tau, int it) {
    return ldexpf(0.1f * (fabsf(tau) + 0.1f), it);
}

__device__ __forceinline__ bf16x8_t as_bf16x8(const uint4& v) {
    return __builtin_bit_cast(bf16x8_t, v);
}

// ------------------------------------------------------- dictionary layout
// W_enc is kept in HBM in a tiled layout matched to the encode GEMMs, built
// once when an SAE app is loaded.  The unit is a 16-byte piece (8 bf16 of
// one latent row).  Latent j = 256*mt + 32*w + r and row element
// i = 64*kc + 16*s + 8*g + e (e < 8) live in piece
//     (kc*n_mt + mt)*2048 + w*256 + s*64 + (r + 32*g)
// so the 32 KB of a 256-latent slice per K chunk of 64 are contiguous,
// every wave-wide 16-byte load is 1 KB contiguous (the A operand of one
// 32x32x16 MFMA step s: lane r + 32*g holds elements 16*s + 8*g .. + 7),
// each half chunk (steps 0-1, steps 2-3) is 2 KB contiguous per 32
// latents, and at each K step the whole grid streams one contiguous region
// (chunk-major order spreads concurrent workgroups over all HBM channels).
__device__ __forceinline__ int64_t packed_piece(int32_t j, int32_t i, int32_t n_mt) {
    const int32_t mt = j >> 8, jr = j & 255;
    const int32_t w = jr >> 5, r = jr & 31;
    const int32_t kc = i >> 6, s = (i >> 4) & 3, g = (i >> 3) & 1;
    return (static_cast<int64_t>(kc) * n_mt + mt) * 2048 + w * 256 + s * 64 + r + 32 * g;
}

__global__ void __launch_bounds__(256)
sae_pack_kernel(const uint16_t* __restrict__ W, int32_t m, int32_t d, uint16_t* __restrict__ Wp) {
    const int32_t pieces_per_row = d / 8;
    const int64_t q = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (q >= static_cast<int64_t>(m) * pieces_per_row) return;
    const int32_t j = static_cast<int32_t>(q / pieces_per_row);
    const int32_t i = static_cast<int32_t>(q % pieces_per_row) * 8;
    reinterpret_cast<uint4*>(Wp)[packed_piece(j, i, m / kBM)] =
        reinterpret_cast<const uint4*>(W)[q];
}

// c_fold[j] = b_enc[j] - W_enc[j,:] . b_dec (packed W_enc), one wave per latent.
__global__ void __launch_bounds__(256)
sae_fold_kernel(const uint16_t* __restrict__ Wp, const uint16_t* __restrict__ b_enc,
                const uint16_t* __restrict__ b_dec, int32_t m, int32_t d,
                float* __restrict__ c_fold) {
    const int32_t j = blockIdx.x * 4 + threadIdx.x / kWave;
    if (j >= m) return;
    const int32_t n_mt = m / kBM;
    const uint4* P = reinterpret_cast<const uint4*>(Wp);
    const uint4* bd = reinterpret_cast<const uint4*>(b_dec);
    float acc = 0.0f;
    for (int32_t p = lane_id(); p < d / 8; p += kWave) {
        const uint4 wv = P[packed_piece(j, p * 8, n_mt)], bv = bd[p];
        const uint32_t ww[4] = {wv.x, wv.y, wv.z, wv.w};
        const uint32_t bw[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc = fmaf(lo_bf16(ww[e]), lo_bf16(bw[e]), acc);
            acc = fmaf(hi_bf16(ww[e]), hi_bf16(bw[e]), acc);
        }
    }
    acc = wave_sum(acc);
    if (lane_id() == 0) c_fold[j] = bf16_to_f32(b_enc[j]) - acc;
}

// ------------------------------------------------ wave-local slice selection
// After a tile's K loop, its values are written to LDS token-major and the
// values of a token's slice are taken by a group of LPS lanes of one wave,
// VPL contiguous latents per lane (VPL * LPS = the slice's latents).  The
// threshold search, the counts and the emission prefix then reduce over
// those lanes with DPP moves: no barrier and no LDS atomic between the
// waves.  Each lane works on NT tokens at once (independent chains that
// fill each other's latencies).  A row's stride is 4 words past a multiple
// of the 64 LDS banks, so the 16-byte reads of the 64 lanes at one step
// spread over every bank.
constexpr int kSelStride = 260;  // floats per token row of 256 latents

// Reductions inside groups of LPS lanes (8, 4 or 2) on DPP moves (quad_perm,
// row_half_mirror)
template <int LPS>
__device__ __forceinline__ float sum_g(float v) {
    v += dpp_f<kDppXor1>(v);
    if constexpr (LPS >= 4) v += dpp_f<kDppXor2>(v);
    if constexpr (LPS >= 8) v += dpp_f<kDppHalfMirror>(v);
    return v;
}
template <int LPS>
__device__ __forceinline__ int isum_g(int v) {
    v += dpp_i<kDppXor1>(v);
    if constexpr (LPS >= 4) v += dpp_i<kDppXor2>(v);
    if constexpr (LPS >= 8) v += dpp_i<kDppHalfMirror>(v);
    return v;
}
template <int LPS>
__device__ __forceinline__ float max_g(float v) {
    v = fmaxf(v, dpp_f<kDppXor1>(v));
    if constexpr (LPS >= 4) v = fmaxf(v, dpp_f<kDppXor2>(v));
    if constexpr (LPS >= 8) v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
    return v;
}
// sum over the lanes q' < q of the group (q = lane % LPS)
template <int LPS>
__device__ __forceinline__ int excl_scan_g(int v, int q) {
    int incl = v;
    int y = dpp_i<0x111>(incl);  // row_shr:1
    incl += q >= 1 ? y : 0;
    if constexpr (LPS >= 4) {
        y = dpp_i<0x112>(incl);  // row_shr:2
        incl += q >= 2 ? y : 0;
    }
    if constexpr (LPS >= 8) {
        y = dpp_i<0x114>(incl);  // row_shr:4
        incl += q >= 4 ? y : 0;
    }
    return incl - v;
}

// The selection of NT tokens over one slice each: per token a threshold tau
// with lo_cnt <= count(pre >= tau) <= cap (first guess mean + z * stdev of
// the slice's values, then bisection on the value), and every latent with
// pre >= tau written to dst[t][0 .. count) as (fp32 bits, latent), with the
// count and the slice's bound beside it.  vrow[t]: this lane's VPL values of
// token t in LDS; q: the lane's place in its group;
// lat0: its first latent.  Every lane of the wave calls it (the cross-lane
// steps are wave-wide); the lanes of a token with valid[t] == false take part
// in them and write nothing.  With TRIM, the values beyond mean +- 5 stdev
// are left out of the statistics behind the first guess (a few outlying
// latents would otherwise lift it for the whole slice).
template <bool TRIM, int NT, int VPL, int LPS>
__device__ __forceinline__ void select_slices(const float* const (&vrow)[NT], int q,
                                              const bool (&valid)[NT], float z, int lo_cnt,
                                              int cap, int32_t lat0, uint2* const (&dst)[NT],
                                              int32_t* const (&cnt_out)[NT],
                                              float* const (&tau_out)[NT]) {
    constexpr int kW = VPL * LPS;  // latents of a slice
    float x[NT][VPL];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
#pragma unroll
        for (int i = 0; i < VPL / 4; ++i) {
            const float4 v = reinterpret_cast<const float4*>(vrow[t])[i];
            x[t][4 * i] = v.x;
            x[t][4 * i + 1] = v.y;
            x[t][4 * i + 2] = v.z;
            x[t][4 * i + 3] = v.w;
        }
    }
    // ax[t]: the largest magnitude among the token's values
    float tau[NT], s1[NT], s2[NT], ax[NT], mu[NT], sd[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float a = 0.0f, b = 0.0f, c = 0.0f;
#pragma unroll
        for (int i = 0; i < VPL; ++i) {
            a += x[t][i];
            b = fmaf(x[t][i], x[t][i], b);
            if (TRIM) c = fmaxf(c, fabsf(x[t][i]));
        }
        s1[t] = a;
        s2[t] = b;
        ax[t] = c;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        s1[t] = sum_g<LPS>(s1[t]);
        s2[t] = sum_g<LPS>(s2[t]);
        if (TRIM) ax[t] = max_g<LPS>(ax[t]);
        mu[t] = s1[t] * (1.0f / kW);
        sd[t] = sqrtf(fmaxf(s2[t] * (1.0f / kW) - mu[t] * mu[t], 0.0f));
        tau[t] = mu[t] + z * sd[t];
    }
    if (TRIM) {
        // values more than kTrimZ stdev from the mean on either side: a large
        // value lifts the mean and the spread, a large negative one the
        // spread.  A value that far out has a magnitude above
        // kTrimZ * stdev - |mean|; the pass below leaves out exactly the
        // values beyond the two cuts, so a token it finds none for keeps its
        // guess.
        bool trim[NT], any = false;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            trim[t] = valid[t] && ax[t] + fabsf(mu[t]) > kTrimZ * sd[t];
            any = any || trim[t];
        }
        if (wave_ballot(any)) {  // uniform
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const float cut = mu[t] + kTrimZ * sd[t], cut_lo = mu[t] - kTrimZ * sd[t];
                float e1 = 0.0f, e2 = 0.0f;
                int ne = 0;
#pragma unroll
                for (int i = 0; i < VPL; ++i) {
                    const bool o = x[t][i] > cut || x[t][i] < cut_lo;
                    ne += o ? 1 : 0;
                    e1 += o ? x[t][i] : 0.0f;
                    e2 = fmaf(o ? x[t][i] : 0.0f, x[t][i], e2);
                }
                e1 = sum_g<LPS>(e1);
                e2 = sum_g<LPS>(e2);
                ne = isum_g<LPS>(ne);
                if (trim[t]) tau[t] = trimmed_guess(s1[t] - e1, s2[t] - e2, kW - ne, z);
            }
        }
    }
    float lo[NT], hi[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        lo[t] = -INFINITY;
        hi[t] = INFINITY;
    }
    // m[t]: this lane's latents at or above tau[t], one bit each; the count
    // is its population, so the emission below reuses the last round's masks
    uint32_t m[NT];
    auto masks = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            uint32_t b = 0;
#pragma unroll
            for (int i = 0; i < VPL; ++i) b |= (x[t][i] >= tau[t] ? 1u : 0u) << i;
            m[t] = b;
        }
    };
    bool settled = false;
    for (int it = 0; it < kRefineIters; ++it) {
        masks();
        int c[NT];
        bool bad[NT], any = false;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            c[t] = isum_g<LPS>(__popc(m[t]));
            bad[t] = valid[t] && (c[t] > cap || c[t] < lo_cnt);
            any = any || bad[t];
        }
        if (!wave_ballot(any)) {  // uniform
            settled = true;
            break;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (!bad[t]) continue;
            if (c[t] > cap) lo[t] = tau[t];
            else hi[t] = tau[t];
            if (it == kRefineIters - 1) {
                // out of rounds: a threshold whose count is known to be below
                // lo_cnt (or +inf, count 0); the merge then checks exactness
                tau[t] = hi[t];
            } else if (isfinite(lo[t]) && isfinite(hi[t])) {
                tau[t] = 0.5f * (lo[t] + hi[t]);
            } else {
                const float step = refine_step(tau[t], it);
                tau[t] = isfinite(hi[t]) ? tau[t] - step : tau[t] + step;
            }
        }
    }
    // out of rounds: the final thresholds were set after the last masks
    if (!settled) masks();
    // emission: this lane's selected latents go to the slots after those of
    // the lanes before it in the token's group; nk[t]: the largest of
    // the token's values that are not kept (NaN never counts: it compares
    // below everything)
    int base[NT], total[NT];
    float nk[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int cl = __popc(m[t]);
        base[t] = excl_scan_g<LPS>(cl, q);
        total[t] = isum_g<LPS>(cl);
        float l = -INFINITY;
#pragma unroll
        for (int i = 0; i < VPL; ++i) l = fmaxf(l, x[t][i] >= tau[t] ? -INFINITY : x[t][i]);
        nk[t] = max_g<LPS>(l);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if (!valid[t]) continue;
        uint32_t b = m[t];
        int slot = base[t];
        while (b != 0) {
            const int i = __builtin_ctz(b);
            b &= b - 1;
            if (slot < cap)
                dst[t][slot] = make_uint2(__float_as_uint(vrow[t][i]),
                                          static_cast<uint32_t>(lat0 + i));
            ++slot;
        }
        if (q == 0) {
            *cnt_out[t] = min(total[t], cap);
            // the slice's bound: the next value above the largest one it
            // does not keep (at most tau, and the tightest bound there is;
            // with nothing kept, the next value above its maximum)
            *tau_out[t] = key_f32(f32_key(nk[t]) + 1u);
        }
    }
}

// ---------------------------------------------- GEMM + candidate emission
// The dictionary stream of one workgroup: the first piece of a slice's K
// chunk 0, and the pieces from one K chunk to the next (both the same for
// every lane; each lane adds its own offset when it loads).
struct SliceSrc {
    const uint4* base;
    int64_t stride;
};
__device__ __forceinline__ SliceSrc slice_src(const uint16_t* W, int32_t n_mt, int mt) {
    return {reinterpret_cast<const uint4*>(W) + static_cast<int64_t>(mt) * 2048,
            static_cast<int64_t>(n_mt) * 2048};
}
// operand A of one K chunk at p: this wave's 32 latents of the packed
// slice.  The dictionary is read once per launch: nontemporal loads stream
// it past the caches (about 4 % faster than cached loads at 65536 x 4096).
__device__ __forceinline__ void load_chunk(uint4* a, const uint4* p) {
    const uint32_t off = threadIdx.x & 511;  // wave * 256 + lane: pieces 4 x 64 apart
    const u32x4_t* q = reinterpret_cast<const u32x4_t*>(p) + ((off >> 6) * 256 + (off & 63));
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const u32x4_t v = __builtin_nontemporal_load(q + s * 64);
        a[s] = make_uint4(v.x, v.y, v.z, v.w);
    }
}
// the folded bias of this lane's 16 latents of slice mt
__device__ __forceinline__ void load_bias(float (&cfv)[16], const float* c_fold, int mt) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float* cf = c_fold + mt * kBM + 32 * wave + 4 * (lane >> 5);
#pragma unroll
    for (int r = 0; r < 16; ++r) cfv[r] = cf[8 * (r / 4) + (r % 4)];
}

// Where one app's slices put their candidates, and how they select them:
// per token slot a row of n_sl slices.
struct SliceSink {
    uint2* cand;
    int32_t* tile_cnt;
    float* tile_tau;
    int32_t n_sl, lo_cnt, cap;
    float z;
};

// A buffer offset past every resource (none is larger than 2^31 - 1 bytes), and
// far enough from 2^32 that no scalar offset wraps it.
constexpr uint32_t kOutOfRange = 0x80000000u;

// A 16-byte buffer load; offsets past the resource's end read zero and touch no
// memory, so a load past the K loop's last chunk needs no branch: its resource
// is empty (and its scalar offset zero: the range check subtracts it).
template <int AUX>
__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t r, uint32_t voff,
                                               uint32_t soff) {
    const u32x4_t v = __builtin_bit_cast(
        u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, AUX));
    return make_uint4(v.x, v.y, v.z, v.w);
}
constexpr int kNontemporal = 2;  // cache policy bit of the buffer loads

// A workgroup's LDS: K loop: token chunks, windows or stages; epilogue: the
// selection rows.  16-byte pieces.
constexpr int kLdsMain = kBN * kSelStride / 4;

// The registers of a workgroup's dictionary stream: what is in flight of one tile
// and, past its last chunk, of the next.
constexpr int kRing = 16;

// What slice_tile finds loaded of its slice.
__device__ __forceinline__ void slice_first(uint4 (&ring)[kRing], float (&cfv)[16],
                                            const SliceSrc src, const float* c_fold, int mt) {
#pragma unroll
    for (int c = 0; c < 3; ++c) load_chunk(ring + 4 * c, src.base + c * src.stride);
    load_bias(cfv, c_fold, mt);
}

// The GEMM and candidate emission of latent slice mt over one tile of tokens:
// tl[n0, n0 + ntok) of the app's list, ntok <= kBN.  On entry the ring holds
// the slice's K chunks 0-2 and cfv its folded bias (slice_first).  The K
// loop fetches three chunks ahead; past the slice's last chunk it fetches
// the first chunks of what runs next, slice `nxt` when has_nxt (then also its bias
// from nxt_bias_of(), after this tile's selection), else nothing new (the last
// chunk again, unused; no load where has_nxt is false at compile time).  lds_main is the workgroup's token-chunk and
// selection space; sink_of() is asked for after the K loop, whose scalar
// registers are few.  The candidates are emitted in WK slices of 256 / WK latents.
template <int WK, typename SinkOf, typename BiasOf>
__device__ __forceinline__ void slice_tile(
    uint4* lds_main, const uint16_t* __restrict__ h, int32_t d, const int32_t* tl, int n0,
    int ntok, int mt, const SliceSrc cur, SinkOf sink_of, const SliceSrc nxt, bool has_nxt,
    int nxt_mt, BiasOf nxt_bias_of, uint4 (&ring)[kRing], float (&cfv)[16]) {
    uint4 *wa0 = ring, *wa1 = ring + 4, *wa2 = ring + 8, *wa3 = ring + 12;
    uint4 (*xs)[kBN * 8] = reinterpret_cast<uint4 (*)[kBN * 8]>(lds_main);
    int tid = threadIdx.x;  // opaque (see big_tile)
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 5, j32 = lane & 31;
    const int nK = d / kBK;  // a multiple of 4 (d % 256 == 0)

    // operand B: gathered token rows; padding rows read a valid row and are
    // zeroed when written to LDS
    const int xr = tid >> 3, xc = tid & 7;
    const uint16_t* xrow[2];
    uint32_t xmask[2];
    f32x16_t acc[4];
    uint4 xv0[2], xv1[2];                   // token ring: 2 chunks in flight
    auto load_x = [&](uint4 (&xv)[2], int kc) {
        kc = min(kc, nK - 1);
#pragma unroll
        for (int p = 0; p < 2; ++p) xv[p] = *reinterpret_cast<const uint4*>(xrow[p] + kc * kBK);
    };
    auto store_x = [&](const uint4 (&xv)[2], int buf) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int n = xr + 64 * p;
            const uint4 v = make_uint4(xv[p].x & xmask[p], xv[p].y & xmask[p],
                                       xv[p].z & xmask[p], xv[p].w & xmask[p]);
            xs[buf][n * 8 + (xc ^ ((n >> 1) & 7))] = v;
        }
    };
    auto compute = [&](const uint4* a, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const bf16x8_t A = as_bf16x8(a[s]);
            uint4 bop[4];
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                const int n = 32 * nb + j32;
                const int chunk = 2 * s + g;
                bop[nb] = xs[buf][n * 8 + (chunk ^ ((n >> 1) & 7))];
            }
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
                acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, as_bf16x8(bop[nb]), acc[nb],
                                                                  0, 0, 0);
        }
    };
    // One K chunk (branch-free): issue the token chunk two ahead and the W
    // chunk three ahead (at wp), multiply the current chunk, then publish
    // the next token chunk to the other LDS buffer.  Loads are issued
    // oldest-needed first, so the in-order vmcnt wait for the next token
    // chunk never waits on a W prefetch.
    auto step = [&](int kc, const uint4* cur_w, uint4* wnext, const uint4* wp, uint4 (&xload)[2],
                    const uint4 (&xstore)[2]) __attribute__((always_inline)) {
        load_x(xload, kc + 2);
        __builtin_amdgcn_sched_barrier(0);  // keep the token loads ahead of the W loads
        load_chunk(wnext, wp);
        __syncthreads();
        compute(cur_w, kc & 1);
        store_x(xstore, (kc + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
    };

    const uint4* after = has_nxt ? nxt.base : cur.base + (nK - 1) * cur.stride;
    const int64_t after_stride = has_nxt ? nxt.stride : 0;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int n = xr + 64 * p;
        const bool ok = n < ntok;
        xmask[p] = ok ? 0xFFFFFFFFu : 0u;
        xrow[p] = h + static_cast<int64_t>(tl[n0 + (ok ? n : 0)]) * d + 8 * xc;
    }
    // the accumulators start from the folded bias
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[b][r] = cfv[r];

    load_x(xv0, 0);
    load_x(xv1, 1);
    store_x(xv0, 0);
    // four chunks per round (the W registers rotate); the last round
    // fetches what follows the slice
    auto round4 = [&](int kc, const uint4* p0, const uint4* p1, const uint4* p2,
                      const uint4* p3) {
        step(kc + 0, wa0, wa3, p0, xv0, xv1);
        step(kc + 1, wa1, wa0, p1, xv1, xv0);
        step(kc + 2, wa2, wa1, p2, xv0, xv1);
        step(kc + 3, wa3, wa2, p3, xv1, xv0);
    };
    const uint4* wp = cur.base + 3 * cur.stride;
    const int64_t ws = cur.stride;
    if (nK > 4) {
        // The first round runs apart from the loop: its loads follow the
        // prologue's (whose W chunks may have been issued long before),
        // while every round of the loop follows a round.  So the loop's
        // waits count only a round's loads, and a step waits for its
        // token chunk without waiting for the W chunk issued a step ago.
        round4(0, wp, wp + ws, wp + 2 * ws, wp + 3 * ws);
        wp += 4 * ws;
        for (int kc = 4; kc < nK - 4; kc += 4) {
            round4(kc, wp, wp + ws, wp + 2 * ws, wp + 3 * ws);
            wp += 4 * ws;
        }
    }
    round4(nK - 4, wp, after, after + after_stride, after + 2 * after_stride);
    // wa0..wa2 now hold the first three chunks of what runs next

    // ------------------------------------------------------ epilogue
    // acc[nb][r] holds latent 32*wave + 8*(r/4) + 4*g + r%4 of token
    // 32*nb + j32 (the 32x32 MFMA output layout).  Every lane writes its
    // values to the tile's 128 token rows in LDS; then wave w selects for
    // rows 16w .. 16w + 15, eight lanes per row, two rows per lane.
    __syncthreads();  // every wave is done with the token chunks
    float* V = reinterpret_cast<float*>(lds_main);
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
        float* rowp = V + (32 * nb + j32) * kSelStride + 32 * wave + 4 * g;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            *reinterpret_cast<float4*>(rowp + 8 * j) =
                make_float4(acc[nb][4 * j], acc[nb][4 * j + 1], acc[nb][4 * j + 2],
                            acc[nb][4 * j + 3]);
    }
    __syncthreads();
    const SliceSink sink = sink_of();
    constexpr int LPS = 8 / WK;  // lanes per slice
    const int q = lane & 7;
    const int sl = mt * WK + q / LPS;
    const int r0 = 16 * wave + (lane >> 3), r1 = r0 + 8;
    const int64_t row0 = static_cast<int64_t>(n0 + r0) * sink.n_sl + sl;
    const int64_t row1 = static_cast<int64_t>(n0 + r1) * sink.n_sl + sl;
    const float* const vr[2] = {V + r0 * kSelStride + 32 * q, V + r1 * kSelStride + 32 * q};
    const bool ok[2] = {r0 < ntok, r1 < ntok};
    uint2* const dst[2] = {sink.cand + row0 * sink.cap, sink.cand + row1 * sink.cap};
    int32_t* const co[2] = {sink.tile_cnt + row0, sink.tile_cnt + row1};
    float* const to[2] = {sink.tile_tau + row0, sink.tile_tau + row1};
    select_slices<true, 2, 32, LPS>(vr, q % LPS, ok, sink.z, sink.lo_cnt, sink.cap,
                                    mt * kBM + 32 * q, dst, co, to);
    if (has_nxt) load_bias(cfv, nxt_bias_of(), nxt_mt);
    __syncthreads();  // the rows are read before what runs next
}

// ------------------------------------------------------------ narrow slices
// A dictionary of few 256-latent slices leaves CUs idle when every slice is
// one workgroup, so it is cut finer: a workgroup owns 256 / WK latents.  A K chunk
// of the slice (8 KB for 64 latents, contiguous in the packed layout) and of the
// token rows is shared through LDS, and the chunks after it are in flight in
// registers: the loads of a chunk go out together, so that the in-order wait for
// one leaves the others behind it.  Three LDS buffers: a wave reads the operands of
// the next chunk, step by step, as it multiplies this one's, so that a step is a
// barrier and its chain of MFMAs.  The tile's token rows are 32 * NB: 32, 64 or 128
// by the tokens left, since a batch of a few requests is the usual one here; a wave
// multiplies 32 latents by one or two groups of 32 tokens over the whole of K, and
// waves without such a block only copy.  Every value is summed in the order of K, as
// in the whole and the big tiles, so that a token's candidates do not depend on the
// path.
// Measured against one workgroup per 256 latents, per launch: 9 tokens of width
// 2304, m = 16384 (64 workgroups then, 256 now) 33.8 -> 15.4 us, with the merge 43.4
// -> 26.7, and 100 tokens 47.8 -> 35.4.  With the waves sharing K instead, each
// streaming dictionary chunks of its own, the 9 tokens took 15.4 as well and 100
// tokens 43.1 with the merge; with the operands read after the barrier 19.6 against
// 16.4 us (9 tokens of width 4096, m = 4096), and steps of four chunks were no faster.
template <int WK>
struct Narrow {
    static constexpr int kSW = kBM / WK;       // latents of a slice
    static constexpr int kWL = kSW / 32;       // latent groups of 32
    static constexpr int kStride = kSW + 4;    // floats per selection row
    static constexpr int kCP = kWL * 256;      // 16-byte pieces of a K chunk of the slice
    static constexpr int kCR = kCP / kEncThreads;  // ... per thread
    static constexpr int R = WK == 4 ? 12 : 6;     // K chunks in the ring
    static_assert(R * kCR <= kRing, "the ring holds them");
};

// K chunks c .. c + C - 1 of slice sl into their places of the ring: thread tid takes
// pieces tid + 512 p of a chunk (none past the last one; c is a multiple of C).
template <int WK, int C>
__device__ __forceinline__ void narrow_load(uint4* a, const uint16_t* W, int n_mt, int sl, int c,
                                            int nK) {
    using N = Narrow<WK>;
    const int64_t chunk = static_cast<int64_t>(n_mt) * 32768;  // bytes of one K chunk
    const char* base = reinterpret_cast<const char*>(W) + static_cast<int64_t>(sl / WK) * 32768 +
                       (sl % WK) * (N::kCP * 16) + chunk * min(c, nK - C);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(base), 0,
        c < nK ? static_cast<int>((C - 1) * chunk + N::kCP * 16) : 0, kBufferDword3);
#pragma unroll
    for (int p = 0; p < C * N::kCR; ++p)
        a[p] = buffer_load16<kNontemporal>(
            r, threadIdx.x * 16u,
            c < nK ? static_cast<uint32_t>(p / N::kCR) * static_cast<uint32_t>(chunk) +
                         (p % N::kCR) * (kEncThreads * 16u)
                   : 0u);
}
// The first chunks of slice sl.
template <int WK>
__device__ __forceinline__ void narrow_first(uint4 (&ring)[kRing], const uint16_t* W, int n_mt,
                                             int sl, int d) {
    using N = Narrow<WK>;
    constexpr int C = WK == 4 ? 4 : 2;  // (d / 64 is a multiple of 4)
#pragma unroll
    for (int c = 0; c < N::R; c += C)
        narrow_load<WK, C>(ring + c * N::kCR, W, n_mt, sl, c, d / kBK);
}

// One tile: slice sl over tokens [n0, n0 + 32 * NB) of the app's list.  On
// entry the ring holds the slice's first chunks (narrow_first); on exit
// those of slice `nxt` of dictionary Wn when nxt >= 0.
template <int WK, int NB>
__device__ __forceinline__ void narrow_tile(uint4* lds_main, const uint16_t* __restrict__ h,
                                            uint32_t h_bytes, int32_t d, const int32_t* tl,
                                            int cnt, int n0, int sl,
                                            const uint16_t* __restrict__ W, int n_mt,
                                            const SliceSink sink,
                                            const float* __restrict__ c_fold, int nxt,
                                            const uint16_t* Wn, int n_mtn,
                                            uint4 (&ring)[kRing]) {
    using N = Narrow<WK>;
    constexpr int kWL = N::kWL;
    constexpr int C = NB == 1 || (WK == 4 && NB == 2) ? 2 : 1;  // K chunks of a step
    constexpr int R = N::R / C;                        // steps of the slice in flight
    constexpr int D = WK == 4 && NB == 4 ? R / 2 : R;  // and of the token rows
    constexpr int kRows = 32 * NB;
    constexpr int kPlane = kRows * 8;  // pieces of one chunk of the token rows
    constexpr int kX = (C * kPlane + kEncThreads - 1) / kEncThreads;  // per thread and step
    constexpr int kW = C * N::kCR;
    constexpr int kTB = kWL * NB > kEncWaves ? kWL * NB / kEncWaves : 1;  // token groups per wave
    constexpr int kBuf = C * (N::kCP + kPlane);  // pieces of an LDS buffer
    static_assert(3 * kBuf <= kLdsMain && C * kPlane == kX * kEncThreads,
                  "three buffers fit the LDS, every thread has its pieces");
    int tid = threadIdx.x;  // opaque (see big_tile)
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6;
    const int wl = wave % kWL, tg = wave / kWL * kTB;  // its latent group and first token group
    const int g = lane >> 5, j32 = lane & 31;
    const int nW = d / (C * kBK);
    const int ntok = min(kRows, cnt - n0);
    // piece q of a step's rows: chunk q / kPlane, row (q % kPlane) / 8, 16-byte piece
    // q % 8 of it; thread tid holds q = tid + 512 p
    uint32_t xoff[kX];
#pragma unroll
    for (int p = 0; p < kX; ++p) {
        const int q = tid + kEncThreads * p, n = (q % kPlane) / 8;
        xoff[p] = n < ntok ? static_cast<uint32_t>(tl[n0 + n]) * static_cast<uint32_t>(d) * 2u +
                                 static_cast<uint32_t>(q / kPlane) * 128u + (q & 7) * 16u
                           : kOutOfRange;
    }
    f32x16_t acc[kTB];
    {
        const float* cf = c_fold + sl * N::kSW + 32 * wl + 4 * g;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float c = cf[8 * (r / 4) + (r % 4)];
#pragma unroll
            for (int b = 0; b < kTB; ++b) acc[b][r] = c;
        }
    }
    uint4 xv[D][kX];
    auto load_x = [&](uint4 (&x)[kX], int w) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(h), 0, w < nW ? static_cast<int>(h_bytes) : 0, kBufferDword3);
#pragma unroll
        for (int p = 0; p < kX; ++p)
            x[p] = buffer_load16<0>(r, xoff[p], w < nW ? static_cast<uint32_t>(w) * (C * 128u) : 0u);
    };
    // row n's piece c sits at n*8 + (c ^ ((n >> 1) & 7)) of its chunk's plane; 512 pieces
    // on are 64 rows on, or whole planes
    const int xdst = C * N::kCP + (tid & ~7) + ((tid & 7) ^ ((tid >> 4) & 7));
    auto store = [&](int slot, int slot_x, uint4* buf) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < kX; ++p) buf[xdst + kEncThreads * p] = xv[slot_x][p];
#pragma unroll
        for (int p = 0; p < kW; ++p) buf[tid + kEncThreads * p] = ring[slot * kW + p];
    };
    const int xsrc = C * N::kCP + (32 * tg + j32) * 8, sw = (j32 >> 1) & 7;
    const int wsrc = wl * 256 + lane;
    const bool busy = wave * kTB < kWL * NB;  // (uniform over the wave) it has a block
    uint4 A[4 * C], B[4 * C][kTB];  // a step's operands
    auto read = [&](int s, const uint4* buf) __attribute__((always_inline)) {
        A[s] = buf[(s / 4) * N::kCP + wsrc + (s % 4) * 64];
#pragma unroll
        for (int b = 0; b < kTB; ++b)
            B[s][b] = buf[(s / 4) * kPlane + xsrc + 256 * b + ((2 * (s % 4) + g) ^ sw)];
    };
    // Step w, in slot w % R of the ring: its place there was stored two steps ago and
    // takes step w + R.  Its operands are in registers; the next step's, stored a step
    // ago, are read as they are multiplied, and the one after it is stored to the
    // buffer that every wave has read a step ago.
    uint4 *b0 = lds_main, *b1 = lds_main + kBuf, *b2 = lds_main + 2 * kBuf;  // of w, w + 1, w + 2
    auto step = [&](int w, int slot) __attribute__((always_inline)) {
        load_x(xv[slot % D], w + D);
        narrow_load<WK, C>(ring + slot * kW, W, n_mt, sl, (w + R) * C, nW * C);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        if (busy) {
#pragma unroll
            for (int s = 0; s < 4 * C; ++s) {
#pragma unroll
                for (int b = 0; b < kTB; ++b)
                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        as_bf16x8(A[s]), as_bf16x8(B[s][b]), acc[b], 0, 0, 0);
                read(s, b1);
            }
        }
        store((slot + 2) % R, (slot + 2) % D, b2);
        __builtin_amdgcn_sched_barrier(0);
        uint4* t = b0;
        b0 = b1;
        b1 = b2;
        b2 = t;
    };
#pragma unroll
    for (int w = 0; w < D; ++w) load_x(xv[w], w);
    __builtin_amdgcn_sched_barrier(0);
    store(0, 0, b0);
    store(1, 1, b1);
    __syncthreads();
    if (busy)
#pragma unroll
        for (int s = 0; s < 4 * C; ++s) read(s, b0);
    static_assert(R % D == 0 && D > 2, "the slots of the rings");
    for (int w = 0; w < nW;) {  // any number of steps
#pragma unroll
        for (int r = 0; r < R; ++r) {
            step(w, r);
            if (++w == nW) break;
        }
    }
    if (nxt >= 0) narrow_first<WK>(ring, Wn, n_mtn, nxt, d);  // under the selection
    __syncthreads();  // every wave is done with the windows
    float* V = reinterpret_cast<float*>(lds_main);
    if (busy) {
#pragma unroll
        for (int b = 0; b < kTB; ++b) {
            float* rowp = V + (32 * (tg + b) + j32) * N::kStride + 32 * wl + 4 * g;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                *reinterpret_cast<float4*>(rowp + 8 * j) = make_float4(
                    acc[b][4 * j], acc[b][4 * j + 1], acc[b][4 * j + 2], acc[b][4 * j + 3]);
        }
    }
    __syncthreads();
    // NT rows per lane group: 16 rows a wave in the widest tile, 8 below (every
    // wave then has rows, or only the first ones)
    constexpr int NT = NB == 4 ? 2 : 1;
    if (8 * NT * wave < ntok) {  // uniform over the wave
        constexpr int VPL = N::kSW / 8;
        const int q = lane & 7;
        const float* vr[NT];
        bool ok[NT];
        uint2* dst[NT];
        int32_t* co[NT];
        float* to[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int r = 8 * NT * wave + (lane >> 3) + 8 * t;
            const int64_t row = static_cast<int64_t>(n0 + r) * sink.n_sl + sl;
            ok[t] = r < ntok;
            vr[t] = V + (ok[t] ? r : 0) * N::kStride + VPL * q;
            dst[t] = sink.cand + row * sink.cap;
            co[t] = sink.tile_cnt + row;
            to[t] = sink.tile_tau + row;
        }
        select_slices<true, NT, VPL, 8>(vr, q, ok, sink.z, sink.lo_cnt, sink.cap,
                                        sl * N::kSW + VPL * q, dst, co, to);
    }
    __syncthreads();  // the rows are read before the next tile's tokens land
}

// The tile by the tokens left of the list from n0 on.
template <int WK>
__device__ __forceinline__ void narrow_any(uint4* lds_main, const uint16_t* __restrict__ h,
                                           uint32_t h_bytes, int32_t d, const int32_t* tl,
                                           int cnt, int n0, int sl,
                                           const uint16_t* __restrict__ W, int n_mt,
                                           const SliceSink sink, const float* __restrict__ c_fold,
                                           int nxt, const uint16_t* Wn, int n_mtn, uint4 (&ring)[kRing]) {
    const int left = cnt - n0;
    if (left <= 32)
        narrow_tile<WK, 1>(lds_main, h, h_bytes, d, tl, cnt, n0, sl, W, n_mt, sink, c_fold, nxt,
                           Wn, n_mtn, ring);
    else if (left <= 64)
        narrow_tile<WK, 2>(lds_main, h, h_bytes, d, tl, cnt, n0, sl, W, n_mt, sink, c_fold, nxt,
                           Wn, n_mtn, ring);
    else
        narrow_tile<WK, 4>(lds_main, h, h_bytes, d, tl, cnt, n0, sl, W, n_mt, sink, c_fold, nxt,
                           Wn, n_mtn, ring);
}

// ------------------------------------------------------------- big token tiles
// From 129 live tokens a 128-token tile streams the dictionary more than once
// (or, with few slices, leaves the reuse to chance), and from about 200 the
// matrix cores bound it, not HBM.  Here a workgroup multiplies 256 latents by
// 256 tokens, each of its eight waves 64 x 128 (128 accumulator registers).
// The token rows of two K stages of 32 are shared through LDS (double buffered,
// one barrier a pair, staged in registers, a row's whole 128-byte line at a time);
// the dictionary goes straight into the registers of the two waves that share a
// latent quarter: both operands through LDS are 128 KB of traffic a stage, as long
// as the stage's MFMAs.  The second half of a stage is multiplied after the next
// one's first reads are issued, so that a barrier does not empty the matrix cores.
// Measured per layer with the merge, 391 tokens, m = 32768, d = 4096: 137 us with a
// barrier a stage and nothing carried, 131 so; 256 tokens, m = 65536, d = 8192: 300
// and 279; 900 tokens, m = 16384, d = 2304: 87 and 83.  Before that, per launch: 258
// us as four 128-token tiles in turn, 156 with both operands through LDS.
constexpr int kBigTok = 256;
constexpr int kBigPieces = 1024;  // 16-byte pieces of a stage's token rows; four stages
static_assert(4 * kBigPieces <= kLdsMain, "the stages fit the LDS");

// Stage swizzle: the 16-byte piece c of token n sits at n*4 + (c ^ gsw(n));
// with it the MFMA-layout reads of 16 tokens x 4 pieces hit distinct banks.
__device__ __forceinline__ int gsw(int n) { return ((n >> 3) ^ (n >> 4)) & 3; }

// A value that is the same in every lane, in a scalar register.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The tiles that an app's live tokens are encoded in.  All of them add in the order
// of K, so the choice shows in no result.  It is made by the rounds of units
// (slice, tokens) over 256 CUs, as counted over the apps of the launch:
//  - narrow tiles while they are one round.  One of a slice cut in four takes 0.66 of
//    a whole tile (200 tokens, width 4096, m = 8192: 53 us an encode against 70), but
//    a second round more than one of whole tiles (m = 16384: 90 and 77);
//  - big tiles for more than 128 tokens where whole ones take 5/3 of their rounds or
//    more.  Two rounds of whole tiles are about one of big ones, or up to a quarter
//    more (width 4096: 512 tokens, m = 32768: 153 and 140; m = 65536: 288 and 267; 140
//    tokens: 182 and 147), three rounds less than two (384 tokens, m = 65536: 233 and
//    250), and one round 0.7 of one (500 tokens, m = 8192: 74 and 104);
//  - whole tiles else.
constexpr int kRoundCUs = 256;
enum TileKind { kNarrowTiles, kWholeTiles, kBigTiles };
struct TileUnits {
    int narrow = 0, whole = 0, big = 0;  // of the launch, were all of its tiles such
    __device__ __forceinline__ void add(int cnt, int n_mt, int n_sl) {
        const int t128 = (cnt + kBN - 1) / kBN;
        narrow += n_sl * t128;
        whole += n_mt * t128;
        big += n_mt * ((cnt + kBigTok - 1) / kBigTok);
    }
};
__device__ __forceinline__ int rounds(int units) { return (units + kRoundCUs - 1) / kRoundCUs; }
template <int WK>
__device__ __forceinline__ TileKind tile_kind(int cnt, const TileUnits& u, int d, int T_max) {
    if (WK > 1 && u.narrow <= kRoundCUs) return kNarrowTiles;
    // (the big tiles' buffer offsets are 32 bits)
    if (WK < 4 && cnt > kBN && 3 * rounds(u.whole) >= 5 * rounds(u.big) &&
        static_cast<int64_t>(T_max) * d * 2 <= 0x7FFFFFFF)
        return kBigTiles;
    return kWholeTiles;
}
// Its number of units (slice, tokens), of n slices and n_nt token tiles, and the
// unit u: the token tiles of eight slices together, a slice to each XCD, the
// slices fastest, so that the workgroups that run the tiles of one slice side by
// side draw it through the same L2.
__device__ __forceinline__ void unit_tile(int u, int n, int n_nt, int* slice, int* nt) {
    *slice = u;
    *nt = 0;
    if (n_nt == 1) return;  // uniform
    const int grp = u / (8 * n_nt), r = u - grp * 8 * n_nt, w = min(8, n - 8 * grp);
    *nt = r / w;
    *slice = 8 * grp + r - *nt * w;
}

template <int WK>
__device__ __forceinline__ void big_tile(uint4* lds_main, const uint16_t* __restrict__ h,
                                         uint32_t h_bytes, int32_t d, const int32_t* tl, int cnt,
                                         int nt, int mt, const uint16_t* __restrict__ W, int n_mt,
                                         const SliceSink sink, const float* __restrict__ c_fold) {
    // opaque, so that nothing computed from it here is merged with the other
    // paths' address arithmetic and held in registers across both
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 3, wn = wave >> 2;  // 64 latents, 128 tokens
    const int g = lane >> 5, j32 = lane & 31;
    const int n0 = nt * kBigTok;
    const int ntok = min(kBigTok, cnt - n0);
    const int nS = d / 32;  // a multiple of 8
    uint4* xsb = lds_main;
    // a stage of 32 is half a K chunk: steps 2 hh, 2 hh + 1 of its four; this
    // wave's A operands of step s, latent group a: piece (2 wm + a) * 256 +
    // (2 hh + s) * 64 + lane of the slice's chunk
    const char* Wb = reinterpret_cast<const char*>(W) + static_cast<int64_t>(mt) * 32768;
    const int64_t chunk = static_cast<int64_t>(n_mt) * 32768;
    const uint32_t woff = static_cast<uint32_t>(2 * wm * 256 + lane) * 16u;
    // the token rows of a pair of stages, 128 bytes of each: this thread takes piece
    // xc of rows xn, xn + 64, xn + 128, xn + 192 (their swizzles are the same).  The
    // second stage of a pair keeps row n at n ^ 2, so that the eight lanes of a row
    // write to eight bank groups.
    uint32_t xoff[4];
    const int xn = tid >> 3, xc = tid & 7;
    const int xdst = (xc >> 2) * kBigPieces + (xn ^ ((xc >> 2) << 1)) * 4 + ((xc & 3) ^ gsw(xn));
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int n = xn + 64 * p;
        xoff[p] = n < ntok ? static_cast<uint32_t>(tl[n0 + n]) * static_cast<uint32_t>(d) * 2u +
                                 xc * 16u
                           : kOutOfRange;
    }
    // half of a stage's dictionary operands: those of step s
    auto load_w = [&](uint4 (&w)[4], int j, int s) __attribute__((always_inline)) {
        const int jc = min(j, nS - 1);
        const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char*>(Wb + (jc >> 1) * chunk + (jc & 1) * 2048), 0,
            j < nS ? 32768 - 2048 : 0, kBufferDword3);
#pragma unroll
        for (int a = 0; a < 2; ++a)
            w[2 * s + a] = buffer_load16<0>(wr, woff + a * 4096u + s * 1024u, 0);
    };
    auto load_x = [&](uint4 (&x)[4], int k) __attribute__((always_inline)) {
        const bool in = 2 * k < nS;
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(h), 0, in ? static_cast<int>(h_bytes) : 0, kBufferDword3);
#pragma unroll
        for (int p = 0; p < 4; ++p)
            x[p] = buffer_load16<0>(xr, xoff[p], in ? static_cast<uint32_t>(k) * 128u : 0u);
    };
    auto store_x = [&](const uint4 (&x)[4], int k) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < 4; ++p) xsb[(k & 1) * 2 * kBigPieces + xdst + 256 * p] = x[p];
    };
    f32x16_t acc[2][4];
    {
        const float* cf = c_fold + mt * kBM + 64 * wm + 4 * g;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 c4 = *reinterpret_cast<const float4*>(cf + 32 * a + 8 * q);
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) {
                    acc[a][nb][4 * q + 0] = c4.x;
                    acc[a][nb][4 * q + 1] = c4.y;
                    acc[a][nb][4 * q + 2] = c4.z;
                    acc[a][nb][4 * q + 3] = c4.w;
                }
            }
    }
    auto read_b = [&](uint4 (&B)[4], int j, int s) __attribute__((always_inline)) {
        const uint4* xb = xsb + (j & 3) * kBigPieces;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            const int n = 128 * wn + 32 * nb + j32;
            B[nb] = xb[(n ^ ((j & 1) << 1)) * 4 + ((2 * s + g) ^ gsw(n))];
        }
    };
    auto multiply = [&](const uint4 (&w)[4], int s, const uint4 (&B)[4])
        __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
                acc[a][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    as_bf16x8(w[2 * s + a]), as_bf16x8(B[nb]), acc[a][nb], 0, 0, 0);
    };
    // Stage j, two of them per barrier: its step 0 is read while the step carried
    // over from stage j - 1 is multiplied, its step 1 is read while step 0 is, and
    // carried on, so that the matrix unit has work while the waves meet.  Between a
    // pair's stages the token rows of the next pair move into buffers that every
    // wave left before this pair's barrier, and those of the pair after it are
    // fetched; the dictionary is fetched two stages ahead into the registers just
    // used (wp: stage j - 1's).
    uint4 F[4], P[4], x[4];
    auto stage = [&](int j, uint4 (&w)[4], uint4 (&wp)[4], bool first)
        __attribute__((always_inline)) {
        if ((j & 1) == 0) __syncthreads();
        read_b(F, j, 0);
        if (!first) multiply(wp, 1, P);
        __builtin_amdgcn_sched_barrier(0);
        load_w(wp, j + 1, 1);
        read_b(P, j, 1);
        multiply(w, 0, F);
        __builtin_amdgcn_sched_barrier(0);
        load_w(w, j + 2, 0);
        if ((j & 1) == 0) {
            store_x(x, j / 2 + 1);
            load_x(x, j / 2 + 2);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    uint4 w0[4], w1[4];
    load_x(x, 0);
    load_w(w0, 0, 0);
    load_w(w0, 0, 1);
    load_w(w1, 1, 0);
    store_x(x, 0);
    load_x(x, 1);
    stage(0, w0, w1, true);
    stage(1, w1, w0, false);
    stage(2, w0, w1, false);
    stage(3, w1, w0, false);
    for (int j = 4; j < nS; j += 4) {  // a multiple of eight stages
        stage(j, w0, w1, false);
        stage(j + 1, w1, w0, false);
        stage(j + 2, w0, w1, false);
        stage(j + 3, w1, w0, false);
    }
    multiply(w1, 1, P);

    // acc[a][nb][r] holds latent 64*wm + 32*a + 8*(r/4) + 4*g + r%4 of token
    // 128*wn + 32*nb + j32; the tile's tokens are selected 128 at a time
    float* V = reinterpret_cast<float*>(lds_main);
    for (int half = 0; half < 2; ++half) {
        if (128 * half >= ntok) break;  // uniform
        __syncthreads();  // the stages, or the first half's rows, are read
        if (wn == half) {
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    float* rowp = V + (32 * nb + j32) * kSelStride + 64 * wm + 32 * a + 4 * g;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        *reinterpret_cast<float4*>(rowp + 8 * j) =
                            make_float4(acc[a][nb][4 * j], acc[a][nb][4 * j + 1],
                                        acc[a][nb][4 * j + 2], acc[a][nb][4 * j + 3]);
                }
        }
        __syncthreads();
        if (128 * half + 16 * wave < ntok) {  // uniform over the wave
            constexpr int LPS = 8 / WK;
            const int q8 = lane & 7;
            const int sl = mt * WK + q8 / LPS;
            // one token per lane group at a time: the second half's
            // accumulators are still held
#pragma unroll 1
            for (int r = 16 * wave + (lane >> 3), i = 0; i < 2; r += 8, ++i) {
                const int64_t row = static_cast<int64_t>(n0 + 128 * half + r) * sink.n_sl + sl;
                const float* const vr[1] = {V + r * kSelStride + 32 * q8};
                const bool ok[1] = {128 * half + r < ntok};
                uint2* const dst[1] = {sink.cand + row * sink.cap};
                int32_t* const co[1] = {sink.tile_cnt + row};
                float* const to[1] = {sink.tile_tau + row};
                select_slices<true, 1, 32, LPS>(vr, q8 % LPS, ok, sink.z, sink.lo_cnt,
                                                sink.cap, mt * kBM + 32 * q8, dst, co, to);
            }
        }
    }
    __syncthreads();  // the rows are read before what runs next
}

// Candidates of one app.  WK: the cut of its slices (1: whole ones of 256
// latents); MANY: the batch has more than 128 token slots, so that an app may have
// several token tiles, and big ones.  The app's units (slice, tokens) are dealt to
// the workgroups; the dictionary stream runs on from one unit into the next.
//
// With r_req given, the kernel also builds the step's routing (in place
// of a route-build launch): every workgroup builds its app's token list
// in LDS from the routing inputs staged there (in the space of the K
// loop's token chunks); workgroup a < n_apps publishes app a's list and
// count, and workgroup 0 the token masks and the error word.  A
// workgroup with a slice starts its first dictionary chunks as soon as the
// staged table shows a request subscribed to the app, so that the stream
// runs while the list is built (without a subscriber it reads nothing).
template <int WK, bool MANY>
__global__ void __launch_bounds__(kEncThreads, 1)
sae_stream_kernel(const uint16_t* __restrict__ h, int32_t d,
                  const int32_t* __restrict__ app_count, const int32_t* __restrict__ tok_list,
                  const uint16_t* __restrict__ W, const float* __restrict__ c_fold,
                  int32_t n_mt, int32_t T_max, float z_guess, int32_t lo_cnt, int32_t cap,
                  uint2* __restrict__ cand, int32_t* __restrict__ tile_cnt,
                  float* __restrict__ tile_tau, const int32_t* __restrict__ r_req,
                  const int32_t* __restrict__ r_tvalid, const uint32_t* __restrict__ r_sub,
                  int32_t r_Rmax, int32_t r_napps, int32_t r_bit,
                  uint32_t* __restrict__ r_mask, int32_t* __restrict__ r_count,
                  int32_t* __restrict__ r_lists, uint32_t* __restrict__ r_err) {
    __shared__ uint4 lds_main[kLdsMain];
    __shared__ int32_t list_s[kRouteMaxT];    // the app's token list (in-kernel route build)
    __shared__ int32_t rtot_s[kEncWaves];
    __shared__ int32_t seen_s[kEncWaves];
    const int own = blockIdx.x, G = gridDim.x;
    const int n_sl = n_mt * WK;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint4 ring[kRing];
    float cfv[16];

    const int32_t* tl = tok_list;
    int cnt = 0;
    int started = -1;  // the slice whose first chunks are in flight
    if (r_req) {  // uniform
        static_assert(sizeof(lds_main) >= (kRouteMaxT + kStageSubMax) * 4, "staging fits");
        int32_t* req_s = reinterpret_cast<int32_t*>(lds_main);
        uint32_t* sub_s = reinterpret_cast<uint32_t*>(lds_main) + kRouteMaxT;
        const bool seen = stage_route<kEncThreads>(r_req, T_max, r_sub, r_Rmax, req_s, sub_s,
                                                   1u << r_bit);
        const uint64_t seen_b = wave_ballot(seen);
        if (lane == 0) seen_s[wave] = seen_b != 0;
        uint32_t err = 0;
        const int32_t tv = clamp_t_valid(*r_tvalid, T_max, err);
        const uint32_t keep = r_napps >= 32 ? 0xFFFFFFFFu : ((1u << r_napps) - 1u);
        uint32_t* masks = own == 0 ? r_mask : nullptr;
        __syncthreads();  // the staged inputs
        bool any = false;
#pragma unroll
        for (int w = 0; w < kEncWaves; ++w) any = any || seen_s[w] != 0;
        // no request subscribes to the app: no token is listed, and a
        // workgroup with nothing to publish is done
        if (!any && own >= r_napps) return;  // uniform
        // Slice `own`, the first unit of a single token tile.  With more tiles
        // another slice may come first, or a big tile, and the chunks are read for
        // nothing: not where they are a good part of a row (K chunks 0-2 of d / 64),
        // nor of a cut slice.
        if (own < n_sl && any && (!MANY || (WK == 1 && d >= 1024))) {  // uniform
            if constexpr (WK == 1) slice_first(ring, cfv, slice_src(W, n_mt, own), c_fold, own);
            else narrow_first<WK>(ring, W, n_mt, own, d);
            started = own;
        }
        if (own < r_napps && own != r_bit) {
            const int32_t n = build_token_list<kEncThreads>(req_s, tv, sub_s, r_sub, r_Rmax, keep,
                                                            own, T_max, list_s, rtot_s, masks,
                                                            err);
            masks = nullptr;
            publish_token_list<kEncThreads>(list_s, n, T_max,
                                            r_lists + static_cast<int64_t>(own) * T_max,
                                            r_count + own);
            __syncthreads();  // list_s is rebuilt below
        }
        cnt = build_token_list<kEncThreads>(req_s, tv, sub_s, r_sub, r_Rmax, keep, r_bit, T_max,
                                            list_s, rtot_s, masks, err);
        if (own == r_bit)
            publish_token_list<kEncThreads>(list_s, cnt, T_max,
                                            r_lists + static_cast<int64_t>(r_bit) * T_max,
                                            r_count + r_bit);
        if (own == 0) publish_error(err, r_err);
        tl = list_s;
    } else {
        cnt = *app_count;
    }
    if (cnt <= 0) return;
    const SliceSink sink{cand, tile_cnt, tile_tau, n_sl, lo_cnt, cap, z_guess};
    const uint32_t h_bytes = static_cast<uint32_t>(T_max) * static_cast<uint32_t>(d) * 2u;
    TileUnits tu;
    tu.add(cnt, n_mt, n_sl);
    const TileKind kind = MANY ? tile_kind<WK>(cnt, tu, d, T_max)
                               : WK == 1 ? kWholeTiles : kNarrowTiles;
    const int tok = kind == kBigTiles ? kBigTok : kBN, n_nt = (cnt + tok - 1) / tok;
    const int n = kind == kNarrowTiles ? n_sl : n_mt, units = n * n_nt;
    int u = own, sl, nt;
    if (u >= units) return;
    unit_tile(u, n, n_nt, &sl, &nt);
    if constexpr (MANY && WK < 4) {
        if (kind == kBigTiles) {  // uniform
            for (; u < units; u += G) {
                unit_tile(u, n, n_nt, &sl, &nt);
                big_tile<WK>(lds_main, h, h_bytes, d, tl, cnt, nt, sl, W, n_mt, sink, c_fold);
            }
            return;
        }
    }
    if constexpr (WK > 1) {
        if (!MANY || kind == kNarrowTiles) {  // uniform
            if (started != sl) narrow_first<WK>(ring, W, n_mt, sl, d);
            for (;;) {
                int sn = -1, ntn = 0;
                if ((u += G) < units) unit_tile(u, n, n_nt, &sn, &ntn);
                narrow_any<WK>(lds_main, h, h_bytes, d, tl, cnt, nt * kBN, sl, W, n_mt, sink, c_fold,
                               sn, W, n_mt, ring);
                if (sn < 0) return;
                sl = sn;
                nt = ntn;
            }
        }
    }
    if constexpr (WK == 1 || MANY) {
        SliceSrc src = slice_src(W, n_mt, sl);
        if (WK > 1 || started != sl) slice_first(ring, cfv, src, c_fold, sl);
        const auto sink_of = [&]() __attribute__((always_inline)) { return sink; };
        const auto bias_of = [&]() __attribute__((always_inline)) { return c_fold; };
        for (u += G; u < units; u += G) {
            int sn, ntn;
            unit_tile(u, n, n_nt, &sn, &ntn);
            const SliceSrc nsrc = slice_src(W, n_mt, sn);
            slice_tile<WK>(lds_main, h, d, tl, nt * kBN, min(kBN, cnt - nt * kBN), sl, src, sink_of,
                           nsrc, true, sn, bias_of, ring, cfv);
            src = nsrc;
            sl = sn;
            nt = ntn;
        }
        slice_tile<WK>(lds_main, h, d, tl, nt * kBN, min(kBN, cnt - nt * kBN), sl, src, sink_of, src,
                       false, sl, bias_of, ring, cfv);
    }
}

// Several SAE apps of one hook in one launch, on a persistent grid: the apps'
// units (slice, tokens) are laid end to end, none of an app without a token, and
// workgroup w runs units w, w + G, w + 2G, ... (G the grid, at most one workgroup
// per CU).  The routing inputs are staged once per workgroup, in LDS of their own;
// the dictionary stream runs on from one unit into the next, so the next slice's
// first chunks load while this one's candidates are selected.
struct EncApp {
    const int32_t* app_count;
    const int32_t* tok_list;
    const uint16_t* W;
    const float* c_fold;
    uint2* cand;
    int32_t* tile_cnt;
    float* tile_tau;
    int32_t n_mt, lo_cnt, cap, bit;
    float z;
};
struct EncApps {
    EncApp a[kMultiMax];
    int32_t n;
};

// WK, MANY: as in sae_stream_kernel, the same for every app.
template <int WK, bool MANY>
__global__ void __launch_bounds__(kEncThreads, 1)
sae_stream_apps_kernel(const uint16_t* __restrict__ h, int32_t d, EncApps apps,
                       const int32_t* __restrict__ r_req, const int32_t* __restrict__ r_tvalid,
                       const uint32_t* __restrict__ r_sub, int32_t r_Rmax, int32_t T_max,
                       int32_t r_napps, uint32_t* __restrict__ r_mask,
                       int32_t* __restrict__ r_count, int32_t* __restrict__ r_lists,
                       uint32_t* __restrict__ r_err) {
    __shared__ uint4 lds_main[kLdsMain];
    __shared__ int32_t list_s[kRouteMaxT];
    __shared__ int32_t rtot_s[kEncWaves];
    __shared__ int32_t stage_s[kRouteMaxT + kStageSubMax];
    __shared__ int32_t cnt_s[kMultiMax];
    __shared__ int32_t kind_s[kMultiMax], n_s[kMultiMax], nt_s[kMultiMax];
    const int tid = threadIdx.x, lane = tid & 63;
    const int own = blockIdx.x, G = gridDim.x;

    int32_t* req_s = stage_s;
    uint32_t* sub_s = reinterpret_cast<uint32_t*>(stage_s + kRouteMaxT);
    int32_t tv = 0;
    uint32_t keep = 0;
    if (r_req) {  // uniform
        if (tid < kMultiMax) cnt_s[tid] = 0;
        stage_route<kEncThreads>(r_req, T_max, r_sub, r_Rmax, req_s, sub_s);
        uint32_t err = 0;
        tv = clamp_t_valid(*r_tvalid, T_max, err);
        keep = r_napps >= 32 ? 0xFFFFFFFFu : ((1u << r_napps) - 1u);
        __syncthreads();  // the staged inputs
        // every app's count
        for (int32_t t0 = 0; t0 < T_max; t0 += kEncThreads) {
            const int32_t t = t0 + tid;
            const uint32_t m =
                t < T_max ? slot_mask_staged(req_s, t, tv, sub_s, r_sub, r_Rmax, keep, err) : 0u;
            for (int i = 0; i < apps.n; ++i) {
                const int c = __popcll(wave_ballot((m >> apps.a[i].bit) & 1u));
                if (lane == 0 && c > 0) atomicAdd(&cnt_s[i], c);
            }
        }
        if (own < r_napps) {
            const int32_t n = build_token_list<kEncThreads>(
                req_s, tv, sub_s, r_sub, r_Rmax, keep, own, T_max, list_s, rtot_s,
                own == 0 ? r_mask : nullptr, err);
            publish_token_list<kEncThreads>(list_s, n, T_max,
                                            r_lists + static_cast<int64_t>(own) * T_max,
                                            r_count + own);
        }
        if (own == 0) publish_error(err, r_err);
    } else if (tid < apps.n) {
        cnt_s[tid] = *apps.a[tid].app_count;
    }
    __syncthreads();  // the counts; list_s free
    // each app's kind of tiles, its slices and token tiles (0 without a token)
    if (tid < apps.n) {
        const int c = cnt_s[tid], n_mt = apps.a[tid].n_mt;
        TileUnits tu;
        for (int i = 0; MANY && i < apps.n; ++i)
            tu.add(max(cnt_s[i], 0), apps.a[i].n_mt, apps.a[i].n_mt * WK);
        const TileKind kind = MANY ? tile_kind<WK>(c, tu, d, T_max)
                                   : WK == 1 ? kWholeTiles : kNarrowTiles;
        const int tok = kind == kBigTiles ? kBigTok : kBN;
        kind_s[tid] = kind;
        n_s[tid] = n_mt * (kind == kNarrowTiles ? WK : 1);
        nt_s[tid] = c > 0 ? (c + tok - 1) / tok : 0;
    }
    __syncthreads();
    // The units, laid end to end: narrow tiles of every app, whole ones, big ones,
    // each kind in a loop of its own (together they would not fit the registers).
    // seek moves (i, base), an app and its first unit, to the app of kind `kind`
    // with unit u; false past the last one, with base past them.
    auto seek = [&](int kind, int u, int& i, int& base) {
        for (; i < apps.n; ++i) {
            if (uniform(kind_s[i]) != kind) continue;
            const int n = uniform(n_s[i]) * uniform(nt_s[i]);
            if (u < base + n) return true;
            base += n;
        }
        return false;
    };
    auto place = [&](int u, int i, int base, int* sl, int* nt) {
        *sl = u - base;
        *nt = 0;
        if (MANY) unit_tile(u - base, uniform(n_s[i]), uniform(nt_s[i]), sl, nt);
    };
    int list_app = -1, cnt = 0;
    const int32_t* tl = nullptr;
    auto list_of = [&](int i) {
        if (i == list_app) return;  // uniform
        if (r_req) {
            uint32_t e = 0;
            cnt = build_token_list<kEncThreads>(req_s, tv, sub_s, r_sub, r_Rmax, keep,
                                                apps.a[i].bit, T_max, list_s, rtot_s, nullptr, e);
            tl = list_s;
        } else {
            cnt = uniform(cnt_s[i]);
            tl = apps.a[i].tok_list;
        }
        list_app = i;
    };
    // the descriptors are read again where they are used (an opaque index
    // keeps their fields out of registers until then)
    auto sink_of = [&](int i) __attribute__((always_inline)) {
        asm volatile("" : "+s"(i));
        const EncApp& b = apps.a[i];
        return SliceSink{b.cand, b.tile_cnt, b.tile_tau, b.n_mt * WK, b.lo_cnt, b.cap, b.z};
    };
    const uint32_t h_bytes = static_cast<uint32_t>(T_max) * static_cast<uint32_t>(d) * 2u;
    int u = own, base = 0;
    if constexpr (WK > 1) {
        int i = 0, sl = 0, nt = 0;
        bool more = seek(kNarrowTiles, u, i, base);
        uint4 ring[kRing];
        if (more) {
            place(u, i, base, &sl, &nt);
            narrow_first<WK>(ring, apps.a[i].W, apps.a[i].n_mt, sl, d);
        }
        while (more) {
            list_of(i);
            const EncApp& a = apps.a[i];
            int in = i, sn = -1, ntn = 0;
            u += G;
            more = seek(kNarrowTiles, u, in, base);
            if (more) place(u, in, base, &sn, &ntn);
            const EncApp& b = apps.a[more ? in : i];
            narrow_any<WK>(lds_main, h, h_bytes, d, tl, cnt, nt * kBN, sl, a.W, a.n_mt, sink_of(i),
                           a.c_fold, sn, b.W, b.n_mt, ring);
            i = in;
            sl = sn;
            nt = ntn;
        }
    }
    if constexpr (WK == 1 || MANY) {
        int i = 0, sl = 0, nt = 0;
        bool more = seek(kWholeTiles, u, i, base);
        uint4 ring[kRing];
        float cfv[16];
        SliceSrc src{};
        if (more) {
            place(u, i, base, &sl, &nt);
            // in flight while the list is built
            src = slice_src(apps.a[i].W, apps.a[i].n_mt, sl);
            slice_first(ring, cfv, src, apps.a[i].c_fold, sl);
        }
        while (more) {
            list_of(i);
            int in = i, sn = sl, ntn = 0;
            u += G;
            more = seek(kWholeTiles, u, in, base);
            auto bias_of = [&]() __attribute__((always_inline)) {
                int k = in;
                asm volatile("" : "+s"(k));
                return apps.a[k].c_fold;
            };
            auto sink_i = [&]() __attribute__((always_inline)) { return sink_of(i); };
            if (more) place(u, in, base, &sn, &ntn);
            const SliceSrc nsrc = more ? slice_src(apps.a[in].W, apps.a[in].n_mt, sn) : src;
            slice_tile<WK>(lds_main, h, d, tl, nt * kBN, min(kBN, cnt - nt * kBN), sl, src, sink_i,
                           nsrc, more, sn, bias_of, ring, cfv);
            src = nsrc;
            i = in;
            sl = sn;
            nt = ntn;
        }
    }
    if constexpr (MANY && WK < 4) {
        for (int i = 0; seek(kBigTiles, u, i, base); u += G) {
            int sl, nt;
            place(u, i, base, &sl, &nt);
            list_of(i);
            const EncApp& a = apps.a[i];
            big_tile<WK>(lds_main, h, h_bytes, d, tl, cnt, nt, sl, a.W, a.n_mt, sink_of(i), a.c_fold);
        }
    }
}

// ------------------------------------------ prefill GEMM + candidate emission
// Many subscribed tokens make the encode MFMA-bound.  The token rows are
// first gathered into a staged layout (sae_xstage_kernel): plane j holds
// elements [32j, 32j+32) of every listed token, 64 contiguous bytes per
// token, zero past the subscribed count.  sae_gemm_kernel then runs 4 waves
// (one per SIMD) on a 256-latent x 256-token tile, each wave a 128 x 128
// quarter held in 256 accumulator registers.  Both operands of each K
// stage of 32 (a 16 KB dictionary half chunk, 2 KB contiguous per 32
// latents, and a 16 KB token plane slice) are copied by the load unit
// straight into LDS (global_load_lds, no register staging) into a ring of
// 4 stages.  Per pair of stages a wave waits for its own copies of the
// pair, meets the others at a barrier, refills the pair of buffers freed by
// the previous step, and runs 64 MFMAs whose operands come from LDS; the
// operands of the last step are read before the next barrier and
// multiplied after it, so the matrix unit has work while the waves meet.  The epilogue is the same threshold emission as the decode kernel,
// per token over the tile's 256 latents.
constexpr int kGemmThreads = 256;
constexpr int kGemmTok = 256;       // tokens per tile
constexpr int kStagePieces = 1024;  // 16-byte pieces per operand per stage
constexpr int kPrefillMinT = 1025;  // token slots from which the prefill GEMM runs
constexpr int kGBlkTok = 8;         // XCD block: token tiles
constexpr int kGBlkLat = 4;         // XCD block: latent tiles
constexpr int kSmallTiles = 512;    // most 128-token tiles of a launch

// s_waitcnt: at most n vector-memory operations of this wave outstanding
// and no LDS operation.
#define XMIX_WAIT_VM_LGKM0(n) \
    __builtin_amdgcn_s_waitcnt(((n) & 15) | (7 << 4) | (((n) >> 4) << 14))

__global__ void __launch_bounds__(256)
sae_xstage_kernel(const uint16_t* __restrict__ h, int32_t d, const int32_t* __restrict__ app_count,
                  const int32_t* __restrict__ tok_list, int32_t n_pad, uint16_t* __restrict__ xs) {
    // one 16-byte piece per thread, output order (plane, token, piece)
    const int64_t q = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t total = static_cast<int64_t>(n_pad) * (d / 8);
    if (q >= total) return;
    const int32_t c = static_cast<int32_t>(q & 3);
    const int64_t jn = q >> 2;
    const int32_t n = static_cast<int32_t>(jn % n_pad);
    const int32_t j = static_cast<int32_t>(jn / n_pad);
    const int32_t cnt = *app_count;
    if (n >= (cnt + kGemmTok - 1) / kGemmTok * kGemmTok) return;  // no tile reads it
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (n < cnt)
        v = *reinterpret_cast<const uint4*>(h + static_cast<int64_t>(tok_list[n]) * d + 32 * j + 8 * c);
    reinterpret_cast<uint4*>(xs)[q] = v;
}

// The live count decides the tile: 64 * NB tokens.  256-token tiles feed the
// matrix cores best, but few of them leave CUs idle; a 128-token tile has half the
// MFMAs and the same dictionary copies, so it is taken where its rounds of 256 CUs,
// priced at 0.68 of a round of the large ones, are the cheaper ones (up to 512 of
// them, which the launch has the workgroups for).  A prefill encode of 1318 tokens,
// 4608 latents: 46.9 -> 37.8 us at d = 768, 103 -> 82 at d = 4096; 250 tokens, 16384
// latents, d = 2048: 65 -> 48; three small rounds for two large ones are
// the slower (921 tokens, 18944 latents, d = 1792: 121 and 110 us).
__global__ void __launch_bounds__(kGemmThreads, 1)
sae_gemm_kernel(const uint16_t* __restrict__ xs_g, int32_t d, int32_t n_pad,
                const int32_t* __restrict__ app_count, const uint16_t* __restrict__ W,
                const float* __restrict__ c_fold, int32_t n_mt, int32_t n_nt, float z_guess,
                int32_t lo_cnt, int32_t cap, uint2* __restrict__ cand,
                int32_t* __restrict__ tile_cnt, float* __restrict__ tile_tau) {
    __shared__ uint4 wsA[kStagePieces], wsB[kStagePieces], wsC[kStagePieces], wsD[kStagePieces];
    __shared__ uint4 xsA[kStagePieces], xsB[kStagePieces], xsC[kStagePieces], xsD[kStagePieces];
    __shared__ float red1[2][kGemmTok];
    __shared__ float red2[2][kGemmTok];
    __shared__ int cnt_s[kGemmTok];
    __shared__ int cnt2_s[2][kGemmTok];
    __shared__ float red3[2][kGemmTok];  // per-token maxima
    // One tile: latent slice mt over tokens [n0, n0 + 64 * NB) of the staged
    // list (ntok of them live), NB = 4 or 2.
    auto gemm_tile = [&](auto nb_c, const int mt, const int n0, const int ntok)
        __attribute__((always_inline)) {
    constexpr int NB = decltype(nb_c)::value;
    constexpr int kTok = 64 * NB;    // tokens of the tile
    constexpr int kHalf = 32 * NB;   // tokens of a wave
    int tid = threadIdx.x;  // opaque (see big_tile)
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;  // latent half, token half
    const int g = lane >> 5, j32 = lane & 31;
    const int nS = d / 32;                    // stages, a multiple of 8

    const uint4* W4 = reinterpret_cast<const uint4*>(W);
    const uint4* X4 = reinterpret_cast<const uint4*>(xs_g);
    const int64_t wstride = static_cast<int64_t>(n_mt) * 2048;  // pieces per K chunk of 64
    const int64_t xplane = static_cast<int64_t>(n_pad) * 4;     // pieces per stage plane
    // copy sources, in pieces from the start of the stage's operand block
    // (lane-contiguous LDS destinations q*256 + wave*64 + lane)
    int wsrc[4], xsrc[NB];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int P = q * 256 + wave * 64 + lane;
        wsrc[q] = (P >> 7) * 256 + (P & 127);
        const int n = P >> 2;
        if (q < NB) xsrc[q] = n * 4 + ((P & 3) ^ gsw(n));
    }
    W4 += static_cast<int64_t>(mt) * 2048;  // this tile's latent slice
    X4 += static_cast<int64_t>(n0) * 4;     // this tile's tokens
    // issue the 8 copies of stage j (past the end: the last stage again,
    // which keeps the loop free of branches that would split the schedule).
    // Each copy is a buffer load whose resource covers exactly the stage's
    // operand block (its base and size are scalar), so the per-lane offset is
    // a fixed 32-bit value and an offset outside the block would read zeros.
    auto copy_stage = [&](int j, uint4* wdst, uint4* xdst) __attribute__((always_inline)) {
        j = min(j, nS - 1);
        const int kc = j >> 1, hh = j & 1;
        const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint4*>(W4 + kc * wstride + hh * 128), 0, 2048 * 16, kBufferDword3);
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint4*>(X4 + j * xplane), 0, kTok * 64, kBufferDword3);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                wr, (__attribute__((address_space(3))) void*)(wdst + q * 256 + wave * 64),
                16, static_cast<unsigned>(wsrc[q]) * 16u, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < NB; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                xr, (__attribute__((address_space(3))) void*)(xdst + q * 256 + wave * 64),
                16, static_cast<unsigned>(xsrc[q]) * 16u, 0, 0, 0);
    };

    // accumulators start at the folded bias of their latent:
    // acc[a][nb][r] holds latent 128*wm + 32*a + 8*(r/4) + 4*g + r%4
    f32x16_t acc[4][NB];
    {
        const float* cf = c_fold + mt * 256 + 128 * wm + 4 * g;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 c4 = *reinterpret_cast<const float4*>(cf + 32 * a + 8 * q);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    acc[a][nb][4 * q + 0] = c4.x;
                    acc[a][nb][4 * q + 1] = c4.y;
                    acc[a][nb][4 * q + 2] = c4.z;
                    acc[a][nb][4 * q + 3] = c4.w;
                }
            }
    }

    uint4 FA[4], FB[NB], PA[4], PB[NB];
    auto read_step = [&](const uint4* wb, const uint4* xb, int s, uint4 (&A)[4], uint4 (&B)[NB])
        __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < 4; ++a) A[a] = wb[(4 * wm + a) * 128 + s * 64 + lane];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int n = kHalf * wn + 32 * nb + j32;
            B[nb] = xb[n * 4 + ((2 * s + g) ^ gsw(n))];
        }
    };
    auto mfma_step = [&](const uint4 (&A)[4], const uint4 (&B)[NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                acc[a][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(A[a]),
                                                                     as_bf16x8(B[nb]), acc[a][nb],
                                                                     0, 0, 0);
    };
    // Two stages per barrier.  Wait for this wave's copies of stages j and
    // j + 1 and its LDS reads, then meet at the barrier: every copy of the
    // pair has landed and every wave is done with the pair before it, whose
    // buffers are refilled with stages j + 2 and j + 3 while this pair is
    // multiplied.  In each stage: read step 0, multiply the carried step,
    // read step 1 (carried on), multiply step 0.
    auto stage_pair = [&](int j, const uint4* w0, const uint4* x0, const uint4* w1,
                          const uint4* x1, uint4* wf0, uint4* xf0, uint4* wf1, uint4* xf1,
                          bool first) __attribute__((always_inline)) {
        XMIX_WAIT_VM_LGKM0(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        copy_stage(j + 2, wf0, xf0);
        read_step(w0, x0, 0, FA, FB);
        if (!first) mfma_step(PA, PB);
        read_step(w0, x0, 1, PA, PB);
        mfma_step(FA, FB);
        copy_stage(j + 3, wf1, xf1);
        read_step(w1, x1, 0, FA, FB);
        mfma_step(PA, PB);
        read_step(w1, x1, 1, PA, PB);
        mfma_step(FA, FB);
        // instruction order: first stage's step-0 reads; carried MFMAs with
        // the first refill between them; step-0 MFMAs with step-1 reads;
        // second stage's step-0 reads and the second refill between the
        // carried MFMAs; step-0 MFMAs with step-1 reads
        constexpr int kReads = 4 + NB, kMfma = 4 * NB, kCopies = 4 + NB;
        __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);
        if (!first) {
#pragma unroll
            for (int i = 0; i < kCopies; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, kMfma / 8, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
        } else {
            __builtin_amdgcn_sched_group_barrier(0x020, kCopies, 0);
        }
#pragma unroll
        for (int i = 0; i < kReads; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, kMfma / 8, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        if constexpr (NB == 4) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < kReads; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < kReads; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, kMfma / 8, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    };

    copy_stage(0, wsA, xsA);
    copy_stage(1, wsB, xsB);
    stage_pair(0, wsA, xsA, wsB, xsB, wsC, xsC, wsD, xsD, true);
    stage_pair(2, wsC, xsC, wsD, xsD, wsA, xsA, wsB, xsB, false);
    for (int j = 4; j < nS; j += 4) {
        stage_pair(j + 0, wsA, xsA, wsB, xsB, wsC, xsC, wsD, xsD, false);
        stage_pair(j + 2, wsC, xsC, wsD, xsD, wsA, xsA, wsB, xsB, false);
    }
    mfma_step(PA, PB);
    // every wave's trailing copies have landed and its reads are done before
    // the stage buffers are reused below
    XMIX_WAIT_VM_LGKM0(0);
    __syncthreads();

    // ---------------------------------------------------------- epilogue
    // acc[a][nb][r] holds latent 128*wm + 32*a + 8*(r/4) + 4*g + r%4 of
    // token 128*wn + 32*nb + j32; lanes j32 and j32 + 32 of waves (0, wn)
    // and (1, wn) together hold the 256 latents of one token.  The four
    // token groups nb of a wave go through each phase together, so the
    // waves meet once for the statistics and twice per refinement round
    // (not once per group) and the groups' independent work fills the gaps
    // of a wave that has its SIMD to itself.  Each token's threshold follows
    // the same sequence of guesses as when its group is finished alone: the
    // rounds go on while any token of the tile is outside the window, and a
    // token inside it keeps its threshold.  The count pass keeps a bit mask
    // of the lane's values >= tau; for the emission a group's values are
    // parked in the wave's own part of the (now idle) stage buffers, so that
    // the few selected ones are fetched by index.
    cnt_s[tid] = 0;
    float* park[2] = {reinterpret_cast<float*>(wave == 0 ? wsA : wave == 1 ? wsB : wave == 2 ? wsC : wsD),
                      reinterpret_cast<float*>(wave == 0 ? xsA : wave == 1 ? xsB : wave == 2 ? xsC : xsD)};
    // park the values of group nb in buffer nb % 2 (16-byte groups,
    // lane-contiguous, so the stores are conflict-free)
    auto park_group = [&](int nb) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 16; ++q)
            reinterpret_cast<float4*>(park[nb & 1])[q * 64 + lane] =
                make_float4(acc[q >> 2][nb][4 * (q & 3)], acc[q >> 2][nb][4 * (q & 3) + 1],
                            acc[q >> 2][nb][4 * (q & 3) + 2], acc[q >> 2][nb][4 * (q & 3) + 3]);
    };
    park_group(0);
    park_group(1);
    // mean and variance over the tile's 256 latents, per token, and the
    // largest value
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        float s1 = 0.0f, s2 = 0.0f, mx = -INFINITY;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                s1 += acc[a][nb][r];
                s2 = fmaf(acc[a][nb][r], acc[a][nb][r], s2);
                mx = fmaxf(mx, acc[a][nb][r]);
            }
        s1 += __shfl_xor(s1, 32, kWave);
        s2 += __shfl_xor(s2, 32, kWave);
        mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
        if (g == 0) {
            red1[wm][kHalf * wn + 32 * nb + j32] = s1;
            red2[wm][kHalf * wn + 32 * nb + j32] = s2;
            red3[wm][kHalf * wn + 32 * nb + j32] = mx;
        }
    }
    __syncthreads();
    float tau[NB], lo_b[NB], hi_b[NB], mxv[NB];
    uint32_t m0[NB], m1[NB];  // bit i: value i >= tau (m1: value 32 + i)
    bool bad[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int n = kHalf * wn + 32 * nb + j32;
        const float s1 = red1[0][n] + red1[1][n], s2 = red2[0][n] + red2[1][n];
        const float mu = s1 * (1.0f / 256.0f);
        const float sd = sqrtf(fmaxf(s2 * (1.0f / 256.0f) - mu * mu, 0.0f));
        const float mx = fmaxf(red3[0][n], red3[1][n]);
        mxv[nb] = mx;
        // a strong latent (above mean + 5 stdev, such as a feature clamped
        // high at an earlier layer) would lift the guess for its whole
        // slice: the guess leaves the slice's largest value out then (the
        // decode kernel leaves out every value above the cut; here a second
        // pass over the accumulators would not fit the register file)
        tau[nb] = mx > mu + kTrimZ * sd ? trimmed_guess(s1 - mx, s2 - mx * mx, kBM - 1, z_guess)
                                        : mu + z_guess * sd;
        lo_b[nb] = -INFINITY;
        hi_b[nb] = INFINITY;
        bad[nb] = false;
    }
    auto count_at = [&](int nb) __attribute__((always_inline)) {
        uint32_t b0 = 0, b1 = 0;
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            b0 |= (acc[i >> 4][nb][i & 15] >= tau[nb] ? 1u : 0u) << i;
            b1 |= (acc[2 + (i >> 4)][nb][i & 15] >= tau[nb] ? 1u : 0u) << i;
        }
        m0[nb] = b0;
        m1[nb] = b1;
        return __popc(b0) + __popc(b1);
    };
    // count(pre >= tau) per token; refine tau until lo_cnt <= count <= cap.
    // cnt2_s is written before the round's first barrier and read before its
    // second, so one buffer serves every round.
    bool gave_up = false;
    for (int it = 0; it < kRefineIters; ++it) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int c_lane = count_at(nb);
            const int c = c_lane + __shfl_xor(c_lane, 32, kWave);
            if (g == 0) cnt2_s[wm][kHalf * wn + 32 * nb + j32] = c;
        }
        __syncthreads();
        bool any_bad = false;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int n = kHalf * wn + 32 * nb + j32;
            const int cn = cnt2_s[0][n] + cnt2_s[1][n];
            bad[nb] = false;
            if (n < ntok) {
                if (cn > cap) {
                    lo_b[nb] = tau[nb];
                    bad[nb] = true;
                } else if (cn < lo_cnt) {
                    hi_b[nb] = tau[nb];
                    bad[nb] = true;
                }
            }
            if (bad[nb]) {
                if (isfinite(lo_b[nb]) && isfinite(hi_b[nb])) {
                    tau[nb] = 0.5f * (lo_b[nb] + hi_b[nb]);
                } else {
                    const float step = refine_step(tau[nb], it);
                    tau[nb] = isfinite(hi_b[nb]) ? tau[nb] - step : tau[nb] + step;
                }
            }
            any_bad = any_bad || bad[nb];
        }
        if (!__syncthreads_or(any_bad)) break;
        // out of rounds: a threshold whose count is known to be <= cap
        if (it == kRefineIters - 1) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                if (bad[nb]) tau[nb] = hi_b[nb];
            gave_up = true;
        }
    }
    if (gave_up) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) count_at(nb);
    }
    // emit every latent with pre >= tau: reserve the lane's slots with one
    // LDS atomic, then write one selected (value, latent) pair per round,
    // the value read back from where it was parked
    const int lat0 = mt * 256 + 128 * wm + 4 * g;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int n = kHalf * wn + 32 * nb + j32;
        const float* pk = park[nb & 1];
        uint32_t b0 = n < ntok ? m0[nb] : 0u, b1 = n < ntok ? m1[nb] : 0u;
        const int c = __popc(b0) + __popc(b1);
        int slot = 0;
        if (c > 0) slot = atomicAdd(&cnt_s[n], c);
        const int64_t row = static_cast<int64_t>(n0 + n) * n_mt + mt;
        uint2* dst = cand + row * cap;
        while (__builtin_amdgcn_read_exec() & wave_ballot((b0 | b1) != 0)) {
            if ((b0 | b1) != 0) {
                const int i = b0 ? __builtin_ctz(b0) : 32 + __builtin_ctz(b1);
                if (b0) b0 &= b0 - 1;
                else b1 &= b1 - 1;
                const float val = pk[((i >> 2) * 64 + lane) * 4 + (i & 3)];
                if (slot < cap)
                    dst[slot] = make_uint2(__float_as_uint(val),
                                           static_cast<uint32_t>(lat0 + 32 * (i >> 4) +
                                                                 8 * ((i >> 2) & 3) + (i & 3)));
                ++slot;
            }
        }
        // the slice's bound: tau, or with nothing at or above it the next
        // value above the slice's maximum (the tighter of the two)
        if (n < ntok && wm == 0 && g == 0)
            tile_tau[row] = mxv[nb] < tau[nb] ? key_f32(f32_key(mxv[nb]) + 1u) : tau[nb];
        // the wave's reads of this buffer precede these stores in its LDS queue
        if (nb + 2 < NB) park_group(nb + 2);
    }
    __syncthreads();
    if (tid < ntok) tile_cnt[static_cast<int64_t>(n0 + tid) * n_mt + mt] = min(cnt_s[tid], cap);
    };
    const int cnt = *app_count;
    const int L = blockIdx.x;
    const int t256 = n_mt * ((cnt + 255) / 256), t128 = n_mt * ((cnt + 127) / 128);
    if (t128 <= kSmallTiles && (t128 + 255) / 256 * 68 < (t256 + 255) / 256 * 100) {  // uniform
        if (L >= t128) return;
        const int mt = L % n_mt, n0 = L / n_mt * 128;
        gemm_tile(std::integral_constant<int, 2>{}, mt, n0, min(128, cnt - n0));
        return;
    }

    // Tile order: launch slot L runs on XCD L % 8, which owns the latent
    // tiles [x*M8, (x+1)*M8) and walks them in blocks of 8 token tiles x 4
    // latent tiles (32 consecutive slots, one per CU of the XCD), token
    // blocks fastest, so each stage of a block's operands is fetched into
    // the XCD's L2 once and read by 4 and 8 workgroups.
    const int xcd = L % 8, slot = L / 8;
    const int m8 = (n_mt + 7) / 8;
    const int nbt = (n_nt + kGBlkTok - 1) / kGBlkTok;
    const int b = slot / (kGBlkTok * kGBlkLat), p = slot % (kGBlkTok * kGBlkLat);
    const int bt = b % nbt, bl = b / nbt;
    const int lt = kGBlkLat * bl + p / kGBlkTok;
    const int nt = kGBlkTok * bt + p % kGBlkTok;
    if (nt >= n_nt || lt >= m8) return;
    const int mt = xcd * m8 + lt;
    if (mt >= n_mt) return;
    const int n0 = nt * kGemmTok;
    if (n0 >= cnt) return;
    gemm_tile(std::integral_constant<int, 4>{}, mt, n0, min(kGemmTok, cnt - n0));
}

// ------------------------------------------------------------- final merge
// Keys are order-preserving integer images of the fp32 values and the
// selection order is (key descending, latent ascending).

// Makes this wave's LDS writes visible to its other lanes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int wave_count(bool p) { return __popcll(wave_ballot(p)); }

// Selects the k best of the pool key[0..n) / idx[0..n) (this wave's LDS
// region, n <= 64 * R) and moves them to lanes 0..k-1 (returned in wk/wi,
// in pool order; other lanes get key 0).  The selection is
//   { i : key[i] > tau  or  (key[i] == tau and idx[i] <= cut) }
// with exactly k entries (requires n >= k); tau is returned.  The keys stay
// in registers for the whole selection; the latents are read from LDS only
// where needed (entries tied at tau, and the k taken).  tau is found by
// bisection on the key bits below the highest bit in which the pool's keys
// differ (counts are ballot popcounts), stopping as soon as the count hits k.
template <int R>
__device__ __forceinline__ void wave_select_take(const uint32_t* key, const int32_t* idx, int n,
                                                 int k, uint32_t* stage_k, int32_t* stage_i,
                                                 uint32_t* tau_out, uint32_t* wk, int32_t* wi) {
    const int lane = lane_id();
    uint32_t kr[R];
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = lane + kWave * r;
        kr[r] = i < n ? key[i] : 0u;  // real keys are >= 1; 0 never counts
        if (i < n) {
            kmin = min(kmin, kr[r]);
            kmax = max(kmax, kr[r]);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        kmin = min(kmin, static_cast<uint32_t>(__shfl_xor(static_cast<int>(kmin), off, kWave)));
        kmax = max(kmax, static_cast<uint32_t>(__shfl_xor(static_cast<int>(kmax), off, kWave)));
    }
    // every key shares the bits of kmin above the highest differing bit, so
    // the k-th largest does too: start the bisection below it
    const uint32_t diff = kmin ^ kmax;
    const int top = diff ? 31 - __builtin_clz(diff) : -1;
    uint32_t tau = top < 31 ? (kmin & ~((2u << top) - 1u)) : 0u;
    if (top < 0) tau = kmin;
    bool exact = false;
    for (int bit = top; bit >= 0; --bit) {
        const uint32_t c = tau | (1u << bit);
        int ge = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) ge += wave_count(kr[r] >= c);
        if (ge >= k) {
            tau = c;
            if (ge == k) {  // the k best are exactly the keys >= c
                exact = true;
                break;
            }
        }
    }
    int32_t cut = 0x7FFFFFFF;
    if (!exact) {
        int gt = 0, eq = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            gt += wave_count(kr[r] > tau);
            eq += wave_count(kr[r] == tau);
        }
        const int need = k - gt;
        if (eq > need) {
            // smallest I with #{key == tau and idx <= I} >= need; the tied
            // latents are read from LDS, only in rounds that hold a tie
            int32_t lo = 0;
            for (int bit = 30; bit >= 0; --bit) {
                const int32_t probe = lo | ((1 << bit) - 1);
                int c = 0;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const bool tie = kr[r] == tau;
                    if (wave_ballot(tie)) c += wave_count(tie && idx[lane + kWave * r] <= probe);
                }
                if (c < need) lo |= (1 << bit);
            }
            cut = lo;
        }
    }
    // compact the selection to the front of the stage area
    int base = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = lane + kWave * r;
        bool take = i < n && kr[r] >= tau;
        const uint64_t cand = wave_ballot(take);
        if (cand) {
            int32_t ir = 0;
            if (take) ir = idx[i];
            take = take && (kr[r] > tau || ir <= cut);
            const uint64_t b = wave_ballot(take);
            if (take) {
                stage_k[base + lanes_below(b)] = kr[r];
                stage_i[base + lanes_below(b)] = ir;
            }
            base += __popcll(b);
        }
    }
    wave_sync();
    *tau_out = tau;
    *wk = lane < base ? stage_k[lane] : 0u;
    *wi = lane < base ? stage_i[lane] : 0x7FFFFFFF;
}

// Optional readback of the merged rows into a ring (same row format and
// head protocol as the readback compaction).
struct RingOut {
    uint8_t* slots;     // null: no readback
    uint64_t* head;     // [2]: head, ticket counter (zero between calls)
    int32_t capacity, row_bytes;
    const int32_t* req;
    int32_t layer_id, app_id;
};

// The workgroup's ticket; the last of the `cnt` workgroups that hold a token
// advances the head by `cnt` (each read the head before its ticket) and
// resets the counter.  Workgroups without a token take no ticket, so a step
// with no subscriber costs no atomics.  No fence before the ticket: the rows
// and the head are read by work ordered after the kernel, which its
// completion makes visible.
__device__ __forceinline__ void ring_ticket(const RingOut& ring, uint64_t h0, int cnt) {
    const uint64_t ticket = atomicAdd(reinterpret_cast<unsigned long long*>(&ring.head[1]), 1ull);
    if (ticket == static_cast<uint64_t>(cnt) - 1u) {
        __atomic_store_n(&ring.head[0], h0 + static_cast<uint64_t>(cnt), __ATOMIC_RELAXED);
        atomicExch(reinterpret_cast<unsigned long long*>(&ring.head[1]), 0ull);
    }
}

constexpr int kMergeThreads = 256;
constexpr int kMergeWaves = kMergeThreads / kWave;
constexpr int kMergeR = 32;                        // pool entries per lane
constexpr int kPoolMax = kMergeR * kWave;          // 2048
constexpr int kRepairR = 6;                        // repair pool entries per lane
constexpr int kRepairPool = kRepairR * kWave;      // 384 >= k + one slice
constexpr int kFloorRounds = 3;                    // pool refills above a raised floor

// Wave-wide scans and reductions on DPP lane moves (every lane active):
// within each row of 16 lanes, then across the four rows (row_bcast for the
// scan, lane reads for the reductions, whose results are uniform).
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
    const uint32_t lo = static_cast<uint32_t>(dpp_i<CTRL>(static_cast<int>(v)));
    const uint32_t hi = static_cast<uint32_t>(dpp_i<CTRL>(static_cast<int>(v >> 32)));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}
__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(v), l);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(v >> 32), l);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}
template <bool MAX>
__device__ __forceinline__ uint32_t wave_minmax_u32(uint32_t v) {
    auto op = [](uint32_t a, uint32_t b) { return MAX ? max(a, b) : min(a, b); };
    v = op(v, static_cast<uint32_t>(dpp_i<kDppXor1>(static_cast<int>(v))));
    v = op(v, static_cast<uint32_t>(dpp_i<kDppXor2>(static_cast<int>(v))));
    v = op(v, static_cast<uint32_t>(dpp_i<kDppHalfMirror>(static_cast<int>(v))));
    v = op(v, static_cast<uint32_t>(dpp_i<kDppMirror>(static_cast<int>(v))));
    const int iv = static_cast<int>(v);
    return op(op(__builtin_amdgcn_readlane(iv, 0), __builtin_amdgcn_readlane(iv, 16)),
              op(__builtin_amdgcn_readlane(iv, 32), __builtin_amdgcn_readlane(iv, 48)));
}
template <bool MAX>
__device__ __forceinline__ uint64_t wave_minmax_u64(uint64_t v) {
    auto op = [](uint64_t a, uint64_t b) { return MAX ? max(a, b) : min(a, b); };
    v = op(v, dpp_u64<kDppXor1>(v));
    v = op(v, dpp_u64<kDppXor2>(v));
    v = op(v, dpp_u64<kDppHalfMirror>(v));
    v = op(v, dpp_u64<kDppMirror>(v));
    return op(op(readlane_u64(v, 0), readlane_u64(v, 16)),
              op(readlane_u64(v, 32), readlane_u64(v, 48)));
}

// The pre-activation of latent 256*mt + threadIdx.x for one token, the workgroup
// computing the 256 latents of slice mt together with the encode's own matrix
// instruction in its order (bias first, then K ascending), so that a recomputed
// value has the bits that the encode kernels gave it.  A wave takes 64 latents; the
// token's row is every column of operand B, so a lane's accumulators hold the same
// values in each of the 32 columns.  part: 256 floats of LDS.
//
// One workgroup reads a slice at the latency of its loads; each step's registers
// are filled again for the next chunk as soon as they are read (ten tied slices,
// 128 tokens, d = 4096: the merge 82 us with a chunk loaded and then multiplied,
// 53 with this, 64 with dot products in registers).
__device__ __forceinline__ float slice_pre(const uint16_t* __restrict__ Wp,
                                           const uint16_t* __restrict__ hrow,
                                           const float* __restrict__ c_fold, int32_t mt,
                                           int32_t n_mt, int32_t d, float* part) {
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const int g = lane >> 5, j32 = lane & 31;
    const uint4* P = reinterpret_cast<const uint4*>(Wp) + static_cast<int64_t>(mt) * 2048;
    const int64_t stride = static_cast<int64_t>(n_mt) * 2048;  // pieces per K chunk
    const uint4* hr = reinterpret_cast<const uint4*>(hrow);
    const uint32_t w_off = (2 * wave * 256 + lane) * 16, h_off = g * 16;
    // acc[a][r]: latent 64*wave + 32*a + 8*(r/4) + 4*g + r%4
    const float* cf = c_fold + mt * kBM + 64 * wave + 4 * g;
    f32x16_t acc[2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[a][r] = cf[32 * a + 8 * (r / 4) + r % 4];
    const int nK = d / kBK;
    uint4 hv[4], wv[2][4];
    auto load = [&](int kc, int s) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rh = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint4*>(hr + kc * 8), 0, 128, kBufferDword3);
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint4*>(P + kc * stride), 0, 2048 * 16, kBufferDword3);
        hv[s] = buffer_load16<0>(rh, h_off, s * 32);
#pragma unroll
        for (int a = 0; a < 2; ++a) wv[a][s] = buffer_load16<0>(rw, w_off, a * 4096 + s * 1024);
        asm volatile("" ::: "memory");  // the steps' loads in order, so that a wait is one step's
    };
#pragma unroll
    for (int s = 0; s < 4; ++s) load(0, s);
#pragma unroll 1
    for (int kc = 0; kc < nK; ++kc) {
        const int next = min(kc + 1, nK - 1);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
                acc[a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(wv[a][s]),
                                                                 as_bf16x8(hv[s]), acc[a], 0, 0, 0);
            load(next, s);  // into the registers just read
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (j32 == r) part[64 * wave + 32 * a + 8 * (r / 4) + 4 * g + r % 4] = acc[a][r];
    __syncthreads();
    const float pre = part[tid];
    __syncthreads();  // part is free for the next slice
    return pre;
}

// One workgroup per subscribed token.  Every thread gathers the candidates
// of the slices it owns (count, threshold and the slice's pair block are
// loaded together, so the gather costs one memory round trip), a prefix
// over the workgroup places them in an LDS pool, the workgroup selects the
// k best of it (radix select) and wave 0 checks the certificate; a failed
// check is repaired by the whole workgroup; wave 0 then writes each winner
// at its rank.  When the candidates exceed the pool, the k-th best of the
// first kPoolMax of them is a lower bound of the k-th best of all: the pool
// is filled again with the candidates at or above it (a little below; when
// exact ties leave that value floor
// where it was, the k-th composite (value, latent) itself), up to
// kFloorRounds times.  n: the workgroup's slot of the app's token list.
__device__ __forceinline__ void merge_token(
    int n, const uint2* __restrict__ cand, const int32_t* __restrict__ tile_cnt,
    const float* __restrict__ tile_tau, int32_t n_sl, int32_t n_mt, int32_t cap,
    const int32_t* __restrict__ app_count, const int32_t* __restrict__ tok_list, int32_t k,
    const uint16_t* __restrict__ h, int32_t d, const uint16_t* __restrict__ Wp,
    const float* __restrict__ c_fold, int32_t* __restrict__ idx_out,
    uint16_t* __restrict__ val_out, const RingOut& ring) {
    __shared__ uint32_t K[kPoolMax + kWave];
    __shared__ int32_t I[kPoolMax + kWave];
    __shared__ __align__(16) uint32_t K2[kWave];  // the selected k entries (k <= 64)
    __shared__ __align__(16) int32_t I2[kWave];
    __shared__ __align__(16) int hist_s[3][256];  // radix digit counts, 3 rounds in flight
    __shared__ float part_s[kBM];  // a recomputed slice
    __shared__ uint64_t cmin_s[kMergeWaves], cmax_s[kMergeWaves];
    __shared__ int sel_n_s;
    __shared__ int scan_s[2][kMergeWaves];  // gather rounds alternate between the two
    __shared__ uint32_t tmax_s[2][kMergeWaves];
    __shared__ int pool_n_s;
    __shared__ uint32_t floor_s;
    __shared__ uint64_t rbest_s[kMergeWaves], kth_s;  // repair: next slice, k-th composite
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const int64_t row0 = static_cast<int64_t>(n) * n_sl;
    // The first round of the gather below does not depend on the token
    // count: its loads go out before the count is read (the slot's area
    // exists for every slot below T_max; a slot past the count leaves
    // without using them).
    const int last = cap / 2 - 1;
    uint4 v0[4];
    int c0 = 0;
    float tf0 = 0.0f;
    {
        const bool own = tid < n_sl;
        const int64_t row = row0 + (own ? tid : 0);
        const uint4* src = reinterpret_cast<const uint4*>(cand + row * cap);
#pragma unroll
        for (int u = 0; u < 4; ++u) v0[u] = src[min(u, last)];
        if (own) {
            c0 = tile_cnt[row];
            tf0 = tile_tau[row];
        }
    }
    // readback ring (optional): each workgroup with a token reads the head
    // before it takes a ticket; the one drawing the last ticket advances it.
    // Read with the loads above (after them, so that no wait for those
    // waits for this one); the head was last written by an earlier call.
    uint64_t h0 = 0;
    if (ring.slots && tid == 0) h0 = ring.head[0];
    const int32_t t = tok_list[n];
    const int cnt = *app_count;
    if (n >= cnt) return;  // uniform: no token, no ring row, no ticket

    // Gather: the candidates whose composite (key, ~latent) is >= floor, in
    // slice order, into the pool
    // (the first kPoolMax of them; the rest are counted only).  Returns their
    // number; tau_tiles receives the largest slice bound, and each
    // wave's smallest and largest pool composite go to cmin_s / cmax_s (read
    // after the caller's barrier, with the first radix histogram cleared).
    uint32_t tau_tiles = 0;
    auto gather = [&](uint64_t floor) __attribute__((always_inline)) {
        int total = 0;
        uint64_t cmn = ~0ull, cmx = 0ull;
        for (int t0 = 0; t0 < n_sl; t0 += kMergeThreads) {
            const int tl = t0 + tid;
            const bool own = tl < n_sl;
            const int64_t row = row0 + (own ? tl : 0);
            // count, threshold and the first 8 pairs of the slice, in one round
            // (a slice holds about 2-3 candidates; more are fetched below)
            const uint4* src = reinterpret_cast<const uint4*>(cand + row * cap);
            uint4 v[4];
            int c;
            uint32_t tk;
            if (t0 == 0 && floor == 0) {
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = v0[u];
                c = c0;
                tk = own ? f32_key(tf0) : 0u;
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = src[min(u, last)];
                c = own ? tile_cnt[row] : 0;
                tk = own ? f32_key(tile_tau[row]) : 0u;
            }
            // with a floor, only the candidates at or above it are kept
            int kept = c;
            if (floor != 0) {  // uniform
                kept = 0;
                for (int q0 = 0; q0 < c; q0 += 8) {
                    uint4 x[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) x[u] = q0 == 0 ? v[u] : src[min(q0 / 2 + u, last)];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int q = q0 + 2 * u;
                        const uint64_t ca =
                            (static_cast<uint64_t>(f32_key(__uint_as_float(x[u].x))) << 32) |
                            ~x[u].y;
                        const uint64_t cb =
                            (static_cast<uint64_t>(f32_key(__uint_as_float(x[u].z))) << 32) |
                            ~x[u].w;
                        kept += (q < c && ca >= floor) ? 1 : 0;
                        kept += (q + 1 < c && cb >= floor) ? 1 : 0;
                    }
                }
            }
            // workgroup prefix of the kept counts (the slots of a round were
            // last read before the previous round's barrier)
            const int incl = wave_incl_sum(kept);
            const uint32_t tm = wave_minmax_u32<true>(tk);
            const int par = (t0 / kMergeThreads) & 1;
            if (lane == kWave - 1) scan_s[par][wave] = incl;
            if (lane == 0) tmax_s[par][wave] = tm;
            __syncthreads();
            int base = total, round = 0;
#pragma unroll
            for (int w = 0; w < kMergeWaves; ++w) {
                base += (w < wave) ? scan_s[par][w] : 0;
                round += scan_s[par][w];
                tau_tiles = max(tau_tiles, tmax_s[par][w]);
            }
            int pos = base + incl - kept;
            total += round;
            if (pos >= kPoolMax) continue;  // nothing of this slice fits
            // the entries of this slice, in order (the first kPoolMax overall)
            for (int q0 = 0; q0 < c; q0 += 8) {
                uint4 x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = q0 == 0 ? v[u] : src[min(q0 / 2 + u, last)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int q = q0 + 2 * u;
                    const uint32_t ka = f32_key(__uint_as_float(x[u].x));
                    const uint32_t kb = f32_key(__uint_as_float(x[u].z));
                    if (q < c && ((static_cast<uint64_t>(ka) << 32) | ~x[u].y) >= floor) {
                        if (pos < kPoolMax) {
                            K[pos] = ka;
                            I[pos] = static_cast<int32_t>(x[u].y);
                            const uint64_t cc = (static_cast<uint64_t>(ka) << 32) | ~x[u].y;
                            cmn = min(cmn, cc);
                            cmx = max(cmx, cc);
                        }
                        ++pos;
                    }
                    if (q + 1 < c && ((static_cast<uint64_t>(kb) << 32) | ~x[u].w) >= floor) {
                        if (pos < kPoolMax) {
                            K[pos] = kb;
                            I[pos] = static_cast<int32_t>(x[u].w);
                            const uint64_t cc = (static_cast<uint64_t>(kb) << 32) | ~x[u].w;
                            cmn = min(cmn, cc);
                            cmx = max(cmx, cc);
                        }
                        ++pos;
                    }
                }
            }
        }
        cmn = wave_minmax_u64<false>(cmn);
        cmx = wave_minmax_u64<true>(cmx);
        if (lane == 0) {
            cmin_s[wave] = cmn;
            cmax_s[wave] = cmx;
        }
        hist_s[0][tid] = 0;
        return total;
    };

    // Radix select of the k-th best pool entry (entries 0 .. np - 1, np >= k)
    // by the whole workgroup.  An entry's rank is its 64-bit composite
    // (key, ~latent), so the order key descending, latent ascending has no
    // ties and exactly k entries lie at or above the k-th composite.
    // Starting at the 8-bit digit that holds the highest bit in which the
    // composites differ (from the gather's smallest and largest), each round
    // counts (LDS atomics) the digits of the entries that match the prefix
    // found so far, and every wave finds the digit that holds the k-th entry
    // from the same counts (one barrier per round; the three count buffers
    // rotate, so a buffer is cleared two barriers after its last read); the
    // rounds end as soon as that digit's whole bin is needed.  Returns the
    // prefix (the k best are the entries whose composite >> *shift_out is
    // >= prefix >> *shift_out).
    auto comp = [&](int i) __attribute__((always_inline)) {
        return (static_cast<uint64_t>(K[i]) << 32) | static_cast<uint32_t>(~I[i]);
    };
    auto radix_kth = [&](int np, int* shift_out) __attribute__((always_inline)) {
        uint64_t cmin = cmin_s[0], cmax = cmax_s[0];
#pragma unroll
        for (int w = 1; w < kMergeWaves; ++w) {
            cmin = min(cmin, cmin_s[w]);
            cmax = max(cmax, cmax_s[w]);
        }
        const uint64_t diff = cmin ^ cmax;
        int shift = diff ? ((63 - __clzll(static_cast<long long>(diff))) & ~7) : 0;
        // bits above the first digit are common to every entry
        uint64_t prefix = shift < 56 ? cmin & ~((1ull << (shift + 8)) - 1ull) : 0ull;
        int need = k;
        for (int round = 0;; ++round) {
            int* hc = hist_s[round % 3];
            const uint64_t hi = shift < 56 ? prefix >> (shift + 8) : 0ull;
            for (int i = tid; i < np; i += kMergeThreads) {
                const uint64_t c = comp(i);
                if (shift >= 56 || (c >> (shift + 8)) == hi)
                    atomicAdd(&hc[static_cast<int>(c >> shift) & 255], 1);
            }
            // for the next round; its last reads (two rounds ago) came
            // before the previous round's barrier
            hist_s[(round + 1) % 3][tid] = 0;
            __syncthreads();
            const int4 h4v = reinterpret_cast<const int4*>(hc)[lane];  // bins 4 lane .. + 3
            const int h4[4] = {h4v.x, h4v.y, h4v.z, h4v.w};
            const int ls = (h4[0] + h4[1]) + (h4[2] + h4[3]);
            const int incl = wave_incl_sum(ls);
            // entries in the bins of every higher lane
            int above = __builtin_amdgcn_readlane(incl, kWave - 1) - incl, dl = 0, gl = 0, hl = 0;
            bool found = false;
#pragma unroll
            for (int j = 3; j >= 0; --j) {
                if (above < need && need <= above + h4[j]) {
                    dl = 4 * lane + j;
                    gl = above;
                    hl = h4[j];
                    found = true;
                }
                above += h4[j];
            }
            // exactly one bin holds the need-th entry
            const uint64_t fb = wave_ballot(found);
            const int src = fb ? __ffsll(static_cast<long long>(fb)) - 1 : 0;
            const int D = __builtin_amdgcn_readlane(dl, src),
                      gt = __builtin_amdgcn_readlane(gl, src),
                      hb = __builtin_amdgcn_readlane(hl, src);
            need -= gt;
            prefix |= static_cast<uint64_t>(D) << shift;
            if (hb == need || shift == 0) break;  // uniform
            shift -= 8;
        }
        *shift_out = shift;
        return prefix;
    };

    // Gather, then selection of the k best of the pool (the pool itself is
    // left as it was: the repair below reads it).  While the candidates
    // overflow the pool, the k-th best of its first kPoolMax entries gives
    // the floor of a refill (one gather and one radix select serve every
    // round).
    uint32_t wk = 0;
    int32_t wi = 0x7FFFFFFF;
    uint64_t floor_c = 0;  // composite floor of the refills
    int total = 0;
    bool fits = false;
    for (int fr = 0;; ++fr) {
        total = gather(floor_c);
        __syncthreads();  // the pool is written
        const bool refill = total > kPoolMax && fr < kFloorRounds;  // uniform
        fits = total <= kPoolMax && total >= k;
        if (!refill && !fits) break;
        if (tid == 0) sel_n_s = 0;
        int shift;
        const uint64_t prefix = radix_kth(refill ? kPoolMax : total, &shift);
        if (refill) {
            // the k-th key is >= the prefix's key bits (the bits below its
            // last digit are zero); step a little below it
            const float fv = key_f32(static_cast<uint32_t>(prefix >> 32));
            uint64_t fl = static_cast<uint64_t>(f32_key(fv - fabsf(fv) * 0x1p-11f)) << 32;
            if (fl <= floor_c) {
                // no progress on the value (exact ties at the floor): the
                // k-th composite of the first kPoolMax itself, with exactly k
                // of them at or above it (the latent breaks the ties)
                fl = prefix;
                if (fl <= floor_c) {  // uniform: no progress at all
                    fits = false;
                    break;
                }
            }
            floor_c = fl;
            __syncthreads();  // every read of the pool is done
            continue;
        }
        const uint64_t cut = prefix >> shift;
        for (int i = tid; i < total; i += kMergeThreads) {
            const uint64_t c = comp(i);
            if ((c >> shift) >= cut) {
                const int pos = atomicAdd(&sel_n_s, 1);  // exactly k entries
                if (pos < kWave) {
                    K2[pos] = static_cast<uint32_t>(c >> 32);
                    I2[pos] = static_cast<int32_t>(~static_cast<uint32_t>(c));
                }
            }
        }
        __syncthreads();
        if (lane < k) {
            wk = K2[lane];
            wi = I2[lane];
        }
        break;
    }
    // every wave: the k-th key (the smallest of the selected) and whether
    // the selection stands (0), fails its certificate (1) or was not made (2)
    const uint32_t sel_tau = wave_minmax_u32<false>(lane < k ? wk : 0xFFFFFFFFu);
    const int fix = !fits ? 2 : (tau_tiles <= sel_tau ? 0 : 1);
    if (fix != 0) {  // uniform
        // Repair: whole slices are recomputed (the workgroup streaming each
        // slice once).  A slice hides only
        // values below its threshold, none of them at a latent below its
        // first: that composite bound says whether it can hide a winner.
        // The pool is cut down to what can still reach the top k; then the
        // slices are redone in descending order of their bound, each one's
        // pool entries replaced by its recomputed values above the floor,
        // wave 0 keeping the k best (at most kRepairPool entries) and raising
        // the floor and the k-th composite; the first slice whose bound lies
        // at or below the k-th composite ends the repair, since no later one
        // can hold a winner.  So tied or crowded slices cost the slices that
        // hold the top k, not every slice.  When the pool misses candidates
        // (more than kPoolMax after the refills) or keeps too many entries,
        // every slice is redone from an empty pool.
        const uint16_t* hrow = h + static_cast<int64_t>(t) * d;
        // the k-th selected composite (0: no selection yet)
        uint64_t kth = fix == 1 ? wave_minmax_u64<false>(
                                      lane < k ? (static_cast<uint64_t>(wk) << 32) |
                                                     static_cast<uint32_t>(~wi)
                                               : ~0ull)
                                : 0ull;
        // pool entries of slice q leave the pool (wave 0; q < 0: none), the
        // others from `fl` up stay
        auto cut_pool = [&](int np, uint32_t fl, int q) __attribute__((always_inline)) {
            int out = 0;
            for (int b0 = 0; b0 < np; b0 += kWave) {
                const int i = b0 + lane;
                const uint32_t kk = i < np ? K[i] : 0u;
                const int32_t ii = i < np ? I[i] : 0;
                const bool keep = i < np && kk >= fl && ii / kBM != q;
                const uint64_t bal = wave_ballot(keep);
                wave_sync();  // this round's reads come before its writes
                if (keep) {
                    K[out + lanes_below(bal)] = kk;
                    I[out + lanes_below(bal)] = ii;
                }
                out += __popcll(bal);
            }
            wave_sync();
            return out;
        };
        bool all = total > kPoolMax;  // uniform: the pool misses candidates
        if (!all && wave == 0) {
            // with a selection, its k-th value; without one, the whole pool
            const uint32_t fl = fix == 1 ? sel_tau : 0u;
            const int out = cut_pool(total, fl, -1);
            if (lane == 0) {
                pool_n_s = out;
                floor_s = fl;
            }
        }
        __syncthreads();
        if (!all && pool_n_s > kRepairPool - kBM) all = true;
        if (!all) {
            uint64_t prev = ~0ull;  // the slices with bounds below it are left
            for (;;) {
                uint64_t best = 0ull;
                const int wk = n_sl / n_mt;
                for (int q = tid; q < n_mt; q += kMergeThreads) {
                    // of a cut slice's parts, the highest bound
                    uint64_t bq = 0ull;
                    for (int j = q * wk; j < (q + 1) * wk; ++j) {
                        const uint32_t tk = f32_key(tile_tau[row0 + j]);
                        if (tk != 0u)
                            bq = max(bq, (static_cast<uint64_t>(tk - 1u) << 32) |
                                             static_cast<uint32_t>(~(j * (kBM / wk))));
                    }
                    if (bq < prev) best = max(best, bq);
                }
                best = wave_minmax_u64<true>(best);
                if (lane == 0) rbest_s[wave] = best;
                __syncthreads();
                best = max(max(rbest_s[0], rbest_s[1]), max(rbest_s[2], rbest_s[3]));
                if (best <= kth) break;  // uniform: no slice left can hold a winner
                prev = best;
                const int32_t q = static_cast<int32_t>(~static_cast<uint32_t>(best)) / kBM;
                if (wave == 0) {
                    const int out = cut_pool(pool_n_s, 0u, q);
                    if (lane == 0) pool_n_s = out;
                }
                __syncthreads();
                const int32_t j = q * kBM + tid;
                const uint32_t key = f32_key(slice_pre(Wp, hrow, c_fold, q, n_mt, d, part_s));
                if (key >= floor_s) {
                    const int pos = atomicAdd(&pool_n_s, 1);
                    K[pos] = key;
                    I[pos] = j;
                }
                __syncthreads();
                const int pn = pool_n_s;
                __syncthreads();  // every thread has read the pool size
                if (pn >= k) {
                    if (wave == 0) {
                        uint32_t tk, a;
                        int32_t b;
                        if (pn > k) {
                            wave_select_take<kRepairR>(K, I, pn, k, K + kPoolMax, I + kPoolMax,
                                                       &tk, &a, &b);
                            if (lane < k) {
                                K[lane] = a;
                                I[lane] = b;
                            }
                        } else {
                            a = lane < k ? K[lane] : 0xFFFFFFFFu;
                            b = lane < k ? I[lane] : 0;
                            tk = wave_minmax_u32<false>(a);
                        }
                        const uint64_t kc = wave_minmax_u64<false>(
                            lane < k ? (static_cast<uint64_t>(a) << 32) | static_cast<uint32_t>(~b)
                                     : ~0ull);
                        if (lane == 0) {
                            pool_n_s = k;
                            floor_s = max(floor_s, tk);
                            kth_s = kc;
                        }
                    }
                    __syncthreads();
                    kth = kth_s;
                }
            }
            // the pool holds the k best unless no slice was redone after the cut
            const int pn = pool_n_s;
            if (pn > k && wave == 0) {
                uint32_t tk, a;
                int32_t b;
                wave_select_take<kRepairR>(K, I, pn, k, K + kPoolMax, I + kPoolMax, &tk, &a, &b);
                if (lane < k) {
                    K[lane] = a;
                    I[lane] = b;
                }
            }
            all = pn < k;  // (fewer than k candidates) redo every slice
        }
        if (all) {  // uniform
            __syncthreads();  // every thread has read the pool size
            if (tid == 0) {
                pool_n_s = 0;
                floor_s = 0u;
            }
            __syncthreads();
            for (int q = 0; q < n_mt; ++q) {
                const int32_t j = q * kBM + tid;
                const uint32_t key = f32_key(slice_pre(Wp, hrow, c_fold, q, n_mt, d, part_s));
                if (key >= floor_s) {
                    const int pos = atomicAdd(&pool_n_s, 1);
                    K[pos] = key;
                    I[pos] = j;
                }
                __syncthreads();
                const int pn = pool_n_s;
                __syncthreads();  // every thread has read the pool size
                if (pn > k) {
                    if (wave == 0) {
                        uint32_t tk, a;
                        int32_t b;
                        wave_select_take<kRepairR>(K, I, pn, k, K + kPoolMax, I + kPoolMax, &tk,
                                                   &a, &b);
                        if (lane < k) {
                            K[lane] = a;
                            I[lane] = b;
                        }
                        if (lane == 0) {
                            pool_n_s = k;
                            floor_s = max(floor_s, tk);
                        }
                    }
                    __syncthreads();
                }
            }
        }
        if (wave == 0) {
            wk = lane < k ? K[lane] : 0u;
            wi = lane < k ? I[lane] : 0x7FFFFFFF;
        }
    }
    if (wave != 0) return;
    // write the k winners in the order (value desc, index asc): each lane
    // counts the winners that come before its own (the entries are
    // distinct), reading them back from LDS in broadcast
    if (lane < k) {
        K2[lane] = wk;
        I2[lane] = wi;
    }
    wave_sync();
    const uint64_t mine = (static_cast<uint64_t>(wk) << 32) | static_cast<uint32_t>(~wi);
    int rank = 0;
    for (int j = 0; j < k; ++j) {
        const uint64_t other = (static_cast<uint64_t>(K2[j]) << 32) | static_cast<uint32_t>(~I2[j]);
        rank += other > mine ? 1 : 0;
    }
    const uint16_t vb = f32_to_bf16_rne(fmaxf(key_f32(wk), 0.0f));
    if (lane < k) {
        const int64_t o = static_cast<int64_t>(t) * k + rank;
        idx_out[o] = wi;
        val_out[o] = vb;
    }
    if (ring.slots) {
        // ring row {token, request, layer, app} + idx[k] + val[k]; only the
        // last `capacity` rows of this call are written
        h0 = static_cast<uint64_t>(__shfl(static_cast<long long>(h0), 0, kWave));
        if (static_cast<int64_t>(n) >= static_cast<int64_t>(cnt) - ring.capacity) {
            uint8_t* row = ring.slots + static_cast<int64_t>((h0 + static_cast<uint64_t>(n)) %
                                                             static_cast<uint64_t>(ring.capacity)) *
                                            ring.row_bytes;
            // 16-bit stores: with k odd, every other row starts 2 bytes
            // past a 4-byte boundary
            uint16_t* row16 = reinterpret_cast<uint16_t*>(row);
            if (lane < 8) {
                const int f = lane >> 1;
                const uint32_t hdr = static_cast<uint32_t>(
                    f == 0 ? t : f == 1 ? ring.req[t] : f == 2 ? ring.layer_id : ring.app_id);
                row16[lane] = static_cast<uint16_t>((lane & 1) ? hdr >> 16 : hdr & 0xFFFFu);
            }
            if (lane < k) {
                const uint32_t iv = static_cast<uint32_t>(wi);
                row16[8 + 2 * rank] = static_cast<uint16_t>(iv & 0xFFFFu);
                row16[8 + 2 * rank + 1] = static_cast<uint16_t>(iv >> 16);
                row16[8 + 2 * k + rank] = vb;
            }
        }
        if (lane == 0) ring_ticket(ring, h0, cnt);
    }
}

__global__ void __launch_bounds__(kMergeThreads) __attribute__((amdgpu_waves_per_eu(4)))
sae_merge_kernel(const uint2* __restrict__ cand, const int32_t* __restrict__ tile_cnt,
                 const float* __restrict__ tile_tau, int32_t n_sl, int32_t n_mt, int32_t cap,
                 const int32_t* __restrict__ app_count, const int32_t* __restrict__ tok_list,
                 int32_t k, const uint16_t* __restrict__ h, int32_t d,
                 const uint16_t* __restrict__ Wp, const float* __restrict__ c_fold,
                 int32_t* __restrict__ idx_out, uint16_t* __restrict__ val_out,
                 RingOut ring) {
    merge_token(blockIdx.x, cand, tile_cnt, tile_tau, n_sl, n_mt, cap, app_count, tok_list, k, h, d,
                Wp, c_fold, idx_out, val_out, ring);
}

// One app's merge inputs and outputs in a batched launch.
struct MergeApp {
    const uint2* cand;
    const int32_t* tile_cnt;
    const float* tile_tau;
    const int32_t* app_count;
    const int32_t* tok_list;
    const uint16_t* Wp;
    const float* c_fold;
    int32_t* idx_out;
    uint16_t* val_out;
    RingOut ring;
    int32_t n_sl, n_mt, cap, k;
};
struct MergeApps {
    MergeApp a[kMultiMax];
};

// The merges of a batch of apps on a persistent grid: the pairs (app, slot
// of its token list) of every app's listed tokens, app by app, are dealt to
// the workgroups in turn, so a slot past its app's count costs nothing (no
// workgroup, no gather) and an empty batch costs one read of the counts.
__global__ void __launch_bounds__(kMergeThreads) __attribute__((amdgpu_waves_per_eu(4)))
sae_merge_apps_kernel(const uint16_t* __restrict__ h, int32_t d, int32_t T_max, int32_t n_apps,
                      MergeApps apps) {
    __shared__ int32_t cnt_s[kMultiMax];
    for (int i = 0; i < n_apps; ++i)
        if (threadIdx.x == i) cnt_s[i] = min(max(*apps.a[i].app_count, 0), T_max);
    __syncthreads();
    int32_t start[kMultiMax + 1];
    start[0] = 0;
#pragma unroll
    for (int i = 0; i < kMultiMax; ++i) start[i + 1] = start[i] + (i < n_apps ? cnt_s[i] : 0);
    const int32_t P = start[kMultiMax];
    for (int32_t p = blockIdx.x; p < P; p += gridDim.x) {  // uniform
        int i = 0;
#pragma unroll
        for (int j = 1; j < kMultiMax; ++j) i = j < n_apps && p >= start[j] ? j : i;
        const MergeApp& a = apps.a[i];
        merge_token(p - start[i], a.cand, a.tile_cnt, a.tile_tau, a.n_sl, a.n_mt, a.cap, a.app_count,
                    a.tok_list, a.k, h, d, a.Wp, a.c_fold, a.idx_out, a.val_out, a.ring);
        __syncthreads();  // the token's LDS is read before the next token's gather
    }
}

// ------------------------------------------------------------------ launch
// CUs of the current device (256 if the query fails), looked up once per device.
static int32_t cu_count() {
    constexpr int kDevs = 64;
    static std::atomic<int32_t> cache[kDevs];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevs) return 256;
    int32_t n = cache[dev].load(std::memory_order_relaxed);
    if (n <= 0) {
        int v = 0;
        n = hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
                    v > 0
                ? v
                : 256;
        cache[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Slices that one 256-latent tile is cut into (see narrow_tile), for a launch of
// n_mt tiles: as many as keep the workgroups at 256 or fewer.  A CU alone draws
// about 45 GB/s, so 160 whole slices saturate HBM and more than 128 are left whole;
// the apps of a batched call count together (eight dictionaries of 16384 latents,
// 102 tokens of width 2048 each: 275 us cut by each one's own slices, 148 whole).
// Batches of more than 512 slots keep whole slices too, which keeps the candidate
// area of every call that fitted the static workspace within it.
static int32_t slice_cut(int32_t T_max, int32_t d, int64_t n_mt) {
    static_assert(kMaxCutLatents == 128 * kBM, "the last dictionary that is cut");
    if (T_max > kMaxCutSlots || static_cast<int64_t>(T_max) * d * 2 > 0x7FFFFFFF) return 1;
    return n_mt <= 64 ? 4 : n_mt <= 128 ? 2 : 1;
}

// Whether an app may have several token tiles, big ones among them (whose buffer
// offsets are 32 bits).
static bool many_tiles(int32_t T_max) { return T_max > kBN; }

// Workgroups for an app's candidates: one per unit, at most one per CU where the
// token tiles are several.
static int32_t enc_grid(int32_t T_max, int64_t n_sl) {
    if (!many_tiles(T_max) || n_sl >= cu_count()) return static_cast<int32_t>(n_sl);
    const int64_t units = n_sl * ((T_max + kBN - 1) / kBN);
    return static_cast<int32_t>(units < cu_count() ? units : cu_count());
}

struct CandArea {
    uint2* cand;   // (fp32 bits, latent) pairs, [T_max][n_sl][cap]
    int32_t* cnt;  // [T_max][n_sl]
    float* tau;    // [T_max][n_sl]
};

static CandArea cand_area(void* base, int32_t T_max, int32_t n_sl, int cap) {
    const size_t slots = static_cast<size_t>(T_max) * n_sl;
    CandArea a;
    a.cand = static_cast<uint2*>(base);
    a.cnt = reinterpret_cast<int32_t*>(a.cand + slots * cap);
    a.tau = reinterpret_cast<float*>(a.cnt + slots);
    return a;
}

static int32_t stage_tokens(int32_t T_max) {
    return (T_max + kGemmTok - 1) / kGemmTok * kGemmTok;
}

static size_t area_bytes(int32_t T_max, int32_t m, int32_t k, int32_t cut) {
    const size_t slots = static_cast<size_t>(T_max) * (m / kBM * cut);
    return slots * (static_cast<size_t>(emit_cap(m, k, kBM / cut)) * 8u + 8u);
}

// The cut that an area of `bytes` holds, at most `cut` (a finer one needs more, and
// every accepted area holds whole slices).
static int32_t fit_cut(int32_t T_max, int32_t m, int32_t k, int32_t cut, size_t bytes) {
    while (cut > 1 && area_bytes(T_max, m, k, cut) > bytes) cut /= 2;
    return cut;
}

static size_t sae_bytes(int32_t T_max, int32_t d, int32_t m, int32_t k, int32_t cut) {
    size_t bytes = (area_bytes(T_max, m, k, cut) + 255u) / 256u * 256u;
    if (T_max >= kPrefillMinT)  // staged token rows of the prefill GEMM
        bytes += static_cast<size_t>(stage_tokens(T_max)) * d * sizeof(uint16_t);
    return bytes;
}

size_t sae_whole_bytes(int32_t T_max, int32_t d, int32_t m, int32_t k) {
    return sae_bytes(T_max, d, m, k, 1);
}

size_t sae_candidate_bytes(int32_t T_max, int32_t d, int32_t m, int32_t k) {
    return sae_bytes(T_max, d, m, k, slice_cut(T_max, d, m / kBM));
}

hipError_t launch_sae_pack(const uint16_t* W_enc, int32_t m, int32_t d, uint16_t* W_packed,
                           hipStream_t stream) {
    const int64_t pieces = static_cast<int64_t>(m) * (d / 8);
    hipLaunchKernelGGL(sae_pack_kernel, dim3(static_cast<uint32_t>((pieces + 255) / 256)),
                       dim3(256), 0, stream, W_enc, m, d, W_packed);
    return hipGetLastError();
}

hipError_t launch_sae_fold(const uint16_t* W_enc, const uint16_t* b_enc, const uint16_t* b_dec,
                           int32_t m, int32_t d, float* c_fold, hipStream_t stream) {
    hipLaunchKernelGGL(sae_fold_kernel, dim3((m + 3) / 4), dim3(256), 0, stream, W_enc, b_enc,
                       b_dec, m, d, c_fold);
    return hipGetLastError();
}

hipError_t launch_sae_candidates(const uint16_t* h, int32_t d, int32_t T_max,
                                 const int32_t* app_count, const int32_t* tok_list,
                                 const uint16_t* W_enc, const float* c_fold, int32_t m,
                                 int32_t k, void* cand, size_t cand_bytes, hipStream_t stream,
                                 const RouteIn* route) {
    const int32_t n_mt = m / kBM;
    const int32_t cut = fit_cut(T_max, m, k, slice_cut(T_max, d, n_mt), cand_bytes);
    const int32_t n_sl = n_mt * cut;
    const EmitPlan e = emit_plan(m, k, kBM / cut);
    const CandArea a = cand_area(cand, T_max, n_sl, e.cap);
    const int32_t grid = enc_grid(T_max, n_sl);
    // the decode kernel routes when the batch fits its LDS list and its grid
    // has a workgroup for every app to publish
    if (route && (T_max > kRouteMaxT || grid < route->n_apps)) {
        const hipError_t r = launch_route_build(route->req, route->T_valid, route->sub,
                                                route->R_max, T_max, route->n_apps,
                                                route->tok_mask, route->app_count,
                                                route->app_tokens, route->err_word, stream);
        if (r != hipSuccess) return r;
        route = nullptr;
    }
    if (T_max >= kPrefillMinT) {
        const int32_t n_pad = stage_tokens(T_max);
        uint16_t* xs = reinterpret_cast<uint16_t*>(
            static_cast<char*>(cand) + (area_bytes(T_max, m, k, cut) + 255u) / 256u * 256u);
        const int64_t pieces = static_cast<int64_t>(n_pad) * (d / 8);
        hipLaunchKernelGGL(sae_xstage_kernel, dim3(static_cast<uint32_t>((pieces + 255) / 256)),
                           dim3(256), 0, stream, h, d, app_count, tok_list, n_pad, xs);
        const int32_t n_nt = n_pad / kGemmTok;
        const int m8 = (n_mt + 7) / 8;
        const int nbt = (n_nt + kGBlkTok - 1) / kGBlkTok;
        const int nbl = (m8 + kGBlkLat - 1) / kGBlkLat;
        // workgroups for the blocks of 256-token tiles and for the 128-token
        // tiles that a small live count takes instead
        const int32_t small = 2 * n_mt * n_nt < kSmallTiles ? 2 * n_mt * n_nt : kSmallTiles;
        int32_t grid_g = 8 * nbt * nbl * kGBlkTok * kGBlkLat;
        grid_g = grid_g > small ? grid_g : small;
        hipLaunchKernelGGL(sae_gemm_kernel, dim3(grid_g), dim3(kGemmThreads), 0, stream, xs, d,
                           n_pad, app_count, W_enc, c_fold, n_mt, n_nt, e.z, e.lo, e.cap, a.cand,
                           a.cnt, a.tau);
        return hipGetLastError();
    }
    const RouteIn none{};
    const RouteIn& ri = route ? *route : none;
    const bool many = many_tiles(T_max);
    const auto kernel = cut == 4   ? (many ? sae_stream_kernel<4, true> : sae_stream_kernel<4, false>)
                        : cut == 2 ? (many ? sae_stream_kernel<2, true> : sae_stream_kernel<2, false>)
                                   : (many ? sae_stream_kernel<1, true> : sae_stream_kernel<1, false>);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kEncThreads), 0, stream, h, d, app_count, tok_list,
                       W_enc, c_fold, n_mt, T_max, e.z, e.lo, e.cap, a.cand, a.cnt, a.tau, ri.req,
                       ri.T_valid, ri.sub, ri.R_max, ri.n_apps, ri.app_bit, ri.tok_mask,
                       ri.app_count, ri.app_tokens, ri.err_word);
    return hipGetLastError();
}

hipError_t launch_sae_merge(const uint16_t* h, int32_t d, int32_t T_max,
                            const int32_t* app_count, const int32_t* tok_list,
                            const uint16_t* W_enc, const float* c_fold, int32_t m, int32_t k,
                            int32_t* idx_out, uint16_t* val_out, void* cand, size_t cand_bytes,
                            const MergeRing* ring, hipStream_t stream) {
    const int32_t n_mt = m / kBM;
    const int32_t cut = fit_cut(T_max, m, k, slice_cut(T_max, d, n_mt), cand_bytes);
    const int32_t n_sl = n_mt * cut;
    const int cap = emit_cap(m, k, kBM / cut);
    const CandArea a = cand_area(cand, T_max, n_sl, cap);
    RingOut r{};
    if (ring) {
        r.slots = ring->slots;
        r.head = ring->head;
        r.capacity = ring->capacity;
        r.row_bytes = ring->row_bytes;
        r.req = ring->req;
        r.layer_id = ring->layer_id;
        r.app_id = ring->app_id;
    }
    hipLaunchKernelGGL(sae_merge_kernel, dim3(T_max), dim3(kMergeThreads), 0, stream, a.cand,
                       a.cnt, a.tau, n_sl, n_mt, cap, app_count, tok_list, k, h, d, W_enc,
                       c_fold, idx_out, val_out, r);
    return hipGetLastError();
}

bool sae_multi_supported(int32_t T_max) { return T_max < kPrefillMinT; }

hipError_t launch_sae_encode_multi(const uint16_t* h, int32_t d, int32_t T_max, int32_t n,
                                   const SaeAppIn* apps, hipStream_t stream,
                                   const RouteIn* route) {
    const bool many = many_tiles(T_max);
    for (int32_t c0 = 0; c0 < n; c0 += kMultiMax) {
        const int32_t nc = n - c0 < kMultiMax ? n - c0 : kMultiMax;
        // one cut for all, by the slices of the batch together
        int64_t n_all = 0;
        for (int32_t i = 0; i < nc; ++i) n_all += apps[c0 + i].m / kBM;
        int32_t cut = slice_cut(T_max, d, n_all);
        for (int32_t i = 0; i < nc; ++i)
            cut = fit_cut(T_max, apps[c0 + i].m, apps[c0 + i].k, cut, apps[c0 + i].cand_bytes);
        EncApps ea;
        MergeApps ma;
        memset(&ea, 0, sizeof(ea));
        memset(&ma, 0, sizeof(ma));
        ea.n = nc;
        for (int32_t i = 0; i < nc; ++i) {
            const SaeAppIn& in = apps[c0 + i];
            const int32_t n_mt = in.m / kBM, n_sl = n_mt * cut;
            const EmitPlan e = emit_plan(in.m, in.k, kBM / cut);
            const CandArea a = cand_area(in.cand, T_max, n_sl, e.cap);
            ea.a[i] = EncApp{in.app_count, in.tok_list, in.W, in.c_fold, a.cand, a.cnt, a.tau,
                             n_mt, e.lo, e.cap, in.bit, e.z};
            RingOut r{};
            if (in.ring) {
                r.slots = in.ring->slots;
                r.head = in.ring->head;
                r.capacity = in.ring->capacity;
                r.row_bytes = in.ring->row_bytes;
                r.req = in.ring->req;
                r.layer_id = in.ring->layer_id;
                r.app_id = in.ring->app_id;
            }
            ma.a[i] = MergeApp{a.cand, a.cnt, a.tau, in.app_count, in.tok_list, in.W, in.c_fold,
                               in.idx_out, in.val_out, r, n_sl, n_mt, e.cap, in.k};
        }
        // the first launch builds the routing when the batch fits its LDS list
        const RouteIn* ri = c0 == 0 ? route : nullptr;
        if (ri && T_max > kRouteMaxT) {
            const hipError_t r = launch_route_build(ri->req, ri->T_valid, ri->sub, ri->R_max,
                                                    T_max, ri->n_apps, ri->tok_mask,
                                                    ri->app_count, ri->app_tokens,
                                                    ri->err_word, stream);
            if (r != hipSuccess) return r;
            ri = nullptr;
        }
        const RouteIn none{};
        const RouteIn& rr = ri ? *ri : none;
        // persistent: one workgroup per CU (and one per app to publish)
        const int64_t units = n_all * cut * (many ? (T_max + kBN - 1) / kBN : 1);
        int32_t g = units < cu_count() ? static_cast<int32_t>(units) : cu_count();
        if (ri && g < ri->n_apps) g = ri->n_apps;
        const auto kernel =
            cut == 4   ? (many ? sae_stream_apps_kernel<4, true> : sae_stream_apps_kernel<4, false>)
            : cut == 2 ? (many ? sae_stream_apps_kernel<2, true> : sae_stream_apps_kernel<2, false>)
                       : (many ? sae_stream_apps_kernel<1, true> : sae_stream_apps_kernel<1, false>);
        hipLaunchKernelGGL(kernel, dim3(g), dim3(kEncThreads), 0, stream, h, d, ea, rr.req,
                           rr.T_valid, rr.sub, rr.R_max, T_max, rr.n_apps, rr.tok_mask,
                           rr.app_count, rr.app_tokens, rr.err_word);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        // persistent merges: up to four workgroups per CU
        const int32_t mg = nc * T_max < 4 * cu_count() ? nc * T_max : 4 * cu_count();
        hipLaunchKernelGGL(sae_merge_apps_kernel, dim3(mg), dim3(kMergeThreads), 0, stream, h, d,
                           T_max, nc, ma);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Where the by-value descriptors hold device pointers (for the graph
// executor's redirection).
template <>
struct ArgPointers<RingOut> {
    static std::vector<uint16_t> offsets() {
        return {offsetof(RingOut, slots), offsetof(RingOut, head), offsetof(RingOut, req)};
    }
};
template <>
struct ArgPointers<EncApps> {
    static std::vector<uint16_t> offsets() {
        std::vector<uint16_t> o;
        for (int i = 0; i < kMultiMax; ++i)
            for (const size_t f : {offsetof(EncApp, app_count), offsetof(EncApp, tok_list),
                                   offsetof(EncApp, W), offsetof(EncApp, c_fold),
                                   offsetof(EncApp, cand), offsetof(EncApp, tile_cnt),
                                   offsetof(EncApp, tile_tau)})
                o.push_back(static_cast<uint16_t>(offsetof(EncApps, a) + i * sizeof(EncApp) + f));
        return o;
    }
};
template <>
struct ArgPointers<MergeApps> {
    static std::vector<uint16_t> offsets() {
        std::vector<uint16_t> o;
        for (int i = 0; i < kMultiMax; ++i) {
            const size_t b = offsetof(MergeApps, a) + i * sizeof(MergeApp);
            for (const size_t f : {offsetof(MergeApp, cand), offsetof(MergeApp, tile_cnt),
                                   offsetof(MergeApp, tile_tau), offsetof(MergeApp, app_count),
                                   offsetof(MergeApp, tok_list), offsetof(MergeApp, Wp),
                                   offsetof(MergeApp, c_fold), offsetof(MergeApp, idx_out),
                                   offsetof(MergeApp, val_out)})
                o.push_back(static_cast<uint16_t>(b + f));
            for (const uint16_t f : ArgPointers<RingOut>::offsets())
                o.push_back(static_cast<uint16_t>(b + offsetof(MergeApp, ring) + f));
        }
        return o;
    }
};

void add_sae_kernels(std::vector<KernelInfo>& t) {
    t.push_back(kernel_info(sae_pack_kernel));
    t.push_back(kernel_info(sae_fold_kernel));
    t.push_back(kernel_info(sae_stream_kernel<1, false>));
    t.push_back(kernel_info(sae_stream_kernel<1, true>));
    t.push_back(kernel_info(sae_stream_kernel<2, false>));
    t.push_back(kernel_info(sae_stream_kernel<2, true>));
    t.push_back(kernel_info(sae_stream_kernel<4, false>));
    t.push_back(kernel_info(sae_stream_kernel<4, true>));
    t.push_back(kernel_info(sae_xstage_kernel));
    t.push_back(kernel_info(sae_gemm_kernel));
    t.push_back(kernel_info(sae_merge_kernel));
    t.push_back(kernel_info(sae_merge_apps_kernel));
    t.push_back(kernel_info(sae_stream_apps_kernel<1, false>));
    t.push_back(kernel_info(sae_stream_apps_kernel<1, true>));
    t.push_back(kernel_info(sae_stream_apps_kernel<2, false>));
    t.push_back(kernel_info(sae_stream_apps_kernel<2, true>));
    t.push_back(kernel_info(sae_stream_apps_kernel<4, false>));
    t.push_back(kernel_info(sae_stream_apps_kernel<4, true>));
}

}  // namespace xmix
