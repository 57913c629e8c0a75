// Device helpers shared by the hook-step kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace xmix {

constexpr int kWave = 64;

// Has the kernel arguments named ("s"(x), ...) in scalar registers here.  The
// compiler reads an argument where it is first used, so a short kernel's chain
// holds a round trip to the argument block between each of its steps; with this
// the reads are issued together, and beside the first loads from memory.
#define XMIX_ARGS_NOW(...) asm volatile("" ::__VA_ARGS__)

// Whether a launch of one workgroup per token row reads its rows before it knows
// which ones carry a bit: a step of few rows is a chain of round trips (mask, row,
// result), and reading all of at most 8 MB costs it less than one of them.  The
// fused probe and steering pass with this, its arguments read together and no
// load behind a branch: 32 layers of 256 rows of 8 KB 150 -> 128 us, 16 layers of
// 512 rows of 16 KB 177 -> 143 us (a third of the bits set) and 130 -> 102 (5 %).
// Reading every row is what costs where few carry a bit: 16 layers of 512 fp32
// rows of 8 KB take 52.3 us with it and 50.1 without at 5 % of the bits, 61.7 and
// 64.5 at 40 %; of 1024 such rows, at the line, 62.1 and 59.5, and 78.6 and 82.2.
// The steering kernel keeps to the rows it needs: few rows of a gated step carry
// a bit, and eight such layers took 62 us with this and 56 without.
__host__ __device__ inline bool early_rows(int32_t rows, int32_t nvec) {
    return static_cast<int64_t>(rows) * nvec <= (8 << 20) / 16;
}

// Word 3 of a raw buffer resource (32-bit element format, no swizzle).
constexpr int kBufferDword3 = 0x00020000;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// This lane's 16-byte slice, `off` bytes on, of the n slices at p (both uniform):
// lanes past them read zero, and with n = 0 no memory is touched.  Loads that a
// step may or may not need go out this way without a branch, since a load behind
// one is easily waited for before the next is issued.
__device__ __forceinline__ uint4 slice_load(const uint4* p, int32_t n, uint32_t off) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint4*>(p), 0, n * 16, kBufferDword3);
    const u32x4_t v =
        __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// This lane's element of the n at p (uniform), in the same way: zero past them.
__device__ __forceinline__ int32_t lane_load(const void* p, int32_t n, int lane) {
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, n * 4, kBufferDword3);
    return __builtin_amdgcn_raw_buffer_load_b32(r, lane * 4, 0, 0);
}
__device__ __forceinline__ uint16_t lane_load(const uint16_t* p, int32_t n, int lane) {
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p), 0, n * 2, kBufferDword3);
    return __builtin_amdgcn_raw_buffer_load_b16(r, lane * 2, 0, 0);
}

// ---------------------------------------------------------------- bf16 bits
__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// Round-to-nearest-even of an fp32 value onto bf16, as bits.  Adding
// 0x7FFF plus the lowest kept bit and truncating rounds half to even; it
// carries into the exponent correctly, including the overflow to infinity.
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0;  // NaN
    u += 0x7FFFu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}

// Two bf16 packed in one dword: element 0 in the low half.
__device__ __forceinline__ float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    return static_cast<uint32_t>(f32_to_bf16_rne(a)) |
           (static_cast<uint32_t>(f32_to_bf16_rne(b)) << 16);
}

// Round-to-nearest-even of an fp64 value onto bf16 without double
// rounding: first round to fp32 with round-to-odd (truncate, then set the
// last bit if anything was dropped), which keeps the information a later
// round-to-nearest needs because fp32 carries 16 more bits than bf16; then
// round that fp32 value to bf16.  Any value, subnormal results included.
__device__ __forceinline__ uint16_t f64_to_bf16_rne(double x) {
    float f = __double2float_rz(x);
    if (static_cast<double>(f) != x && x == x) f = __uint_as_float(__float_as_uint(f) | 1u);
    return f32_to_bf16_rne(f);
}
// The same rounding of a value whose bf16 image is a normal number, on the
// high word of the double alone: the low word only matters as "not zero",
// half an ulp of bf16 is bit 12 of the high word, and a carry runs into the
// exponent field as it should.  Seven 32-bit operations instead of the
// conversions above, which run at a fraction of the rate.
__device__ __forceinline__ uint32_t f64_to_bf16_normal(uint32_t hi, uint32_t lo) {
    const uint32_t s = hi | (lo != 0u ? 1u : 0u);
    const uint32_t r = s + 0x0FFFu + ((hi >> 13) & 1u);
    return ((r - (896u << 20)) >> 13 & 0x7FFFu) | (hi >> 16 & 0x8000u);
}
// Two values rounded and packed (a in the low half).  Magnitudes in
// [2^-126, 2^127) take the short form; zeros, subnormal results, values at the
// top of the range, infinities and NaN the general one.
__device__ __forceinline__ uint32_t pack_bf16_from_f64(double a, double b) {
    const uint32_t ah = static_cast<uint32_t>(__double2hiint(a));
    const uint32_t bh = static_cast<uint32_t>(__double2hiint(b));
    uint32_t ra = f64_to_bf16_normal(ah, static_cast<uint32_t>(__double2loint(a)));
    uint32_t rb = f64_to_bf16_normal(bh, static_cast<uint32_t>(__double2loint(b)));
    // exponent fields 897 .. 1149: the images' exponents 1 .. 253
    const bool plain = ((ah & 0x7FFFFFFFu) - (897u << 20)) < (253u << 20) &&
                       ((bh & 0x7FFFFFFFu) - (897u << 20)) < (253u << 20);
    if (!plain) {
        ra = f64_to_bf16_rne(a);
        rb = f64_to_bf16_rne(b);
    }
    return ra | (rb << 16);
}

// Order-preserving map of fp32 onto uint32: a < b  <=>  key(a) < key(b).
__device__ __forceinline__ uint32_t f32_key(float f) {
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_f32(uint32_t k) {
    uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
    return __uint_as_float(u);
}

// ----------------------------------------------------------- wave helpers
__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Number of lanes below this one whose bit is set in `ballot`.
__device__ __forceinline__ int lanes_below(uint64_t ballot) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(ballot >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(ballot), 0));
}

__device__ __forceinline__ uint64_t wave_ballot(bool p) { return __ballot(p); }

// Butterfly sum over the 64 lanes; every lane receives the total.  The
// combination order is fixed, so the result is bit-reproducible.
// DPP lane moves (every source lane active): quad_perm [1,0,3,2] and
// [2,3,0,1], row_half_mirror and row_mirror inside each row of 16 lanes.
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(dpp_i<CTRL>(__float_as_int(v)));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;
__device__ __forceinline__ float readlane_f(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// The sum over the 64 lanes of a wave, the same value in every lane (every
// lane active): DPP moves add within each row of 16 lanes, then the four row
// sums are added in a fixed order.
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_f<kDppXor1>(v);
    v += dpp_f<kDppXor2>(v);
    v += dpp_f<kDppHalfMirror>(v);
    v += dpp_f<kDppMirror>(v);
    return (readlane_f(v, 0) + readlane_f(v, 16)) + (readlane_f(v, 32) + readlane_f(v, 48));
}

// Inclusive prefix sum over the lanes of a wave (every lane active), on the
// DPP row shifts and broadcasts described below.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_rows(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false);
}
// row_shr 1, 2, 4, 8 inside each row
// (a lane with no source adds 0), then row_bcast:15 adds row 0's total to
// row 1 and row 2's to row 3, and row_bcast:31 the total of rows 0-1 to
// rows 2 and 3
__device__ __forceinline__ int wave_incl_sum(int v) {
    v += dpp_rows<0x111, 0xF>(v);
    v += dpp_rows<0x112, 0xF>(v);
    v += dpp_rows<0x114, 0xF>(v);
    v += dpp_rows<0x118, 0xF>(v);
    v += dpp_rows<0x142, 0xA>(v);
    v += dpp_rows<0x143, 0xC>(v);
    return v;
}
__device__ __forceinline__ float logistic(float x) { return 1.0f / (1.0f + expf(-x)); }

}  // namespace xmix
