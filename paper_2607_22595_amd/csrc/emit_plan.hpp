// Candidate emission parameters (host code): how many values a tile of a
// dictionary is asked for, and with which first threshold.
#pragma once

#include <math.h>
#include <stdint.h>

namespace xmix {

constexpr int kMaxCap = 64;  // most candidate pairs one tile may emit

// For a dictionary of m latents in tiles of `width`, and top-k: the per-tile
// capacity, the lower count bound, and the standard normal quantile of the first
// threshold guess.
struct EmitPlan {
    int cap, lo;
    float z;
};

// Pairs one tile may emit: four times a target of twice the tile's share of
// the k winners, plus one.
inline int emit_cap(int32_t m, int32_t k, int32_t width) {
    const int t = (2 * k * width + m - 1) / m + 1;
    const int cap = 4 * (t < 2 ? 2 : t);
    return cap < kMaxCap ? cap : kMaxCap;
}

// 0.5 * erfc(z / sqrt 2): the share of a standard normal above z
inline double upper_tail(double z) { return 0.5 * erfc(z / sqrt(2.0)); }

// z with f(z) = want for an f that falls with z, by bisection
template <typename F>
inline double falling_root(F f, double want) {
    double a = -8.0, b = 8.0;
    for (int i = 0; i < 40; ++i) {
        const double mid = 0.5 * (a + b);
        if (f(mid) > want) a = mid;
        else b = mid;
    }
    return 0.5 * (a + b);
}

// The guess mean + z * stdev comes from the tile's own values, so of 256 of
// them it is off by about sqrt(1/256 + z^2/512) stdev.  A tile whose guess ends up
// above the token's k-th value hides a winner and sends the token to the
// repair (50 us of one workgroup), so the guess is aimed five such errors
// below the k-th value's quantile, and at two values a tile or more.  Measured:
// 391 tokens, m = 32768, k = 64 (repairs in most launches when it was aimed at 2 a
// tile) merge 62 -> 9 us; 1777 tokens of width 2304, m = 16384, k = 64 prefill GEMM
// 240 -> 146 us (every tile was searched for exactly 12 values).
//
// A lower bound on the count is set only where the tiles together might not
// supply k values, their total less than four Poisson deviations above k: a tile
// that misses it searches, a prefill tile until its last token has settled, while
// a short total is rare and costs one token a repair.  The bound is the tile's
// share of the k, or a quarter of the capacity (a tile whose guess lies too high
// hides winners), so that it leaves a wide window below the capacity.  With the
// bound at k (8 of 8 here) and set from six deviations, a prefill encode of 8192
// tokens of width 2048, m = 5120, k = 8 took 347 us and takes 235; m = 512,
// k = 64, d = 768: 171 and 129.
inline EmitPlan emit_plan(int32_t m, int32_t k, int32_t width) {
    const int n = m / width;
    EmitPlan e;
    e.cap = emit_cap(m, k, width);
    const double share = static_cast<double>(k) / m;  // k <= 64 of 256 or more
    const double zk = falling_root(upper_tail, share);
    const double z = falling_root(
        [width](double q) { return -(q + 5.0 * sqrt((1.0 + 0.5 * q * q) / width)); }, -zk);
    double target = width * upper_tail(z);
    // room for the counts' own spread below the capacity
    const double most = e.cap < kMaxCap ? e.cap - 1.8 * sqrt(e.cap) : 45.0;
    target = target < most ? target : most;
    target = target < 2.0 ? 2.0 : target;
    const double total = n * target;
    const int part = (k + n - 1) / n, quarter = e.cap / 4;
    const int lo = part > quarter ? part : quarter;
    e.lo = total - k >= 4.0 * sqrt(total) ? 0 : lo < k ? lo : k;
    const double want = e.lo ? 0.5 * (e.lo + e.cap) : target;
    e.z = static_cast<float>(falling_root(upper_tail, want / width));
    return e;
}

}  // namespace xmix
