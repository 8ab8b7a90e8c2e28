// Taps and weights of the antialiased filters, shared by their kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xr_device.hpp"

namespace xr {
namespace dev {

// Taps of output index x for an antialiased filter of radius R (1 bilinear,
// 2 Keys): sigma = max(1, n_in / n_out), every source i with
// s - R sigma < i <= s + R sigma inside [0, n_in - 1], from exact integers
// (s = num / (2 n_out), num = (2x + 1) n_in - n_out). Not in the paper: the
// usual remedy for aliasing when shrinking.
// All in unsigned 32 bits: (2x + 1) n_in <= 2^31 for sides up to 32768.
__device__ __forceinline__ void aa_range(int32_t x, int32_t n_in, int32_t n_out, int32_t r,
                                         int32_t &lo, int32_t &hi)
{
    const uint32_t a = (2u * static_cast<uint32_t>(x) + 1u) * static_cast<uint32_t>(n_in);
    const uint32_t den = 2u * static_cast<uint32_t>(n_out);
    const uint32_t reach = 2u * static_cast<uint32_t>(r) * static_cast<uint32_t>(n_in > n_out ? n_in : n_out);
    const uint32_t b = static_cast<uint32_t>(n_out) + reach;
    lo = a >= b ? static_cast<int32_t>((a - b) / den) + 1 : 0;
    hi = min(static_cast<int32_t>((a + (reach - static_cast<uint32_t>(n_out))) / den), n_in - 1);
}

// K(d) in factored forms whose factors do not cancel: 1 - u; Keys a = -1/2
// as (1 - u)(1 + u (1 - 3u/2)) for u <= 1 and -(u - 1)(u - 2)^2 / 2 for
// 1 < u < 2 (u - 1 and u - 2 are exact there).
template <int R>
__device__ __forceinline__ float aa_kernel(float d)
{
    const float u = fabsf(d);
    if constexpr (R == 1) {
        return u < 1.0f ? 1.0f - u : 0.0f;
    } else {
        if (u <= 1.0f)
            return (1.0f - u) * (1.0f + u * (1.0f - 1.5f * u));
        if (u < 2.0f) {
            const float v = u - 2.0f;
            return (-0.5f * (u - 1.0f)) * (v * v);
        }
        return 0.0f;
    }
}

// Normalised weights of the n taps lo .. lo + n - 1 of output index x: the
// kernel values K((i - s) / sigma), then each divided by their sum (summed in
// ascending i); w(k) is the place of weight k.
template <int R, class W>
__device__ __forceinline__ void aa_weights(int32_t x, int32_t n_in, int32_t n_out, int32_t lo, int32_t n, W w)
{
    // (i - s) / sigma = (2 i n_out - num) / (2 max(n_in, n_out)) from exact
    // integers: one rounding, no cancellation (the difference is at most
    // 2 R max(n_in, n_out), so 32 bits that wrap hold it; div_rcp equals the
    // IEEE quotient for every |a| <= 2 b and even b up to 65536, checked
    // exhaustively on the host)
    const uint32_t num = (2u * static_cast<uint32_t>(x) + 1u) * static_cast<uint32_t>(n_in) -
                         static_cast<uint32_t>(n_out);
    const float den = static_cast<float>(2 * (n_in > n_out ? n_in : n_out));
    const float rcp = __fdiv_rn(1.0f, den);
    uint32_t dn = 2u * static_cast<uint32_t>(lo) * static_cast<uint32_t>(n_out) - num;
    float sum = 0.0f;
    for (int32_t k = 0; k < n; ++k) {
        const float v = aa_kernel<R>(div_rcp(static_cast<float>(static_cast<int32_t>(dn)), den, rcp));
        w(k) = v;
        sum += v;
        dn += 2u * static_cast<uint32_t>(n_out);
    }
    const float inv = 1.0f / sum;
    for (int32_t k = 0; k < n; ++k)
        w(k) *= inv;
}

// The same in registers, for n <= N; zero past the n taps.
template <int R, int N>
__device__ __forceinline__ void aa_weights(int32_t x, int32_t n_in, int32_t n_out, int32_t lo, int32_t n,
                                           float (&w)[N])
{
    const uint32_t num = (2u * static_cast<uint32_t>(x) + 1u) * static_cast<uint32_t>(n_in) -
                         static_cast<uint32_t>(n_out);
    const float den = static_cast<float>(2 * (n_in > n_out ? n_in : n_out));
    const float rcp = __fdiv_rn(1.0f, den);
    uint32_t dn = 2u * static_cast<uint32_t>(lo) * static_cast<uint32_t>(n_out) - num;
    float sum = 0.0f;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const float v = aa_kernel<R>(div_rcp(static_cast<float>(static_cast<int32_t>(dn)), den, rcp));
        w[k] = k < n ? v : 0.0f;
        sum += w[k];
        dn += 2u * static_cast<uint32_t>(n_out);
    }
    const float inv = 1.0f / sum;
#pragma unroll
    for (int k = 0; k < N; ++k)
        w[k] *= inv;
}

// First tap, number of taps (at most kmax) and weights into an LDS table.
template <int R>
__device__ __forceinline__ void aa_table(int32_t x, int32_t n_in, int32_t n_out, int32_t kmax,
                                         int32_t *lo_out, int32_t *n_out_taps, float *w)
{
    int32_t lo, hi;
    aa_range(x, n_in, n_out, R, lo, hi);
    const int32_t n = min(hi - lo + 1, kmax);
    aa_weights<R>(x, n_in, n_out, lo, n, [w](int32_t k) -> float & { return w[k]; });
    *lo_out = lo;
    *n_out_taps = n;
}

}  // namespace dev
}  // namespace xr
