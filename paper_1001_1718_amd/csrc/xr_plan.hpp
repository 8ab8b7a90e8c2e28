// Strip heights of the kernels that address a strip's rows by 32-bit offsets
// into a buffer resource (host arithmetic only, no HIP).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace xr {

// A resource spans less than 2 GiB: stores that a kernel drops go to offsets
// of 2^31 and more, which a longer one would hold.
constexpr int64_t kResourceBytes = int64_t(1) << 31;

// Output rows of a batched job's strip, for a tile of ppt_y rows: a strip
// walks about ppt_y source rows or ppt_y output rows, whichever is fewer output
// rows, so shrinking jobs do not make long tiles. Its source rows,
// (strip - 1) in_h / out_h + K + 1 at most, and its output rows stay below
// 2^31 bytes.
inline int32_t batch_strip(int32_t ppt_y, int32_t in_h, int32_t out_h, int64_t src_pitch, int64_t dst_pitch)
{
    int64_t strip = std::min<int64_t>(ppt_y, (static_cast<int64_t>(ppt_y) * out_h + in_h - 1) / in_h);
    strip = std::min(strip, (kResourceBytes / src_pitch - 6) * out_h / in_h);
    strip = std::min(strip, (kResourceBytes - 1) / dst_pitch);
    return static_cast<int32_t>(std::max<int64_t>(1, strip));
}

// Strips of the exact-ratio walks, in output row pairs (x2), output rows (x0.5)
// and source rows (the adjoint at x2) for a tile of ppt_y rows: whole steps of
// the kernel's loop, shortened until the strip's rows and the few around it
// stay well inside a resource; 0 where even the shortest strip does not (the
// general kernels then take the call). `pitch` is the longer of both images'.
inline int32_t exact_strip(int64_t least, int64_t strip, int64_t pitch)
{
    while (strip > least && (2 * strip + 8) * pitch >= kResourceBytes / 2)
        strip -= least;
    return (2 * strip + 8) * pitch < kResourceBytes ? static_cast<int32_t>(strip) : 0;
}
inline int32_t x2_pairs(int32_t ppt_y, int64_t pitch)
{
    return exact_strip(4, std::max<int64_t>(4, (static_cast<int64_t>(ppt_y) + 7) / 8 * 4), pitch);
}
inline int32_t x05_rows(int32_t ppt_y, int64_t pitch)
{
    return exact_strip(2, std::max<int64_t>(2, (static_cast<int64_t>(ppt_y) + 1) / 2 * 2), pitch);
}
inline int32_t bwd_x2_rows(int64_t pitch) { return exact_strip(4, 8, pitch); }

}  // namespace xr
