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

}  // namespace xr
