// Internal interface between the C-ABI layer (xr_api.cpp) and the kernels
// (xr_forward.hip, xr_backward.hip). Not installed; callers use include/xresize.h.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/xresize.h"

namespace xr {

// One resize job, resolved to byte addresses and validated on the host.
// `src` / `dst` point at the first stored row of plane 0.
struct ResizeArgs {
    const unsigned char *src;
    unsigned char *dst;
    int64_t src_pitch, src_plane_pitch;
    int64_t dst_pitch, dst_plane_pitch;
    int32_t in_w, in_h;      // full logical source size
    int32_t out_w, out_h;    // full logical destination size
    int32_t src_row0;        // logical row stored first in src
    int32_t src_rows;        // logical rows stored in src
    int32_t dst_row0;        // first logical output row to compute
    int32_t dst_rows;        // number of output rows to compute
    int32_t planes;
    int32_t aligned16;       // src, dst and pitches are 16-byte aligned
    int32_t map_off;         // 1: pixel-centre map; 0: the map eq. 1 prints
};

// Entry of the device job table of the batched launch.
struct BatchJob {
    ResizeArgs a;
    int32_t tiles_x;         // tiles per row of the output (per plane)
    int32_t tiles_y;         // tiles per column of the output (per plane)
    int64_t tile_begin;      // tiles of the jobs of the same kind before this one
    int32_t strip_h;         // output rows per thread strip of this job
    int32_t kind;            // launch of the job (kBatchKinds)
    int32_t kind_fc;         // 2 * (bicubic) + (four channels)
    int16_t waves_w;         // wavefronts of a workgroup that walk a tile of
    int16_t waves_h;         // this job: side by side, below one another
};

// Kinds of batched jobs; those of the kinds 0-3 share one launch. Kinds 0-3
// are 2 * (bicubic) + (four channels); kind 4 holds the jobs whose output is
// narrower than the staged walk's run or whose staged rows are too long.
constexpr int32_t kBatchKinds = 5;
constexpr int32_t kBatchNarrow = 4;

// Header of the batched workspace; jobs follow at offset kBatchHeaderBytes,
// grouped by kind.
struct BatchHeader {
    int32_t n_jobs;
    int32_t dtype;
    int32_t block_w;         // threads per workgroup along x
    int32_t block_h;         // thread rows per workgroup
    int32_t ppt_y;           // rows per thread strip (before per-job scaling)
    int32_t lds_bytes;       // LDS of a workgroup of the staged walk
    int32_t job_lo[kBatchKinds];    // jobs [job_lo, job_hi) are of kind k
    int32_t job_hi[kBatchKinds];
    int64_t tiles[kBatchKinds];     // tiles of kind k, a workgroup each
};
constexpr size_t kBatchHeaderBytes = 256;
static_assert(sizeof(BatchHeader) <= kBatchHeaderBytes, "batch header");

// Longest thread strip of the batched walk.
constexpr int32_t kBatchMaxStrip = 256;

// Output columns per thread of the staged walk, by channels and bytes per
// pixel: runs of 4 to 16 bytes, as many columns as the ring of filtered rows
// leaves registers for.
constexpr int32_t walk_ppx(int32_t channels, int32_t pixel_bytes)
{
    return channels == 1 ? 4 : pixel_bytes == 16 ? 1 : 2;
}
// Outputs of fewer runs (of 256 columns, 128 of RGBA, in one row) than this
// take the per-tap strips by default, which start without tables or staged rows.
// Measured, the walk's speed over theirs at 2200 / 2700 / 3300 / 4000 runs, over
// six ratios from 0.35 to 2.5: RGBA uint8 nearest 0.82 to 0.95, 0.90 to 1.00, 0.94 to
// 1.09, 1.01 to 1.17, float16 alike; float16 bilinear 0.86 to 1.05, 0.96 to 1.07;
// float16 bicubic below x2 0.81 to 0.95, 0.86 to 0.94, 0.92 to 1.02, 0.99 to 1.11, at
// x2.5 1.09 up; float32 bilinear at x1 to x1.25 0.85, 0.88, 0.94, 1.05 to 1.21, else
// 1.0 up; one-channel nearest of bytes and halves 0.90 to 1.21, 1.00 to 1.37; all
// others 0.92 (one) to 2.33, and 0.60 to 0.96 below their line.
inline int64_t walk_least_runs(int32_t filter, int32_t dtype, int32_t channels, int32_t in_w, int32_t out_w)
{
    const bool twice = out_w / 2 >= in_w;
    if (channels == 1)
        return filter == XR_NEAREST && dtype != XR_F32 ? 2600 : 1700;
    if (dtype == XR_F32)
        return filter == XR_BILINEAR && out_w >= in_w && !twice ? 3500 : 2100;
    if (filter == XR_NEAREST)
        return 3400;
    return dtype == XR_U8 ? 2100 : filter == XR_BILINEAR ? 2600 : twice ? 2100 : 3500;
}
inline bool walk_default(int32_t filter, int32_t dtype, int32_t channels, int32_t in_w, int32_t out_w, int64_t rows,
                         int64_t planes)
{
    const int64_t wide = channels == 4 ? 128 : 256;
    return (out_w + wide - 1) / wide * rows * planes >= walk_least_runs(filter, dtype, channels, in_w, out_w);
}
// In a batch, whose launches hold many tiles at a time, twice as many where a
// run stays within 16 bytes and registers allow (256 uneven uint8 images up to
// 2048^2: 8 columns of one channel and 4 bilinear RGBA ones 987 us, 4 and 2 998;
// 64 up to 700^2 58 and 56).
constexpr int32_t batch_ppx(int32_t filter, int32_t dtype, int32_t channels)
{
    if (dtype == XR_U8)
        return channels == 1 ? 8 : filter == XR_BILINEAR ? 4 : 2;
    return walk_ppx(channels, channels * (dtype == XR_F16 ? 2 : 4));
}

// Shape of an axis that a kernel can specialise on.
enum AxisMode : int32_t { kGeneral = 0, kUp2 = 1, kDown2 = 2 };

// The kernel that a call runs. The launches below take a Route to fill in: given
// one they only name the kernel, so tests can ask for it without a GPU.
enum Route : int32_t {
    kRouteGather = 1, kRouteStrip, kRouteWalk, kRouteX2, kRouteX05,
    kRouteAaGather, kRouteAaTile, kRouteAaWalk,
    kRouteBwdX2, kRouteBwdOwner, kRouteBwdWalk,
};
inline bool just_named(Route *only, Route r)
{
    if (only)
        *only = r;
    return only != nullptr;
}

hipError_t launch_forward(const ResizeArgs &a, int32_t filter, int32_t dtype, int32_t channels,
                          const xr_tile &tile, int32_t mode, hipStream_t stream, Route *only = nullptr);
hipError_t launch_antialiased(const ResizeArgs &a, int32_t filter, int32_t dtype, int32_t channels,
                              const xr_tile &tile, hipStream_t stream, Route *only);
// True when that launch of an LDS tile takes the gather walk, which needs no
// block of its own to fit.
bool antialiased_walk_supported(const ResizeArgs &a, int32_t filter, int32_t dtype, int32_t channels);
// The staged walk at any ratio (xr_walk.hip); `taken` stays false where it
// does not apply (staged rows too long for LDS, outputs narrower than a run,
// runs it is not built for, pitches past 4 MiB).
hipError_t launch_walk(const ResizeArgs &a, int32_t filter, int32_t dtype, int32_t channels, const xr_tile &tile,
                       hipStream_t stream, bool &taken, Route *only);
// True when the walk with its own columns per thread (walk_ppx) can stage its
// rows for an in_w -> out_w resize.
bool walk_fits(int32_t filter, int32_t dtype, int32_t channels, int32_t in_w, int32_t out_w);
// True when the walk is built for runs of ppx columns per thread.
bool walk_built(int32_t filter, int32_t dtype, int32_t channels, int32_t ppx);

// Launches of a prepared batch: workgroups per kind, LDS of those that walk.
struct BatchLaunch {
    int32_t block_w, block_h;
    int32_t grid[kBatchKinds];
    int32_t lds_bytes;
};
// The grid of `tiles` workgroups, in rows of at most 2^22 (a launch holds
// fewer than 2^32 threads along x).
inline dim3 batch_grid(int32_t tiles)
{
    const int32_t row = std::min<int32_t>(tiles, 1 << 22);
    return dim3(static_cast<uint32_t>(row), static_cast<uint32_t>((tiles + static_cast<int64_t>(row) - 1) / row));
}
// LDS of a wavefront that walks a job in strips of `strip` rows; ok = false
// where the staged walk does not apply.
struct BatchWalkNeed {
    int32_t win_bytes, wave_bytes;  // the staged rows; with the row table
    bool ok;
};
BatchWalkNeed batch_walk_need(const ResizeArgs &a, int32_t filter, int32_t dtype, int32_t channels, int32_t strip);
// The batched launches of a prepared workspace: the jobs that walk, and the others.
hipError_t launch_batched(const void *ws, int32_t dtype, const BatchLaunch &l, hipStream_t stream);
// Direct-to-LDS loads take the place of their data from the low 16 bits of M0:
// workgroups that stage rows stay within 64 KiB of LDS.
constexpr int64_t kStageMaxLds = 64 * 1024;
hipError_t launch_batch_narrow(const void *ws, int32_t dtype, dim3 block, int32_t grid, hipStream_t stream);
hipError_t launch_backward(const ResizeArgs &a, int32_t filter, int32_t dtype, int32_t channels,
                           hipStream_t stream, Route *only = nullptr);
// False when the adjoint's smallest LDS tile cannot hold the output rows of
// one source row and the column tables (upscales beyond roughly 190x rows or
// a few hundred x columns).
bool backward_supported(const ResizeArgs &a, int32_t filter, int32_t channels);

// Weight tables of the antialiased kernel: at most kx (ky) taps per output
// column (row), floor(2 R sigma) + 1 with sigma = max(1, n_in / n_out), and
// the LDS bytes of one workgroup's tables.
struct AaPlan {
    int32_t kx, ky;
    int64_t lds_bytes;
    int32_t win_w = 0, win_h = 0;  // source window of the LDS-tiled kernel
};
inline AaPlan aa_plan(int32_t in_w, int32_t in_h, int32_t out_w, int32_t out_h, int32_t r,
                      int32_t block_w, int32_t block_h)
{
    const auto taps = [r](int64_t n_in, int64_t n_out) {
        return static_cast<int32_t>((n_in > n_out ? (2 * r * n_in) / n_out : 2 * r) + 1);
    };
    AaPlan p;
    p.kx = taps(in_w, out_w);
    p.ky = taps(in_h, out_h);
    p.lds_bytes = 4 * (2 * static_cast<int64_t>(block_w) + 2 * block_h +
                       static_cast<int64_t>(block_w) * p.kx + static_cast<int64_t>(block_h) * p.ky);
    return p;
}
// gfx950 gives a workgroup up to 160 KiB of LDS; 96 KiB admits the taller
// blocks of the LDS-tiled kernel (bilinear x0.25: 64x8 blocks, 11% faster than
// the 16x16 that fits 64 KiB)
constexpr int64_t kAaLdsBudget = 96 * 1024;
// The LDS-tiled antialiased kernel adds the tile's source window (pixels of
// pb bytes) and one float32 row buffer per window row: a block of bw output
// columns reads at most floor(((bw - 1) n_in + 2 R max(n_in, n_out)) / n_out) + 2
// source columns (its first and last columns' tap ranges, eq. 1).
inline AaPlan aa_tile_plan(int32_t in_w, int32_t in_h, int32_t out_w, int32_t out_h, int32_t r,
                           int32_t block_w, int32_t block_h, int32_t pb, int32_t channels)
{
    AaPlan p = aa_plan(in_w, in_h, out_w, out_h, r, block_w, block_h);
    const auto span = [r](int64_t n, int64_t n_in, int64_t n_out) {
        return static_cast<int32_t>(((n - 1) * n_in + 2 * r * (n_in > n_out ? n_in : n_out)) / n_out + 2);
    };
    p.win_w = std::min<int32_t>(span(block_w, in_w, out_w), in_w);
    p.win_h = std::min<int32_t>(span(block_h, in_h, out_h), in_h);
    const int64_t tables = (p.lds_bytes + 15) / 16 * 16;
    const int64_t window = (static_cast<int64_t>(p.win_w) * p.win_h * pb + 15) / 16 * 16;
    const int64_t rows = static_cast<int64_t>(p.win_h) * block_w * channels * 4;
    p.lds_bytes = tables + window + rows;
    return p;
}

// Pixels per thread along x that the strip kernel is instantiated for.
bool strip_ppx_supported(int32_t dtype, int32_t channels, int32_t ppx);

}  // namespace xr
