// Antialiased resize kernels for gfx950 (the filter stretched when shrinking).
//
//  k_gather_walk  (xr_gather_walk.hpp) one column per lane, the source rows
//                 staged in LDS and walked once per strip; rows shrinking or
//                 equal
//  k_tile_aa      a block's source window in LDS, filtered separably; the
//                 remaining shapes
//  k_gather_aa    one pixel per thread, every tap from memory
//
// All three evaluate a pixel with the same float32 operation sequence.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "xr_aa.hpp"
#include "xr_buffer.hpp"
#include "xr_device.hpp"
#include "xr_gather_walk.hpp"
#include "xr_internal.h"

namespace xr {
using namespace dev;

// ---------------------------------------------------------------------------
// k_gather_aa (antialiased: filter stretched by the shrink factor)
// ---------------------------------------------------------------------------

// One output pixel per thread in a block_w x block_h tile (the paper's
// tiling, eq. 6). The workgroup first fills LDS tables of taps and weights
// for its block_w columns and block_h rows (kx / ky weights each), then every
// thread sums its window: per source row the taps ascending (multiply, then
// FMAs), then the rows ascending.
template <int R, typename T, int C>
__global__ void __launch_bounds__(1024) k_gather_aa(ResizeArgs a, int32_t kx, int32_t ky)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int32_t bw = static_cast<int32_t>(blockDim.x), bh = static_cast<int32_t>(blockDim.y);
    int32_t *xlo = reinterpret_cast<int32_t *>(lds);
    int32_t *xn = xlo + bw;
    int32_t *ylo = xn + bw;
    int32_t *yn = ylo + bh;
    float *xw = reinterpret_cast<float *>(yn + bh);
    float *yw = xw + bw * kx;
    const int32_t tid = threadIdx.y * bw + threadIdx.x;
    for (int32_t t = tid; t < bw + bh; t += bw * bh) {
        if (t < bw) {
            const int32_t x = min(static_cast<int32_t>(blockIdx.x) * bw + t, a.out_w - 1);
            aa_table<R>(x, a.in_w, a.out_w, kx, xlo + t, xn + t, xw + t * kx);
        } else {
            const int32_t u = t - bw;
            const int32_t y = a.dst_row0 + min(static_cast<int32_t>(blockIdx.y) * bh + u, a.dst_rows - 1);
            aa_table<R>(y, a.in_h, a.out_h, ky, ylo + u, yn + u, yw + u * ky);
        }
    }
    __syncthreads();
    const int32_t px = blockIdx.x * bw + threadIdx.x;
    const int32_t py = blockIdx.y * bh + threadIdx.y;
    if (px >= a.out_w || py >= a.dst_rows)
        return;
    const unsigned char *src = a.src + static_cast<int64_t>(blockIdx.z) * a.src_plane_pitch;
    const int32_t x0 = xlo[threadIdx.x], nx = xn[threadIdx.x];
    const int32_t y0 = ylo[threadIdx.y], ny = yn[threadIdx.y];
    const float *wxr = xw + threadIdx.x * kx;
    const float *wyr = yw + threadIdx.y * ky;
    float acc[C];
    for (int32_t j = 0; j < ny; ++j) {
        const unsigned char *row = src + static_cast<int64_t>(y0 + j - a.src_row0) * a.src_pitch;
        float h[C], p[C];
        Pix<T, C>::load(row, x0, p);
        fma_first(h, wxr[0], p);
        for (int32_t i = 1; i < nx; ++i) {
            Pix<T, C>::load(row, x0 + i, p);
            fma_next(h, wxr[i], p);
        }
        if (j == 0)
            fma_first(acc, wyr[0], h);
        else
            fma_next(acc, wyr[j], h);
    }
    unsigned char *dst = a.dst + static_cast<int64_t>(blockIdx.z) * a.dst_plane_pitch +
                         static_cast<int64_t>(py) * a.dst_pitch;
    Pix<T, C>::store(dst, px, acc);
}

// ---------------------------------------------------------------------------
// k_tile_aa
// ---------------------------------------------------------------------------

// The antialiased filter on block_w x block_h tiles of output pixels with
// the source window staged in LDS (separable). A workgroup takes `tpb`
// vertically adjacent tiles of one tile column: the column tables (taps and
// kx weights per output column, the same as k_gather_aa's) are built once,
// the row tables once per tile. Per tile the source window (rows ylo(first)
// .. yhi(last), columns xlo(first) .. xhi(last)) is copied to LDS with
// coalesced loads, the horizontal pass filters every window row for every
// tile column into an LDS row buffer, and each thread then sums its rows. Per
// pixel the float32 sequence is exactly k_gather_aa's (taps ascending per
// row, rows ascending), so the two kernels agree bit for bit. The window is
// at most win_w x win_h pixels (bounded on the host from the scale).
constexpr int kAaRegTaps = 12;  // register-held horizontal weights (bicubic to 1/2.75)
constexpr int32_t kAaTilesPerBlock = 4;  // most tiles a workgroup walks down its column
constexpr int64_t kAaMinBlocks = 1024;    // workgroups the multi-tile grid keeps

template <int R, typename T, int C>
__global__ void __launch_bounds__(1024) k_tile_aa(ResizeArgs a, int32_t kx, int32_t ky, int32_t win_w,
                                                  int32_t win_h, int32_t tpb)
{
    constexpr int PB = Pix<T, C>::kBytes;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int32_t bw = static_cast<int32_t>(blockDim.x), bh = static_cast<int32_t>(blockDim.y);
    const int32_t nthreads = bw * bh;
    int32_t *xlo = reinterpret_cast<int32_t *>(lds);
    int32_t *xn = xlo + bw;
    int32_t *ylo = xn + bw;
    int32_t *yn = ylo + bh;
    float *xw = reinterpret_cast<float *>(yn + bh);
    float *yw = xw + bw * kx;
    const int64_t table_bytes = 4 * (2 * static_cast<int64_t>(bw) + 2 * bh +
                                     static_cast<int64_t>(bw) * kx + static_cast<int64_t>(bh) * ky);
    unsigned char *win = lds + (table_bytes + 15) / 16 * 16;
    float *hbuf = reinterpret_cast<float *>(win + (static_cast<int64_t>(win_w) * win_h * PB + 15) / 16 * 16);
    const int32_t tid = threadIdx.y * bw + threadIdx.x;
    const unsigned char *src = a.src + static_cast<int64_t>(blockIdx.z) * a.src_plane_pitch;
    const int32_t n_tiles_y = (a.dst_rows + bh - 1) / bh;
    const int32_t tile_end = min(static_cast<int32_t>(blockIdx.y + 1) * tpb, n_tiles_y);
    // Every bound below is uniform over the workgroup, and no thread leaves
    // the loop early, so every thread reaches every barrier.
    for (int32_t by = static_cast<int32_t>(blockIdx.y) * tpb; by < tile_end; ++by) {
        const bool first = by == static_cast<int32_t>(blockIdx.y) * tpb;
        for (int32_t t = tid + (first ? 0 : bw); t < bw + bh; t += nthreads) {
            if (t < bw) {
                const int32_t x = min(static_cast<int32_t>(blockIdx.x) * bw + t, a.out_w - 1);
                aa_table<R>(x, a.in_w, a.out_w, kx, xlo + t, xn + t, xw + t * kx);
            } else {
                const int32_t u = t - bw;
                const int32_t y = a.dst_row0 + min(by * bh + u, a.dst_rows - 1);
                aa_table<R>(y, a.in_h, a.out_h, ky, ylo + u, yn + u, yw + u * ky);
            }
        }
        __syncthreads();
        // the tile's source window (tap ranges are monotone in x and y)
        const int32_t wx0 = xlo[0];
        const int32_t ww = min(xlo[bw - 1] + xn[bw - 1] - wx0, win_w);
        const int32_t wy0 = ylo[0];
        const int32_t wh = min(ylo[bh - 1] + yn[bh - 1] - wy0, win_h);
        // NB loads in flight per thread before any LDS store. Element i of the
        // window is (i / ww, i % ww); a thread's elements step by nthreads,
        // i.e. by dr rows and dc columns with a carry, so no division per
        // element.
        constexpr int NB = 8;
        const int32_t total = ww * wh;
        const int32_t dr = nthreads / ww, dc = nthreads - dr * ww;
        int32_t r = tid / ww, c = tid - (tid / ww) * ww;
        const unsigned char *wsrc = src + static_cast<int64_t>(wy0 - a.src_row0) * a.src_pitch +
                                    static_cast<int64_t>(wx0) * PB;
        for (int32_t base = tid; base < total; base += nthreads * NB) {
            RawBuf<PB, PB> v[NB];
            int32_t off[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                // past the end: reload the window's last element (a valid address)
                const bool in = base + k * nthreads < total;
                const int32_t rr = in ? r : wh - 1, cc = in ? c : ww - 1;
                off[k] = (rr * win_w + cc) * PB;
                v[k] = load_raw<PB, PB>(wsrc + static_cast<int64_t>(rr) * a.src_pitch + cc * PB);
                c += dc;
                r += dr + (c >= ww ? 1 : 0);
                c -= c >= ww ? ww : 0;
            }
#pragma unroll
            for (int k = 0; k < NB; ++k)
                if (base + k * nthreads < total)
                    store_raw<PB, PB>(win + off[k], v[k]);
        }
        __syncthreads();
        // horizontal pass: window row r, tile column hc (threads of one
        // column take rows ty, ty + bh, ...). A column's weights are the same
        // on every row, so up to kAaRegTaps of them are held in registers.
        const int32_t hc = threadIdx.x;
        const int32_t hx0 = xlo[hc] - wx0, hnx = xn[hc];
        const float *hwx = xw + hc * kx;
        if (kx <= kAaRegTaps) {
            float wr[kAaRegTaps];
#pragma unroll
            for (int k = 0; k < kAaRegTaps; ++k)
                wr[k] = k < hnx ? hwx[k] : 0.0f;
            for (int32_t rr = threadIdx.y; rr < wh; rr += bh) {
                const unsigned char *wrow = win + static_cast<int64_t>(rr) * win_w * PB;
                float h[C], p[C];
                Pix<T, C>::load(wrow, hx0, p);
                fma_first(h, wr[0], p);
#pragma unroll
                for (int k = 1; k < kAaRegTaps; ++k) {
                    if (k < hnx) {
                        Pix<T, C>::load(wrow, hx0 + k, p);
                        fma_next(h, wr[k], p);
                    }
                }
                float *hp = hbuf + (static_cast<int64_t>(rr) * bw + hc) * C;
#pragma unroll
                for (int ch = 0; ch < C; ++ch)
                    hp[ch] = h[ch];
            }
        } else {
            for (int32_t rr = threadIdx.y; rr < wh; rr += bh) {
                const unsigned char *wrow = win + static_cast<int64_t>(rr) * win_w * PB;
                float h[C], p[C];
                Pix<T, C>::load(wrow, hx0, p);
                fma_first(h, hwx[0], p);
                for (int32_t k = 1; k < hnx; ++k) {
                    Pix<T, C>::load(wrow, hx0 + k, p);
                    fma_next(h, hwx[k], p);
                }
                float *hp = hbuf + (static_cast<int64_t>(rr) * bw + hc) * C;
#pragma unroll
                for (int ch = 0; ch < C; ++ch)
                    hp[ch] = h[ch];
            }
        }
        __syncthreads();
        const int32_t px = blockIdx.x * bw + threadIdx.x;
        const int32_t py = by * bh + threadIdx.y;
        if (px < a.out_w && py < a.dst_rows) {
            const int32_t r0 = ylo[threadIdx.y] - wy0, ny = yn[threadIdx.y];
            const float *wyr = yw + threadIdx.y * ky;
            float acc[C], h[C];
            for (int32_t j = 0; j < ny; ++j) {
                const float *hp = hbuf + (static_cast<int64_t>(r0 + j) * bw + threadIdx.x) * C;
#pragma unroll
                for (int ch = 0; ch < C; ++ch)
                    h[ch] = hp[ch];
                if (j == 0)
                    fma_first(acc, wyr[0], h);
                else
                    fma_next(acc, wyr[j], h);
            }
            unsigned char *dst = a.dst + static_cast<int64_t>(blockIdx.z) * a.dst_plane_pitch +
                                 static_cast<int64_t>(py) * a.dst_pitch;
            Pix<T, C>::store(dst, px, acc);
        }
        // the next tile rewrites the row tables, the window and the row buffer
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// k_gather_walk's policy
// ---------------------------------------------------------------------------

// The antialiased filters as a gather walk (rows shrinking or equal).
template <int R>
struct AaWalk {
    static constexpr int kSlots = 2 * R;  // |i - s_y| < R sigma, the s_y sigma apart
    static constexpr bool kFirstMul = true;
    static constexpr bool kRowRegs = true;
    __device__ __forceinline__ static int32_t result_w(const ResizeArgs &a) { return a.out_w; }
    __device__ __forceinline__ static int32_t result_rows(const ResizeArgs &a) { return a.dst_rows; }
    __device__ __forceinline__ static int32_t walked_w(const ResizeArgs &a) { return a.in_w; }
    __device__ __forceinline__ static int32_t stored_row(const ResizeArgs &a, int32_t r) { return r - a.src_row0; }
    __device__ __forceinline__ static void range_x(const ResizeArgs &a, int32_t x, int32_t &lo, int32_t &n)
    {
        int32_t hi;
        aa_range(x, a.in_w, a.out_w, R, lo, hi);
        n = hi - lo + 1;
    }
    __device__ __forceinline__ static void range_y(const ResizeArgs &a, int32_t y, int32_t &lo, int32_t &n)
    {
        int32_t hi;
        aa_range(a.dst_row0 + y, a.in_h, a.out_h, R, lo, hi);
        n = hi - lo + 1;
    }
    template <class W>
    __device__ __forceinline__ static void weights_x(const ResizeArgs &a, int32_t x, int32_t lo, int32_t n, W w)
    {
        aa_weights<R>(x, a.in_w, a.out_w, lo, n, w);
    }
    template <int N>
    __device__ __forceinline__ static void weights_x(const ResizeArgs &a, int32_t x, int32_t lo, int32_t n,
                                                     float (&w)[N])
    {
        aa_weights<R, N>(x, a.in_w, a.out_w, lo, n, w);
    }
    template <int N>
    __device__ __forceinline__ static void weights_y(const ResizeArgs &a, int32_t y, int32_t lo, int32_t n,
                                                     float (&w)[N])
    {
        aa_weights<R, N>(a.dst_row0 + y, a.in_h, a.out_h, lo, n, w);
    }
    template <class W>
    __device__ __forceinline__ static void weights_y(const ResizeArgs &a, int32_t y, int32_t lo, int32_t n, W w)
    {
        aa_weights<R>(a.dst_row0 + y, a.in_h, a.out_h, lo, n, w);
    }
};

namespace {
// Launch of the gather walk for an antialiased filter: false where it does
// not apply (rows growing, whose sample rows reach more result rows; pitches
// past 4 MiB; tables or windows too large for LDS) or too few strips make it
// the slower one.
template <int R, typename T, int C>
bool aa_walk_shape(const ResizeArgs &a, GatherShape &g)
{
    if (a.in_h < a.out_h || a.src_pitch > kStageMaxPitch)
        return false;
    const AaPlan p = aa_tile_plan(a.in_w, a.in_h, a.out_w, a.out_h, R, gather_cols(C), 1, Pix<T, C>::kBytes, C);
    const auto cap = [&](int64_t strip) {
        return std::min<int64_t>(((strip - 1) * a.in_h + 2 * R * static_cast<int64_t>(a.in_h)) / a.out_h + 2, a.in_h);
    };
    // a row of the table form costs as much for a few columns as for a
    // wavefront's (1024 bilinear planes 274 x 144 -> 27 x 14: 232 us so, 182 in
    // tiles; 512 bicubic planes 300 x 90 -> 60 x 30: 69 and 105)
    if (p.kx > kGatherRegTaps && a.out_w < 24)
        return false;
    // One-channel columns of several samples, two to a lane, need more results
    // than others to pay. The walk's speed over the tiles' at 280 / 340 / 420 / 520 /
    // 700 thousand of one image: bicubic x0.35 (12 samples, from the table) float32
    // 0.56 0.60 0.79 0.90 0.97, float16 0.60 0.65 0.86 0.98 1.06, uint8 0.82 0.88 1.16;
    // x0.25 (17) float32 0.71 0.72 0.97 1.08, float16 0.64 0.87 0.95 1.07, uint8 0.86
    // 0.97 1.29; x0.5 (9) float32 0.75 0.83 1.05, float16 0.84 0.92 1.11, uint8 1.15;
    // bilinear x0.25 (9) float32 0.75 0.99 1.06; bicubic x0.15 (27) 1.27 up. In a stack
    // of 24 planes bilinear 1.06 up. RGBA bicubic x0.7 and x0.9 of halves and floats
    // 0.87 to 0.95, 1.14 up.
    int64_t least = kGatherLeast;
    const int size = static_cast<int>(sizeof(T));
    const bool stack = a.planes >= 8;
    if (C == 1 && R == 2 && p.kx > kGatherRegTaps)
        least += p.kx > 20 ? 0 : size == 1 ? least / 2 : p.kx > 14 ? (size == 4 ? 3 * least / 4 : least / 2) : size == 4 ? 3 * least / 2 : 7 * least / 8;
    else if (C == 1 && R == 2)
        least += size == 1 ? 0 : least / 2;
    else if (C == 1)
        least += p.kx > 6 && p.kx <= kGatherRegTaps && size == 4 && !stack ? least / 4 : 0;
    else if (R == 2)
        least += p.kx <= 7 && size > 1 && !stack ? least / 5 : 0;
    const int64_t strip = gather_strip(C, a.out_w, a.dst_rows, a.planes, a.src_pitch, least, cap);
    return strip > 0 && gather_shape(g, C, AaWalk<R>::kSlots, p.kx, p.win_w, Pix<T, C>::kBytes, strip, cap);
}

template <int R, typename T, int C>
hipError_t launch_aa_typed(const ResizeArgs &a, const xr_tile &tile, hipStream_t stream, Route *only)
{
    const dim3 block(tile.block_w, tile.block_h, 1);
    const dim3 grid((a.out_w + tile.block_w - 1) / tile.block_w,
                    (a.dst_rows + tile.block_h - 1) / tile.block_h, a.planes);
    if (tile.kernel == XR_KERNEL_GATHER) {
        if (just_named(only, kRouteAaGather))
            return hipSuccess;
        const AaPlan plan = aa_plan(a.in_w, a.in_h, a.out_w, a.out_h, R, tile.block_w, tile.block_h);
        hipLaunchKernelGGL((k_gather_aa<R, T, C>), grid, block, plan.lds_bytes, stream, a, plan.kx, plan.ky);
        return hipGetLastError();
    }
    GatherShape g;
    if (aa_walk_shape<R, T, C>(a, g))
        return just_named(only, kRouteAaWalk) ? hipSuccess
                                              : launch_gather_walk<AaWalk<R>, T, C>(a, g, a.out_w, a.dst_rows, stream);
    if (just_named(only, kRouteAaTile))
        return hipSuccess;
    const AaPlan plan = aa_tile_plan(a.in_w, a.in_h, a.out_w, a.out_h, R, tile.block_w, tile.block_h,
                                     Pix<T, C>::kBytes, C);
    // tiles per workgroup down a tile column: the column tables are then
    // built once per tpb tiles, while the grid keeps kAaMinBlocks
    // workgroups
    const int64_t cols = static_cast<int64_t>(grid.x) * grid.z;
    int32_t tpb = 1;
    while (tpb < kAaTilesPerBlock && cols * ((grid.y + 2 * tpb - 1) / (2 * tpb)) >= kAaMinBlocks)
        tpb *= 2;
    const dim3 grid_t(grid.x, (grid.y + tpb - 1) / tpb, grid.z);
    hipLaunchKernelGGL((k_tile_aa<R, T, C>), grid_t, block, plan.lds_bytes, stream, a, plan.kx, plan.ky,
                       plan.win_w, plan.win_h, tpb);
    return hipGetLastError();
}

template <int R>
hipError_t launch_aa(const ResizeArgs &a, int32_t dtype, int32_t channels, const xr_tile &tile,
                     hipStream_t stream, Route *only)
{
    switch (dtype) {
    case XR_U8:
        return channels == 4 ? launch_aa_typed<R, uint8_t, 4>(a, tile, stream, only)
                             : launch_aa_typed<R, uint8_t, 1>(a, tile, stream, only);
    case XR_F16:
        return channels == 4 ? launch_aa_typed<R, _Float16, 4>(a, tile, stream, only)
                             : launch_aa_typed<R, _Float16, 1>(a, tile, stream, only);
    case XR_F32:
        return channels == 4 ? launch_aa_typed<R, float, 4>(a, tile, stream, only)
                             : launch_aa_typed<R, float, 1>(a, tile, stream, only);
    default:
        return hipErrorInvalidValue;
    }
}
}  // namespace

namespace {
template <int R, int C>
bool walk_supported(const ResizeArgs &a, int32_t dtype)
{
    GatherShape g;
    return dtype == XR_U8    ? aa_walk_shape<R, uint8_t, C>(a, g)
           : dtype == XR_F16 ? aa_walk_shape<R, _Float16, C>(a, g)
                             : aa_walk_shape<R, float, C>(a, g);
}
}  // namespace

bool antialiased_walk_supported(const ResizeArgs &a, int32_t filter, int32_t dtype, int32_t channels)
{
    if (filter == XR_BILINEAR_AA)
        return channels == 4 ? walk_supported<1, 4>(a, dtype) : walk_supported<1, 1>(a, dtype);
    return channels == 4 ? walk_supported<2, 4>(a, dtype) : walk_supported<2, 1>(a, dtype);
}

hipError_t launch_antialiased(const ResizeArgs &a, int32_t filter, int32_t dtype, int32_t channels,
                              const xr_tile &tile, hipStream_t stream, Route *only)
{
    return filter == XR_BILINEAR_AA ? launch_aa<1>(a, dtype, channels, tile, stream, only)
                                    : launch_aa<2>(a, dtype, channels, tile, stream, only);
}

}  // namespace xr
