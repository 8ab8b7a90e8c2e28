// Forward resize kernels for gfx950.
//
//  k_gather     one thread per output pixel; a workgroup of block_w x block_h
//               threads covers a block_w x block_h tile (paper section III.A,
//               eq. 6). Every tap is read from memory. Kept as the paper's
//               own tiling, for the tile-shape study and as a reference
//               launch shape.
//  k_strip      each thread owns ppt_x adjacent output columns and walks a
//               strip of ppt_y output rows. The horizontally filtered source
//               rows (the inner sums of eq. 5) are kept in a ring of K
//               registers and reused by every output row that needs them, so
//               a source row is filtered once per strip instead of K times.
//  k_x2         the walk specialised for an exact x2 upscale on both axes:
//               output columns/rows alternate between t = 3/4 and t = 1/4, a
//               thread's ppt_x columns read one contiguous run of ppt_x/2 + K
//               source pixels, every source row completes a pair of output
//               rows, and every memory access goes through a buffer resource
//               so no branch separates the walk's loads and stores.
//  k_x05        the walk for an exact x0.5 on both axes: t = 1/2
//               everywhere, a contiguous run of 2 ppt_x - 2 + K source
//               pixels per row, two source rows per output row, with the
//               buffer-resource loads and stores of k_x2.
//  k_batch_narrow the batched jobs that the staged walk leaves.
//
// Other ratios run the staged walk (xr_walk.hip), antialiased filters the
// kernels of xr_aa.hip. The bilinear and bicubic kernels evaluate each output
// with the same float32 operation sequence (xr_device.hpp), so their results
// are bit-identical.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "xr_buffer.hpp"
#include "xr_device.hpp"
#include "xr_internal.h"
#include "xr_plan.hpp"

namespace xr {
using namespace dev;

// ---------------------------------------------------------------------------
// helpers: contiguous runs of pixels
// ---------------------------------------------------------------------------

// Storage type code of a pixel type.
template <typename T>
struct DType;
template <>
struct DType<uint8_t> {
    static constexpr int32_t kCode = XR_U8;
};
template <>
struct DType<_Float16> {
    static constexpr int32_t kCode = XR_F16;
};
template <>
struct DType<float> {
    static constexpr int32_t kCode = XR_F32;
};

template <typename T, int C>
struct PixRaw {
    static constexpr int kBytes = Pix<T, C>::kBytes;
};

// Decode pixel `i` of a byte buffer into floats.
template <typename T, int C>
__device__ __forceinline__ void decode(const unsigned char *buf, int i, float (&v)[C])
{
    Pix<T, C>::load(buf, i, v);
}


// Store of an output run that is written once and not read back by this
// launch: non-temporal vector stores (they do not keep the lines in the
// caches, which leaves room there for the source rows that neighbouring
// strips re-read; measured faster for the x2 walk).
template <int BYTES, int ALIGN>
__device__ __forceinline__ void store_stream(unsigned char *p, const RawBuf<BYTES, ALIGN> &v)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    if constexpr (ALIGN >= 16 && BYTES % 16 == 0) {
#pragma unroll
        for (int i = 0; i < BYTES / 16; ++i)
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(v.b + 16 * i),
                                        reinterpret_cast<u32x4 *>(__builtin_assume_aligned(p, 16)) + i);
    } else if constexpr (ALIGN >= 8 && BYTES % 8 == 0) {
#pragma unroll
        for (int i = 0; i < BYTES / 8; ++i)
            __builtin_nontemporal_store(*reinterpret_cast<const u32x2 *>(v.b + 8 * i),
                                        reinterpret_cast<u32x2 *>(__builtin_assume_aligned(p, 8)) + i);
    } else if constexpr (ALIGN >= 4 && BYTES % 4 == 0) {
#pragma unroll
        for (int i = 0; i < BYTES / 4; ++i)
            __builtin_nontemporal_store(*reinterpret_cast<const uint32_t *>(v.b + 4 * i),
                                        reinterpret_cast<uint32_t *>(__builtin_assume_aligned(p, 4)) + i);
    } else {
        store_raw<BYTES, ALIGN>(p, v);
    }
}


// ---------------------------------------------------------------------------
// k_gather
// ---------------------------------------------------------------------------

template <int FILTER, typename T, int C>
__global__ void __launch_bounds__(1024) k_gather(ResizeArgs a)
{
    using TP = Taps<FILTER>;
    constexpr int K = TP::K;
    const int32_t px = blockIdx.x * blockDim.x + threadIdx.x;  // eq. 6
    const int32_t py = blockIdx.y * blockDim.y + threadIdx.y;
    if (px >= a.out_w || py >= a.dst_rows)
        return;
    const int32_t plane = blockIdx.z;
    int32_t x0, y0;
    float tx, ty, ux, uy;
    source_tap<FILTER>(px, a.in_w, a.out_w, a.map_off, x0, tx, ux);
    source_tap<FILTER>(a.dst_row0 + py, a.in_h, a.out_h, a.map_off, y0, ty, uy);
    float wx[K], wy[K];
    weights<FILTER>(tx, ux, wx);
    weights<FILTER>(ty, uy, wy);
    int32_t ix[K];
#pragma unroll
    for (int i = 0; i < K; ++i)
        ix[i] = clampi(x0 + TP::LO + i, 0, a.in_w - 1);
    const unsigned char *src = a.src + static_cast<int64_t>(plane) * a.src_plane_pitch;
    float acc[C];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const int32_t r = clampi(y0 + TP::LO + j, 0, a.in_h - 1) - a.src_row0;
        const unsigned char *row = src + static_cast<int64_t>(r) * a.src_pitch;
        float h[C], p[C];
        Pix<T, C>::load(row, ix[0], p);
        fma_first(h, wx[0], p);
#pragma unroll
        for (int i = 1; i < K; ++i) {
            Pix<T, C>::load(row, ix[i], p);
            fma_next(h, wx[i], p);
        }
        if (j == 0)
            fma_first(acc, wy[0], h);
        else
            fma_next(acc, wy[j], h);
    }
    unsigned char *dst = a.dst + static_cast<int64_t>(plane) * a.dst_plane_pitch +
                         static_cast<int64_t>(py) * a.dst_pitch;
    Pix<T, C>::store(dst, px, acc);
}

// ---------------------------------------------------------------------------
// k_strip (any scale)
// ---------------------------------------------------------------------------

// Copy one pixel of PB bytes between PB-aligned addresses.
template <int PB>
__device__ __forceinline__ void copy_pixel(unsigned char *dst, const unsigned char *src)
{
    if constexpr (PB == 1) {
        *dst = *src;
    } else if constexpr (PB == 2) {
        *reinterpret_cast<uint16_t *>(dst) = *reinterpret_cast<const uint16_t *>(src);
    } else if constexpr (PB == 4) {
        *reinterpret_cast<uint32_t *>(dst) = *reinterpret_cast<const uint32_t *>(src);
    } else if constexpr (PB == 8) {
        *reinterpret_cast<uint2 *>(dst) = *reinterpret_cast<const uint2 *>(src);
    } else {
        *reinterpret_cast<uint4 *>(dst) = *reinterpret_cast<const uint4 *>(src);
    }
}

// Any scale: a thread owns PPX adjacent output columns (each with its own
// taps) and walks the source rows its strip of output rows reads, in order.
// Each source row is filtered once into ring slot (row - first row) mod K;
// an output row is emitted as soon as its last tap row has been filtered,
// reading its K rows from slots that are constants of the 4-row unrolled
// walk. The PPX*K tap pixels of the row PD rows ahead are requested before
// the current row is filtered.
template <int FILTER, typename T, int C, int PPX>
struct StripBody {
    using TP = Taps<FILTER>;
    static constexpr int K = TP::K;
    static constexpr int PB = Pix<T, C>::kBytes;
    static constexpr int ROWB = PPX * K * PB;       // tap bytes per source row
    static constexpr int PD = ROWB <= 32 ? 3 : 1;   // prefetch distance in rows
    static constexpr int Q = PD + 1;                // divides 4
    using Raw = RawBuf<ROWB, PB>;

    int32_t ixb[PPX][K];  // byte offsets of the clamped tap columns
    float wx[PPX][K];
    float ring[K][PPX][C];
    Raw rawq[Q];

    __device__ __forceinline__ Raw load_row(const ResizeArgs &a, const unsigned char *src,
                                            int32_t r) const
    {
        // clamped into the stored band (which holds every needed row)
        const int32_t rr = clampi(r, a.src_row0, a.src_row0 + a.src_rows - 1) - a.src_row0;
        const unsigned char *row = src + static_cast<int64_t>(rr) * a.src_pitch;
        Raw raw;
#pragma unroll
        for (int c = 0; c < PPX; ++c)
#pragma unroll
            for (int i = 0; i < K; ++i)
                copy_pixel<PB>(raw.b + (c * K + i) * PB, row + ixb[c][i]);
        return raw;
    }

    __device__ __forceinline__ void hfilter(const Raw &raw, float (&out)[PPX][C]) const
    {
#pragma unroll
        for (int c = 0; c < PPX; ++c) {
            float p[C];
            decode<T, C>(raw.b, c * K, p);
            fma_first(out[c], wx[c][0], p);
#pragma unroll
            for (int i = 1; i < K; ++i) {
                decode<T, C>(raw.b, c * K + i, p);
                fma_next(out[c], wx[c][i], p);
            }
        }
    }

    // Process output rows [r_begin, r_end) (band coordinates) of one plane for
    // the PPX columns starting at col0.
    __device__ __forceinline__ void run(const ResizeArgs &a, int32_t plane, int32_t col0,
                                        int32_t r_begin, int32_t r_end)
    {
#pragma unroll
        for (int c = 0; c < PPX; ++c) {
            const int32_t x = min(col0 + c, a.out_w - 1);
            int32_t x0;
            float t, u;
            source_tap<FILTER>(x, a.in_w, a.out_w, a.map_off, x0, t, u);
            weights<FILTER>(t, u, wx[c]);
#pragma unroll
            for (int i = 0; i < K; ++i)
                ixb[c][i] = clampi(x0 + TP::LO + i, 0, a.in_w - 1) * PB;
        }
        const unsigned char *src = a.src + static_cast<int64_t>(plane) * a.src_plane_pitch;
        unsigned char *dst = a.dst + static_cast<int64_t>(plane) * a.dst_plane_pitch;
        const int32_t ncols = min(PPX, a.out_w - col0);
        // the whole run of PPX pixels is inside the row and aligned for one
        // vector store (PPX * PB bytes at a multiple of that size)
        const bool full_run = ncols == PPX && a.aligned16;

        int32_t y = a.dst_row0 + r_begin;  // next output row to emit (logical)
        const int32_t y_end = a.dst_row0 + r_end;
        int32_t y0, y0_last;
        float ty, uy, tl, ul;
        // one division per strip: the rows' taps use its reciprocal
        const float rcp_h = __fdiv_rn(1.0f, static_cast<float>(2 * a.out_h));
        source_tap_rcp<FILTER>(y, a.in_h, a.out_h, a.map_off, rcp_h, y0, ty, uy);
        source_tap_rcp<FILTER>(y_end - 1, a.in_h, a.out_h, a.map_off, rcp_h, y0_last, tl, ul);
        float wy[K];
        weights<FILTER>(ty, uy, wy);
        int32_t last = y0 + TP::LO + K - 1;  // last tap row of output y
        const int32_t rho0 = y0 + TP::LO;
        const int32_t rho1 = y0_last + TP::LO + K - 1;

        // emit every output row whose last tap row is rho (ring slot I of rho)
        auto emit_all = [&](auto slot_tag, int32_t rho) {
            constexpr int I = decltype(slot_tag)::value;
            while (y < y_end && last == rho) {
                unsigned char *drow = dst + static_cast<int64_t>(y - a.dst_row0) * a.dst_pitch;
                float v[PPX][C];
#pragma unroll
                for (int c = 0; c < PPX; ++c) {
                    fma_first(v[c], wy[0], ring[(I + 1) % K][c]);
#pragma unroll
                    for (int j = 1; j < K; ++j)
                        fma_next(v[c], wy[j], ring[(I + 1 + j) % K][c]);
                }
                if (full_run) {
                    RawBuf<PPX * PB, cmin(16, PPX * PB)> out;
                    encode_run<T, C, PPX>(v, out);
                    store_stream<PPX * PB, cmin(16, PPX * PB)>(drow + static_cast<int64_t>(col0) * PB, out);
                } else {
#pragma unroll
                    for (int c = 0; c < PPX; ++c)
                        if (c < ncols)
                            Pix<T, C>::store(drow, col0 + c, v[c]);
                }
                ++y;
                if (y < y_end) {
                    source_tap_rcp<FILTER>(y, a.in_h, a.out_h, a.map_off, rcp_h, y0, ty, uy);
                    weights<FILTER>(ty, uy, wy);
                    last = y0 + TP::LO + K - 1;
                }
            }
        };
        // Requests past the last needed row re-read that row (a cache hit)
        // instead of fetching rows this strip never uses.
        auto step = [&](auto slot_tag, int32_t rho) {
            constexpr int I = decltype(slot_tag)::value;
            rawq[(I + PD) % Q] = load_row(a, src, min(rho + PD, rho1));
            if (rho <= rho1) {
                hfilter(rawq[I % Q], ring[I % K]);
                emit_all(slot_tag, rho);
            }
        };
#pragma unroll
        for (int i = 0; i < PD; ++i)
            rawq[i % Q] = load_row(a, src, min(rho0 + i, rho1));
        for (int32_t rho = rho0; rho <= rho1; rho += 4) {
            step(std::integral_constant<int, 0>{}, rho);
            step(std::integral_constant<int, 1>{}, rho + 1);
            step(std::integral_constant<int, 2>{}, rho + 2);
            step(std::integral_constant<int, 3>{}, rho + 3);
        }
    }
};

// Row strip of a thread: threadIdx.y selects one of blockDim.y strips stacked
// vertically in the tile. blockDim.x is a multiple of the wavefront size, so
// the strip is uniform across a wavefront.
__device__ __forceinline__ int32_t strip_begin(int32_t by, int32_t strip_h)
{
    return __builtin_amdgcn_readfirstlane((by * static_cast<int32_t>(blockDim.y) + threadIdx.y) * strip_h);
}

template <int FILTER, typename T, int C, int PPX>
__global__ void __launch_bounds__(512) k_strip(ResizeArgs a, int32_t strip_h, int32_t order)
{
    int32_t bx, by;
    tile_coords(order, bx, by);
    const int32_t col0 = (bx * static_cast<int32_t>(blockDim.x) + threadIdx.x) * PPX;
    const int32_t r_begin = strip_begin(by, strip_h);
    if (col0 >= a.out_w || r_begin >= a.dst_rows)
        return;
    const int32_t r_end = min(r_begin + strip_h, a.dst_rows);
    StripBody<FILTER, T, C, PPX> body;
    body.run(a, blockIdx.z, col0, r_begin, r_end);
}

// ---------------------------------------------------------------------------
// edge runs of the exact-ratio walks
// ---------------------------------------------------------------------------
//
// A thread at the image's left or right edge loads its run of N pixels
// (pixels of a multiple of 4 bytes) from column ld0, clamped so the load stays
// inside the row (0 for images narrower than the run). Pixel s of the run
// must be column clamp(run0 + s, 0, in_w - 1): first every loaded pixel past
// the last column repeats its left neighbour, then the window moves right by
// ld0 - run0 pixels (at most MAXL) repeating its first pixel, or left by
// run0 - ld0 (at most MAXR) repeating its last. Lane values only select,
// never index, so the rebuild stays in registers.
template <int N, int PB, int MAXL, int MAXR, int LBYTES>
__device__ __forceinline__ RawBuf<LBYTES, 4> clamp_window(const RawBuf<LBYTES, 4> &in, int32_t run0,
                                                         int32_t ld0, int32_t in_w)
{
    static_assert(PB % 4 == 0 && N * PB <= LBYTES, "whole-dword pixels");
    constexpr int DW = PB / 4;
    uint32_t w[N][DW];
    __builtin_memcpy(w, in.b, N * PB);
    const int32_t last = in_w - 1 - ld0;
#pragma unroll
    for (int t = 1; t < N; ++t)
#pragma unroll
        for (int d = 0; d < DW; ++d)
            w[t][d] = t > last ? w[t - 1][d] : w[t][d];
    const int32_t sh = run0 - ld0;
#pragma unroll
    for (int step = 0; step < MAXL; ++step) {
        const bool go = step < -sh;
#pragma unroll
        for (int t = N - 1; t > 0; --t)
#pragma unroll
            for (int d = 0; d < DW; ++d)
                w[t][d] = go ? w[t - 1][d] : w[t][d];
    }
#pragma unroll
    for (int step = 0; step < MAXR; ++step) {
        const bool go = step < sh;
#pragma unroll
        for (int t = 0; t + 1 < N; ++t)
#pragma unroll
            for (int d = 0; d < DW; ++d)
                w[t][d] = go ? w[t + 1][d] : w[t][d];
    }
    RawBuf<LBYTES, 4> out = in;
    __builtin_memcpy(out.b, w, N * PB);
    return out;
}

// ---------------------------------------------------------------------------
// k_x2 (exact x2 upscale on both axes)
// ---------------------------------------------------------------------------
//
// Output rows pair up as (2m+1, 2m+2): both tap the K source rows
// m+LO .. m+LO+K-1, with t = 1/4 and t = 3/4 (s(y) = (2y - 1)/4). A strip of
// np pairs (np a multiple of 4) filters np + K - 1 source rows, the first
// K - 1 before its first pair, and emits both rows of every pair. A thread
// owns PPX output columns (PPX/2 source columns plus the K/2 taps on either
// side: a run of SPAN source pixels per row).
//
// Every load and store is issued on every step, so the compiler's counts of
// memory operations in flight are exact and each wait covers only the row it
// needs (loads run PD rows ahead):
// * source rows are clamped to the image and the stored band;
// * output rows outside the caller's band fall outside the store resource
//   and are dropped;
// * a thread whose run crosses the left or right image edge loads the run
//   clamped into the row and rebuilds the edge-replicated pixels in
//   registers (pixels of 4 bytes or more), or loads each pixel from its
//   clamped column (1- and 2-byte pixels);
// * a thread whose output run crosses the right image edge has its run store
//   dropped (offset moved past the resource) and stores its pixels one by
//   one.
// The output stores stream past the L2 (kStoreStream). The float32 operation
// order per pixel is the one every kernel uses.
template <int FILTER, typename T, int C, int PPX, int PD>
struct X2Walk {
    using TP = Taps<FILTER>;
    static constexpr int K = TP::K;
    static constexpr int LO = TP::LO;
    static constexpr int M = PPX / 2;
    static constexpr int SPAN = M + K;
    static constexpr int PB = Pix<T, C>::kBytes;
    // a run starts at source column M t - K/2; loads start MIS bytes lower so
    // that they begin on a dword (the same MIS for every interior thread)
    static_assert((M * PB) % 4 == 0, "a thread's run must advance by whole dwords");
    static constexpr int MIS = (4 - ((K / 2) * PB) % 4) % 4;
    static constexpr int LB = (MIS + SPAN * PB + 3) / 4 * 4;  // bytes loaded per row
    static constexpr int OB = PPX * PB;                         // bytes stored per row
    static constexpr int Q = PD + 1;
    static_assert(4 % K == 0 && 4 % Q == 0, "slots repeat every 4 rows");
    using Raw = RawBuf<LB, 4>;

    __amdgpu_buffer_rsrc_t srsrc;
    int32_t row_first;   // logical source row of window row 0 of the strip
    int32_t row_lo, row_hi;  // clamp range (row_lo: the source resource's first row)
    int64_t src_pitch, dst_pitch;
    uint32_t lane_src;   // byte offset of this thread's load within a row (dword aligned)
    int32_t run0, ld0, in_w;  // run: columns run0 .. run0 + SPAN - 1 clamped; edge load at ld0
    bool edge;
    RunStore<T, C, PPX> st;
    int32_t dst_row_off; // strip row of the store resource's first row
    float we[K], wo[K];
    float ring[K][PPX][C];
    Raw rawq[Q];

    __device__ __forceinline__ Raw load_row(int32_t j) const
    {
        const int32_t r = clampi(row_first + j, row_lo, row_hi) - row_lo;
        const uint32_t roff = static_cast<uint32_t>(static_cast<int64_t>(r) * src_pitch);
        Raw raw;
        if constexpr (PB % 4 == 0) {
            buf_load<LB>(raw.b, srsrc, roff + lane_src);
        } else {
            if (!edge) {
                buf_load<LB>(raw.b, srsrc, roff + lane_src);
            } else {
#pragma unroll
                for (int s = 0; s < SPAN; ++s)
                    buf_load_px<PB>(raw.b + MIS + s * PB, srsrc,
                                    roff + static_cast<uint32_t>(clampi(run0 + s, 0, in_w - 1) * PB));
            }
        }
        return raw;
    }

    __device__ __forceinline__ void hfilter(const Raw &loaded, float (&out)[PPX][C]) const
    {
        Raw raw = loaded;
        if constexpr (PB % 4 == 0) {
            if (edge)  // image edge: rebuild the replicated pixels in registers
                raw = clamp_window<SPAN, PB, K / 2, M + K / 2>(loaded, run0, ld0, in_w);
        }
        float p[SPAN][C];
#pragma unroll
        for (int s = 0; s < SPAN; ++s)
            decode<T, C>(raw.b + MIS, s, p[s]);
#pragma unroll
        for (int q = 0; q < M; ++q) {
            fma_first(out[2 * q], we[0], p[q]);
#pragma unroll
            for (int i = 1; i < K; ++i)
                fma_next(out[2 * q], we[i], p[q + i]);
            fma_first(out[2 * q + 1], wo[0], p[q + 1]);
#pragma unroll
            for (int i = 1; i < K; ++i)
                fma_next(out[2 * q + 1], wo[i], p[q + 1 + i]);
        }
    }

    // strip row `row` (0-based; it may lie outside the band) from the window
    // whose oldest row sits in ring slot OLD
    template <int OLD>
    __device__ __forceinline__ void emit_row(int32_t row, const float (&w)[K]) const
    {
        float v[PPX][C];
#pragma unroll
        for (int c = 0; c < PPX; ++c) {
            fma_first(v[c], w[0], ring[OLD % K][c]);
#pragma unroll
            for (int j = 1; j < K; ++j)
                fma_next(v[c], w[j], ring[(OLD + j) % K][c]);
        }
        RawBuf<OB, cmin(16, OB)> out;
        encode_run<T, C, PPX>(v, out);
        st.store(static_cast<uint32_t>(static_cast<int64_t>(row - dst_row_off) * dst_pitch), out);
    }

    // pair k of the strip: source row k + K - 1 completes its window
    template <int I>
    __device__ __forceinline__ void step(int32_t k, int32_t np)
    {
        constexpr int J = I + K - 1;  // window row index mod 4
        rawq[(J + PD) % Q] = load_row(min(k + K - 1 + PD, np + K - 2));
        __builtin_amdgcn_sched_barrier(0);
        hfilter(rawq[J % Q], ring[J % K]);
        emit_row<I>(2 * k, wo);      // row 2m+1, t = 1/4
        emit_row<I>(2 * k + 1, we);  // row 2m+2, t = 3/4
        __builtin_amdgcn_sched_barrier(0);
    }

    __device__ __forceinline__ void run(int32_t np)
    {
        weights<FILTER>(0.75f, 0.25f, we);
        weights<FILTER>(0.25f, 0.75f, wo);
#pragma unroll
        for (int i = 0; i < PD; ++i)
            rawq[i % Q] = load_row(min(i, np + K - 2));
#pragma unroll
        for (int j = 0; j + 1 < K; ++j) {
            rawq[(j + PD) % Q] = load_row(min(j + PD, np + K - 2));
            hfilter(rawq[j % Q], ring[j % K]);
        }
        // the first four pairs ahead of the loop: the loop's waits then see
        // the same rows of loads and stores in flight on every iteration
        step<0>(0, np);
        step<1>(1, np);
        step<2>(2, np);
        step<3>(3, np);
        for (int32_t k = 4; k < np; k += 4) {
            step<0>(k, np);
            step<1>(k + 1, np);
            step<2>(k + 2, np);
            step<3>(k + 3, np);
        }
    }
};

// Rows ahead of use that the x2 walk loads (one row keeps a 4-byte RGBA walk
// at 98 VGPRs, five wavefronts per SIMD; three rows measured the same)
constexpr int kX2Prefetch = 1;

// Strip s of np pairs covers logical output rows [2 s np - 1, 2 (s+1) np - 1);
// threadIdx.y picks one of blockDim.y consecutive strips from s_first on.
template <int FILTER, typename T, int C, int PPX>
__global__ void __launch_bounds__(512) k_x2(ResizeArgs a, int32_t np, int32_t s_first, int32_t order)
{
    int32_t bx, by;
    tile_coords(order, bx, by);
    using W = X2Walk<FILTER, T, C, PPX, kX2Prefetch>;
    constexpr int K = W::K, LO = W::LO, SPAN = W::SPAN, PB = W::PB;
    const int32_t col0 = (bx * static_cast<int32_t>(blockDim.x) + static_cast<int32_t>(threadIdx.x)) * PPX;
    if (!RunStore<T, C, PPX>::kExchange && col0 >= a.out_w)  // (an exchange needs every lane)
        return;
    const int32_t s = s_first + __builtin_amdgcn_readfirstlane(by * static_cast<int32_t>(blockDim.y) +
                                                               static_cast<int32_t>(threadIdx.y));
    const int32_t ys = 2 * s * np - 1;
    const int32_t y_lo = max(ys, max(a.dst_row0, 0));
    const int32_t y_hi = min(ys + 2 * np, min(a.dst_row0 + a.dst_rows, a.out_h));
    if (y_lo >= y_hi)
        return;
    W w;
    // source: the stored band's rows from the strip's first clamped row on
    const int32_t band_lo = max(0, a.src_row0);
    const int32_t band_hi = min(a.in_h - 1, a.src_row0 + a.src_rows - 1);
    w.row_first = s * np - 1 + LO;
    w.row_lo = clampi(w.row_first, band_lo, band_hi);
    w.row_hi = clampi(w.row_first + np + K - 2, band_lo, band_hi);  // the strip's last source row
    w.src_pitch = a.src_pitch;
    const unsigned char *src = a.src + static_cast<int64_t>(blockIdx.z) * a.src_plane_pitch +
                               static_cast<int64_t>(w.row_lo - a.src_row0) * a.src_pitch;
    w.srsrc = buf_rsrc(src, static_cast<uint32_t>(static_cast<int64_t>(w.row_hi - w.row_lo) * a.src_pitch +
                                                  static_cast<int64_t>(a.in_w) * PB));
    w.run0 = col0 / 2 - K / 2;
    w.in_w = a.in_w;
    w.edge = w.run0 < 0 || w.run0 + SPAN > a.in_w;
    w.ld0 = max(0, min(w.run0, a.in_w - SPAN));
    w.lane_src = static_cast<uint32_t>((w.edge && PB % 4 == 0) ? w.ld0 * PB : w.run0 * PB - W::MIS);
    // destination: rows [y_lo, y_hi) of the band
    unsigned char *dst = a.dst + static_cast<int64_t>(blockIdx.z) * a.dst_plane_pitch +
                         static_cast<int64_t>(y_lo - a.dst_row0) * a.dst_pitch;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    w.st.init(buf_rsrc(dst, static_cast<uint32_t>(static_cast<int64_t>(y_hi - y_lo) * a.dst_pitch)), col0,
              a.out_w, static_cast<int32_t>(threadIdx.y * blockDim.x + threadIdx.x), lds);
    w.dst_pitch = a.dst_pitch;
    w.dst_row_off = y_lo - ys;
    w.run(np);
}

// ---------------------------------------------------------------------------
// k_x05 (exact x0.5 on both axes)
// ---------------------------------------------------------------------------
//
// For out = in / 2 every output column and row has s = 2x + 1/2: x0 = 2x and
// t = 1/2, so output x taps source 2x + LO + i with the weights of t = 1/2
// (bicubic (-1, 9, 9, -1) / 16, bilinear (1/2, 1/2)). A thread's PPX columns
// read one run of NEED = 2 PPX - 2 + K source pixels per row; output row y
// reads the K source rows from 2y + LO on, so a strip of nr output rows (nr
// even) filters 2 nr + K - 2 source rows, K - 2 before its first output row,
// into a ring of K, two per output row. Loads and stores are issued on every
// step, through buffer resources, with the edge rules of k_x2: rows clamped on
// load, output rows outside the band dropped by the store resource, edge runs
// rebuilt in registers (or loaded pixel by pixel for 1- and 2-byte pixels),
// right-edge output runs stored pixel by pixel.
template <int FILTER, typename T, int C, int PPX, int PD>
struct D2Walk {
    using TP = Taps<FILTER>;
    static constexpr int K = TP::K;
    static constexpr int LO = TP::LO;
    static constexpr int PB = Pix<T, C>::kBytes;
    static constexpr int NEED = 2 * PPX - 2 + K;
    // a run starts at column 2 col0 + LO; loads start MIS bytes lower, on a dword
    static_assert((2 * PPX * PB) % 4 == 0, "a thread's run must advance by whole dwords");
    static constexpr int MIS = (4 - ((-LO) * PB) % 4) % 4;
    static constexpr int LB = (MIS + NEED * PB + 3) / 4 * 4;
    static constexpr int OB = PPX * PB;
    static constexpr int Q = PD + 1;
    static_assert(4 % K == 0 && 4 % Q == 0, "slots repeat every 4 rows");
    using Raw = RawBuf<LB, 4>;

    __amdgpu_buffer_rsrc_t srsrc;
    int32_t row_first, row_lo, row_hi;
    int64_t src_pitch, dst_pitch;
    uint32_t lane_src;
    int32_t run0, ld0, in_w, dst_row_off;
    bool edge;
    RunStore<T, C, PPX> st;
    float w[K];
    float ring[K][PPX][C];
    Raw rawq[Q];

    __device__ __forceinline__ Raw load_row(int32_t j) const
    {
        const int32_t r = clampi(row_first + j, row_lo, row_hi) - row_lo;
        const uint32_t roff = static_cast<uint32_t>(static_cast<int64_t>(r) * src_pitch);
        Raw raw;
        if constexpr (PB % 4 == 0) {
            buf_load<LB>(raw.b, srsrc, roff + lane_src);
        } else {
            if (!edge) {
                buf_load<LB>(raw.b, srsrc, roff + lane_src);
            } else {
#pragma unroll
                for (int s = 0; s < NEED; ++s)
                    buf_load_px<PB>(raw.b + MIS + s * PB, srsrc,
                                    roff + static_cast<uint32_t>(clampi(run0 + s, 0, in_w - 1) * PB));
            }
        }
        return raw;
    }

    __device__ __forceinline__ void hfilter(const Raw &loaded, float (&out)[PPX][C]) const
    {
        Raw raw = loaded;
        if constexpr (PB % 4 == 0) {
            if (edge)
                raw = clamp_window<NEED, PB, -LO, NEED>(loaded, run0, ld0, in_w);
        }
        float p[NEED][C];
#pragma unroll
        for (int s = 0; s < NEED; ++s)
            decode<T, C>(raw.b + MIS, s, p[s]);
#pragma unroll
        for (int c = 0; c < PPX; ++c) {
            fma_first(out[c], w[0], p[2 * c]);
#pragma unroll
            for (int i = 1; i < K; ++i)
                fma_next(out[c], w[i], p[2 * c + i]);
        }
    }

    // strip row `row` from the window whose oldest row sits in ring slot OLD
    template <int OLD>
    __device__ __forceinline__ void emit_row(int32_t row) const
    {
        float v[PPX][C];
#pragma unroll
        for (int c = 0; c < PPX; ++c) {
            fma_first(v[c], w[0], ring[OLD % K][c]);
#pragma unroll
            for (int j = 1; j < K; ++j)
                fma_next(v[c], w[j], ring[(OLD + j) % K][c]);
        }
        RawBuf<OB, cmin(16, OB)> out;
        encode_run<T, C, PPX>(v, out);
        st.store(static_cast<uint32_t>(static_cast<int64_t>(row - dst_row_off) * dst_pitch), out);
    }

    // filter window row j (slot J mod K), requesting row j + PD first
    template <int J>
    __device__ __forceinline__ void filter(int32_t j, int32_t last)
    {
        rawq[(J + PD) % Q] = load_row(min(j + PD, last));
        __builtin_amdgcn_sched_barrier(0);
        hfilter(rawq[J % Q], ring[J % K]);
    }

    // output row k of the strip: window rows 2k + K - 2 and 2k + K - 1 complete it
    template <int I>  // k mod 2
    __device__ __forceinline__ void step(int32_t k, int32_t last)
    {
        constexpr int J0 = 2 * I + K - 2;  // window row index mod 4
        filter<J0>(2 * k + K - 2, last);
        filter<J0 + 1>(2 * k + K - 1, last);
        emit_row<2 * I>(k);
        __builtin_amdgcn_sched_barrier(0);
    }

    __device__ __forceinline__ void run(int32_t nr)
    {
        weights<FILTER>(0.5f, 0.5f, w);
        const int32_t last = 2 * nr + K - 3;  // the strip's last window row
#pragma unroll
        for (int i = 0; i < PD; ++i)
            rawq[i % Q] = load_row(min(i, last));
        if constexpr (K == 4) {
            filter<0>(0, last);
            filter<1>(1, last);
        }
        step<0>(0, last);
        step<1>(1, last);
        for (int32_t k = 2; k < nr; k += 2) {
            step<0>(k, last);
            step<1>(k + 1, last);
        }
    }
};

constexpr int kX05Prefetch = 1;

// Strip s covers logical output rows [s nr, (s + 1) nr); threadIdx.y picks
// one of blockDim.y consecutive strips from s_first on.
template <int FILTER, typename T, int C, int PPX>
__global__ void __launch_bounds__(512) k_x05(ResizeArgs a, int32_t nr, int32_t s_first, int32_t order)
{
    int32_t bx, by;
    tile_coords(order, bx, by);
    using W = D2Walk<FILTER, T, C, PPX, kX05Prefetch>;
    constexpr int K = W::K, LO = W::LO, NEED = W::NEED, PB = W::PB;
    const int32_t col0 = (bx * static_cast<int32_t>(blockDim.x) + static_cast<int32_t>(threadIdx.x)) * PPX;
    if (!RunStore<T, C, PPX>::kExchange && col0 >= a.out_w)  // (an exchange needs every lane)
        return;
    const int32_t s = s_first + __builtin_amdgcn_readfirstlane(by * static_cast<int32_t>(blockDim.y) +
                                                               static_cast<int32_t>(threadIdx.y));
    const int32_t ys = s * nr;
    const int32_t y_lo = max(ys, max(a.dst_row0, 0));
    const int32_t y_hi = min(ys + nr, min(a.dst_row0 + a.dst_rows, a.out_h));
    if (y_lo >= y_hi)
        return;
    W w;
    const int32_t band_lo = max(0, a.src_row0);
    const int32_t band_hi = min(a.in_h - 1, a.src_row0 + a.src_rows - 1);
    w.row_first = 2 * ys + LO;
    w.row_lo = clampi(w.row_first, band_lo, band_hi);
    w.row_hi = clampi(w.row_first + 2 * nr + K - 3, band_lo, band_hi);
    w.src_pitch = a.src_pitch;
    const unsigned char *src = a.src + static_cast<int64_t>(blockIdx.z) * a.src_plane_pitch +
                               static_cast<int64_t>(w.row_lo - a.src_row0) * a.src_pitch;
    w.srsrc = buf_rsrc(src, static_cast<uint32_t>(static_cast<int64_t>(w.row_hi - w.row_lo) * a.src_pitch +
                                                  static_cast<int64_t>(a.in_w) * PB));
    w.run0 = 2 * col0 + LO;
    w.in_w = a.in_w;
    w.edge = w.run0 < 0 || w.run0 + NEED > a.in_w;
    w.ld0 = max(0, min(w.run0, a.in_w - NEED));
    w.lane_src = static_cast<uint32_t>((w.edge && PB % 4 == 0) ? w.ld0 * PB : w.run0 * PB - W::MIS);
    unsigned char *dst = a.dst + static_cast<int64_t>(blockIdx.z) * a.dst_plane_pitch +
                         static_cast<int64_t>(y_lo - a.dst_row0) * a.dst_pitch;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    w.st.init(buf_rsrc(dst, static_cast<uint32_t>(static_cast<int64_t>(y_hi - y_lo) * a.dst_pitch)), col0,
              a.out_w, static_cast<int32_t>(threadIdx.y * blockDim.x + threadIdx.x), lds);
    w.dst_pitch = a.dst_pitch;
    w.dst_row_off = y_lo - ys;
    w.run(nr);
}

// ---------------------------------------------------------------------------
// k_batch_narrow: the batched jobs that the staged walk (xr_walk.hip) leaves
// ---------------------------------------------------------------------------

// Jobs whose output is narrower than the staged walk's run or whose staged
// rows are too long for it (any filter and channel count): the per-tap strip
// walk, one column per thread, a workgroup per tile.
template <typename T>
__global__ void __launch_bounds__(256) k_batch_narrow(const unsigned char *__restrict__ ws)
{
    int32_t plane, tx, ty;
    BatchJob job;
    if (!batch_tile(ws, kBatchNarrow, batch_block(), job, plane, tx, ty))
        return;
    const ResizeArgs &a = job.a;
    const int32_t col0 = tx * static_cast<int32_t>(blockDim.x) + static_cast<int32_t>(threadIdx.x);
    const int32_t r_begin =
        __builtin_amdgcn_readfirstlane((ty * static_cast<int32_t>(blockDim.y) + threadIdx.y) * job.strip_h);
    if (col0 >= a.out_w || r_begin >= a.dst_rows)
        return;
    const int32_t r_end = min(r_begin + job.strip_h, a.dst_rows);
    switch (job.kind_fc) {
    case 0: {
        StripBody<kBilinear, T, 1, 1> b;
        b.run(a, plane, col0, r_begin, r_end);
        break;
    }
    case 1: {
        StripBody<kBilinear, T, 4, 1> b;
        b.run(a, plane, col0, r_begin, r_end);
        break;
    }
    case 2: {
        StripBody<kBicubic, T, 1, 1> b;
        b.run(a, plane, col0, r_begin, r_end);
        break;
    }
    default: {
        StripBody<kBicubic, T, 4, 1> b;
        b.run(a, plane, col0, r_begin, r_end);
        break;
    }
    }
}

hipError_t launch_batch_narrow(const void *ws, int32_t dtype, dim3 block, int32_t grid, hipStream_t stream)
{
    const unsigned char *p = static_cast<const unsigned char *>(ws);
    if (dtype == XR_U8)
        hipLaunchKernelGGL(k_batch_narrow<uint8_t>, batch_grid(grid), block, 0, stream, p);
    else if (dtype == XR_F16)
        hipLaunchKernelGGL(k_batch_narrow<_Float16>, batch_grid(grid), block, 0, stream, p);
    else
        hipLaunchKernelGGL(k_batch_narrow<float>, batch_grid(grid), block, 0, stream, p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// dispatch
// ---------------------------------------------------------------------------

bool strip_ppx_supported(int32_t dtype, int32_t channels, int32_t ppx)
{
    (void)dtype;
    if (channels == 4)
        return ppx == 1 || ppx == 2 || ppx == 4 || ppx == 8;
    return ppx == 4 || ppx == 8 || ppx == 16;
}

namespace {

// The x2 walk needs whole-dword runs: (PPX/2) pixels of a thread a multiple
// of 4 bytes (one-byte pixels: PPX 8 or 16).
// Runs of more than 64 output bytes per thread (float32 RGBA with 8 columns)
// take the general walk: their rings exceed the register file.
template <typename T, int C, int PPX>
constexpr bool x2_ppx_ok()
{
    return PPX % 2 == 0 && ((PPX / 2) * Pix<T, C>::kBytes) % 4 == 0 && PPX * Pix<T, C>::kBytes <= 64;
}

// Strips of 2 np output rows, np = ppt_y / 2 rounded up to a multiple of 4
// (at least 4; see x2_pairs).
template <int FILTER, typename T, int C, int PPX>
hipError_t launch_x2(const ResizeArgs &a, const xr_tile &tile, int64_t np, hipStream_t stream, Route *only)
{
    if (just_named(only, kRouteX2))
        return hipSuccess;
    const int64_t s_first = (static_cast<int64_t>(a.dst_row0) + 1) / (2 * np);
    const int64_t s_last = (static_cast<int64_t>(a.dst_row0) + a.dst_rows) / (2 * np);
    const int64_t strips = s_last - s_first + 1;
    const int32_t cols_per_block = tile.block_w * PPX;
    const dim3 block(tile.block_w, tile.block_h, 1);
    const dim3 grid((a.out_w + cols_per_block - 1) / cols_per_block,
                    static_cast<uint32_t>((strips + tile.block_h - 1) / tile.block_h), a.planes);
    const size_t lds = run_store_lds<T, C, PPX>(tile.block_w * tile.block_h);
    hipLaunchKernelGGL((k_x2<FILTER, T, C, PPX>), grid, block, lds, stream, a, static_cast<int32_t>(np),
                       static_cast<int32_t>(s_first), tile.order);
    return hipGetLastError();
}

// Strips of nr output rows, nr = ppt_y rounded up to an even count (x05_rows).
template <int FILTER, typename T, int C, int PPX>
hipError_t launch_x05(const ResizeArgs &a, const xr_tile &tile, int64_t nr, hipStream_t stream, Route *only)
{
    if (just_named(only, kRouteX05))
        return hipSuccess;
    const int64_t s_first = static_cast<int64_t>(a.dst_row0) / nr;
    const int64_t s_last = (static_cast<int64_t>(a.dst_row0) + a.dst_rows - 1) / nr;
    const int64_t strips = s_last - s_first + 1;
    const int32_t cols_per_block = tile.block_w * PPX;
    const dim3 block(tile.block_w, tile.block_h, 1);
    const dim3 grid((a.out_w + cols_per_block - 1) / cols_per_block,
                    static_cast<uint32_t>((strips + tile.block_h - 1) / tile.block_h), a.planes);
    const size_t lds = run_store_lds<T, C, PPX>(tile.block_w * tile.block_h);
    hipLaunchKernelGGL((k_x05<FILTER, T, C, PPX>), grid, block, lds, stream, a, static_cast<int32_t>(nr),
                       static_cast<int32_t>(s_first), tile.order);
    return hipGetLastError();
}

template <int FILTER, typename T, int C>
hipError_t launch_typed(const ResizeArgs &a, const xr_tile &tile, int32_t mode, hipStream_t stream, Route *only)
{
    if (tile.kernel == XR_KERNEL_GATHER) {
        if (just_named(only, kRouteGather))
            return hipSuccess;
        const dim3 block(tile.block_w, tile.block_h, 1);
        const dim3 grid((a.out_w + tile.block_w - 1) / tile.block_w,
                        (a.dst_rows + tile.block_h - 1) / tile.block_h, a.planes);
        hipLaunchKernelGGL((k_gather<FILTER, T, C>), grid, block, 0, stream, a);
        return hipGetLastError();
    }
    const int64_t pitch = std::max(a.src_pitch, a.dst_pitch);
    const int32_t cols_per_block = tile.block_w * tile.ppt_x;
    const int32_t rows_per_block = tile.block_h * tile.ppt_y;
    const dim3 block(tile.block_w, tile.block_h, 1);
    const dim3 grid((a.out_w + cols_per_block - 1) / cols_per_block,
                    (a.dst_rows + rows_per_block - 1) / rows_per_block, a.planes);
#define XR_STRIP_CASE(P)                                                                        \
    case P:                                                                                     \
        if constexpr (FILTER != kNearest) {                                                     \
            if (mode == kUp2 && x2_pairs(tile.ppt_y, pitch) > 0) {                              \
                if constexpr (x2_ppx_ok<T, C, P>())                                             \
                    return launch_x2<FILTER, T, C, P>(a, tile, x2_pairs(tile.ppt_y, pitch), stream, only); \
            }                                                                                   \
            if (mode == kDown2 && x05_rows(tile.ppt_y, pitch) > 0) {                            \
                if constexpr ((2 * P * Pix<T, C>::kBytes) % 4 == 0 && P * Pix<T, C>::kBytes <= 64) \
                    return launch_x05<FILTER, T, C, P>(a, tile, x05_rows(tile.ppt_y, pitch), stream, only); \
            }                                                                                   \
        }                                                                                       \
        if (tile.kernel != XR_KERNEL_STRIP_ANY) {                                               \
            bool taken = false;                                                                 \
            const hipError_t e = launch_walk(a, FILTER == kBicubic ? XR_BICUBIC                 \
                                                : FILTER == kNearest ? XR_NEAREST : XR_BILINEAR, \
                                             DType<T>::kCode, C, tile, stream, taken, only);    \
            if (taken)                                                                          \
                return e;                                                                       \
        }                                                                                       \
        if (just_named(only, kRouteStrip))                                                      \
            return hipSuccess;                                                                  \
        hipLaunchKernelGGL((k_strip<FILTER, T, C, P>), grid, block, 0, stream, a, tile.ppt_y,   \
                           tile.order);                                                         \
        return hipGetLastError();
    if constexpr (C == 4) {
        switch (tile.ppt_x) {
            XR_STRIP_CASE(1)
            XR_STRIP_CASE(2)
            XR_STRIP_CASE(4)
            XR_STRIP_CASE(8)
        default:
            return hipErrorInvalidValue;
        }
    } else {
        switch (tile.ppt_x) {
            XR_STRIP_CASE(4)
            XR_STRIP_CASE(8)
            XR_STRIP_CASE(16)
        default:
            return hipErrorInvalidValue;
        }
    }
#undef XR_STRIP_CASE
}

template <int FILTER>
hipError_t launch_filter(const ResizeArgs &a, int32_t dtype, int32_t channels, const xr_tile &tile,
                         int32_t mode, hipStream_t stream, Route *only)
{
    switch (dtype) {
    case XR_U8:
        return channels == 4 ? launch_typed<FILTER, uint8_t, 4>(a, tile, mode, stream, only)
                             : launch_typed<FILTER, uint8_t, 1>(a, tile, mode, stream, only);
    case XR_F16:
        return channels == 4 ? launch_typed<FILTER, _Float16, 4>(a, tile, mode, stream, only)
                             : launch_typed<FILTER, _Float16, 1>(a, tile, mode, stream, only);
    case XR_F32:
        return channels == 4 ? launch_typed<FILTER, float, 4>(a, tile, mode, stream, only)
                             : launch_typed<FILTER, float, 1>(a, tile, mode, stream, only);
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_forward(const ResizeArgs &a, int32_t filter, int32_t dtype, int32_t channels,
                          const xr_tile &tile, int32_t mode, hipStream_t stream, Route *only)
{
    if (filter == XR_BILINEAR_AA || filter == XR_BICUBIC_AA)
        return launch_antialiased(a, filter, dtype, channels, tile, stream, only);
    if (filter == XR_BICUBIC)
        return launch_filter<kBicubic>(a, dtype, channels, tile, mode, stream, only);
    if (filter == XR_NEAREST)
        return launch_filter<kNearest>(a, dtype, channels, tile, mode, stream, only);
    return launch_filter<kBilinear>(a, dtype, channels, tile, mode, stream, only);
}

}  // namespace xr
