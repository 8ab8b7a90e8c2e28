// Walk of the filters whose results gather a varying number of samples: the
// antialiased forward filters and the adjoint at any ratio.
//
// A result value is sum_j wy_j (sum_k wx_k v[j][k]) over a contiguous range
// of samples per axis, columns first, both in ascending order. A wavefront
// owns 64 result columns (128 of a one-channel image) and a strip of result
// rows, and walks the sample rows the strip reads, each once, in order:
//  * the rows are staged in LDS some 8 KiB ahead (xr_stage.hpp);
//  * a lane filters its columns' samples of RB staged rows at a time, all
//    their LDS reads first, with the columns' weights in registers (past
//    kGatherRegTaps samples: an LDS table of the workgroup);
//  * a filtered row is added at once to the result rows it belongs to: at
//    most kSlots consecutive ones, held in registers at slot
//    (row mod kSlots), each stored when its last sample row has been added.
//    So the filtered rows need no buffer, and a sample row is filtered once
//    per strip instead of once per tile of a few rows.
// The row side is a table of the wavefront in LDS with one entry per sample
// row: the weight per slot, and which slots are active, new and complete.
//
// What bounds it: instruction issue (bicubic x0.5 of a 4096^2 RGBA uint8 image:
// 99.3 us with a block's window and filtered rows in LDS, 35.4 us so, 2.4 TB/s;
// of a wavefront's time a tenth goes into its tables; 192 bilinear uint8 planes
// 375 x 500 -> 224^2: 135.0 to 24.5 us, 29.8 with one column per lane; the
// bicubic x1.5 adjoint of 48 float32 planes 512^2: 96.1 to 43.3 us, 46.7
// with one column; 41.6 in a trace of warm steps). Measured and left out: two windows a wavefront, the next rows
// arriving while the staged ones are filtered (34.9 to 36.4 us against 36.4,
// planes 32 against 30).
//
// A policy P supplies the tap ranges and weights:
//   kSlots      power of two, at least the result rows a sample row reaches
//   kFirstMul   the first term of a row sum is a product (else a fused
//               multiply-add onto zero)
//   the geometry, and per axis the first sample and count of a result index
//   (range_x, range_y) and its weights (weights_x, weights_y into w(k), and
//   weights_x and, with kRowRegs, weights_y into an array, zero past the count)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "xr_device.hpp"
#include "xr_internal.h"
#include "xr_stage.hpp"

namespace xr {

// LDS layout and strip of a launch (host side, see gather_shape).
struct GatherShape {
    int32_t waves;       // wavefronts per workgroup (strips below one another)
    int32_t strip;       // result rows per wavefront, at most 64
    int32_t rows_cap;    // sample rows of a strip, at most
    int32_t kx;          // column weights per column, at most (a multiple of 4)
    int32_t big;         // more of them than a walk holds in registers
    int32_t col_bytes;   // column table of the workgroup (big)
    int32_t wave_bytes;  // row table and window of a wavefront
    int32_t win_off, win_bytes;
    int32_t lds_bytes;   // dynamic LDS of a workgroup
};

// Result columns of a wavefront: two per lane for one-channel images, whose
// rows else carry as many instructions for the walk as for the filter.
constexpr int32_t gather_cols(int32_t channels) { return channels == 1 ? 128 : 64; }
constexpr int32_t kGatherWaves = 4;
constexpr int32_t kGatherRegTaps = 10;
constexpr int64_t kGatherWindow = 8192;

// Strips are the tallest of 64 .. 4 rows that give gather_min_waves wavefronts
// (12 per compute unit, 8 where a lane holds two columns): a strip re-filters
// the sample rows it shares with the next one, but a wavefront alone on its
// SIMD issues at most every fourth cycle and waits for each load. Bicubic x0.5
// of a 4096^2 RGBA image (2048 wavefronts at 32 rows, 4096 at 16): 38.4 and
// 37.3 us; 192 bilinear planes 375 x 500 -> 224^2 (1536 at 64 rows, 2688 at
// 32, 5376 at 16): 34.9, 24.8 and 27.5 us.
//
// 0: fewer than `least` results, too few wavefronts to hide that latency even at
// 4 rows; kernels that spread one tile's rows over a workgroup are then faster
// (0.48x to 0.79x their speed below 130 K results where a walk was forced). From
// kGatherLeast on the walk is at 1.0x to 18x for RGBA and for one-channel images
// but those for which its caller names more.
constexpr int64_t gather_min_waves(int32_t channels) { return channels == 1 ? 2048 : 3072; }
constexpr int64_t kGatherLeast = 1 << 18;
template <class RowsCap>
inline int64_t gather_strip(int32_t channels, int64_t res_w, int64_t res_rows, int64_t planes, int64_t pitch,
                            int64_t least, RowsCap rows_cap)
{
    const int64_t wide = gather_cols(channels);
    const auto waves = [&](int64_t strip) {
        return ((res_w + wide - 1) / wide) * ((res_rows + strip - 1) / strip) * planes;
    };
    int64_t strip = 64;
    while (strip > 4 && (waves(strip) < gather_min_waves(channels) || rows_cap(strip) * pitch >= (int64_t(1) << 31)))
        strip /= 2;
    return res_w * res_rows * planes < least || rows_cap(strip) * pitch >= (int64_t(1) << 31) ? 0 : strip;
}

// The launch of a walk whose sample rows hold at most win_px samples of
// px_bytes and whose strips of n result rows read at most rows_cap(n) sample
// rows; false when a workgroup's LDS would not fit.
template <class RowsCap>
inline bool gather_shape(GatherShape &g, int32_t channels, int32_t slots, int32_t kx, int32_t win_px,
                         int32_t px_bytes, int64_t strip, RowsCap rows_cap)
{
    if (kx > 1024)
        return false;
    g.kx = (kx + 3) / 4 * 4;
    g.strip = static_cast<int32_t>(strip);
    g.big = kx > kGatherRegTaps;
    g.col_bytes = g.big ? gather_cols(channels) * 4 * g.kx : 0;
    const int64_t row_bytes = (static_cast<int64_t>(win_px) * px_bytes + 30) / 16 * 16;
    const int64_t cap = rows_cap(strip);
    g.rows_cap = static_cast<int32_t>(cap);
    g.win_off = static_cast<int32_t>((cap * 4 * (slots + 1) + 15) / 16 * 16);
    g.win_bytes = static_cast<int32_t>(row_bytes * std::max<int64_t>(1, std::min(cap, kGatherWindow / row_bytes)));
    // a column with fewer taps than its neighbours reads as many samples
    g.wave_bytes = g.win_off + g.win_bytes + (g.kx * px_bytes + 8 + 15) / 16 * 16;
    for (g.waves = kGatherWaves; g.waves > 1 && g.col_bytes + g.waves * g.wave_bytes > kStageMaxLds;)
        g.waves /= 2;
    g.lds_bytes = g.col_bytes + g.waves * g.wave_bytes;
    return g.lds_bytes <= kStageMaxLds;
}

// BIG: more than kGatherRegTaps samples per column; the column weights then
// come from an LDS table of the workgroup instead of registers.
template <class P, typename T, int C, bool BIG>
__global__ void __launch_bounds__(256, 4) k_gather_walk(ResizeArgs a, GatherShape g)
{
    using namespace dev;
    constexpr int S = P::kSlots;
    constexpr int PB = Pix<T, C>::kBytes;
    constexpr int NC = gather_cols(C) / 64;  // columns per lane, 64 apart
    constexpr bool kBytes = std::is_same_v<T, uint8_t>;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int32_t lane = static_cast<int32_t>(threadIdx.x);
    const int32_t wave = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(threadIdx.y));
    const int32_t plane = blockIdx.z;
    const int32_t res_w = P::result_w(a);
    const int32_t c_first = static_cast<int32_t>(blockIdx.x) * (64 * NC);

    float *colw = reinterpret_cast<float *>(lds);  // BIG: [kx][64 NC]
    unsigned char *mine = lds + g.col_bytes + wave * g.wave_bytes;
    float *roww = reinterpret_cast<float *>(mine);                        // [rows_cap][S]
    uint32_t *rowf = reinterpret_cast<uint32_t *>(roww + g.rows_cap * S); // [rows_cap]
    unsigned char *win = mine + g.win_off;

    // the lane's columns: samples [lo, lo + cnt)
    int32_t x[NC], lo[NC], cnt[NC];
    bool inside[NC];
    int32_t most = 0, fewest = g.kx;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int32_t xc = c_first + lane + 64 * c;
        inside[c] = xc < res_w;
        x[c] = min(xc, res_w - 1);
        P::range_x(a, x[c], lo[c], cnt[c]);
        cnt[c] = min(cnt[c], g.kx);
        most = max(most, cnt[c]);
        fewest = min(fewest, cnt[c]);
    }
    int32_t kn = g.kx, kmin = 0;  // most and fewest samples of a column of this tile
    while (kn > 0 && __builtin_amdgcn_ballot_w64(most >= kn) == 0)
        --kn;
    while (kmin < kn && __builtin_amdgcn_ballot_w64(fewest <= kmin) == 0)
        ++kmin;
    if constexpr (BIG) {
        if (wave == 0) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                float *wc = colw + lane + 64 * c;
                P::weights_x(a, x[c], lo[c], cnt[c], [&](int32_t k) -> float & { return wc[k * 64 * NC]; });
                for (int32_t k = 0; k < g.kx; ++k)
                    wc[k * 64 * NC] = k < cnt[c] ? wc[k * 64 * NC] * sample_scale<T, C>(k) : 0.0f;
            }
        }
        __syncthreads();
    }

    // the strip's result rows y_a .. y_b - 1 and sample rows r_lo .. r_lo + rows - 1
    const int32_t y_a = static_cast<int32_t>(blockIdx.y * blockDim.y + wave) * g.strip;
    const int32_t y_b = min(y_a + g.strip, P::result_rows(a));
    if (y_a >= y_b)
        return;
    const int32_t o = min(y_a + lane, y_b - 1);  // (strips of up to 64 rows: a result row per lane)
    int32_t o_lo, o_n;
    P::range_y(a, o, o_lo, o_n);
    const int32_t r_lo = __builtin_amdgcn_readfirstlane(o_lo);
    const int32_t rows = min(__builtin_amdgcn_readlane(o_lo + o_n, 63) - r_lo, g.rows_cap);

    const int32_t seg0 = min(__builtin_amdgcn_readfirstlane(lo[0]), P::walked_w(a) - 1);
    const int32_t seg1 = max(__builtin_amdgcn_readlane(lo[NC - 1] + cnt[NC - 1] - 1, 63), seg0);
    uint32_t loff[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
        loff[c] = static_cast<uint32_t>((lo[c] - seg0) * PB);
    const unsigned char *src = a.src + static_cast<int64_t>(plane) * a.src_plane_pitch +
                               static_cast<int64_t>(P::stored_row(a, r_lo)) * a.src_pitch +
                               static_cast<int64_t>(seg0) * PB;
    RowStage st;
    st.init(src, static_cast<uint32_t>(a.src_pitch), (seg1 - seg0 + 1) * PB, 0, 0);
    const uint32_t lp = st.lds_pitch();
    int32_t rc = min(max(g.win_bytes / static_cast<int32_t>(lp), 1), 64);  // (a lane holds a row's flags)
    rc = rc > 4 ? rc / 4 * 4 : rc;
    if (rows > 0)
        st.request(win, 0, min(rc, rows), lane);  // in flight while the tables are built

    // row table
    o_lo -= r_lo;
    o_n = min(o_n, rows - o_lo);
    for (int32_t i = lane; i < rows * S; i += 64)
        roww[i] = 0.0f;
    for (int32_t i = lane; i < rows; i += 64)
        rowf[i] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const bool mine_o = y_a + lane < y_b;
    if (mine_o) {
        const int32_t slot = lane & (S - 1);
        // active, new (first sample row), complete (last one)
        const auto flag = [&](int32_t k) {
            atomicOr(&rowf[o_lo + k], ((k == 0 ? 0x101u : 0x1u) << slot) | (k == o_n - 1 ? 0x10000u << slot : 0u));
        };
        bool wide = true;
        if constexpr (P::kRowRegs) {  // few weights: written once instead of passed over in LDS
            wide = __builtin_amdgcn_ballot_w64(o_n > kGatherRegTaps) != 0;
            if (!wide) {
                float w[kGatherRegTaps];
                P::weights_y(a, o, o_lo + r_lo, o_n, w);
#pragma unroll
                for (int k = 0; k < kGatherRegTaps; ++k)
                    if (k < o_n) {
                        roww[(o_lo + k) * S + slot] = kBytes ? w[k] * 0x1p23f : w[k];
                        flag(k);
                    }
            }
        }
        if (wide) {
            P::weights_y(a, o, o_lo + r_lo, o_n, [&](int32_t k) -> float & { return roww[(o_lo + k) * S + slot]; });
            for (int32_t k = 0; k < o_n; ++k) {
                if (kBytes)
                    roww[(o_lo + k) * S + slot] *= 0x1p23f;
                flag(k);
            }
        }
        // a row without samples follows the sample row before its place
        if (o_n == 0 && o_lo > 0)
            atomicAdd(&rowf[o_lo - 1], 0x1000000u);
    }
    // rows without samples before the first sample row
    const int32_t lead =
        __builtin_popcountll(__builtin_amdgcn_ballot_w64(mine_o && o_lo + o_n <= 0));

    unsigned char *const dst = a.dst + static_cast<int64_t>(plane) * a.dst_plane_pitch +
                               static_cast<int64_t>(y_a) * a.dst_pitch +
                               static_cast<int64_t>(c_first) * PB;
    float acc[NC][S][C];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int ch = 0; ch < C; ++ch)
                acc[c][s][ch] = 0.0f;
    int32_t y = 0;  // rows of the strip that are stored
    auto store_row = [&](int32_t row, auto value) __attribute__((always_inline)) {
        unsigned char *d = dst + static_cast<int64_t>(row) * a.dst_pitch;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (inside[c])
                Pix<T, C>::store(d, lane + 64 * c, value(c));
    };
    auto zeros = [&](int32_t m) __attribute__((always_inline)) {
        for (; m > 0; --m, ++y) {
            const float z[C] = {};
            store_row(y, [&](int) -> const float(&)[C] { return z; });
        }
    };
    zeros(lead);

    // add filtered row h of the strip (flags f, weights w) to its result rows
    // and store those that it completes
    auto add_row = [&](uint32_t f, const float (&w)[S], const float (&h)[NC][C]) __attribute__((always_inline)) {
        if (kBytes || (f & ((1u << S) - 1u) & ~(P::kFirstMul ? f >> 8 : 0u)) == (1u << S) - 1u) {
            // every slot takes the row (the usual case)
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    fma_next(acc[c][s], w[s], h[c]);
        } else {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                if (P::kFirstMul && (f >> (8 + s)) & 1u) {
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        fma_first(acc[c][s], w[s], h[c]);
                } else if ((f >> s) & 1u) {
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        fma_next(acc[c][s], w[s], h[c]);
                }
            }
        }
        if (f >= 0x10000u) {
            const int32_t y0 = y;
#pragma unroll
            for (int s = 0; s < S; ++s)
                if ((f >> (16 + s)) & 1u) {
                    store_row(y0 + ((s - y0) & (S - 1)), [&](int c) -> const float(&)[C] { return acc[c][s]; });
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int ch = 0; ch < C; ++ch)
                            acc[c][s][ch] = 0.0f;
                    ++y;
                }
            zeros(static_cast<int32_t>(f >> 24));
        }
    };

    // every sample row of the strip: filter(rows of the chunk from i0 on,
    // their LDS offsets) gives RB filtered rows
    auto walk = [&](auto rb_tag, auto filter) __attribute__((always_inline)) {
        constexpr int RB = decltype(rb_tag)::value;
        for (int32_t base = 0; base < rows; base += rc) {
            const int32_t n = min(rc, rows - base);
            if (base > 0) {
                RowStage::drain_lds();
                st.request(win, base, n, lane);
            }
            RowStage::wait();
            const int32_t li = min(lane, n - 1);  // lane i holds row i's flags and place
            const uint32_t flags = rowf[base + li];
            const uint32_t place = static_cast<uint32_t>(li) * lp + st.start(base + li);
            for (int32_t i0 = 0; i0 < n; i0 += RB) {
                float wr[RB][S];
                uint32_t at[RB];
#pragma unroll
                for (int q = 0; q < RB; ++q) {
                    const int32_t i = min(i0 + q, n - 1);
                    at[q] = __builtin_amdgcn_readlane(place, i);
                    __builtin_memcpy(wr[q], __builtin_assume_aligned(roww + (base + i) * S, 4 * S), 4 * S);
                }
                float h[RB][NC][C];
                filter(at, h);
#pragma unroll
                for (int q = 0; q < RB; ++q)
                    if (i0 + q < n)
                        add_row(__builtin_amdgcn_readlane(flags, i0 + q), wr[q], h[q]);
            }
        }
    };

    if constexpr (!BIG) {
        // up to 2 NP samples per column, their weights in registers
        auto run = [&](auto np_tag) __attribute__((always_inline)) {
            constexpr int N = 2 * decltype(np_tag)::value;
            // rows filtered at a time: their samples take up to 32 registers
            constexpr int W = NC * ((N * PB + 3) / 4 + (PB < 4 ? 1 : 0));
            constexpr int RB = C == 1 && 8 * W <= 32 ? 8 : 4 * W <= 32 ? 4 : 2 * W <= 36 ? 2 : 1;
            float wt[NC][N][C];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                float w[N];
                P::weights_x(a, x[c], lo[c], cnt[c], w);
#pragma unroll
                for (int t = 0; t < N; ++t)
                    sample_weights<T, C>(w[t] * sample_scale<T, C>(t), wt[c][t]);
            }
            walk(std::integral_constant<int, RB>{},
                 [&](const uint32_t (&at)[RB], float (&h)[RB][NC][C]) __attribute__((always_inline)) {
                     SampleRun<T, C, N> run[RB][NC];
#pragma unroll
                     for (int q = 0; q < RB; ++q)
#pragma unroll
                         for (int c = 0; c < NC; ++c)
                             run[q][c].load(win, at[q] + loff[c]);
                     __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                     for (int q = 0; q < RB; ++q)
#pragma unroll
                         for (int c = 0; c < NC; ++c)
#pragma unroll
                             for (int ch = 0; ch < C; ++ch)
                                 h[q][c][ch] = 0.0f;
#pragma unroll
                     for (int t = 0; t < N; ++t)
#pragma unroll
                         for (int c = 0; c < NC; ++c) {
                             // (bytes: the weights past a column's samples are zero)
                             if (kBytes || t < kmin || t < cnt[c]) {
#pragma unroll
                                 for (int q = 0; q < RB; ++q) {
                                     float v[C];
                                     run[q][c].terms(t, v);
#pragma unroll
                                     for (int ch = 0; ch < C; ++ch)
                                         h[q][c][ch] = t == 0 ? wt[c][t][ch] * v[ch]
                                                              : __builtin_fmaf(wt[c][t][ch], v[ch], h[q][c][ch]);
                                 }
                             }
                         }
                 });
        };
        switch ((kn + 1) / 2) {
        case 0:
        case 1:
            run(std::integral_constant<int, 1>{});
            break;
        case 2:
            run(std::integral_constant<int, 2>{});
            break;
        case 3:
            run(std::integral_constant<int, 3>{});
            break;
        case 4:
            run(std::integral_constant<int, 4>{});
            break;
        default:
            run(std::integral_constant<int, 5>{});
            break;
        }
    } else {
        constexpr int RB = NC * PB >= 8 ? 2 : 4;
        walk(std::integral_constant<int, RB>{},
             [&](const uint32_t (&at)[RB], float (&h)[RB][NC][C]) __attribute__((always_inline)) {
#pragma unroll
                 for (int q = 0; q < RB; ++q)
#pragma unroll
                     for (int c = 0; c < NC; ++c)
#pragma unroll
                         for (int ch = 0; ch < C; ++ch)
                             h[q][c][ch] = 0.0f;
                 auto group = [&](auto first_tag, int32_t k) __attribute__((always_inline)) {
                     SampleRun<T, C, 4> run[RB][NC];
                     float wt[NC][4][C];
#pragma unroll
                     for (int c = 0; c < NC; ++c)
#pragma unroll
                         for (int t = 0; t < 4; ++t)
                             sample_weights<T, C>(colw[(k + t) * 64 * NC + 64 * c + lane], wt[c][t]);
#pragma unroll
                     for (int q = 0; q < RB; ++q)
#pragma unroll
                         for (int c = 0; c < NC; ++c)
                             run[q][c].load(win, at[q] + loff[c] + static_cast<uint32_t>(k * PB));
#pragma unroll
                     for (int t = 0; t < 4; ++t)
#pragma unroll
                         for (int c = 0; c < NC; ++c)
                             if (kBytes || k + t < kmin || k + t < cnt[c]) {
#pragma unroll
                                 for (int q = 0; q < RB; ++q) {
                                     float v[C];
                                     run[q][c].terms(t, v);
#pragma unroll
                                     for (int ch = 0; ch < C; ++ch)
                                         h[q][c][ch] = decltype(first_tag)::value && t == 0
                                                           ? wt[c][t][ch] * v[ch]
                                                           : __builtin_fmaf(wt[c][t][ch], v[ch], h[q][c][ch]);
                                 }
                             }
                 };
                 group(std::true_type{}, 0);
                 for (int32_t k = 4; k < kn; k += 4)
                     group(std::false_type{}, k);
             });
    }
    zeros(y_b - y_a - y);  // a strip without sample rows
}

// grid: column tiles x (strips / wavefronts) x planes
template <class P, typename T, int C>
inline hipError_t launch_gather_walk(const ResizeArgs &a, const GatherShape &g, int32_t res_w, int32_t res_rows,
                                     hipStream_t stream)
{
    const int32_t rows = g.strip * g.waves;
    constexpr int32_t wide = gather_cols(C);
    const dim3 grid((res_w + wide - 1) / wide, (res_rows + rows - 1) / rows, a.planes);
    if (g.big)
        hipLaunchKernelGGL((k_gather_walk<P, T, C, true>), grid, dim3(64, g.waves), g.lds_bytes, stream, a, g);
    else
        hipLaunchKernelGGL((k_gather_walk<P, T, C, false>), grid, dim3(64, g.waves), g.lds_bytes, stream, a, g);
    return hipGetLastError();
}

}  // namespace xr
