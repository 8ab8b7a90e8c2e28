// Forward resize at any ratio for gfx950: the staged walk, for single images
// (k_walk) and for batches of uneven jobs (k_batch_walk).
//
// A wavefront owns 64 PPX adjacent output columns and a strip of output rows:
//  * it copies the next source rows of its window into its own LDS area,
//    several at a time and straight from memory (xr_stage.hpp), waits for
//    them once and filters them from LDS. Columns whose taps lie outside the
//    image read pixels that were replicated behind the staged row's ends, so
//    every column reads its K taps as one run. Where rows shrink so far that
//    the taps of adjacent output rows do not meet, only the rows with taps
//    are staged;
//  * each staged row is filtered once into ring slot (row mod K), all LDS
//    reads of RB rows ahead of their arithmetic, and every output row is
//    emitted as soon as its last tap row is filtered, from slots that are
//    constants of the code;
//  * the output rows' weights are computed once per strip, one row per lane,
//    into a table in LDS that is read a row ahead as a broadcast;
//  * the last run of an image row is moved left to end at the image's edge
//    (its pixels are computed twice, to the same bits), so every store writes
//    a whole run.
// The float32 sequence per output value is the one every kernel uses.
//
// Against the walks it replaced (taps loaded from memory per row between the
// stores of the rows before, whose completion every such load then waits for):
// bicubic x1.3 of a 2479 x 3507 gray uint8 page 58.7 -> 13.0 us, bicubic x1.5 of
// 48 float32 planes of 512^2 196 -> 36 us (4.5 TB/s), bicubic x0.36 of a
// 4000 x 3000 float32 RGBA photo 64.8 -> 44.7 us (4.8 TB/s), bilinear x6 of an
// 800^2 RGBA uint8 image 26.2 -> 21.1 us (4.5 TB/s). Long outputs are bound by
// memory, small ones by the time to a wavefront's first rows.
//
// Batches: the jobs are grouped by kind (filter x channel count), and one launch
// has a workgroup per tile of all of them. The hardware hands the
// tiles out in order; a kind's jobs are ordered largest first, so long tiles
// start early and short ones fill the tail. (Persistent workgroups that drew
// tiles from a counter in memory were bound by it, some 10 ns a tile: 256
// uneven uint8 images up to 2048^2 1,216 us against 975, 32 up to 357^2 102
// against 36.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "xr_buffer.hpp"
#include "xr_device.hpp"
#include "xr_internal.h"
#include "xr_plan.hpp"
#include "xr_stage.hpp"

namespace xr {
using namespace dev;

namespace {

constexpr int32_t kWalkWindow = 6 * 1024;       // bytes of staged rows per wavefront ...
constexpr int32_t kWalkMaxWindow = 17 * 1024;   // ... or four rows, up to this
constexpr int32_t kWalkMaxStrip = 256;          // output rows per strip
constexpr int32_t kWalkSlack = 16;              // bytes read past the last staged row

// Granules (16 bytes) left free at either end of a staged row for the two
// pixels that replicate the image's edge.
constexpr int32_t pad_granules(int32_t pb) { return (2 * pb + 15) / 16; }

// Bytes of one staged row of a wavefront of 64 ppx output columns, at most:
// columns c1 <= c2 have first taps at most floor((c2 - c1) in / out) + 1 apart.
inline int64_t walk_row_bytes(int32_t taps, int32_t pb, int32_t ppx, int64_t in_w, int64_t out_w)
{
    const int64_t px = std::min<int64_t>((64 * ppx - 1) * in_w / out_w + taps + 1, in_w);
    return ((px * pb + 30) / 16 + 2 * pad_granules(pb)) * 16;
}

inline int32_t walk_window(int64_t row_bytes)
{
    return static_cast<int32_t>(std::max<int64_t>(4 * row_bytes, kWalkWindow / (4 * row_bytes) * 4 * row_bytes));
}

// Bytes of the weight table of a strip.
__host__ __device__ constexpr int32_t walk_table(int32_t taps, int32_t rows)
{
    return ((taps + 1) * 4 * rows + 15) / 16 * 16;
}

}  // namespace

// An axis index's base tap and offset by one division, then one step of
// n_in / n_out per index: x0 = q, t = rem / den, as source_tap.
template <int FILTER>
struct AxisSteps {
    int32_t q, rem, den, sq, sr;
    float d, rcp;

    __device__ __forceinline__ void init(int32_t x, int32_t n_in, int32_t n_out, int32_t o)
    {
        den = 2 * n_out;
        const int32_t num = (2 * x + o) * n_in - (FILTER == kNearest ? 0 : o * n_out);
        q = num / den;
        rem = num - q * den;
        if (rem < 0) {
            q -= 1;
            rem += den;
        }
        sq = 2 * n_in / den;
        sr = 2 * n_in - sq * den;
        d = static_cast<float>(den);
        rcp = __fdiv_rn(1.0f, d);
    }
    __device__ __forceinline__ void step()
    {
        q += sq;
        rem += sr;
        if (rem >= den) {
            rem -= den;
            ++q;
        }
    }
    __device__ __forceinline__ void get(float (&w)[Taps<FILTER>::K]) const
    {
        if constexpr (FILTER == kNearest)
            weights<FILTER>(0.0f, 1.0f, w);
        else
            weights<FILTER>(div_rcp(static_cast<float>(rem), d, rcp), div_rcp(static_cast<float>(den - rem), d, rcp), w);
    }
};

// Cache policy of the walk's output stores: non-temporal only. Rows may start
// at any byte offset, so a wavefront's run covers partial lines at both ends;
// measured on uneven batches (plain non-temporal, streaming past the L2 as in the
// exact walks, write-back): 256 uint8 images up to 2048^2 987, 1003 and 913 us,
// 128 float16 ones 805, 915 and 883, 64 float32 ones up to 1500^2 497, 480 and 468.
constexpr int kWalkStore = 2;

template <int FILTER, typename T, int C, int PPX>
struct StagedWalk {
    using TP = Taps<FILTER>;
    static constexpr int K = TP::K, LO = TP::LO;
    static constexpr int PB = Pix<T, C>::kBytes;
    static constexpr int OB = PPX * PB;
    static constexpr bool kBytes = std::is_same_v<T, uint8_t>;
    using Run = SampleRun<T, C, K>;
    // rows whose taps are read ahead of their arithmetic: 4, 2 or 1, within
    // about 40 registers
    static constexpr int kRowWords = PPX * ((K * PB + 3) / 4 + (PB < 4 ? 1 : 0));
    static constexpr int RB = kRowWords <= 10 ? 4 : kRowWords <= 20 ? 2 : 1;

    float wt[PPX][K][C];  // column weights (scaled for bytes, xr_stage.hpp)
    uint32_t off[PPX];    // first tap of each column in a staged row
    float ring[K][PPX][C];
    float wcur[K], wnext[K];
    const float *table;   // [rows][K]
    __amdgpu_buffer_rsrc_t drsrc;
    uint32_t lane_off, dst_off, dst_pitch;
    int32_t yi, rows;     // next output row of the strip, rows of the strip
    int32_t q, rem, den, sq, sr;  // its base tap in walked rows, and the step to the next
    int32_t last;         // walked row that completes it

    __device__ __forceinline__ void read_weights(float (&w)[K], int32_t y) const
    {
        __builtin_memcpy(w, table + min(y, rows - 1) * K, 4 * K);
    }

    template <int I>
    __device__ __forceinline__ void emit()
    {
        float v[PPX][C];
#pragma unroll
        for (int c = 0; c < PPX; ++c) {
            fma_first(v[c], wcur[0], ring[(I + 1) % K][c]);
#pragma unroll
            for (int j = 1; j < K; ++j)
                fma_next(v[c], wcur[j], ring[(I + 1 + j) % K][c]);
        }
        RawBuf<OB, cmin(16, cgcd(OB, 16))> out;
        encode_run<T, C, PPX>(v, out);
        buf_store<OB, kWalkStore>(out.b, drsrc, dst_off + lane_off);
        dst_off += dst_pitch;
        ++yi;
#pragma unroll
        for (int j = 0; j < K; ++j)
            wcur[j] = wnext[j];
        read_weights(wnext, yi + 1);
        q += sq;
        rem += sr;
        if (rem >= den) {
            rem -= den;
            ++q;
        }
        last = q + K - 1;
    }

    // walked row n, read into run, goes to ring slot I
    template <int I>
    __device__ __forceinline__ void step(int32_t n, const Run (&run)[PPX])
    {
#pragma unroll
        for (int c = 0; c < PPX; ++c)
#pragma unroll
            for (int t = 0; t < K; ++t) {
                float v[C];
                run[c].terms(t, v);
#pragma unroll
                for (int ch = 0; ch < C; ++ch) {
                    float &h = ring[I % K][c][ch];
                    h = t == 0 ? wt[c][t][ch] * v[ch] : __builtin_fmaf(wt[c][t][ch], v[ch], h);
                }
            }
        while (last == n && yi < rows)
            emit<I>();
    }

    // Output rows [r_begin, r_end) (band coordinates) of one plane, columns
    // from wave_col0 on; `lds`: this wavefront's walk_table + window bytes.
    __device__ __forceinline__ void run(const ResizeArgs &a, int32_t plane, int32_t wave_col0, int32_t r_begin,
                                        int32_t r_end, unsigned char *lds, int32_t table_bytes, int32_t win_bytes,
                                        int32_t lane)
    {
        const int32_t col0 = wave_col0 + lane * PPX;
        const int32_t c0 = min(col0, a.out_w - PPX);
        lane_off = col0 < a.out_w ? static_cast<uint32_t>(c0 * PB) : 0x80000000u;  // dropped by the resource
        int32_t f[PPX];
        AxisSteps<FILTER> ax;
        ax.init(c0, a.in_w, a.out_w, a.map_off);
        f[0] = ax.q + LO;
#pragma unroll
        for (int c = 1; c < PPX; ++c) {
            int32_t ql = ax.q, rl = ax.rem;
#pragma unroll
            for (int k = 0; k < c; ++k) {
                ql += ax.sq;
                rl += ax.sr;
                if (rl >= ax.den) {
                    rl -= ax.den;
                    ++ql;
                }
            }
            f[c] = ql + LO;
        }
        // the window's columns, and where the strip starts and ends
        const int32_t f_lo = __builtin_amdgcn_readfirstlane(f[0]);
        const int32_t f_hi = __builtin_amdgcn_readlane(f[PPX - 1], 63) + K - 1;
        const int32_t seg0 = clampi(f_lo, 0, a.in_w - 1), seg1 = clampi(f_hi, 0, a.in_w - 1);
        const bool left = f_lo < 0, right = f_hi > a.in_w - 1;
        rows = r_end - r_begin;
        const int32_t y_first = a.dst_row0 + r_begin;
        AxisSteps<FILTER> ay;
        ay.init(y_first, a.in_h, a.out_h, a.map_off);
        AxisSteps<FILTER> az;
        az.init(y_first + rows - 1, a.in_h, a.out_h, a.map_off);
        const int32_t rho0 = __builtin_amdgcn_readfirstlane(ay.q) + LO;
        const int32_t rho1 = __builtin_amdgcn_readfirstlane(az.q) + LO + K - 1;
        // walked rows: every source row from rho0 to rho1, or (gap) the K tap
        // rows of each output row one after the other
        const bool gap = a.in_h > K * a.out_h;
        const int32_t walked = gap ? K * rows : rho1 - rho0 + 1;
        den = ay.den;
        rem = gap ? 0 : __builtin_amdgcn_readfirstlane(ay.rem);
        sr = gap ? 0 : ay.sr;
        sq = gap ? K : ay.sq;
        q = 0;
        last = K - 1;

        float *wtab = reinterpret_cast<float *>(lds);           // [rows][K]
        int32_t *firsts = reinterpret_cast<int32_t *>(wtab + rows * K);
        unsigned char *const win = lds + table_bytes;
        const int32_t band_lo = a.src_row0, band_hi = a.src_row0 + a.src_rows - 1;
        const int32_t r_base = clampi(rho0, band_lo, band_hi);
        RowStage st;
        st.init(a.src + static_cast<int64_t>(plane) * a.src_plane_pitch +
                    static_cast<int64_t>(r_base - a.src_row0) * a.src_pitch + static_cast<int64_t>(seg0) * PB,
                static_cast<uint32_t>(a.src_pitch), (seg1 - seg0 + 1) * PB, left ? pad_granules(PB) : 0,
                right ? pad_granules(PB) : 0);
        const uint32_t lp = st.lds_pitch();
        const int32_t rc = min(win_bytes / static_cast<int32_t>(lp) / 4 * 4, 64);
        // source row of walked row n, counted from r_base
        const auto row_of = [&](int32_t n) {
            const int32_t rho = gap ? firsts[n / K] + n % K : rho0 + n;
            return clampi(rho, band_lo, band_hi) - r_base;
        };

        // row weights (and first tap rows), one output row per lane
        for (int32_t base = 0; base < rows; base += 64) {
            const int32_t i = min(base + lane, rows - 1);
            AxisSteps<FILTER> ar;
            ar.init(y_first + i, a.in_h, a.out_h, a.map_off);
            float w[K];
            ar.get(w);
#pragma unroll
            for (int j = 0; j < K; ++j)
                wtab[i * K + j] = kBytes ? w[j] * 0x1p23f : w[j];
            firsts[i] = ar.q + LO;
        }
        RowStage::drain_lds();
        st.request_rows(win, min(rc, walked), lane, row_of);

        // column weights, while the first rows arrive
#pragma unroll
        for (int c = 0; c < PPX; ++c) {
            float w[K];
            ax.get(w);
            ax.step();
#pragma unroll
            for (int t = 0; t < K; ++t)
                sample_weights<T, C>(w[t] * sample_scale<T, C>(t), wt[c][t]);
            off[c] = static_cast<uint32_t>((f[c] - seg0) * PB);
        }
        table = wtab;
        yi = 0;
        read_weights(wcur, 0);
        read_weights(wnext, 1);
        unsigned char *dbase = a.dst + static_cast<int64_t>(plane) * a.dst_plane_pitch +
                               static_cast<int64_t>(r_begin) * a.dst_pitch;
        drsrc = buf_rsrc(dbase, static_cast<uint32_t>(static_cast<int64_t>(rows) * a.dst_pitch));
        dst_pitch = static_cast<uint32_t>(a.dst_pitch);
        dst_off = 0;

        for (int32_t base = 0; base < walked; base += rc) {
            const int32_t n = min(rc, walked - base);
            if (base > 0) {
                RowStage::drain_lds();
                st.request_rows(win, n, lane, [&](int32_t i) { return row_of(base + i); });
            }
            RowStage::wait();
            const int32_t li = min(lane, n - 1);  // lane i holds where staged row i starts
            const uint32_t place = static_cast<uint32_t>(li) * lp + st.start(row_of(base + li));
            if (left || right) {  // replicate the image's edge pixels
                if (lane < n) {
                    unsigned char *p = win + place;
                    unsigned char *e = p + (seg1 - seg0) * PB;
#pragma unroll
                    for (int k = 1; k <= 2; ++k) {
                        if (left)
                            store_raw<PB, PB>(p - k * PB, load_raw<PB, PB>(p));
                        if (right)
                            store_raw<PB, PB>(e + k * PB, load_raw<PB, PB>(e));
                    }
                }
                RowStage::drain_lds();
            }
            for (int32_t i = 0; i < n; i += 4) {
                // slots are walked row mod 4 (K divides 4, chunks hold whole fours)
                auto block = [&](auto first_tag) __attribute__((always_inline)) {
                    constexpr int Q = decltype(first_tag)::value;
                    if (i + Q >= n)
                        return;
                    Run run[RB][PPX];
#pragma unroll
                    for (int b = 0; b < RB; ++b) {
                        const uint32_t at = __builtin_amdgcn_readlane(place, min(i + Q + b, n - 1));
#pragma unroll
                        for (int c = 0; c < PPX; ++c)
                            run[b][c].load(win, at + off[c]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    step<Q>(base + i + Q, run[0]);
                    if constexpr (RB > 1) {
                        if (i + Q + 1 < n)
                            step<Q + 1>(base + i + Q + 1, run[1]);
                    }
                    if constexpr (RB > 2) {
                        if (i + Q + 2 < n)
                            step<Q + 2>(base + i + Q + 2, run[2]);
                        if (i + Q + 3 < n)
                            step<Q + 3>(base + i + Q + 3, run[3]);
                    }
                };
                block(std::integral_constant<int, 0>{});
                if constexpr (RB == 1)
                    block(std::integral_constant<int, 1>{});
                if constexpr (RB <= 2)
                    block(std::integral_constant<int, 2>{});
                if constexpr (RB == 1)
                    block(std::integral_constant<int, 3>{});
            }
        }
    }
};

template <int FILTER, typename T, int C, int PPX>
__global__ void __launch_bounds__(512, 4) k_walk(ResizeArgs a, int32_t strip_h, int32_t order, int32_t table_bytes,
                                                 int32_t win_bytes)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    int32_t bx, by;
    tile_coords(order, bx, by);
    const int32_t lane = static_cast<int32_t>(threadIdx.x) & 63;
    const int32_t wx = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(threadIdx.x) >> 6);
    const int32_t wy = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(threadIdx.y));
    const int32_t bw = static_cast<int32_t>(blockDim.x);
    const int32_t col0 = (bx * bw + wx * 64) * PPX;
    const int32_t r_begin = (by * static_cast<int32_t>(blockDim.y) + wy) * strip_h;
    if (col0 >= a.out_w || r_begin >= a.dst_rows)
        return;
    const int32_t wave = wy * (bw >> 6) + wx;
    StagedWalk<FILTER, T, C, PPX> w;
    w.run(a, blockIdx.z, col0, r_begin, min(r_begin + strip_h, a.dst_rows),
          lds + wave * (table_bytes + win_bytes + kWalkSlack), table_bytes, win_bytes, lane);
}

// kind = 2 * bicubic + four channels
constexpr int32_t batch_kind(int filter, int channels) { return (filter == kBicubic ? 2 : 0) + (channels == 4 ? 1 : 0); }

// A workgroup's tile of the jobs of one kind: waves_w x waves_h strips of
// 64 PPX columns by strip_h rows of one plane of one job. The wavefronts share
// the workgroup's LDS; a job of long staged rows leaves some of them idle.
template <int FILTER, typename T, int C>
__device__ __forceinline__ void batch_walk_tile(const unsigned char *__restrict__ ws, int64_t tile,
                                                unsigned char *lds)
{
    constexpr int32_t kind = batch_kind(FILTER, C);
    constexpr int PPX = batch_ppx(FILTER == kBicubic ? XR_BICUBIC : XR_BILINEAR,
                                  std::is_same_v<T, uint8_t> ? XR_U8 : std::is_same_v<T, float> ? XR_F32 : XR_F16, C);
    const int32_t tid = static_cast<int32_t>(threadIdx.y * blockDim.x + threadIdx.x);
    const int32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int32_t plane, tx, ty;
    BatchJob job;
    if (!batch_tile(ws, kind, tile, job, plane, tx, ty))
        return;
    const ResizeArgs &a = job.a;
    int32_t wx = wave, wy = 0;
    while (wx >= job.waves_w) {
        wx -= job.waves_w;
        ++wy;
    }
    const int32_t col0 = (tx * job.waves_w + wx) * 64 * PPX;
    const int32_t r_begin = (ty * job.waves_h + wy) * job.strip_h;
    if (wy < job.waves_h && col0 < a.out_w && r_begin < a.dst_rows) {
        const int32_t mine = reinterpret_cast<const BatchHeader *>(ws)->lds_bytes / (job.waves_w * job.waves_h) / 16 * 16;
        const int32_t table_bytes = walk_table(Taps<FILTER>::K, job.strip_h);
        StagedWalk<FILTER, T, C, PPX> w;
        w.run(a, plane, col0, r_begin, min(r_begin + job.strip_h, a.dst_rows),
              lds + wave * mine, table_bytes, mine - table_bytes - kWalkSlack, tid & 63);
    }
}

// Batches of one kind: a workgroup per tile.
template <int FILTER, typename T, int C>
__global__ void __launch_bounds__(256, 4) k_batch_walk(const unsigned char *__restrict__ ws)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    batch_walk_tile<FILTER, T, C>(ws, batch_block(), lds);
}

// Two series of tiles in one: of n in all, a of the first, spread evenly.
struct Interleave {
    uint64_t step;  // ceil(2^32 a / n)
    uint32_t a;

    void init(int64_t a_, int64_t n)
    {
        a = static_cast<uint32_t>(a_);
        step = n > 0 ? ((static_cast<uint64_t>(a_) << 32) + n - 1) / n : 0;
    }
    // tile `t` (below n < 2^31) is of the first series; t becomes its place in
    // its own. min(a, floor(t step / 2^32)) of the tiles below t are.
    __device__ __forceinline__ bool first(uint32_t &t) const
    {
        const uint32_t lo = min(a, static_cast<uint32_t>((t * step) >> 32));
        const uint32_t hi = min(a, static_cast<uint32_t>((t * step + step) >> 32));
        const bool mine = hi > lo;
        t = mine ? lo : t - lo;
        return mine;
    }
};

// Batches of several kinds: one launch of all their tiles, the kinds
// interleaved, so that a batch has one last wave instead of four and the
// one-channel and bicubic tiles, which instructions bound, share the chip with
// the bilinear RGBA ones, which memory bounds. Launched kind by kind and so, in
// processes in turn: 16 uneven uint8 images up to 256^2 29.3 and 11.2 us, 64 up to
// 700^2 75 and 57, 128 up to 1200^2 240 and 201, 128 up to 2048^2 493 and 424, 256
// up to 2048^2 984 to 995 and 955; float16 64 up to 1000^2 135 and 124, 128 up to
// 2048^2 913 and 790; float32 64 up to 1500^2 502 and 496, 256 up to 2048^2 2853
// and 2640. (The 256 uint8 images take 940 to 990 us by card and process, for a
// cause not found: kind by kind 980 to 1010.)
// A batch of one kind has its own kernel, of fewer registers.
struct BatchMix {
    Interleave four, cubic1, cubic4;  // RGBA of all, bicubic of the one-channel and of the RGBA tiles
    int32_t tiles;
};
template <typename T>
__global__ void __launch_bounds__(256, 4) k_batch_mix(const unsigned char *__restrict__ ws, BatchMix mix)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int64_t block = batch_block();
    if (block >= mix.tiles)
        return;
    uint32_t t = static_cast<uint32_t>(block);
    if (mix.four.first(t)) {
        if (mix.cubic4.first(t))
            batch_walk_tile<kBicubic, T, 4>(ws, t, lds);
        else
            batch_walk_tile<kBilinear, T, 4>(ws, t, lds);
    } else {
        if (mix.cubic1.first(t))
            batch_walk_tile<kBicubic, T, 1>(ws, t, lds);
        else
            batch_walk_tile<kBilinear, T, 1>(ws, t, lds);
    }
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------

namespace {

// Output columns per thread that the walk is built for: runs of up to 16
// bytes, and few enough that the ring of filtered rows stays in registers.
constexpr bool walk_ppx_ok(int32_t taps, int32_t channels, int32_t pixel_bytes, int32_t ppx)
{
    return ppx * pixel_bytes <= 16 && (channels == 4 ? ppx <= 4 : ppx >= 4) && ppx * channels * taps <= 32;
}

template <int FILTER, typename T, int C, int PPX>
hipError_t launch_walk_ppx(const ResizeArgs &a, const xr_tile &tile, hipStream_t stream, bool &taken, Route *only)
{
    constexpr int K = Taps<FILTER>::K, PB = Pix<T, C>::kBytes;
    constexpr int32_t kType = std::is_same_v<T, uint8_t> ? XR_U8 : std::is_same_v<T, float> ? XR_F32 : XR_F16;
    constexpr int32_t kFilter = FILTER == kBicubic ? XR_BICUBIC : FILTER == kNearest ? XR_NEAREST : XR_BILINEAR;
    const int64_t row_bytes = walk_row_bytes(K, PB, PPX, a.in_w, a.out_w);
    // source rows a strip reads; offsets within them stay below 2^31
    const auto src_rows = [&](int64_t rows) { return std::min<int64_t>((rows - 1) * a.in_h / a.out_h + K + 1, a.in_h); };
    int64_t strip = std::min<int64_t>(tile.ppt_y, kWalkMaxStrip);
    const int64_t pitch = std::max(a.src_pitch, a.dst_pitch);
    while (strip > 1 && std::max(src_rows(strip), strip) * pitch >= (int64_t(1) << 30))
        strip /= 2;
    const int32_t table = walk_table(K, static_cast<int32_t>(strip));
    const int32_t win = walk_window(row_bytes);
    if (pitch > kStageMaxPitch || 4 * row_bytes > kWalkMaxWindow || a.out_w < PPX)
        return hipSuccess;
    // A named strip tile on an output too small for the walk's default: the
    // per-tap strips start without tables or staged rows, which pays where a
    // column has four channels, or a strip of more than two output rows walks
    // several source rows for each. Measured as named, 156 small resizes: 16-
    // and 8-byte-run RGBA tiles ran at 0.63 to 1.03 of the per-tap speed (2 of
    // 44 above), shrinking float16 and float32 ones of one channel in taller
    // strips at 0.79 to 1.13 (one above); the other one-channel tiles at 0.96 to
    // 2.4, and so they walk.
    if (tile.kernel == XR_KERNEL_STRIP && !walk_default(kFilter, kType, C, a.in_w, a.out_w, a.dst_rows, a.planes) &&
        (C == 4 || (PB > 1 && a.in_h > a.out_h && tile.ppt_y > 2)))
        return hipSuccess;
    // fewer wavefronts a workgroup where those of the tile pass the LDS limit
    // (one fits always: 17 KiB and a table of 5)
    int32_t block_w = tile.block_w, block_h = tile.block_h;
    const auto lds = [&] { return static_cast<int64_t>(block_w / 64 * block_h) * (table + win + kWalkSlack); };
    while (lds() > kStageMaxLds) {
        int32_t &side = block_h > 1 ? block_h : block_w;
        side = block_h > 1 ? side / 2 : side / 128 * 64;
    }
    const int64_t rows_per_block = strip * block_h;
    const int64_t gy = (a.dst_rows + rows_per_block - 1) / rows_per_block;
    if (gy > 65535)
        return hipSuccess;
    taken = true;
    if (just_named(only, kRouteWalk))
        return hipSuccess;
    const int32_t cols_per_block = block_w * PPX;
    hipLaunchKernelGGL((k_walk<FILTER, T, C, PPX>),
                       dim3((a.out_w + cols_per_block - 1) / cols_per_block, static_cast<uint32_t>(gy), a.planes),
                       dim3(block_w, block_h), static_cast<size_t>(lds()), stream, a,
                       static_cast<int32_t>(strip), tile.order, table, win);
    return hipGetLastError();
}

template <int FILTER, typename T, int C>
hipError_t launch_walk_typed(const ResizeArgs &a, const xr_tile &tile, hipStream_t stream, bool &taken, Route *only)
{
    // the LDS strip shapes name the columns of a workgroup, not of a thread
    const int32_t ppx = tile.kernel == XR_KERNEL_STRIP_LDS ? walk_ppx(C, Pix<T, C>::kBytes) : tile.ppt_x;
#define XR_WALK_CASE(P)                                                              \
    case P:                                                                          \
        if constexpr (walk_ppx_ok(Taps<FILTER>::K, C, Pix<T, C>::kBytes, P))             \
            return launch_walk_ppx<FILTER, T, C, P>(a, tile, stream, taken, only);   \
        return hipSuccess;
    switch (ppx) {
        XR_WALK_CASE(1)
        XR_WALK_CASE(2)
        XR_WALK_CASE(4)
        XR_WALK_CASE(8)
        XR_WALK_CASE(16)
    default:
        return hipSuccess;
    }
#undef XR_WALK_CASE
}

template <int FILTER>
hipError_t launch_walk_filter(const ResizeArgs &a, int32_t dtype, int32_t channels, const xr_tile &tile,
                              hipStream_t stream, bool &taken, Route *only)
{
    switch (dtype) {
    case XR_U8:
        return channels == 4 ? launch_walk_typed<FILTER, uint8_t, 4>(a, tile, stream, taken, only)
                             : launch_walk_typed<FILTER, uint8_t, 1>(a, tile, stream, taken, only);
    case XR_F16:
        return channels == 4 ? launch_walk_typed<FILTER, _Float16, 4>(a, tile, stream, taken, only)
                             : launch_walk_typed<FILTER, _Float16, 1>(a, tile, stream, taken, only);
    default:
        return channels == 4 ? launch_walk_typed<FILTER, float, 4>(a, tile, stream, taken, only)
                             : launch_walk_typed<FILTER, float, 1>(a, tile, stream, taken, only);
    }
}

template <typename T, int FILTER, int C>
struct BatchKind {
    static constexpr int32_t kKind = batch_kind(FILTER, C);
    static void launch(const unsigned char *ws, dim3 block, const BatchLaunch &l, hipStream_t stream)
    {
        if (l.grid[kKind] > 0)
            hipLaunchKernelGGL((k_batch_walk<FILTER, T, C>), batch_grid(l.grid[kKind]), block, l.lds_bytes, stream, ws);
    }
};

template <typename T>
void launch_kinds(const unsigned char *ws, dim3 block, const BatchLaunch &l, hipStream_t stream)
{
    const int64_t one = int64_t(l.grid[0]) + l.grid[2], four = int64_t(l.grid[1]) + l.grid[3];
    int kinds = 0;
    for (int32_t k = 0; k < kBatchNarrow; ++k)
        kinds += l.grid[k] > 0;
    if (kinds > 1 && one + four < (int64_t(1) << 31)) {
        BatchMix mix;
        mix.four.init(four, one + four);
        mix.cubic1.init(l.grid[2], one);
        mix.cubic4.init(l.grid[3], four);
        mix.tiles = static_cast<int32_t>(one + four);
        hipLaunchKernelGGL(k_batch_mix<T>, batch_grid(mix.tiles), block, l.lds_bytes, stream, ws, mix);
        return;
    }
    BatchKind<T, kBilinear, 1>::launch(ws, block, l, stream);
    BatchKind<T, kBilinear, 4>::launch(ws, block, l, stream);
    BatchKind<T, kBicubic, 1>::launch(ws, block, l, stream);
    BatchKind<T, kBicubic, 4>::launch(ws, block, l, stream);
}

}  // namespace

hipError_t launch_walk(const ResizeArgs &a, int32_t filter, int32_t dtype, int32_t channels, const xr_tile &tile,
                       hipStream_t stream, bool &taken, Route *only)
{
    if (filter == XR_BICUBIC)
        return launch_walk_filter<kBicubic>(a, dtype, channels, tile, stream, taken, only);
    if (filter == XR_NEAREST)
        return launch_walk_filter<kNearest>(a, dtype, channels, tile, stream, taken, only);
    return launch_walk_filter<kBilinear>(a, dtype, channels, tile, stream, taken, only);
}

bool walk_fits(int32_t filter, int32_t dtype, int32_t channels, int32_t in_w, int32_t out_w)
{
    const int32_t taps = filter == XR_BICUBIC ? 4 : filter == XR_NEAREST ? 1 : 2;
    const int32_t pb = (dtype == XR_U8 ? 1 : dtype == XR_F16 ? 2 : 4) * channels;
    const int32_t ppx = walk_ppx(channels, pb);
    return out_w >= ppx && 4 * walk_row_bytes(taps, pb, ppx, in_w, out_w) <= kWalkMaxWindow;
}

bool walk_built(int32_t filter, int32_t dtype, int32_t channels, int32_t ppx)
{
    return walk_ppx_ok(filter == XR_BICUBIC ? 4 : filter == XR_NEAREST ? 1 : 2, channels,
                       (dtype == XR_U8 ? 1 : dtype == XR_F16 ? 2 : 4) * channels, ppx);
}

BatchWalkNeed batch_walk_need(const ResizeArgs &a, int32_t filter, int32_t dtype, int32_t channels, int32_t strip)
{
    const int32_t taps = filter == XR_BICUBIC ? 4 : 2;
    const int32_t pb = (dtype == XR_U8 ? 1 : dtype == XR_F16 ? 2 : 4) * channels;
    const int32_t ppx = batch_ppx(filter, dtype, channels);
    const int64_t row_bytes = walk_row_bytes(taps, pb, ppx, a.in_w, a.out_w);
    BatchWalkNeed n;
    // (the walk stores through a resource of its strip: one row has to fit)
    n.ok = a.out_w >= ppx && 4 * row_bytes <= kWalkMaxWindow && a.src_pitch <= kStageMaxPitch &&
           a.dst_pitch < kResourceBytes;
    n.win_bytes = walk_window(row_bytes);
    n.wave_bytes = (walk_table(taps, strip) + n.win_bytes + kWalkSlack + 15) / 16 * 16;
    return n;
}

hipError_t launch_batched(const void *ws, int32_t dtype, const BatchLaunch &l, hipStream_t stream)
{
    const unsigned char *p = static_cast<const unsigned char *>(ws);
    const dim3 block(l.block_w, l.block_h, 1);
    if (dtype == XR_U8)
        launch_kinds<uint8_t>(p, block, l, stream);
    else if (dtype == XR_F16)
        launch_kinds<_Float16>(p, block, l, stream);
    else
        launch_kinds<float>(p, block, l, stream);
    if (l.grid[kBatchNarrow] > 0)
        return launch_batch_narrow(p, dtype, block, l.grid[kBatchNarrow], stream);
    return hipGetLastError();
}

}  // namespace xr
