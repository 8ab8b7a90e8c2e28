// Source rows staged in LDS by one wavefront.
//
// A walk's wavefront owns an area of LDS and copies the next rows of its
// source window there with direct loads from memory (16 bytes a lane, no
// registers and no branch per load), waits for them once, and filters every
// staged row from LDS. Loads and stores share one counter on gfx950: a walk that
// loads row by row between its stores waits for those stores at every row; this
// one waits for a chunk's stores once, with the next chunk's rows, and where one
// chunk holds a strip, never. Wavefronts are independent (no workgroup barrier), and the rows in flight are bounded by
// LDS, not by registers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "xr_device.hpp"

namespace xr {
namespace dev {

typedef const void __attribute__((address_space(1))) *gptr_t;
typedef void __attribute__((address_space(3))) *lptr_t;

// Pitches that the staged walks take: offsets of a strip's rows stay within
// 32 bits (an image row of 32768 float32 RGBA pixels is 2^19 bytes).
constexpr int64_t kStageMaxPitch = int64_t(1) << 22;

// The window: `bytes` bytes of every source row, from the byte `p` points at
// in row 0 on. Rows lie in LDS as whole 16-byte granules of memory, so row r
// starts mis(r) bytes into its LDS row; a granule is read when it holds at
// least one byte of the window (it cannot cross a page, and the bytes around
// the window are never used).
struct RowStage {
    const unsigned char *base;  // p rounded down to 16 bytes
    uint32_t m0, pitch;
    int32_t bytes, nch;         // window bytes, granules per LDS row
    int32_t front;              // granules left free in front of a row

    __device__ __forceinline__ void init(const unsigned char *p, uint32_t pitch_, int32_t bytes_, int32_t front_,
                                         int32_t back)
    {
        const uint64_t q = reinterpret_cast<uint64_t>(p);
        base = reinterpret_cast<const unsigned char *>(q & ~uint64_t(15));
        m0 = static_cast<uint32_t>(q & 15);
        pitch = pitch_;
        bytes = bytes_;
        front = front_;
        nch = front + back + static_cast<int32_t>(((pitch % 16 == 0 ? m0 : 15u) + static_cast<uint32_t>(bytes) + 15u) / 16u);
    }

    // bytes of an LDS row, and where the window of row r starts in its row
    __device__ __forceinline__ uint32_t lds_pitch() const { return 16u * static_cast<uint32_t>(nch); }
    __device__ __forceinline__ uint32_t start(int32_t r) const
    {
        return 16u * static_cast<uint32_t>(front) + ((m0 + static_cast<uint32_t>(r) * pitch) & 15u);
    }

    // Request rows first .. first + n - 1 into the wavefront's area (n * nch
    // granules). All earlier reads of the area must have returned.
    __device__ __forceinline__ void request(unsigned char *area, int32_t first, int32_t n, int32_t lane) const
    {
        if (pitch % 16 != 0 || front > 0) {  // (rows with free granules have them at both ends)
            request_rows(area, n, lane, [&](int32_t i) { return first + i; });
            return;
        }
        // rows start at one place of a granule and every granule holds window
        // bytes: a lane's next granule is one constant step on, or two
        const int32_t total = n * nch;
        const int32_t dr = 64 / nch, dc = 64 - dr * nch;
        const int32_t r = lane / nch;
        int32_t c = lane - r * nch;
        uint32_t o = static_cast<uint32_t>(first + r) * pitch + 16u * static_cast<uint32_t>(c);
        const uint32_t step = static_cast<uint32_t>(dr) * pitch + 16u * static_cast<uint32_t>(dc);
        const uint32_t wrap = pitch - 16u * static_cast<uint32_t>(nch);
        for (int32_t g = 0; g < total; g += 64) {
            if (g + lane < total)
                __builtin_amdgcn_global_load_lds((gptr_t)(base + o), (lptr_t)(area + 16 * g), 16, 0, 0);
            c += dc;
            o += step;
            if (c >= nch) {
                c -= nch;
                o += wrap;
            }
        }
    }

    // The same for the rows row_of(i), i < n.
    template <class RowOf>
    __device__ __forceinline__ void request_rows(unsigned char *area, int32_t n, int32_t lane, RowOf row_of) const
    {
        const int32_t total = n * nch;
        const int32_t dr = 64 / nch, dc = 64 - dr * nch;
        int32_t r = lane / nch, c = lane - r * nch;
        for (int32_t g = 0; g < total; g += 64) {
            if (g + lane < total) {
                const uint32_t o = m0 + static_cast<uint32_t>(row_of(r)) * pitch;
                const int32_t j = min(max(c - front, 0),
                                      static_cast<int32_t>(((o & 15u) + static_cast<uint32_t>(bytes) - 1u) >> 4));
                __builtin_amdgcn_global_load_lds((gptr_t)(base + ((o & ~15u) + 16u * static_cast<uint32_t>(j))),
                                                 (lptr_t)(area + 16 * g), 16, 0, 0);
            }
            c += dc;
            r += dr;
            if (c >= nch) {
                c -= nch;
                ++r;
            }
        }
    }

    // every load and store of this wavefront has completed
    __device__ __forceinline__ static void wait()
    {
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }

    // every LDS access of this wavefront has completed
    __device__ __forceinline__ static void drain_lds()
    {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
        __builtin_amdgcn_wave_barrier();
    }
};

// BYTES bytes from byte offset `at` of an LDS area into `dst` (whole dwords),
// `at` a multiple of ALIGN. One- and two-byte samples are read as aligned
// dwords, one more than the run holds, and shifted together: an LDS read that
// is not aligned to its size costs many times an aligned one (bilinear
// antialiased planes 375 x 500 -> 224^2: 92 us with unaligned dword reads,
// 39 us so).
template <int BYTES, int ALIGN>
__device__ __forceinline__ void lds_run(unsigned char *dst, const unsigned char *area, uint32_t at)
{
    if constexpr (ALIGN >= 4) {
        __builtin_memcpy(dst, __builtin_assume_aligned(area + at, ALIGN), BYTES);
    } else {
        constexpr int N = (BYTES + 3) / 4;
        uint32_t d[N + 1];
        __builtin_memcpy(d, __builtin_assume_aligned(area + (at & ~3u), 4), 4 * (N + 1));
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const uint32_t x = __builtin_amdgcn_alignbyte(d[j + 1], d[j], at);
            __builtin_memcpy(dst + 4 * j, &x, 4);
        }
    }
}

// Bytes as float32 operands without a conversion: byte j of a dword, masked
// in place, is the bit pattern of the number (byte 2^(8j)) 2^-149 (j < 3; the
// exponent field holds at most 1), the last one after a shift as j = 0. With
// the weight scaled by 2^(126 - 8j) the product is the byte's, times 2^-23,
// and every sum of such products rounds as the unscaled one does (nothing
// here is small enough to lose bits); the row weights carry the 2^23. On
// gfx950 the mask takes a 2-cycle issue slot, v_cvt_f32_ubyte a 4-cycle one
// (measured), and a multiply-add takes 2 with either operand.

// Samples of one staged row that belong to a lane's column: N samples of T, C
// from LDS, then sample t as C operands and their weights.
template <typename T, int C, int N>
struct SampleRun {
    static constexpr int PB = Pix<T, C>::kBytes;
    static constexpr bool kBytes = std::is_same_v<T, uint8_t>;
    unsigned char b[(N * PB + 3) / 4 * 4];

    __device__ __forceinline__ void load(const unsigned char *win, uint32_t at)
    {
        lds_run<N * PB, PB>(b, win, at);
    }
    __device__ __forceinline__ void terms(int t, float (&v)[C]) const
    {
        if constexpr (kBytes && C == 4) {
            uint32_t d;
            __builtin_memcpy(&d, b + 4 * t, 4);
            v[0] = __builtin_bit_cast(float, d & 0xffu);
            v[1] = __builtin_bit_cast(float, d & 0xff00u);
            v[2] = __builtin_bit_cast(float, d & 0xff0000u);
            v[3] = __builtin_bit_cast(float, d >> 24);
        } else if constexpr (kBytes) {
            uint32_t d;
            __builtin_memcpy(&d, b + t / 4 * 4, 4);
            v[0] = __builtin_bit_cast(float, t % 4 == 3 ? d >> 24 : d & (0xffu << (8 * (t % 4))));
        } else {
            Pix<T, C>::load(b, t, v);
        }
    }
};

// Weight of sample t (held as scale<T, C>(t) times the weight) for channel ch.
template <typename T, int C>
__device__ __forceinline__ float sample_scale(int t)
{
    if (!std::is_same_v<T, uint8_t>)
        return 1.0f;
    return C == 4 ? 0x1p110f : t % 4 == 1 ? 0x1p118f : t % 4 == 2 ? 0x1p110f : 0x1p126f;
}
template <typename T, int C>
__device__ __forceinline__ void sample_weights(float w, float (&wt)[C])
{
#pragma unroll
    for (int ch = 0; ch < C; ++ch)
        wt[ch] = !(std::is_same_v<T, uint8_t> && C == 4) ? w
                 : ch == 1                                ? w * 0x1p8f
                 : ch == 2                                ? w
                                                          : w * 0x1p16f;
}

}  // namespace dev
}  // namespace xr
