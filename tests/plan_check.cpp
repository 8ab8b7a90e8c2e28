// Host check of the strip heights: for every tile height, row ratio and a
// sweep of row pitches, the output rows of a strip stay below 2^31 bytes (the
// offset of a dropped store) wherever one row does, and so do its source rows
// wherever K + 2 of them do. Exit status 0 when all hold.
#include <stdio.h>

#include "../paper_1001_1718_amd/csrc/xr_plan.hpp"

int main()
{
    long long bad = 0, total = 0;
    const int sides[] = {1, 2, 3, 7, 30, 224, 1000, 4096, 32767, 32768};
    for (int64_t base = 16; base < (int64_t(1) << 31); base *= 2)
        for (int64_t pitch : {base, base + base / 2, 2 * base - 4})
            for (int32_t ppt : {1, 2, 8, 14, 24, 190, 256})
                for (int in_h : sides)
                    for (int out_h : sides) {
                        const int64_t by_dst = xr::batch_strip(ppt, in_h, out_h, 16, pitch);
                        const int64_t by_src = xr::batch_strip(ppt, in_h, out_h, pitch, 16);
                        const int64_t rows = (by_src - 1) * in_h / out_h + 5;
                        bad += by_dst < 1 || by_dst > ppt || by_dst * pitch >= (int64_t(1) << 31);
                        bad += by_src < 1 || by_src > ppt || (by_src > 1 && rows * pitch >= (int64_t(1) << 31));
                        total += 2;
                    }
    // the exact-ratio walks: whole steps, and 2 strip + 8 rows below 2^31 bytes
    // or no strip at all, which only pitches of 2^27 bytes and more get
    for (int64_t base = 16; base < (int64_t(1) << 33); base *= 2)
        for (int64_t pitch : {base, base + base / 2, 2 * base - 4})
            for (int32_t ppt = 1; ppt <= 4096; ppt = ppt * 3 / 2 + 1) {
                const auto check = [&](int64_t strip, int64_t step) {
                    bad += strip % step != 0 || (strip == 0 && pitch < (int64_t(1) << 27)) ||
                           (strip > 0 && (2 * strip + 8) * pitch >= (int64_t(1) << 31));
                    ++total;
                };
                check(xr::x2_pairs(ppt, pitch), 4);
                check(xr::x05_rows(ppt, pitch), 2);
                check(xr::bwd_x2_rows(pitch), 4);
            }
    printf("checked %lld strips, %lld too long\n", total, bad);
    return bad != 0;
}
