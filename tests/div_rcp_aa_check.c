// Exhaustive host check of the division in the antialiased weights: for all
// even 2 <= b <= 65536 and integers 0 <= a <= 2 b (every |2 i n_out - num| and
// 2 max(n_in, n_out) with sides up to 32768 and radius up to 2), is
// fma(fma(-q0, b, a), y, q0) with y = RN(1/b), q0 = RN(a y) equal to the
// correctly rounded a / b? Exit status 0 when every pair agrees.
#include <math.h>
#include <stdint.h>
#include <stdio.h>
int main(void)
{
    long long bad = 0, total = 0;
    for (int32_t b = 2; b <= 65536; b += 2) {
        const float bf = (float)b, y = 1.0f / bf;
        long long wrong = 0;
        for (int32_t a = 0; a <= 2 * b; ++a) {
            const float af = (float)a, q0 = af * y;
            const float q = fmaf(fmaf(-q0, bf, af), y, q0);
            wrong += q != af / bf;
        }
        bad += wrong;
        total += 2 * b + 1;
    }
    printf("checked %lld pairs, %lld mismatches\n", total, bad);
    return bad != 0;
}
