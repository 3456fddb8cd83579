// Host-logic checks of the structure-aware initialisation's workspace (csrc/sa_layout.h), on the CPU:
// the bytes used fit in the bytes asked for, which stay what they have always been.
#include "sa_layout.h"

#include <stdio.h>

namespace {

int failures = 0;

size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

void check(int H, int W)
{
    const dbmp::SaLayout L = dbmp::sa_layout(H, W);
    const size_t n = (size_t)H * W, nb = (n + 4095) / 4096;
    const size_t want = 256 + up256(16 * ((((size_t)W + 15) / 16) * (((size_t)H + 15) / 16))) +
                        2 * up256(8 * n) + up256(8 * ((n + 2047) / 2048));
    dbmp::lv_shape(H, W);
    const size_t rows = (size_t)dbmp::lv_rows(H, W);
    const size_t nblk = (((size_t)W + 63) / 64) * (((size_t)H + rows - 1) / rows);
    const bool ok = L.total == want && L.used <= L.total && L.minmax == 0 && L.bmm >= 16 &&
                    L.lv >= L.bmm + 16 * nblk && L.gsum >= L.lv + 8 * n &&
                    L.bsum >= L.gsum + 8 * 64 * nb && L.used == L.bsum + 8 * nb &&
                    ((L.bmm | L.lv | L.gsum | L.bsum) & 15) == 0;
    if (!ok) {
        if (failures < 20) fprintf(stderr, "FAILED %d x %d: used %zu of %zu\n", H, W, L.used, want);
        ++failures;
    }
}

}  // namespace

int main()
{
    for (int H = 1; H <= 300; ++H)
        for (int W = 1; W <= 300; ++W) check(H, W);
    for (int s = 1; s <= 1024; s = s * 5 / 4 + 1)  // thin and large ones, up to 2^31 - 1 pixels
        for (long long k = 1; k * s < 2147483647LL; k = k * 9 / 8 + 1) {
            check((int)k, s);
            check(s, (int)k);
        }
    for (long long a = 1025; a < 46340; a = a * 9 / 8 + 1)
        for (long long b = 1025; a * b < 2147483647LL; b = b * 9 / 8 + 1) check((int)a, (int)b);
    check(1, 2147483646);
    check(2147483646, 1);
    if (failures) return 1;
    printf("sa layout checks passed\n");
    return 0;
}
