// The default tiles over sizes, numbers of states, precisions and numbers of systems.
#include <stdio.h>

#include "tile_rule.h"

static int bad = 0;
#define CHECK(c)                                                                                             \
    do {                                                                                                     \
        if (!(c) && ++bad < 20)                                                                              \
            printf("%s: M=%lld Bp=%d precision=%d R=%d: rows %d kslab %d waves %d\n", #c, (long long)M, Bp, \
                   precision, R, t.rows, t.kslab, t.waves);                                                  \
    } while (0)

// bytes of one system's plan on the matrix-core path
static int64_t plan_bytes(int64_t M, int Bp, int precision, const lb_tile& t) {
    auto up = [](int64_t x, int64_t a) { return (x + a - 1) / a * a; };
    const int64_t Mp = up(M, 16), nslab = (M + t.kslab - 1) / t.kslab;
    int64_t b = up(8 * 5, 256);
    for (int i = 0; i < 3; ++i) b = up(b + 8 * up(Mp * Bp, 64), 256);
    if (precision == LB_FP32) b = up(b + 4 * up(Mp * Bp, 128), 256);
    return up(b + 8 * nslab * Mp * Bp, 256);
}

int main() {
    long n = 0;
    for (int Bp : {16, 32, 64})
        for (int precision : {LB_FP64, LB_FP32})
            for (int64_t M = 2; M <= 46340; M += M < 9000 ? 1 : 37) {
                const lb_tile one = lb_default_tile(M, Bp, precision, 1);
                for (int R : {1, 2, 3, 16, 65535}) {
                    const lb_tile t = lb_default_tile(M, Bp, precision, R);
                    ++n;
                    // what the kernels are compiled for
                    CHECK(t.rows == 16 || t.rows == 32 || t.rows == 64);
                    CHECK(t.waves == 1 || t.waves == 2 || t.waves == 4);
                    CHECK(t.kslab > 0 && t.kslab % 32 == 0);
                    // the order of a sum does not depend on what shares the launch
                    CHECK(t.kslab == one.kslab);
                    // 32-bit slab numbers and columns, and no slab beyond the last column
                    CHECK((int64_t)((M + t.kslab - 1) / t.kslab - 1) * t.kslab < M);
                    // FP32 sums a slab in FP32: never a longer one than the long rule's
                    if (precision == LB_FP32) CHECK(t.kslab <= limit_tile(M, Bp).kslab);
                    // what the allocation-free call takes with the long slabs it takes with these
                    if (plan_bytes(M, Bp, precision, limit_tile(M, Bp)) <= (int64_t)LB_NOALLOC_SCRATCH_BYTES)
                        CHECK(plan_bytes(M, Bp, precision, t) <= (int64_t)LB_NOALLOC_SCRATCH_BYTES);
                    // the row thresholds
                    if (precision == LB_FP64 && M < 32768) {
                        if (M >= 8200 && Bp < 64) CHECK(t.rows == 64);
                        if (M >= 3000 && M < 8200) CHECK(t.rows == 32);
                        if (M < 3000 && t.rows != 16) CHECK(t.rows == 32 && M > 2000 && (R > 1 || Bp == 32));
                    }
                    if (precision == LB_FP32 && M < 32768)
                        CHECK(t.rows == (M < 2500 ? 16 : M < 8200 ? 32 : 64));
                }
            }
    printf("%ld tiles, %d bad\n", n, bad);
    return bad != 0;
}
