// The default tile of a block of states and the limits that go with it: plain host code,
// so that its properties are checked without a device.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "../../include/lindblad.h"

struct lb_tile {
    int rows;   // rows per wave (multiple of 16)
    int kslab;  // columns per split-K slab (multiple of 16)
    int waves;  // waves per workgroup
};

// Slabs of at least 256 columns (384 for 64 states), for about 2500 row-waves x
// slabs (5000 for 32 and 64 states) with tiles of 64 (32) rows: the slab length
// of large M, and the measure of the allocation-free call's limit.
static inline int64_t long_slabs(int64_t M, int Bp) {
    const int CT = Bp / 16;
    const int64_t rowwaves = CT == 1 ? (M + 63) / 64 : (M + 31) / 32;
    const int64_t target = CT == 1 ? 2500 : 5000;
    const int64_t maxslab = std::max<int64_t>(1, M / (CT == 4 ? 384 : 256));
    return std::max<int64_t>(1, std::min((target + rowwaves - 1) / rowwaves, maxslab));
}

// FP64 blocks up to this size run a stage as one launch (k_block64) unless a tile was
// set for them. A workgroup per 16 rows fills the chip in whole rounds: up to 128 row
// tiles two systems fit one round and up to 169 three of them fit two; beyond, two or
// three systems lose more than one gains (64 states, which keep a CU busier, from 128
// on). In us a stage, GEMM and combination / one launch:
//   16 states:  N = 17  9.8 / 6.2    N = 30  12.3 / 9.1    N = 45  18.0 / 14.6
//   64 states:  N = 17  12.1 / 8.1   N = 30  17.5 / 14.8   N = 45  29.4 / 26.4
//   N = 51, 32 states, 1, 2, 3 systems:  25.5 / 23.6  40.0 / 37.4  59.1 / 40.1
//   N = 49, 64 states, 2 systems 53 / 56; N = 58, 32 states, 3 systems 78 / 90
static inline int64_t whole_limit(int Bp) { return Bp == 64 ? 2048 : 2704; }

// Default tile from sweeps on MI355X (LDS-staged kernels). A stage of one system
// is fastest with one wave per SIMD (1024, just under rather than just over) and
// as few slabs as that takes: more waves mean more partial sums, more rows in
// flight at once and a second round that is nearly empty. With 16 states, in us
// a stage (2500 waves of 64 rows before / now):
//   N = 20   16 rows   25 / 9.4       N = 80   32 rows   81 / 58
//   N = 30   16 rows   22 / 11        N = 100  64 rows  162 / 132
//   N = 60   32 rows   36 / 27        N = 128  64 rows  409 / 333
// (k_block64 takes the smallest of these sizes where no tile is asked for; a server's
// mixed batches and stage timings still run them as tiles).
// Hence tiles of 16 rows below M = 3000 (FP32: 2500), of 32 below 8200, of 64 beyond
// (32 for 64 states in FP64, which fits two waves of that size on a SIMD), and as many
// slabs as keep row tiles x slabs within 1024, or within 2048 where that fills
// the last round better. From M = 32768 on the waves of one system fill the chip
// several times over and the stage runs at the read stream's rate: about 2500
// waves there (N = 200, two systems: 3857 us a stage; with 1875 waves 3932).
// Several systems of M = 2000 to 3000 have waves enough with tiles of 32 rows, one to a
// workgroup (16 states, N = 53, R = 4: 62 us with the long slabs' 64 rows, 60 with 16,
// 54 with 32); 64 states then need the long rule's slabs, up to six of them (N = 51,
// R = 1, 2, 3: 43, 51, 75 us with the long rule's tile, 35, 58, 83 with five slabs of 16
// rows, 31, 48, 74 now), and 32 states have no better tile there than the long rule's.
// FP32 keeps the long rule's slabs at every size: a slab is summed in FP32, so its
// length is the sum's accuracy (N = 99, 50 states: with 6 slabs instead of 17 the
// stage is 1.3 times as fast and the error 1.7 times as large).
// Slabs are a multiple of 32 columns (128 bytes of FP32, 256 of FP64) so that
// every slab starts on a line. The slab length fixes the summation order, so it
// depends on (M, Bp) and the precision only and never on how many systems share
// a launch: a system's result is bit-identical alone and batched.
static inline lb_tile lb_default_tile(int64_t M, int Bp, int precision, int R) {
    lb_tile t;
    const int CT = Bp / 16;
    t.rows = M < (precision == LB_FP32 ? 2500 : 3000) ? 16 : M < 8200 ? 32 : 64;
    t.waves = 4;
    int64_t nslab;
    if (M >= 32768) {
        t.rows = CT == 1 || precision == LB_FP32 ? 64 : 32;
        t.waves = CT == 1 ? 2 : 1;
        nslab = long_slabs(M, Bp);
    } else if (precision == LB_FP32) {
        t.waves = 1;
        nslab = long_slabs(M, Bp);
    } else {
        const int64_t tiles = (M + t.rows - 1) / t.rows, groups = (tiles + 3) / 4;
        if (t.rows == 16) {
            nslab = std::min<int64_t>(5, (M + 63) / 64);
            if (M > whole_limit(Bp)) {
                if (CT == 4) nslab = std::min(long_slabs(M, Bp), std::max<int64_t>(5, 1024 / tiles));
                if (CT == 2) nslab = long_slabs(M, Bp);
            }
        } else {
            const int64_t n1 = std::max<int64_t>(1, 1024 / tiles), n2 = std::max<int64_t>(1, 2048 / tiles);
            // two rounds, with twice the partial sums, where they are filled 15 % better than one
            nslab = std::min<int64_t>(t.rows == 64 && n2 * 100 > n1 * 2 * 115 ? n2 : n1, 9);
        }
        // workgroups of four waves (they share X's lines) where those do not start another round
        if (groups * nslab > 256 * ((tiles * nslab + 1023) / 1024)) t.waves = 1;
        // no more partial sums than the allocation-free call holds, where the longer slabs fit it
        // (three and a half packed states besides them)
        const int64_t lim = (((int64_t)LB_NOALLOC_SCRATCH_BYTES - 4096) / (4 * (M + 16) * Bp) - 7) / 2;
        nslab = std::min(nslab, std::max(lim, long_slabs(M, Bp)));
        if (CT == 4 && t.rows == 64) t.rows = 32;
        if (t.rows == 16 && M > 2000 && (R > 1 || (CT == 2 && M > whole_limit(Bp)))) {
            t.rows = 32;
            t.waves = 1;
        }
    }
    int64_t ks = (M + nslab - 1) / nslab;
    ks = (ks + 31) / 32 * 32;
    t.kslab = (int)ks;
    return t;
}

// The tile whose scratch the allocation-free call's limit is stated for: the long
// slabs, whatever the default tile of that size (a size refused stays refused).
static inline lb_tile limit_tile(int64_t M, int Bp) {
    lb_tile t;
    t.rows = Bp == 16 ? 64 : 32;
    t.waves = 1;
    const int64_t ns = long_slabs(M, Bp);
    t.kslab = (int)(((M + ns - 1) / ns + 31) / 32 * 32);
    return t;
}
