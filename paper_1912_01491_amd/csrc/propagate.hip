// RK4 integration of dv/dt = Q v + K (Eq. (10); Table 1 step 3.1).
//
// Classic fourth-order Runge-Kutta with constant K:
//   k1 = f(v), k2 = f(v + h/2 k1), k3 = f(v + h/2 k2), k4 = f(v + h k3),
//   v <- v + h/6 (k1 + 2 k2 + 2 k3 + k4),   f(x) = Q x + K.
// Every stage streams Q once, so the integrator is bound by HBM bandwidth for
// a few states and by the matrix cores for many.
//
// Dense paths (per stage):
//   * B = 1: k_gemv -- one wavefront per group of rows, lanes along the row,
//     cross-lane reduction, stage combine fused into the same kernel; for one
//     system of 256 < M <= 4096, rk4_resident.h -- one launch runs all steps
//     with Q on the chip.
//   * B >= 2: k_gemm64 / k_gemm32 -- split-K GEMM on the matrix cores
//     (v_mfma_f64_16x16x4f64, v_mfma_f32_16x16x4f32) writing per-slab
//     partial sums, followed by k_stage which reduces the slabs in a fixed
//     order (deterministic, no atomics) and applies the RK4 combination.
//     FP64 up to M = 2704 (2048 for more than 32 states): k_block64 -- the whole
//     stage in one launch, a workgroup per 16 rows.
//   * M <= 256 and B*M <= 4096: rk4_small.h -- one workgroup per state runs
//     all steps with Q in registers.
// State layout inside the library: states are padded to Bp in {16, 32, 64}
// columns and stored "pair-interleaved", X[(k>>1)*2Bp + 2b + (k&1)], so that
// the 16-byte load a lane issues holds two consecutive k of one state -- the
// B-operand of two MFMAs whose A-operand is the two consecutive Q columns the
// same lane loaded. The FP32 path interleaves by four.
#include <mutex>

#include "lb_internal.h"
#include "rk4_resident.h"
#include "rk4_small.h"
#include "rowdot.h"
#include "sell.h"

#include <math.h>

#include <algorithm>
#include <type_traits>
#include <cstring>
#include <stdio.h>
#include <stdlib.h>

typedef double lb_double4 __attribute__((ext_vector_type(4)));
typedef float lb_float4 __attribute__((ext_vector_type(4)));
typedef unsigned int lb_u4 __attribute__((ext_vector_type(4)));

namespace {

__host__ __device__ __forceinline__ int64_t ilv2(int64_t k, int b, int Bp) { return (k >> 1) * (2 * Bp) + 2 * b + (k & 1); }
__host__ __device__ __forceinline__ int64_t ilv4(int64_t k, int b, int Bp) { return (k >> 2) * (4 * Bp) + 4 * b + (k & 3); }

// Work decomposition of a stage GEMM launch: gx row blocks x nslab k-slabs x R
// systems, launched as a 1-D grid. Workgroups are handed to the 8 XCDs round
// robin by workgroup id, so workgroup b runs on XCD b % 8; it is given work item
// w = (b % 8) * per_xcd + b / 8, i.e. each XCD walks one contiguous range of
// the slab-major work list and keeps the few X slabs it is reading resident in
// its own L2.
struct GemmGrid {
    int gx, nslab, R;
    int64_t per_xcd;
};

__device__ __forceinline__ bool gemm_work(const GemmGrid& g, int& x, int& slab, int& r) {
    const int64_t b = blockIdx.x;
    const int64_t w = (b & 7) * g.per_xcd + (b >> 3);
    if (w >= (int64_t)g.gx * g.nslab * g.R) return false;
    x = (int)(w % g.gx);
    const int64_t cmb = w / g.gx;
    slab = (int)(cmb % g.nslab);
    r = (int)(cmb / g.nslab);
    return true;
}

// ---------------------------------------------------------------------------
// Matrix-core stage GEMM, FP64: Part[slab] = Q[:, slab] X[slab, :]
// ---------------------------------------------------------------------------
// A wave owns RT row tiles of 16 rows and CT column tiles of 16 states over one
// k-slab. Lane l loads Q[row0 + 16t + (l%16)][kc + 2(l/16) + {0,1}] (16 bytes)
// and X[kc + 2(l/16) + {0,1}][16c + (l%16)]; the MFMA k-index j = l/16 maps to
// column kc + 2j (first MFMA) and kc + 2j + 1 (second).
template <int RT, int CT, bool ALIGNED>
__global__ __launch_bounds__(256) void k_gemm64(const double* const* Qs, int64_t M, int64_t Mp, int64_t ldq,
                                                const double* Xall, int64_t xstride, double* Pall,
                                                int64_t pstride, int kslab, GemmGrid gg) {
    constexpr int Bp = 16 * CT;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    int bx, slab, r;
    if (!gemm_work(gg, bx, slab, r)) return;
    const double* Q = Qs[r];
    const double* X = Xall + r * xstride;
    double* Part = Pall + r * pstride + (int64_t)slab * Mp * Bp;
    const int64_t row0 = ((int64_t)bx * (blockDim.x >> 6) + wave) * (16 * RT);
    if (row0 >= M) return;
    const int64_t k0 = (int64_t)slab * kslab;
    const int64_t k1 = k0 + kslab < M ? k0 + kslab : M;

    const double* qrow[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        int64_t row = row0 + 16 * t + lr;
        row = row < M ? row : M - 1;
        qrow[t] = Q + row * ldq;
    }
    lb_double4 acc[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[t][c] = lb_double4{0, 0, 0, 0};

    int64_t kc = k0;
    for (; kc + 16 <= k1; kc += 16) {
        double2 qa[RT], qb[RT], xa[CT], xb[CT];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const double* p = qrow[t] + kc + 2 * lk;
            if (ALIGNED) {
                qa[t] = *reinterpret_cast<const double2*>(p);
                qb[t] = *reinterpret_cast<const double2*>(p + 8);
            } else {
                qa[t] = make_double2(p[0], p[1]);
                qb[t] = make_double2(p[8], p[9]);
            }
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            xa[c] = *reinterpret_cast<const double2*>(X + ((kc >> 1) + lk) * (2 * Bp) + 2 * (16 * c + lr));
            xb[c] = *reinterpret_cast<const double2*>(X + (((kc + 8) >> 1) + lk) * (2 * Bp) + 2 * (16 * c + lr));
        }
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[t].x, xa[c].x, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[t].y, xa[c].y, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qb[t].x, xb[c].x, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qb[t].y, xb[c].y, acc[t][c], 0, 0, 0);
            }
    }
    if (kc < k1) {  // ragged tail: guarded scalar loads, zero beyond M
        double qa[RT][4], xa[CT][4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int64_t k = kc + 2 * lk + (h & 1) + 8 * (h >> 1);
            const bool ok = k < k1;
#pragma unroll
            for (int t = 0; t < RT; ++t) qa[t][h] = ok ? qrow[t][k] : 0.0;
#pragma unroll
            for (int c = 0; c < CT; ++c) xa[c][h] = ok ? X[ilv2(k, 16 * c + lr, Bp)] : 0.0;
        }
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[t][h], xa[c][h], acc[t][c], 0, 0, 0);
    }
    // D layout of v_mfma_f64_16x16x4f64: lane l, element j -> row 4j + l/16,
    // column l%16 (the FP32 variant below uses row 4(l/16) + j)
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t row = row0 + 16 * t + 4 * j + lk;
                if (row < M) Part[ilv2(row, 16 * c + lr, Bp)] = acc[t][c][j];
            }
}

// ---------------------------------------------------------------------------
// Matrix-core stage GEMM, FP32 operands: Q32 and X32 in FP32, FP32 products and
// accumulation within a k-slab, FP64 sums across slabs. A slab's sum is an FP32
// value and is stored as one (17 of them at N = 99: 43 MB a stage instead of 85).
// ---------------------------------------------------------------------------
template <int RT, int CT, bool ALIGNED>
__global__ __launch_bounds__(256) void k_gemm32(const float* const* Qs, int64_t M, int64_t Mp, int64_t ldq,
                                                const float* Xall, int64_t xstride, float* Pall,
                                                int64_t pstride, int kslab, GemmGrid gg) {
    constexpr int Bp = 16 * CT;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    int bx, slab, r;
    if (!gemm_work(gg, bx, slab, r)) return;
    const float* Q = Qs[r];
    const float* X = Xall + r * xstride;
    float* Part = Pall + r * pstride + (int64_t)slab * Mp * Bp;
    const int64_t row0 = ((int64_t)bx * (blockDim.x >> 6) + wave) * (16 * RT);
    if (row0 >= M) return;
    const int64_t k0 = (int64_t)slab * kslab;
    const int64_t k1 = k0 + kslab < M ? k0 + kslab : M;

    const float* qrow[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        int64_t row = row0 + 16 * t + lr;
        row = row < M ? row : M - 1;
        qrow[t] = Q + row * ldq;
    }
    lb_float4 acc[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[t][c] = lb_float4{0, 0, 0, 0};

    // 32 columns (128 bytes of each row) per iteration, as two 16-byte loads per
    // lane: columns kc + 4(l/16) + {0..3} and kc + 16 + 4(l/16) + {0..3}
    int64_t kc = k0;
    for (; kc + 32 <= k1; kc += 32) {
        float4 qa[RT], qb[RT], xa[CT], xb[CT];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const float* p = qrow[t] + kc + 4 * lk;
            if (ALIGNED) {
                qa[t] = *reinterpret_cast<const float4*>(p);
                qb[t] = *reinterpret_cast<const float4*>(p + 16);
            } else {
                qa[t] = make_float4(p[0], p[1], p[2], p[3]);
                qb[t] = make_float4(p[16], p[17], p[18], p[19]);
            }
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            xa[c] = *reinterpret_cast<const float4*>(X + ((kc >> 2) + lk) * (4 * Bp) + 4 * (16 * c + lr));
            xb[c] = *reinterpret_cast<const float4*>(X + (((kc + 16) >> 2) + lk) * (4 * Bp) + 4 * (16 * c + lr));
        }
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].x, xa[c].x, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].y, xa[c].y, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].z, xa[c].z, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].w, xa[c].w, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qb[t].x, xb[c].x, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qb[t].y, xb[c].y, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qb[t].z, xb[c].z, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qb[t].w, xb[c].w, acc[t][c], 0, 0, 0);
            }
    }
    for (; kc + 16 <= k1; kc += 16) {
        float4 qa[RT], xa[CT];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const float* p = qrow[t] + kc + 4 * lk;
            if (ALIGNED) qa[t] = *reinterpret_cast<const float4*>(p);
            else qa[t] = make_float4(p[0], p[1], p[2], p[3]);
        }
#pragma unroll
        for (int c = 0; c < CT; ++c)
            xa[c] = *reinterpret_cast<const float4*>(X + ((kc >> 2) + lk) * (4 * Bp) + 4 * (16 * c + lr));
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].x, xa[c].x, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].y, xa[c].y, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].z, xa[c].z, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].w, xa[c].w, acc[t][c], 0, 0, 0);
            }
    }
    if (kc < k1) {
        float qa[RT][4], xa[CT][4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int64_t k = kc + 4 * lk + h;
            const bool ok = k < k1;
#pragma unroll
            for (int t = 0; t < RT; ++t) qa[t][h] = ok ? qrow[t][k] : 0.0f;
#pragma unroll
            for (int c = 0; c < CT; ++c) xa[c][h] = ok ? X[ilv4(k, 16 * c + lr, Bp)] : 0.0f;
        }
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t][h], xa[c][h], acc[t][c], 0, 0, 0);
    }
    // D layout of v_mfma_f32_16x16x4f32: lane l, element j -> row 4(l/16) + j
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int j = 0; j < 4; j += 2) {
                const int64_t row = row0 + 16 * t + 4 * lk + j;
                float* o = Part + ilv2(row, 16 * c + lr, Bp);
                if (row + 1 < M) *reinterpret_cast<float2*>(o) = make_float2(acc[t][c][j], acc[t][c][j + 1]);
                else if (row < M) *o = acc[t][c][j];
            }
}

// ---------------------------------------------------------------------------
// LDS-staged variants of the two stage GEMMs (rows of Q 128-byte aligned).
// ---------------------------------------------------------------------------
// The matrix-core A operand wants lane l to hold row l%16 of a 16-row tile, so
// a direct 16-byte load per lane touches 16 rows per quarter-wave and splits
// every 128-byte line of Q between two load instructions. Here a wave instead
// reads its 16*RT rows x 128 bytes (16 FP64 / 32 FP32 columns) as 2*RT loads of
// 8 complete lines (lane L: row L/8 of the group, 16-byte piece (L%8) ^ (L/8)),
// with the nontemporal hint since Q is streamed once per stage, writes the
// pieces to a wave-private LDS buffer (slot g*64 + L), and reads the operands
// back in the matrix-core layout: row r, piece c sits in slot
// (r/8)*64 + (r%8)*8 + (c ^ (r%8)), which keeps each group of 8 lanes of a
// 16-byte LDS read on distinct banks. Two chunks of loads are kept in flight.
// The columns each MFMA consumes are the same as in the direct kernels, so the
// results are bit-identical to theirs.

__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Per-lane byte offsets (from the wave's first row) of the lane's 16-byte piece
// in each of the 2*RT groups of 8 rows; rows past M re-read row M-1.
template <int G>
__device__ __forceinline__ void stage_offsets(uint32_t (&off)[G], int64_t row0, int64_t M, int64_t rowbytes,
                                              int lane) {
    const int wr = lane >> 3, wc = (lane & 7) ^ wr;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        int64_t row = row0 + 8 * g + wr;
        row = row < M ? row : M - 1;
        off[g] = (uint32_t)((row - row0) * rowbytes + 16 * wc);
    }
}

typedef const lb_u4 __attribute__((address_space(1)))* lb_gu4;

template <int G>
__device__ __forceinline__ void stage_load(lb_u4 (&q)[G], const char* p, const uint32_t (&off)[G]) {
#pragma unroll
    for (int g = 0; g < G; ++g) q[g] = __builtin_nontemporal_load((lb_gu4)(p + off[g]));
}

// The B operand (states) of one chunk for CT column tiles, loaded together with
// the chunk's Q so that waiting for it never waits for a later prefetch.
template <int CT>
__device__ __forceinline__ void stage_xload(lb_u4 (&xa)[CT], lb_u4 (&xb)[CT], const char* x0, const char* x1) {
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        xa[c] = *(lb_gu4)(x0 + 256 * c);
        xb[c] = *(lb_gu4)(x1 + 256 * c);
    }
}

template <int G>
__device__ __forceinline__ void stage_put(lb_u4* lds, const lb_u4 (&q)[G], int lane) {
#pragma unroll
    for (int g = 0; g < G; ++g) lds[g * 64 + lane] = q[g];
}

template <int RT, int CT>
__global__ __launch_bounds__(256) void k_gemm64s(const double* const* Qs, int64_t M, int64_t Mp, int64_t ldq,
                                                 const double* Xall, int64_t xstride, double* Pall,
                                                 int64_t pstride, int kslab, GemmGrid gg) {
    extern __shared__ lb_u4 stage_lds[];
    constexpr int Bp = 16 * CT;
    constexpr int G = 2 * RT;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    int bx, slab, r;
    if (!gemm_work(gg, bx, slab, r)) return;
    const double* Q = Qs[r];
    const double* X = Xall + r * xstride;
    double* Part = Pall + r * pstride + (int64_t)slab * Mp * Bp;
    const int64_t row0 = ((int64_t)bx * (blockDim.x >> 6) + wave) * (16 * RT);
    if (row0 >= M) return;
    const int64_t k0 = (int64_t)slab * kslab;
    const int64_t k1 = k0 + kslab < M ? k0 + kslab : M;
    lb_u4* lds = stage_lds + wave * (G * 64);
    const char* qbase = reinterpret_cast<const char*>(Q + row0 * ldq);
    uint32_t off[G];
    stage_offsets<G>(off, row0, M, ldq * 8, lane);
    const int rr = lr & 7;
    const int s0 = (lr >> 3) * 64 + rr * 8 + (lk ^ rr);

    lb_double4 acc[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[t][c] = lb_double4{0, 0, 0, 0};

    // X of chunk kc for column tile c: lane's double2 at ((kc>>1) + lk)*2Bp + 2(16c + lr); the
    // chunk's second half (columns kc+8..) starts 4*2Bp doubles later.
    const char* xlane = reinterpret_cast<const char*>(X + lk * (2 * Bp) + 2 * lr);
    auto xaddr = [&](int64_t kc) { return xlane + (kc >> 1) * (2 * Bp) * 8; };
    auto mma = [&](const lb_u4 (&xa)[CT], const lb_u4 (&xb)[CT]) {
        lb_double2v qa[RT], qb[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            qa[t] = __builtin_bit_cast(lb_double2v, lds[128 * t + s0]);
            qb[t] = __builtin_bit_cast(lb_double2v, lds[(128 * t + s0) ^ 4]);
        }
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const lb_double2v x0 = __builtin_bit_cast(lb_double2v, xa[c]);
                const lb_double2v x1 = __builtin_bit_cast(lb_double2v, xb[c]);
                acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[t].x, x0.x, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[t].y, x0.y, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qb[t].x, x1.x, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qb[t].y, x1.y, acc[t][c], 0, 0, 0);
            }
    };

    // two chunks in flight: (qA, xA) holds chunk j, (qB, xB) chunk j+1
    const int64_t nch = (k1 - k0) / 16;
    lb_u4 qA[G], qB[G], xA0[CT], xA1[CT], xB0[CT], xB1[CT];
    // the scheduling barriers keep each chunk's loads where they are issued here,
    // ahead of the next chunk's, instead of next to their first use
    auto fetch = [&](lb_u4 (&q)[G], lb_u4 (&x0)[CT], lb_u4 (&x1)[CT], int64_t kc) {
        __builtin_amdgcn_sched_barrier(0);
        stage_xload<CT>(x0, x1, xaddr(kc), xaddr(kc + 8));
        stage_load<G>(q, qbase + kc * 8, off);
        __builtin_amdgcn_sched_barrier(0);
    };
    // Every pass issues both prefetches (chunk indices past the end re-read the
    // last chunk), so the same loads are in flight at every loop iteration.
    auto kcl = [&](int64_t ch) { return k0 + 16 * (ch < nch ? ch : nch - 1); };
    if (nch > 0) {
        fetch(qA, xA0, xA1, kcl(0));
        fetch(qB, xB0, xB1, kcl(1));
        int64_t j = 0;
        for (; j + 1 < nch; j += 2) {
            stage_put<G>(lds, qA, lane);
            wave_lds_fence();
            mma(xA0, xA1);
            wave_lds_fence();
            fetch(qA, xA0, xA1, kcl(j + 2));
            stage_put<G>(lds, qB, lane);
            wave_lds_fence();
            mma(xB0, xB1);
            wave_lds_fence();
            fetch(qB, xB0, xB1, kcl(j + 3));
        }
        if (j < nch) {
            stage_put<G>(lds, qA, lane);
            wave_lds_fence();
            mma(xA0, xA1);
            wave_lds_fence();
        }
    }
    const int64_t kc = k0 + 16 * nch;
    if (kc < k1) {  // ragged tail: guarded scalar loads, zero beyond M
        double qa[RT][4], xa[CT][4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int64_t k = kc + 2 * lk + (h & 1) + 8 * (h >> 1);
            const bool ok = k < k1;
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                int64_t row = row0 + 16 * t + lr;
                row = row < M ? row : M - 1;
                qa[t][h] = ok ? Q[row * ldq + k] : 0.0;
            }
#pragma unroll
            for (int c = 0; c < CT; ++c) xa[c][h] = ok ? X[ilv2(k, 16 * c + lr, Bp)] : 0.0;
        }
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[t][h], xa[c][h], acc[t][c], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t row = row0 + 16 * t + 4 * j + lk;
                if (row < M) Part[ilv2(row, 16 * c + lr, Bp)] = acc[t][c][j];
            }
}

template <int RT, int CT>
__global__ __launch_bounds__(256) void k_gemm32s(const float* const* Qs, int64_t M, int64_t Mp, int64_t ldq,
                                                 const float* Xall, int64_t xstride, float* Pall,
                                                 int64_t pstride, int kslab, GemmGrid gg) {
    extern __shared__ lb_u4 stage_lds[];
    constexpr int Bp = 16 * CT;
    constexpr int G = 2 * RT;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    int bx, slab, r;
    if (!gemm_work(gg, bx, slab, r)) return;
    const float* Q = Qs[r];
    const float* X = Xall + r * xstride;
    float* Part = Pall + r * pstride + (int64_t)slab * Mp * Bp;
    const int64_t row0 = ((int64_t)bx * (blockDim.x >> 6) + wave) * (16 * RT);
    if (row0 >= M) return;
    const int64_t k0 = (int64_t)slab * kslab;
    const int64_t k1 = k0 + kslab < M ? k0 + kslab : M;
    lb_u4* lds = stage_lds + wave * (G * 64);
    const char* qbase = reinterpret_cast<const char*>(Q + row0 * ldq);
    uint32_t off[G];
    stage_offsets<G>(off, row0, M, ldq * 4, lane);
    const int rr = lr & 7;
    const int s0 = (lr >> 3) * 64 + rr * 8 + (lk ^ rr);

    lb_float4 acc[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[t][c] = lb_float4{0, 0, 0, 0};

    // X of chunk kc for column tile c: lane's float4 at ((kc>>2) + lk)*4Bp + 4(16c + lr); the
    // chunk's second half (columns kc+16..) starts 4*4Bp floats later.
    const char* xlane = reinterpret_cast<const char*>(X + lk * (4 * Bp) + 4 * lr);
    auto xaddr = [&](int64_t kc) { return xlane + (kc >> 2) * (4 * Bp) * 4; };
    auto mma = [&](const lb_u4 (&xa)[CT], const lb_u4 (&xb)[CT]) {
        lb_float4 qa[RT], qb[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            qa[t] = __builtin_bit_cast(lb_float4, lds[128 * t + s0]);
            qb[t] = __builtin_bit_cast(lb_float4, lds[(128 * t + s0) ^ 4]);
        }
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const lb_float4 x0 = __builtin_bit_cast(lb_float4, xa[c]);
                const lb_float4 x1 = __builtin_bit_cast(lb_float4, xb[c]);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].x, x0.x, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].y, x0.y, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].z, x0.z, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].w, x0.w, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qb[t].x, x1.x, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qb[t].y, x1.y, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qb[t].z, x1.z, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qb[t].w, x1.w, acc[t][c], 0, 0, 0);
            }
    };

    const int64_t nch = (k1 - k0) / 32;
    lb_u4 qA[G], qB[G], xA0[CT], xA1[CT], xB0[CT], xB1[CT];
    auto fetch = [&](lb_u4 (&q)[G], lb_u4 (&x0)[CT], lb_u4 (&x1)[CT], int64_t kc) {
        __builtin_amdgcn_sched_barrier(0);
        stage_xload<CT>(x0, x1, xaddr(kc), xaddr(kc + 16));
        stage_load<G>(q, qbase + kc * 4, off);
        __builtin_amdgcn_sched_barrier(0);
    };
    // Every pass issues both prefetches (chunk indices past the end re-read the
    // last chunk), so the same loads are in flight at every loop iteration.
    auto kcl = [&](int64_t ch) { return k0 + 32 * (ch < nch ? ch : nch - 1); };
    if (nch > 0) {
        fetch(qA, xA0, xA1, kcl(0));
        fetch(qB, xB0, xB1, kcl(1));
        int64_t j = 0;
        for (; j + 1 < nch; j += 2) {
            stage_put<G>(lds, qA, lane);
            wave_lds_fence();
            mma(xA0, xA1);
            wave_lds_fence();
            fetch(qA, xA0, xA1, kcl(j + 2));
            stage_put<G>(lds, qB, lane);
            wave_lds_fence();
            mma(xB0, xB1);
            wave_lds_fence();
            fetch(qB, xB0, xB1, kcl(j + 3));
        }
        if (j < nch) {
            stage_put<G>(lds, qA, lane);
            wave_lds_fence();
            mma(xA0, xA1);
            wave_lds_fence();
        }
    }
    // remainder (< 32 columns, last slab only): direct loads as in k_gemm32
    const float* qrow[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        int64_t row = row0 + 16 * t + lr;
        row = row < M ? row : M - 1;
        qrow[t] = Q + row * ldq;
    }
    int64_t kc = k0 + 32 * nch;
    if (kc + 16 <= k1) {
        float4 qa[RT], xa[CT];
#pragma unroll
        for (int t = 0; t < RT; ++t) qa[t] = *reinterpret_cast<const float4*>(qrow[t] + kc + 4 * lk);
#pragma unroll
        for (int c = 0; c < CT; ++c)
            xa[c] = *reinterpret_cast<const float4*>(X + ((kc >> 2) + lk) * (4 * Bp) + 4 * (16 * c + lr));
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].x, xa[c].x, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].y, xa[c].y, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].z, xa[c].z, acc[t][c], 0, 0, 0);
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t].w, xa[c].w, acc[t][c], 0, 0, 0);
            }
        kc += 16;
    }
    if (kc < k1) {
        float qa[RT][4], xa[CT][4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int64_t k = kc + 4 * lk + h;
            const bool ok = k < k1;
#pragma unroll
            for (int t = 0; t < RT; ++t) qa[t][h] = ok ? qrow[t][k] : 0.0f;
#pragma unroll
            for (int c = 0; c < CT; ++c) xa[c][h] = ok ? X[ilv4(k, 16 * c + lr, Bp)] : 0.0f;
        }
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t][h], xa[c][h], acc[t][c], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int j = 0; j < 4; j += 2) {
                const int64_t row = row0 + 16 * t + 4 * lk + j;
                float* o = Part + ilv2(row, 16 * c + lr, Bp);
                if (row + 1 < M) *reinterpret_cast<float2*>(o) = make_float2(acc[t][c][j], acc[t][c][j + 1]);
                else if (row < M) *o = acc[t][c][j];
            }
}

// ---------------------------------------------------------------------------
// Stage combine: k_i = sum_slab Part + K, then the RK4 update of that stage.
// ---------------------------------------------------------------------------
struct StageArgs {
    const double* const* Ks;
    double* V;       // + r*sstride
    double* Acc;
    double* X;
    float* X32;      // may be null
    int64_t sstride; // per-system stride of V/Acc/X (doubles)
    int64_t s32stride;
    const void* Part;  // partial sums: double, or float in FP32
    int64_t pstride;
    int nslab;
    int64_t M, Mp;
    int Bp;
    double dt;
};

// The stage combination of two rows of a state: k = (Q x + K); returns the next
// stage's x. Without a second row (two false) that element stays zero.
__device__ __forceinline__ lb_double2v stage_pair(int stage, double h, lb_double2v k, bool two, lb_double2v* V,
                                                  lb_double2v* Acc) {
    const lb_double2v v = *V;
    lb_double2v x;
    if (stage == 1) {
        *Acc = k;
        x = v + 0.5 * h * k;
    } else if (stage == 2) {
        *Acc = *Acc + 2.0 * k;
        x = v + 0.5 * h * k;
    } else if (stage == 3) {
        *Acc = *Acc + 2.0 * k;
        x = v + h * k;
    } else {
        x = v + h / 6.0 * (*Acc + k);
        if (!two) x.y = 0.0;
        *V = x;
    }
    if (!two) x.y = 0.0;
    return x;
}

// A thread takes two rows of one state: they are neighbours in every array but the
// user's, so all of it moves in pairs, 16 bytes a lane in FP64 (one element a lane
// left half of each line to another wave: 19.7 us at N = 99, 50 states, 17 slabs,
// now 11.2; 10.9 at N = 100, 64 states, 5 slabs in FP64, now 8.8). T: type of the
// partial sums.
template <typename T>
__global__ __launch_bounds__(256) void k_stage(StageArgs a, int stage) {
    typedef T pair __attribute__((ext_vector_type(2)));
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // (row pair, b) in row-major
    const int r = blockIdx.y;
    const int64_t row = e / a.Bp * 2;
    if (row >= a.M) return;
    const int b = (int)(e % a.Bp);
    const int64_t idx = ilv2(row, b, a.Bp);
    const bool two = row + 1 < a.M;
    const T* part = (const T*)a.Part + r * a.pstride + idx;
    lb_double2v k = {0.0, 0.0};
#pragma unroll 4
    for (int s = 0; s < a.nslab; ++s) {
        const pair q = *reinterpret_cast<const pair*>(part + (int64_t)s * a.Mp * a.Bp);
        k.x += (double)q.x;
        k.y += (double)q.y;
    }
    k.x += a.Ks[r][row];
    if (two) k.y += a.Ks[r][row + 1];
    lb_double2v* V = reinterpret_cast<lb_double2v*>(a.V + r * a.sstride + idx);
    lb_double2v* Acc = reinterpret_cast<lb_double2v*>(a.Acc + r * a.sstride + idx);
    lb_double2v* X = reinterpret_cast<lb_double2v*>(a.X + r * a.sstride + idx);
    const lb_double2v x = stage_pair(stage, a.dt, k, two, V, Acc);
    *X = x;
    if (a.X32)
        *reinterpret_cast<float2*>(a.X32 + r * a.s32stride + ilv4(row, b, a.Bp)) = make_float2((float)x.x, (float)x.y);
}

// ---------------------------------------------------------------------------
// A whole stage of a small system in one launch (FP64, 2 to 64 states): a workgroup
// owns RT tiles of 16 rows, its eight waves an eighth of the columns each (lane mapping as in
// k_gemm64), their sums meet in LDS in the order of the waves and the stage
// combination follows at once. x is read from one buffer and written to another,
// since other workgroups may still be reading. What a stage costs at this size is
// launches and latency, and this is one launch instead of two, without partial sums
// in memory. The columns' split depends on M alone, so a system's bits do not depend
// on what shares the launch, nor on RT: two tiles read x once for 32 rows where there
// are workgroups enough (block_rows).
// ---------------------------------------------------------------------------
constexpr int kBlockWaves = 8;

// Columns of a wave, the length of a slab that gives the same sums (plan_make): whole
// lines of 16 where such slabs are used (M = 2208, 2600 and 2703 take up to 3 % longer for
// it alone and 6 % for two or three systems, the other N^2 - 1 have that length anyway).
static int64_t block_columns(int64_t M) {
    return M > 2048 ? (M + 16 * kBlockWaves - 1) / (16 * kBlockWaves) * 16
                    : (M + 8 * kBlockWaves - 1) / (8 * kBlockWaves) * 8;
}

struct BlockArgs {
    const double* const* Qs;
    const double* const* Ks;
    int64_t M, ldq, kw;  // kw: block_columns(M)
    double *V, *Acc;
    int64_t sstride;
    const double* Xin;
    double* Xout;
    int64_t in_stride, out_stride;
    double h;
};

template <int CT, int RT, bool ALIGNED>
__global__ __launch_bounds__(64 * kBlockWaves, RT == 1 ? 2 : 4) void k_block64(BlockArgs a, int stage) {
    constexpr int Bp = 16 * CT;
    __shared__ double red[kBlockWaves][CT * 256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const int r = blockIdx.y;
    const int64_t M = a.M, row0 = (int64_t)blockIdx.x * (16 * RT);
    const double* X = a.Xin + r * a.in_stride + 2 * lr;
    const double* q[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int64_t row = row0 + 16 * t + lr;
        q[t] = a.Qs[r] + (row < M ? row : M - 1) * a.ldq;
    }
    const int64_t k0 = wave * a.kw, k1 = k0 + a.kw < M ? k0 + a.kw : M;
    lb_double4 acc[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[t][c] = lb_double4{0, 0, 0, 0};
    // U steps of 8 columns, all loads first
    auto steps = [&](auto U, int64_t kc) __attribute__((always_inline)) {
        constexpr int n = decltype(U)::value;
        lb_double2v qa[n][RT], xa[n][CT];
#pragma unroll
        for (int u = 0; u < n; ++u) {
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                const double* p = q[t] + kc + 8 * u + 2 * lk;
                qa[u][t] = ALIGNED ? *reinterpret_cast<const lb_double2v*>(p) : lb_double2v{p[0], p[1]};
            }
#pragma unroll
            for (int c = 0; c < CT; ++c)
                xa[u][c] = *reinterpret_cast<const lb_double2v*>(X + (((kc + 8 * u) >> 1) + lk) * (2 * Bp) + 32 * c);
        }
#pragma unroll
        for (int u = 0; u < n; ++u)
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[u][t].x, xa[u][c].x, acc[t][c], 0, 0, 0);
                    acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[u][t].y, xa[u][c].y, acc[t][c], 0, 0, 0);
                }
    };
    int64_t kc = k0;
    for (; kc + 32 <= k1; kc += 32) steps(std::integral_constant<int, 4>(), kc);
    for (; kc + 8 <= k1; kc += 8) steps(std::integral_constant<int, 1>(), kc);
    if (kc < k1) {  // fewer than 8 columns, at the end of the row: nothing beyond M is read
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int64_t k = kc + 2 * lk + e;
            const bool ok = k < k1;
            double xv[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) xv[c] = ok ? X[(k >> 1) * (2 * Bp) + (k & 1) + 32 * c] : 0.0;
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                const double qv = ok ? q[t][k] : 0.0;
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(qv, xv[c], acc[t][c], 0, 0, 0);
            }
        }
    }
    const int b = threadIdx.x % Bp, rp = threadIdx.x / Bp;
    const int i = (b >> 4) * 256 + 32 * rp + (b & 15);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        if (t > 0) __syncthreads();  // the last tile's sums are still being read
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) red[wave][256 * c + 64 * j + lane] = acc[t][c][j];  // (row 4j + l/16, column l%16)
        __syncthreads();
        const int64_t row = row0 + 16 * t + 2 * rp;
        if (rp < 8 && row < M) {
            const bool two = row + 1 < M;
            lb_double2v k = {red[0][i], red[0][i + 16]};
#pragma unroll
            for (int w = 1; w < kBlockWaves; ++w) {
                k.x += red[w][i];
                k.y += red[w][i + 16];
            }
            k.x += a.Ks[r][row];
            if (two) k.y += a.Ks[r][row + 1];
            const int64_t idx = ilv2(row, b, Bp);
            *reinterpret_cast<lb_double2v*>(a.Xout + r * a.out_stride + idx) =
                stage_pair(stage, a.h, k, two, reinterpret_cast<lb_double2v*>(a.V + r * a.sstride + idx),
                           reinterpret_cast<lb_double2v*>(a.Acc + r * a.sstride + idx));
        }
    }
}

// user layout (B, M) -> interleaved padded (Mp, Bp); padding rows/columns zero
__global__ void k_pack(const double* const* Vu, int64_t M, int64_t Mp, int B, int Bp, double* V, double* X,
                       float* X32, int64_t sstride, int64_t s32stride) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int r = blockIdx.y;
    if (e >= Mp * Bp) return;
    const int64_t row = e / Bp;
    const int b = (int)(e % Bp);
    const double v = (row < M && b < B) ? Vu[r][(int64_t)b * M + row] : 0.0;
    const int64_t idx = ilv2(row, b, Bp);
    V[r * sstride + idx] = v;
    X[r * sstride + idx] = v;
    if (X32) X32[r * s32stride + ilv4(row, b, Bp)] = (float)v;
}

__global__ void k_unpack(double* const* Vu, int64_t M, int B, int Bp, const double* V, int64_t sstride) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int r = blockIdx.y;
    if (e >= M * B) return;
    const int b = (int)(e / M);
    const int64_t row = e % M;
    Vu[r][e] = V[r * sstride + ilv2(row, b, Bp)];
}

// ---------------------------------------------------------------------------
// One state: GEMV with the stage combine fused in (rows are complete per wave).
// A wave owns R rows; lanes read 16 bytes each along the row, so one load
// instruction covers 1 KB of a row (full lines when rows are 128-byte aligned,
// then read with the nontemporal hint where Q exceeds the last-level cache). A row's
// sum does not depend on R, so R only trades waves for loads in flight.
// ---------------------------------------------------------------------------
template <int R, bool ALIGNED, bool NT>
__global__ __launch_bounds__(256) void k_gemv(const double* const* Qs, const double* const* Ks,
                                              double* const* Vs, int64_t M, int64_t ldq, double* Wall,
                                              int64_t wstride, int stage, double h) {
    // W layout per system: [Acc | Xa | Xb], each Ma = M rounded up to 32
    // doubles; stage i reads X from Xa when i is odd and Xb when even, and
    // writes the other one.
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int r = blockIdx.y;
    const int64_t row0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + wave) * R;
    if (row0 >= M) return;
    const double* Q = Qs[r];
    double* W = Wall + r * wstride;
    const int64_t Ma = (M + 31) / 32 * 32;
    double* Acc = W;
    const double* Xin = (stage & 1) ? W + Ma : W + 2 * Ma;
    double* Xout = (stage & 1) ? W + 2 * Ma : W + Ma;
    double acc[R];
    const double* qrow[R];
#pragma unroll
    for (int t = 0; t < R; ++t) {
        int64_t row = row0 + t;
        qrow[t] = Q + (row < M ? row : M - 1) * ldq;
    }
    wave_rowdots<R, ALIGNED, NT>(qrow, Xin, M, lane, acc);
    if (lane < R) {
        double kv = 0.0;
#pragma unroll
        for (int t = 0; t < R; ++t)
            if (t == lane) kv = acc[t];
        const int64_t row = row0 + lane;
        if (row < M) {
            const double k = kv + Ks[r][row];
            double* V = Vs[r];
            double x;
            if (stage == 1) {
                Acc[row] = k;
                x = V[row] + 0.5 * h * k;
            } else if (stage == 2) {
                Acc[row] = Acc[row] + 2.0 * k;
                x = V[row] + 0.5 * h * k;
            } else if (stage == 3) {
                Acc[row] = Acc[row] + 2.0 * k;
                x = V[row] + h * k;
            } else {
                x = V[row] + h / 6.0 * (Acc[row] + k);
                V[row] = x;
            }
            Xout[row] = x;
        }
    }
}

__global__ void k_gemv_init(double* const* Vs, int64_t M, double* Wall, int64_t wstride) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int r = blockIdx.y;
    if (e >= M) return;
    Wall[r * wstride + (M + 31) / 32 * 32 + e] = Vs[r][e];  // Xa = v
}

// ---------------------------------------------------------------------------
// Sparse RK4 stage: one launch per stage with the stage combination fused in,
// over the slice layout of sell.h (one wavefront per 64-row slice, one block of
// 256 threads per long row).
// ---------------------------------------------------------------------------

// RK4 stage combination for one element, given k = (Q x + K)_i and the values
// of v and of the accumulator loaded beforehand; h: the stage's factor. Product
// and sum rounded separately, whatever the code around makes of it.
__device__ __forceinline__ void rk4_update(int stage, double h, double k, double v, double acc, int64_t i, double* V,
                                           double* Acc, double* Xout) {
#pragma clang fp contract(off)
    if (stage == 4) {
        V[i] = v + h * (acc + k);
        return;
    }
    Acc[i] = stage == 1 ? k : acc + 2.0 * k;
    Xout[i] = v + h * k;
}

// The stage vectors of a sparse integration, M*B each: stage 1 reads x from V, stage 4 writes only V.
struct SellStage {
    int B, stage;
    double h;  // dt/2, dt/2, dt, dt/6
    const double* K;
    double* V;
    double* acc;
    const double* xin;
    double* xout;
};

// DRIVE: k = (Q0 x) + eps (Q1 x) + K, the two sums formed separately.
// SB: states per pass over a slice (1 for a single state, 4 for batches).
// A few us long at small sizes, so what precedes the loads of x counts: the stage's pointers and
// factor come from the host, K is read in the loop over states (read before it, the loop's first
// loads wait for it), and a single state has no loop. N = 100, us a stage: 4.6 -> 4.2 static,
// 5.5 -> 5.2 rocked; N = 1000: 19.5 -> 19.2 and 38.4 -> 38.4.
template <bool DRIVE, int SB>
__global__ __launch_bounds__(256) void k_sell_stage(SellMat a, SellStage st, double eps) {
    const int64_t M = a.M;
    const int B = SB == 1 ? 1 : st.B;
    const int stage = st.stage;
    const double h = st.h;
    double* Acc = st.acc;
    const double* Xin = st.xin;
    double* Xout = st.xout;
    const int wk = sell_work(a);
    if (wk < 0) return;
    if (wk < a.nlong) {
        const LongRowPtr lr = (LongRowPtr)(a.longrows + wk);
        const int64_t row = lr->row;
        const double kr = st.K[row];
        for (int b = 0; b < B; ++b) {
            const int64_t i = (int64_t)b * M + row;
            const double v = st.V[i], acc = stage > 1 ? Acc[i] : 0.0;
            double q0, q1;
            block_row_dots<DRIVE>(a, lr, Xin + (int64_t)b * M, q0, q1);
            if (threadIdx.x == 0) {
                double k = q0;
                if (DRIVE) k += eps * q1;
                k += kr;
                rk4_update(stage, h, k, v, acc, i, st.V, Acc, Xout);
            }
        }
        return;
    }
    // one slice per wavefront; the slice index is wave-uniform
    const int sl = __builtin_amdgcn_readfirstlane((wk - a.nlong) * 4 + (int)(threadIdx.x >> 6));
    if (sl >= a.S) return;
    const int lane = threadIdx.x & (kSlice - 1);
    const int64_t r = (int64_t)sl * kSlice + lane;
    const SellHeadPtr head = (SellHeadPtr)(a.head0 + sl);
    const SellFirst first = sell_first(head);
    SellHeadPtr head1 = nullptr;
    SellFirst first1;
    if (DRIVE) {
        head1 = (SellHeadPtr)(a.head1 + sl);
        first1 = sell_first(head1);
    }
    const bool mine = r < M && !((first.lmask >> lane) & 1);
    for (int b0 = 0; b0 < B; b0 += SB) {
        const int nb = min(SB, B - b0);
        const double kr = mine ? st.K[r] : 0.0;
        double vv[SB], aa[SB], acc[SB], accd[SB];
#pragma unroll
        for (int j = 0; j < SB; ++j) {
            vv[j] = aa[j] = acc[j] = accd[j] = 0.0;
            if (j < nb && mine) {
                const int64_t i = (int64_t)(b0 + j) * M + r;
                vv[j] = st.V[i];
                if (stage > 1) aa[j] = Acc[i];
            }
        }
        const double* xb = Xin + (int64_t)b0 * M;
        sell_row<SB>(first, head, a.scol0, a.sval0, lane, xb, M, nb, acc);
        if (DRIVE) sell_row<SB>(first1, head1, a.scol1, a.sval1, lane, xb, M, nb, accd);
#pragma unroll
        for (int j = 0; j < SB; ++j)
            if (j < nb && mine) {
                double k = acc[j];
                if (DRIVE) k += eps * accd[j];
                rk4_update(stage, h, k + kr, vv[j], aa[j], (int64_t)(b0 + j) * M + r, st.V, Acc, Xout);
            }
    }
}

__global__ void k_to_f32(const double* Q, float* Q32, int64_t n) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) Q32[e] = (float)Q[e];
}

// ---------------------------------------------------------------------------
// Kernel selection
// ---------------------------------------------------------------------------

typedef void (*gemm64_fn)(const double* const*, int64_t, int64_t, int64_t, const double*, int64_t, double*,
                          int64_t, int, GemmGrid);
typedef void (*gemm32_fn)(const float* const*, int64_t, int64_t, int64_t, const float*, int64_t, float*,
                          int64_t, int, GemmGrid);

template <bool AL>
gemm64_fn pick64(int RT, int CT) {
    if (CT == 1) {
        if (RT == 1) return k_gemm64<1, 1, AL>;
        if (RT == 2) return k_gemm64<2, 1, AL>;
        if (RT == 4) return k_gemm64<4, 1, AL>;
        if (RT == 8) return k_gemm64<8, 1, AL>;
    } else if (CT == 2) {
        if (RT == 1) return k_gemm64<1, 2, AL>;
        if (RT == 2) return k_gemm64<2, 2, AL>;
        if (RT == 4) return k_gemm64<4, 2, AL>;
    } else if (CT == 4) {
        if (RT == 1) return k_gemm64<1, 4, AL>;
        if (RT == 2) return k_gemm64<2, 4, AL>;
        if (RT == 4) return k_gemm64<4, 4, AL>;
    }
    return nullptr;
}

template <bool AL>
gemm32_fn pick32(int RT, int CT) {
    if (CT == 1) {
        if (RT == 1) return k_gemm32<1, 1, AL>;
        if (RT == 2) return k_gemm32<2, 1, AL>;
        if (RT == 4) return k_gemm32<4, 1, AL>;
        if (RT == 8) return k_gemm32<8, 1, AL>;
    } else if (CT == 2) {
        if (RT == 1) return k_gemm32<1, 2, AL>;
        if (RT == 2) return k_gemm32<2, 2, AL>;
        if (RT == 4) return k_gemm32<4, 2, AL>;
    } else if (CT == 4) {
        if (RT == 1) return k_gemm32<1, 4, AL>;
        if (RT == 2) return k_gemm32<2, 4, AL>;
        if (RT == 4) return k_gemm32<4, 4, AL>;
    }
    return nullptr;
}

gemm64_fn pick64s(int RT, int CT) {
    if (CT == 1) {
        if (RT == 1) return k_gemm64s<1, 1>;
        if (RT == 2) return k_gemm64s<2, 1>;
        if (RT == 4) return k_gemm64s<4, 1>;
    } else if (CT == 2) {
        if (RT == 1) return k_gemm64s<1, 2>;
        if (RT == 2) return k_gemm64s<2, 2>;
        if (RT == 4) return k_gemm64s<4, 2>;
    } else if (CT == 4) {
        if (RT == 1) return k_gemm64s<1, 4>;
        if (RT == 2) return k_gemm64s<2, 4>;
        if (RT == 4) return k_gemm64s<4, 4>;
    }
    return nullptr;
}

gemm32_fn pick32s(int RT, int CT) {
    if (CT == 1) {
        if (RT == 1) return k_gemm32s<1, 1>;
        if (RT == 2) return k_gemm32s<2, 1>;
        if (RT == 4) return k_gemm32s<4, 1>;
    } else if (CT == 2) {
        if (RT == 1) return k_gemm32s<1, 2>;
        if (RT == 2) return k_gemm32s<2, 2>;
        if (RT == 4) return k_gemm32s<4, 2>;
    } else if (CT == 4) {
        if (RT == 1) return k_gemm32s<1, 4>;
        if (RT == 2) return k_gemm32s<2, 4>;
        if (RT == 4) return k_gemm32s<4, 4>;
    }
    return nullptr;
}

int bpad(int B) { return B <= 16 ? 16 : (B <= 32 ? 32 : 64); }

}  // namespace

// Tile-cache file (LB_TUNE_CACHE): one line "M Bp precision rows kslab waves". Read once
// per context, before the first tile is set, tuned, asked for or used, so that it never
// takes the place of one that was set.
void lb_load_tune_cache(lb_ctx* c) {
    if (c->cache_loaded) return;
    c->cache_loaded = true;
    const char* path = getenv("LB_TUNE_CACHE");
    if (!path) return;
    FILE* f = fopen(path, "r");
    if (!f) return;
    long long M;
    int Bp, prec, rows, ks, waves;
    while (fscanf(f, "%lld %d %d %d %d %d", &M, &Bp, &prec, &rows, &ks, &waves) == 6) {
        c->tuned[std::make_tuple((int64_t)M, Bp, prec)] = lb_tile{rows, ks, waves};
        c->measured.insert(std::make_tuple((int64_t)M, Bp, prec));
    }
    fclose(f);
}

static lb_tile choose_tile(lb_ctx* c, int64_t M, int Bp, int precision, int R) {
    lb_load_tune_cache(c);
    auto it = c->tuned.find(std::make_tuple(M, Bp, precision));
    if (it != c->tuned.end()) return it->second;
    return lb_default_tile(M, Bp, precision, R);
}

// Whether choose_tile's answer was set or tuned (after it: the cache file is loaded then),
// and whether it was set: the fastest of several tiles gives way to a stage in one launch.
static bool has_tile(lb_ctx* c, int64_t M, int Bp, int precision) {
    return c->tuned.count(std::make_tuple(M, Bp, precision)) != 0;
}
static bool asked_tile(lb_ctx* c, int64_t M, int Bp, int precision) {
    return has_tile(c, M, Bp, precision) && !c->measured.count(std::make_tuple(M, Bp, precision));
}

int lb_impl_q_to_f32(lb_ctx* c, int64_t M, const double* Q, int64_t ldq, float* Q32) {
    const int64_t n = M * ldq;
    hipLaunchKernelGGL(k_to_f32, dim3(lb_blocks(n, 256)), dim3(256), 0, c->stream, Q, Q32, n);
    LB_CHECK_LAUNCH();
    return LB_OK;
}

// ---------------------------------------------------------------------------
// Propagation plan: path selection, buffer layout, kernel enqueueing.
// ---------------------------------------------------------------------------

namespace {

// The load of Q, the arrivals and the two launches around them: a whole call of two
// steps, a launch per stage / resident, in us: N = 17 75 / 49, N = 37 71 / 61, N = 64
// 207 / 113.
constexpr int64_t kResidentSteps = 2;
// Steps of a piece of a long run: 30 to 100 ms, of which the load of Q and the launches
// are less than a thousandth.
constexpr int64_t kResidentPiece = 4096;
// The wait for the chip is no longer than about what a launch per stage takes more in the
// run's steps: 40 us each.
constexpr int64_t kResidentStepTicks = 4000;

constexpr int kMaxDevices = 64;

enum PathKind { PATH_SMALL, PATH_GEMV, PATH_MFMA };

struct Plan {
    PathKind kind;
    int R;
    int64_t M, Mp, ldq;
    int B, Bp, precision;
    lb_tile tile;
    int nslab;
    int64_t sstride, s32stride, pstride, wstride;
    size_t o_ptr, o_v, o_acc, o_x, o_x32, o_part, o_w, bytes;
    Rk4Small small;
    bool aligned;
    bool whole;   // a stage is one launch of k_block64
    bool staged;  // every Q and every row of Q 128-byte aligned: LDS-staged GEMM, streaming GEMV loads
    const void** d;
    double *V, *Acc, *X, *Part, *W;
    float* X32;
};

// Many systems of M > 2048 whose Q exceed the last-level cache are read from memory each
// stage, faster by the LDS-staged GEMM with a slab for each of k_block64's waves (same
// sums, same bits), unless the workgroups of 32 rows fit the chip two to a CU (256
// CUs). In us a stage, k_block64 / GEMM and combination:
//   16 states:  N = 46, R = 8  75 / 65   R = 16  144 / 130   N = 48, R = 7 (504 workgroups)  60 / 64
//               N = 50, R = 7  95 / 79   R = 10  134 / 117   R = 20  236 / 226
//   32 states:  N = 48, R = 8  103 / 97  R = 12  142 / 136   N = 50, R = 10  152 / 138
// Smaller systems have fewer columns in a slab: N = 42, 16 states, R = 14 92 / 88, R = 32
// 181 / 189; N = 37, R = 64 216 / 224.
static bool many_blocks(const Plan& p) {
    return p.Bp <= 32 && p.M > 2048 && p.R * ((p.M + 31) / 32) > 512 &&
           (size_t)p.R * p.M * p.ldq * sizeof(double) > ((size_t)256 << 20);
}

// allow_small: a whole run in one launch where M is small; own_tile: the tile was asked
// for, and is used.
static int plan_make(Plan& p, int R, int64_t M, int64_t ldq, int B, int precision, const lb_tile& tile,
                     bool allow_small, bool own_tile) {
    p = Plan();
    p.R = R;
    p.M = M;
    p.ldq = ldq;
    p.B = B;
    p.precision = precision;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = lb_align(off + bytes, 256);
        return o;
    };
    p.o_ptr = take(sizeof(void*) * 5 * R);
    if (allow_small && M <= 256 && (int64_t)B * M <= 4096 && precision == LB_FP64) {
        p.kind = PATH_SMALL;
        p.small = rk4_small_pick((int)M);
    } else if (B == 1 && precision == LB_FP64) {
        p.kind = PATH_GEMV;
        p.aligned = ldq % 2 == 0;
        p.wstride = 3 * (int64_t)lb_align(M, 32);
        p.o_w = take(sizeof(double) * p.wstride * R + (R == 1 && rk4_resident_range(M) ? rk4_resident_bytes(M) : 0));
    } else {
        p.kind = PATH_MFMA;
        p.Bp = bpad(B);
        p.whole = !own_tile && precision == LB_FP64 && M <= whole_limit(p.Bp);
        p.tile = p.whole && many_blocks(p) ? lb_tile{64, (int)block_columns(M), 1} : tile;
        p.whole = p.whole && !many_blocks(p);
        p.Mp = (M + 15) / 16 * 16;
        p.nslab = (int)((M + p.tile.kslab - 1) / p.tile.kslab);
        p.sstride = lb_align(p.Mp * p.Bp, 64);
        p.s32stride = lb_align(p.Mp * p.Bp, 128);
        p.pstride = (int64_t)p.nslab * p.Mp * p.Bp;
        p.aligned = precision == LB_FP32 ? (ldq % 4 == 0) : (ldq % 2 == 0);
        p.o_v = take(sizeof(double) * p.sstride * R);
        p.o_acc = take(sizeof(double) * p.sstride * R);
        p.o_x = take(sizeof(double) * p.sstride * R);
        if (precision == LB_FP32) p.o_x32 = take(sizeof(float) * p.s32stride * R);
        p.o_part = take(sizeof(double) * p.pstride * R);
        const int RT = tile.rows / 16, CT = p.Bp / 16;
        if (tile.rows % 16 || tile.kslab % 16 || tile.kslab <= 0 || tile.waves < 1 || tile.waves > 4 ||
            (precision == LB_FP64 ? (p.aligned ? pick64<true>(RT, CT) : pick64<false>(RT, CT)) == nullptr
                                  : (p.aligned ? pick32<true>(RT, CT) : pick32<false>(RT, CT)) == nullptr))
            return lb_fail(LB_ERR_INVALID_ARG, "unsupported tile rows=%d kslab=%d waves=%d for Bp=%d", tile.rows,
                           tile.kslab, tile.waves, p.Bp);
    }
    p.bytes = off;
    return LB_OK;
}

// Kernel choice that depends on the operands' alignment (the LDS-staged
// forms need 128-byte rows); rejects Q that is not 16-byte aligned.
static int plan_align(Plan& p, const lb_prop_sys* sys) {
    const int R = p.R;
    const int64_t es = p.precision == LB_FP32 ? 4 : 8;
    p.staged = (p.kind == PATH_MFMA || p.kind == PATH_GEMV) && (p.ldq * es) % 128 == 0;
    for (int r = 0; r < R; ++r) {
        const void* qp = p.precision == LB_FP32 ? (const void*)sys[r].Q32 : (const void*)sys[r].Q;
        if (p.kind != PATH_SMALL && ((uintptr_t)qp) % 16) return lb_fail(LB_ERR_INVALID_ARG, "Q must be 16-byte aligned");
        if (((uintptr_t)qp) % 128) p.staged = false;
    }
    if (p.staged && p.kind == PATH_MFMA) {
        const int RT = p.tile.rows / 16, CT = p.Bp / 16;
        if (p.precision == LB_FP64 ? pick64s(RT, CT) == nullptr : pick32s(RT, CT) == nullptr) p.staged = false;
    }
    return LB_OK;
}

// Points the plan's buffers into device memory `base` (p.bytes).
static void plan_buffers(Plan& p, char* base) {
    p.d = (const void**)(base + p.o_ptr);
    if (p.kind == PATH_GEMV) p.W = (double*)(base + p.o_w);
    if (p.kind == PATH_MFMA) {
        p.V = (double*)(base + p.o_v);
        p.Acc = (double*)(base + p.o_acc);
        p.X = (double*)(base + p.o_x);
        p.X32 = p.precision == LB_FP32 ? (float*)(base + p.o_x32) : nullptr;
        p.Part = (double*)(base + p.o_part);
    }
}

// Binds the plan to device memory `base` (p.bytes) and uploads the per-system
// pointer arrays through the context's pinned staging buffer. Synchronizes.
static int plan_bind(lb_ctx* c, Plan& p, char* base, const lb_prop_sys* sys) {
    const int R = p.R;
    int rc = plan_align(p, sys);
    if (rc) return rc;
    rc = lb_host_reserve(c, sizeof(void*) * 5 * R);
    if (rc) return rc;
    LB_HIP(hipStreamSynchronize(c->stream));
    const void** h = (const void**)c->host;
    for (int r = 0; r < R; ++r) {
        h[r] = sys[r].Q;
        h[R + r] = sys[r].Q32;
        h[2 * R + r] = sys[r].K;
        h[3 * R + r] = sys[r].V;
        h[4 * R + r] = sys[r].V;
    }
    LB_HIP(hipMemcpyAsync(base + p.o_ptr, h, sizeof(void*) * 5 * R, hipMemcpyHostToDevice, c->stream));
    LB_HIP(hipStreamSynchronize(c->stream));
    plan_buffers(p, base);
    return LB_OK;
}

static StageArgs stage_args(const Plan& p, double dt) {
    StageArgs sa;
    sa.Ks = (const double* const*)(p.d + 2 * p.R);
    sa.V = p.V;
    sa.Acc = p.Acc;
    sa.X = p.X;
    sa.X32 = p.X32;
    sa.sstride = p.sstride;
    sa.s32stride = p.s32stride;
    sa.Part = p.Part;
    sa.pstride = p.pstride;
    sa.nslab = p.nslab;
    sa.M = p.M;
    sa.Mp = p.Mp;
    sa.Bp = p.Bp;
    sa.dt = dt;
    return sa;
}

// One launch of the stage GEMM (MFMA path) or the stage GEMV (stage 1).
static int plan_gemm(const Plan& p, hipStream_t s, int stage, double dt) {
    if (p.kind == PATH_GEMV) {
        // rows per wave: as many as keep at least ~8192 waves in the launch, and two of
        // the long rows from M = 9000 on, where x is a second stream per wave (one row
        // and two, in us a stage: N = 90 88 / 92, N = 97 118 / 110, N = 128 338 / 323)
        const int64_t rows_total = p.M * p.R;
        const int RW = rows_total >= 8 * 8192 ? 8 : rows_total >= 4 * 8192 ? 4 : rows_total >= 2 * 8192 || p.M >= 9000 ? 2 : 1;
        const unsigned gx = lb_blocks((p.M + RW - 1) / RW, 4);
        // The nontemporal hint pays once the systems' Q no longer fit the last-level
        // cache (256 MB), where a stage evicts what the next one reads first. One
        // stage with and without it: N = 70 (192 MB) 33.0 and 29.8 us, N = 75
        // (253 MB) 43.2 and 38.1, N = 80 (328 MB) 56.3 and 59.6.
        const bool streamed = (size_t)p.R * p.M * p.ldq * sizeof(double) > (256u << 20);
        typedef void (*gemv_fn)(const double* const*, const double* const*, double* const*, int64_t, int64_t,
                                double*, int64_t, int, double);
        gemv_fn fn;
        if (!p.aligned) fn = RW == 8 ? k_gemv<8, false, false> : RW == 4 ? k_gemv<4, false, false>
                           : RW == 2 ? k_gemv<2, false, false> : k_gemv<1, false, false>;
        else if (p.staged && streamed) fn = RW == 8 ? k_gemv<8, true, true> : RW == 4 ? k_gemv<4, true, true>
                              : RW == 2 ? k_gemv<2, true, true> : k_gemv<1, true, true>;
        else fn = RW == 8 ? k_gemv<8, true, false> : RW == 4 ? k_gemv<4, true, false>
                : RW == 2 ? k_gemv<2, true, false> : k_gemv<1, true, false>;
        hipLaunchKernelGGL(fn, dim3(gx, p.R), dim3(256), 0, s, (const double* const*)p.d,
                           (const double* const*)(p.d + 2 * p.R), (double* const*)(p.d + 3 * p.R), p.M, p.ldq, p.W,
                           p.wstride, stage, dt);
        LB_CHECK_LAUNCH();
        return LB_OK;
    }
    const int RT = p.tile.rows / 16, CT = p.Bp / 16;
    const int64_t rowwaves = (p.M + p.tile.rows - 1) / p.tile.rows;
    GemmGrid gg;
    gg.gx = (int)((rowwaves + p.tile.waves - 1) / p.tile.waves);
    gg.nslab = p.nslab;
    gg.R = p.R;
    const int64_t total = (int64_t)gg.gx * gg.nslab * gg.R;
    gg.per_xcd = (total + 7) / 8;
    const dim3 ggrid((unsigned)(8 * gg.per_xcd));
    const dim3 gblock(64 * p.tile.waves);
    // staged kernels: 2*RT KiB of LDS per wave
    const size_t shm = p.staged ? (size_t)p.tile.waves * 2 * RT * 1024 : 0;
    if (p.precision == LB_FP64) {
        gemm64_fn fn = p.staged ? pick64s(RT, CT) : (p.aligned ? pick64<true>(RT, CT) : pick64<false>(RT, CT));
        hipLaunchKernelGGL(fn, ggrid, gblock, shm, s, (const double* const*)p.d, p.M, p.Mp, p.ldq, (const double*)p.X,
                           p.sstride, p.Part, p.pstride, p.tile.kslab, gg);
    } else {
        gemm32_fn fn = p.staged ? pick32s(RT, CT) : (p.aligned ? pick32<true>(RT, CT) : pick32<false>(RT, CT));
        hipLaunchKernelGGL(fn, ggrid, gblock, shm, s, (const float* const*)(p.d + p.R), p.M, p.Mp, p.ldq,
                           (const float*)p.X32, p.s32stride, (float*)p.Part, p.pstride, p.tile.kslab, gg);
    }
    LB_CHECK_LAUNCH();
    return LB_OK;
}

static int plan_init_state(const Plan& p, hipStream_t s) {
    if (p.kind == PATH_GEMV) {
        hipLaunchKernelGGL(k_gemv_init, dim3(lb_blocks(p.M, 256), p.R), dim3(256), 0, s,
                           (double* const*)(p.d + 3 * p.R), p.M, p.W, p.wstride);
        LB_CHECK_LAUNCH();
    } else if (p.kind == PATH_MFMA) {
        hipLaunchKernelGGL(k_pack, dim3(lb_blocks(p.Mp * p.Bp, 256), p.R), dim3(256), 0, s,
                           (const double* const*)(p.d + 3 * p.R), p.M, p.Mp, p.B, p.Bp, p.V, p.X, p.X32, p.sstride,
                           p.s32stride);
        LB_CHECK_LAUNCH();
    }
    return LB_OK;
}

static int plan_unpack(const Plan& p, hipStream_t s) {
    hipLaunchKernelGGL(k_unpack, dim3(lb_blocks(p.M * p.B, 256), p.R), dim3(256), 0, s,
                       (double* const*)(p.d + 4 * p.R), p.M, p.B, p.Bp, (const double*)p.V, p.sstride);
    LB_CHECK_LAUNCH();
    return LB_OK;
}

// Rows of a workgroup of k_block64. Of many systems two tiles are faster. With 64
// states x is four times Q's traffic and the eight waves of one tile keep a CU to
// themselves: from three rounds of such workgroups on. With fewer, where the systems' Q
// no longer fit the last-level cache (256 MB). In us a stage, tile GEMM of 64 (32)
// rows / one tile / two:
//   64 states:  N = 30, R = 12  73 / 46 / 47   R = 16  80 / 60 / 50   R = 64  193 / 261 / 205
//               N = 37, R = 8   78 / 57 / 60   R = 16  111 / 128 / 98  R = 128  739 / 972 / 718
//   16 states:  N = 37, R = 16  64 / 58 / 59   R = 64  238 / 259 / 235
//               N = 52, R = 4   60 / 46 / 55   R = 6   88 / 90 / 82    R = 8  117 / 131 / 119
//   32 states:  N = 40, R = 12  84 / 66 / 74   R = 64  391 / 407 / 375
// Behind the GEMM remain up to M = 2048 (larger ones: many_blocks) some numbers of systems
// of 256 to 400 MB, which fill the last round badly either way: 16 states, N = 40, R = 16
// 78 / 86 / 86; N = 42, R = 14 84 against 92, 64 states, N = 33, R = 40 144 against 157.
static int block_rows(const Plan& p) {
    if (p.Bp == 64) return (int64_t)p.R * (p.Mp / 16) > 768 ? 32 : 16;
    return (size_t)p.R * p.M * p.ldq * sizeof(double) > ((size_t)256 << 20) ? 32 : 16;
}
typedef void (*block_fn)(BlockArgs, int);
template <bool AL>
static block_fn pick_block(int CT, int rows) {
    if (rows == 32) return CT == 1 ? k_block64<1, 2, AL> : CT == 2 ? k_block64<2, 2, AL> : k_block64<4, 2, AL>;
    return CT == 1 ? k_block64<1, 1, AL> : CT == 2 ? k_block64<2, 1, AL> : k_block64<4, 1, AL>;
}

// One stage in one launch; x alternates between its buffer and that of the partial
// sums, which are not needed.
static int plan_block(const Plan& p, hipStream_t s, int stage, double dt) {
    const int CT = p.Bp / 16, rows = block_rows(p);
    const block_fn fn = p.aligned ? pick_block<true>(CT, rows) : pick_block<false>(CT, rows);
    const bool odd = stage & 1;
    BlockArgs a;
    a.Qs = (const double* const*)p.d;
    a.Ks = (const double* const*)(p.d + 2 * p.R);
    a.M = p.M;
    a.ldq = p.ldq;
    a.kw = block_columns(p.M);
    a.V = p.V;
    a.Acc = p.Acc;
    a.sstride = p.sstride;
    a.Xin = odd ? p.X : p.Part;
    a.Xout = odd ? p.Part : p.X;
    a.in_stride = odd ? p.sstride : p.pstride;
    a.out_stride = odd ? p.pstride : p.sstride;
    a.h = dt;
    hipLaunchKernelGGL(fn, dim3(lb_blocks(p.M, rows), p.R), dim3(64 * kBlockWaves), 0, s, a, stage);
    LB_CHECK_LAUNCH();
    return LB_OK;
}

// The resident run and what follows it (finish: without it V stays as it is). Two that
// need more than half of the chip each could both be on it in part and wait in vain
// until one gives way, so those of a device are enqueued one behind the other, whatever
// their streams.
struct WideOrder {
    std::mutex mu;
    hipEvent_t last = nullptr;
};
WideOrder g_wide[kMaxDevices];

static int resident_piece(const Plan& p, hipStream_t s, double dt, int64_t steps, const Rk4Resident& res, bool finish) {
    const int64_t stride = rk4_resident_stride(p.M), n = 3 * stride;
    double* out = p.W + n;
    ResidentCtl* ctl = (ResidentCtl*)(out + stride);
    const double* const* q = (const double* const*)p.d;
    const double* const* k = (const double* const*)(p.d + 2 * p.R);
    double* const* v = (double* const*)(p.d + 3 * p.R);
    const int64_t start = std::min(res.start, steps * kResidentStepTicks);
    WideOrder& wide = g_wide[res.device];
    std::unique_lock<std::mutex> lk(wide.mu, std::defer_lock);
    if (res.wide) {
        lk.lock();
        LB_HIP(hipStreamWaitEvent(s, wide.last, 0));
    }
    hipLaunchKernelGGL(k_resident_init, dim3(lb_blocks(n, 256)), dim3(256), 0, s, p.W, n, ctl);
    LB_CHECK_LAUNCH();
    hipLaunchKernelGGL(res.fn, dim3(res.grid), dim3(256), 0, s, q, k, v, (int)p.M, p.ldq, p.W, stride, dt, steps, out,
                       ctl, start, res.run);
    LB_CHECK_LAUNCH();
    if (res.wide) LB_HIP(hipEventRecord(wide.last, s));
    if (!finish) return LB_OK;
    hipLaunchKernelGGL(p.aligned ? k_resident_end<true> : k_resident_end<false>, dim3(res.grid), dim3(1024), 0, s, q, k,
                       v, (int)p.M, p.ldq, p.W, stride, dt, steps, (const double*)out, ctl);
    LB_CHECK_LAUNCH();
    return LB_OK;
}

// A long run in pieces, so that a chip that is not free when it starts costs it one of
// them and not the whole run, and another that has to wait for the chip gets a turn.
static int resident_launch(const Plan& p, hipStream_t s, double dt, int64_t steps, const Rk4Resident& res) {
    while (steps > 0) {
        const int64_t pieces = (steps + kResidentPiece - 1) / kResidentPiece, n = (steps + pieces - 1) / pieces;
        const int rc = resident_piece(p, s, dt, n, res, true);
        if (rc) return rc;
        steps -= n;
    }
    return LB_OK;
}

// Enqueues the whole integration (kernels only: no synchronization, no copies),
// so it can be recorded into a graph.
static int plan_launch(const Plan& p, hipStream_t s, double dt, int64_t steps, const Rk4Resident& res) {
    if (steps == 0) return LB_OK;
    if (res.fn) return resident_launch(p, s, dt, steps, res);
    if (p.kind == PATH_SMALL) {
        hipLaunchKernelGGL(p.small.fn, dim3(p.R, p.B), dim3(p.small.threads), 0, s, (const double* const*)p.d,
                           (const double* const*)(p.d + 2 * p.R), (double* const*)(p.d + 3 * p.R), (int)p.M, p.ldq,
                           dt, steps);
        LB_CHECK_LAUNCH();
        return LB_OK;
    }
    int rc = plan_init_state(p, s);
    if (rc) return rc;
    if (p.kind == PATH_GEMV) {
        for (int64_t st = 0; st < steps; ++st)
            for (int stage = 1; stage <= 4; ++stage) {
                rc = plan_gemm(p, s, stage, dt);
                if (rc) return rc;
            }
        return LB_OK;
    }
    if (p.whole) {
        for (int64_t st = 0; st < steps; ++st)
            for (int stage = 1; stage <= 4; ++stage) {
                rc = plan_block(p, s, stage, dt);
                if (rc) return rc;
            }
        return plan_unpack(p, s);
    }
    const StageArgs sa = stage_args(p, dt);
    const dim3 sgrid(lb_blocks((p.M + 1) / 2 * p.Bp, 256), p.R);
    for (int64_t st = 0; st < steps; ++st)
        for (int stage = 1; stage <= 4; ++stage) {
            rc = plan_gemm(p, s, stage, dt);
            if (rc) return rc;
            hipLaunchKernelGGL(p.precision == LB_FP64 ? k_stage<double> : k_stage<float>, sgrid, dim3(256), 0, s, sa, stage);
            LB_CHECK_LAUNCH();
        }
    return plan_unpack(p, s);
}

// Stage time of a run with Q on the chip: a run of 2 + iters steps less one of 2. went: both
// were carried out (a chip that is not free ends them early) and the longer one took longer.
static int time_resident(const Plan& p, hipStream_t s, int iters, const Rk4Resident& res, double* ms, bool* went) {
    int rc = resident_piece(p, s, 0.0, 2, res, false);  // warm-up
    if (rc) return rc;
    const ResidentCtl* ctl = (const ResidentCtl*)(p.W + 4 * rk4_resident_stride(p.M));
    float t[2] = {0, 0};
    *went = true;
    hipEvent_t e[2];
    for (hipEvent_t& ev : e) LB_HIP(hipEventCreate(&ev));
    for (int i = 0; i < 2 && *went && !rc; ++i) {
        unsigned decision = 0;
        LB_HIP(hipEventRecord(e[0], s));
        rc = resident_piece(p, s, 0.0, i == 0 ? 2 : 2 + (int64_t)iters, res, false);
        LB_HIP(hipEventRecord(e[1], s));
        LB_HIP(hipMemcpyAsync(&decision, &ctl->decision, sizeof(decision), hipMemcpyDeviceToHost, s));
        LB_HIP(hipStreamSynchronize(s));
        LB_HIP(hipEventElapsedTime(&t[i], e[0], e[1]));
        *went = decision == kGo;
    }
    for (hipEvent_t ev : e) (void)hipEventDestroy(ev);
    *went = *went && t[1] > t[0];
    *ms = ((double)t[1] - t[0]) / (4.0 * iters);
    return rc;
}

// Average duration (ms) of a stage over `iters` launches of the kernel that is most or
// all of it, measured with HIP events on the context stream; with Q on the chip, of the
// stages by which a run of iters steps more is longer. The states are packed
// first; the kernel reads them but the timing loop does not advance them.
static int plan_time(lb_ctx* c, const Plan& p, int iters, const Rk4Resident& res, double* ms) {
    hipStream_t s = c->stream;
    int rc = LB_OK;
    if (res.fn) {
        bool went = false;
        rc = time_resident(p, s, iters, res, ms, &went);
        if (rc || went) return rc;
    }
    rc = plan_init_state(p, s);
    if (rc) return rc;
    auto launch = [&](int i) {
        return p.kind == PATH_GEMV ? plan_gemm(p, s, 1 + (i & 1), 0.0)
               : p.whole           ? plan_block(p, s, 1, 0.0)
                                   : plan_gemm(p, s, 1, 0.0);
    };
    rc = launch(0);  // warm-up
    if (rc) return rc;
    hipEvent_t e0, e1;
    LB_HIP(hipEventCreate(&e0));
    LB_HIP(hipEventCreate(&e1));
    LB_HIP(hipEventRecord(e0, s));
    for (int i = 0; i < iters && !rc; ++i) rc = launch(i);
    LB_HIP(hipEventRecord(e1, s));
    LB_HIP(hipEventSynchronize(e1));
    float t = 0;
    LB_HIP(hipEventElapsedTime(&t, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    *ms = (double)t / iters;
    return LB_OK;
}

static int plan_for(lb_ctx* c, Plan& p, int R, int64_t M, const lb_prop_sys* sys, int64_t ldq, int B, int precision,
                    const lb_tile* force_tile, bool allow_small) {
    const lb_tile tile = force_tile ? *force_tile : choose_tile(c, M, bpad(B), precision, R);
    int rc = plan_make(p, R, M, ldq, B, precision, tile, allow_small && force_tile == nullptr,
                       force_tile != nullptr || asked_tile(c, M, bpad(B), precision));
    if (rc) return rc;
    rc = lb_ws_reserve(c, p.bytes);
    if (rc) return rc;
    return plan_bind(c, p, (char*)c->ws, sys);
}

// The resident kernel for this plan, or none: one system, one state, enough steps
// to pay for the load of Q and two more launches, a stream that is not being captured,
// and not switched off for the context. It sums a row as k_gemv does: the same bits either way.
static Rk4Resident plan_resident(lb_ctx* c, const Plan& p, int64_t steps) {
    Rk4Resident r;
    if (p.kind != PATH_GEMV || p.R != 1 || steps < kResidentSteps || c->resident_start < 0) return r;
    r = rk4_resident_pick(p.M);
    if (!r.fn) return r;
    r.device = c->device;
    r.start = c->resident_start;
    r.run = c->resident_run;
    const unsigned cus = (unsigned)rk4_compute_units(c->device);
    r.wide = 2 * r.grid > cus;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &cap) != hipSuccess) (void)hipGetLastError();
    if (cap != hipStreamCaptureStatusNone || r.grid > cus) r.fn = nullptr;
    return r;
}

}  // namespace

// R systems of size M, B states each.
int lb_impl_propagate(lb_ctx* c, int R, int64_t M, const lb_prop_sys* sys, int64_t ldq, int B, double dt,
                      int64_t steps, int precision, const lb_tile* force_tile) {
    if (steps == 0) return LB_OK;
    Plan p;
    int rc = plan_for(c, p, R, M, sys, ldq, B, precision, force_tile, true);
    if (rc) return rc;
    return plan_launch(p, c->stream, dt, steps, plan_resident(c, p, steps));
}

int lb_impl_time_stage(lb_ctx* c, int R, int64_t M, const lb_prop_sys* sys, int64_t ldq, int B, int precision,
                       int iters, double* ms, const lb_tile* force_tile) {
    Plan p;
    int rc = plan_for(c, p, R, M, sys, ldq, B, precision, force_tile, false);
    if (rc) return rc;
    return plan_time(c, p, iters, plan_resident(c, p, 2 + (int64_t)iters), ms);
}

// ---------------------------------------------------------------------------
// Allocation-free propagation (one system): the plan's buffers -- packed
// states, stage accumulators, split-K partials, the pointer table -- live in a
// static device array instead of the context workspace, and the pointer table
// is written by a kernel instead of a staged host copy, so the call allocates
// nothing (no device, no pinned host memory) and never synchronizes. Each GPU
// holds its own copy of the array from module load until the process ends;
// every call on a GPU shares it (nothing in it must start at zero: the plan
// writes every element it reads), so calls that overlap on one GPU race.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = (size_t)LB_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) double scratch[kScratchBytes / sizeof(double)];

namespace {

std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices];  // device address of `scratch` on each GPU

__global__ void k_set_ptrs(const void** d, const void* q, const void* q32, const void* k, void* v) {
    if (threadIdx.x == 0) {
        d[0] = q;
        d[1] = q32;
        d[2] = k;
        d[3] = v;
        d[4] = v;
    }
}

}  // namespace

// Looks up the array's device address once per device, and makes the event that orders the wide
// resident runs there, so that no later call has to; `device` must be current.
int lb_scratch_init(int device) {
    if (device < 0 || device >= kMaxDevices) return lb_fail(LB_ERR_UNSUPPORTED, "device %d beyond %d", device, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch[device]) return LB_OK;
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
        return lb_fail(LB_ERR_DEVICE, "hipGetSymbolAddress(scratch) on device %d: %s", device, hipGetErrorString(e));
    LB_HIP(hipEventCreateWithFlags(&g_wide[device].last, hipEventDisableTiming));
    g_scratch[device] = ptr;
    return LB_OK;
}

int lb_impl_propagate_noalloc(lb_ctx* c, int64_t M, const lb_prop_sys* sys, int64_t ldq, int B, double dt,
                              int64_t steps, int precision) {
    if (steps == 0) return LB_OK;
    void* base = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_scratch_mu);
        base = c->device >= 0 && c->device < kMaxDevices ? g_scratch[c->device] : nullptr;
    }
    if (!base) return lb_fail(LB_ERR_DEVICE, "the static scratch of device %d is not set up", c->device);
    Plan p;
    const int Bp = bpad(B);
    const lb_tile tile = choose_tile(c, M, Bp, precision, 1);
    const bool own = has_tile(c, M, Bp, precision);
    int rc = plan_make(p, 1, M, ldq, B, precision, tile, true, asked_tile(c, M, Bp, precision));
    if (rc) return rc;
    size_t need = p.bytes;
    if (p.kind == PATH_MFMA && !own) {
        Plan lim;
        rc = plan_make(lim, 1, M, ldq, B, precision, limit_tile(M, Bp), true, own);
        if (rc) return rc;
        need = std::max(need, lim.bytes);
    }
    if (need > kScratchBytes)
        return lb_fail(LB_ERR_UNSUPPORTED,
                       "M=%lld with %d states needs %zu bytes of scratch; the allocation-free propagate holds %zu",
                       (long long)M, B, need, kScratchBytes);
    rc = plan_align(p, sys);
    if (rc) return rc;
    plan_buffers(p, (char*)base);
    hipLaunchKernelGGL(k_set_ptrs, dim3(1), dim3(64), 0, c->stream, p.d, (const void*)sys->Q, (const void*)sys->Q32,
                       (const void*)sys->K, (void*)sys->V);
    LB_CHECK_LAUNCH();
    return plan_launch(p, c->stream, dt, steps, plan_resident(c, p, steps));
}

struct lb_graph_entry {
    Plan plan;
    void* mem = nullptr;
    hipGraphExec_t exec = nullptr;
    uint64_t last_use = 0;
};

// Captured graphs kept per context (least recently used evicted first): each
// holds its plan buffers and the raw operand pointers it was captured with.
constexpr size_t kMaxGraphs = 8;

void lb_graph_free(lb_graph_entry* g) {
    if (!g) return;
    if (g->exec) (void)hipGraphExecDestroy(g->exec);
    if (g->mem) (void)hipFree(g->mem);
    delete g;
}

int lb_impl_propagate_graph(lb_ctx* c, int64_t M, const lb_prop_sys* sys, int64_t ldq, int B, double dt,
                            int64_t steps, int precision) {
    if (steps == 0) return LB_OK;
    lb_graph_key key{M, ldq, B, precision, sys->Q, sys->Q32, sys->K, sys->V, dt, steps};
    auto it = c->graphs.find(key);
    if (it == c->graphs.end()) {
        if (c->graphs.size() >= kMaxGraphs) {
            auto lru = c->graphs.begin();
            for (auto jt = c->graphs.begin(); jt != c->graphs.end(); ++jt)
                if (jt->second->last_use < lru->second->last_use) lru = jt;
            LB_HIP(hipStreamSynchronize(c->stream));  // its last launch may still run
            lb_graph_free(lru->second);
            c->graphs.erase(lru);
        }
        lb_graph_entry* g = new lb_graph_entry();
        const lb_tile tile = choose_tile(c, M, bpad(B), precision, 1);
        int rc = plan_make(g->plan, 1, M, ldq, B, precision, tile, true, asked_tile(c, M, bpad(B), precision));
        if (rc) {
            delete g;
            return rc;
        }
        hipError_t e = hipMalloc(&g->mem, g->plan.bytes);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            delete g;
            return lb_fail(LB_ERR_OOM, "graph buffers (%zu bytes): %s", g->plan.bytes, hipGetErrorString(e));
        }
        rc = plan_bind(c, g->plan, (char*)g->mem, sys);
        if (rc) {
            lb_graph_free(g);
            return rc;
        }
        hipStream_t cs;
        e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking);
        if (e != hipSuccess) {
            lb_graph_free(g);
            return lb_fail(LB_ERR_DEVICE, "hipStreamCreate: %s", hipGetErrorString(e));
        }
        hipGraph_t graph = nullptr;
        e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
        if (e == hipSuccess) {
            rc = plan_launch(g->plan, cs, dt, steps, Rk4Resident());
            hipError_t e2 = hipStreamEndCapture(cs, &graph);
            if (!rc && e2 != hipSuccess) rc = lb_fail(LB_ERR_DEVICE, "hipStreamEndCapture: %s", hipGetErrorString(e2));
        } else {
            rc = lb_fail(LB_ERR_DEVICE, "hipStreamBeginCapture: %s", hipGetErrorString(e));
        }
        (void)hipStreamDestroy(cs);
        if (!rc) {
            e = hipGraphInstantiate(&g->exec, graph, nullptr, nullptr, 0);
            if (e != hipSuccess) rc = lb_fail(LB_ERR_DEVICE, "hipGraphInstantiate: %s", hipGetErrorString(e));
        }
        if (graph) (void)hipGraphDestroy(graph);
        if (rc) {
            lb_graph_free(g);
            return rc;
        }
        it = c->graphs.emplace(key, g).first;
    }
    it->second->last_use = ++c->graph_clock;
    LB_HIP(hipGraphLaunch(it->second->exec, c->stream));
    return LB_OK;
}

// Tries tile shapes on the context stream and keeps the fastest stage kernel.
int lb_impl_autotune(lb_ctx* c, int64_t M, const lb_prop_sys* sys, int64_t ldq, int B, int precision) {
    const int Bp = bpad(B);
    if (B == 1 && precision == LB_FP64) return LB_OK;  // GEMV path has no tile
    const int CT = Bp / 16;
    std::vector<int> rows_c = CT == 1 ? std::vector<int>{32, 64} : std::vector<int>{16, 32};
    std::vector<int> waves_c = {1, 2, 4};
    std::vector<int> target_c = {1, 1250, 2500, 5000, 10000};  // 1: one slab per row block
    lb_tile best = lb_default_tile(M, Bp, precision, 1);
    double best_ms = 1e30, ms0 = 0;
    if (!lb_impl_time_stage(c, 1, M, sys, ldq, B, precision, 3, &ms0, &best)) best_ms = ms0;
    for (int rows : rows_c)
        for (int waves : waves_c)
            for (int target : target_c) {
                lb_tile t;
                t.rows = rows;
                t.waves = waves;
                const int64_t rowwaves = (M + rows - 1) / rows;
                int64_t nslab = (target + rowwaves - 1) / rowwaves;
                const int64_t maxslab = (M + 255) / 256;
                nslab = nslab < 1 ? 1 : (nslab > maxslab ? maxslab : nslab);
                int64_t ks = (M + nslab - 1) / nslab;
                t.kslab = (int)((ks + 31) / 32 * 32);
                double ms = 0;
                int rc = lb_impl_time_stage(c, 1, M, sys, ldq, B, precision, 3, &ms, &t);
                if (rc) continue;
                if (ms < best_ms) {
                    best_ms = ms;
                    best = t;
                }
            }
    lb_load_tune_cache(c);
    c->tuned[std::make_tuple(M, Bp, precision)] = best;
    c->measured.insert(std::make_tuple(M, Bp, precision));
    if (const char* path = getenv("LB_TUNE_CACHE")) {
        FILE* f = fopen(path, "a");
        if (f) {
            fprintf(f, "%lld %d %d %d %d %d\n", (long long)M, Bp, precision, best.rows, best.kslab, best.waves);
            fclose(f);
        }
    }
    return LB_OK;
}

// The square-wave drive eps(t) = E + A Theta(t), Theta = +1 on [0, T/2) and
// -1 on [T/2, T), of the rocked dimer (Sec. 3). `left` gives the limit from
// the left (at a switch: the half period that ends there).
static double drive_value(double t, double E, double A, double T, bool left) {
    double r = fmod(t, T);
    if (left) {
        if (r <= 0) r += T;
        return r <= 0.5 * T ? E + A : E - A;
    }
    if (r < 0) r += T;
    return r < 0.5 * T ? E + A : E - A;
}

// Stage time t0 + (k + c) dt as one product and one sum.
static double stage_time(double t0, int64_t k, double c, double dt) {
    const double kc = (double)k + c;
    volatile double p = kc * dt;
    return t0 + p;
}

static int csr_propagate(lb_ctx* c, int64_t M, const int64_t* rowptr, const int64_t* col, const double* val,
                         const int64_t* rowptr1, const int64_t* col1, const double* val1, const double* K, double* V,
                         int B, double dt, int64_t steps, double t0, int64_t k0, double E, double A, double T) {
    hipStream_t s = c->stream;
    if (steps == 0) return LB_OK;
    const bool drive = rowptr1 != nullptr;
    const int64_t n = M * B;
    SellMat m;
    size_t o_w = 0;
    int rc = sell_build(c, M, rowptr, col, val, rowptr1, col1, val1, sizeof(double) * 3 * (size_t)n, &m, &o_w);
    if (rc) return rc;
    double* W = (double*)((char*)c->ws + o_w);
    // W: accumulator, x of the odd stages, x of the even ones
    const double* xin[4] = {V, W + 2 * n, W + n, W + 2 * n};
    double* xout[4] = {W + 2 * n, W + n, W + 2 * n, nullptr};
    const double h[4] = {0.5 * dt, 0.5 * dt, dt, dt / 6.0};
    const unsigned grid = (unsigned)m.nlong8 + 8u * (unsigned)m.per_xcd;
    typedef void (*stage_fn)(SellMat, SellStage, double);
    const stage_fn fn = drive ? (B == 1 ? k_sell_stage<true, 1> : k_sell_stage<true, 4>)
                              : (B == 1 ? k_sell_stage<false, 1> : k_sell_stage<false, 4>);
    for (int64_t k = 0; k < steps; ++k)
        for (int stage = 1; stage <= 4; ++stage) {
            double eps = 0.0;
            if (drive) {
                // stages seen from inside the step: t_k and t_k + dt/2 from the right, t_k + dt from the left
                const double cst = stage == 1 ? 0.0 : (stage == 4 ? 1.0 : 0.5);
                eps = drive_value(stage_time(t0, k0 + k, cst, dt), E, A, T, stage == 4);
            }
            const SellStage st{B, stage, h[stage - 1], K, V, W, xin[stage - 1], xout[stage - 1]};
            hipLaunchKernelGGL(fn, dim3(grid), dim3(256), 0, s, m, st, eps);
            LB_CHECK_LAUNCH();
        }
    return LB_OK;
}

int lb_impl_propagate_csr(lb_ctx* c, int64_t M, const int64_t* rowptr, const int64_t* col, const double* val,
                          const double* K, double* V, int B, double dt, int64_t steps) {
    return csr_propagate(c, M, rowptr, col, val, nullptr, nullptr, nullptr, K, V, B, dt, steps, 0.0, 0, 0.0, 0.0, 1.0);
}

int lb_impl_propagate_csr_drive(lb_ctx* c, int64_t M, const int64_t* rowptr0, const int64_t* col0,
                                const double* val0, const int64_t* rowptr1, const int64_t* col1, const double* val1,
                                const double* K, double* V, int B, double dt, int64_t steps, double t0, int64_t k0,
                                double E, double A, double T) {
    return csr_propagate(c, M, rowptr0, col0, val0, rowptr1, col1, val1, K, V, B, dt, steps, t0, k0, E, A, T);
}
