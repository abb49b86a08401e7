// RK4 of small dense systems (M <= 256): one workgroup integrates one state of
// one system over all steps, with Q in its registers for the whole run.
//
// A stage of such a system is a few thousand multiply-adds, so its cost is the
// latency of one pass around the workgroup. The earlier form (one thread per
// row, all states of a system in one workgroup, Q reread from LDS or L2 every
// stage) spent 2.8 us a stage on one state of 63 unknowns and 11.1 us on 16.
// Here a workgroup per state keeps 16 states as fast as one (a launch has 256
// compute units to fill and the states do not interact), and a stage is: 16
// multiply-adds per row tile on registers, one LDS write of the partial row
// sums, one barrier, and the sum of the partials: 0.21 us a stage at 63 unknowns
// (1000 steps 0.84 ms, was 11.1 ms with one state and 44.8 ms with 16).
#pragma once

#include "lb_internal.h"

namespace {

// The stage combination on registers: k = (Q x + K)_i; returns the next stage's x_i.
// The fused multiply-adds are written out: what the compiler makes of sums and
// products depends on whether it knows the stage, and the bits with it.
__device__ __forceinline__ double rk4_next(int stage, double h, double k, double& v, double& acc) {
    if (stage == 1) {
        acc = k;
        return fma(0.5 * h, k, v);
    }
    if (stage == 2) {
        acc = fma(2.0, k, acc);
        return fma(0.5 * h, k, v);
    }
    if (stage == 3) {
        acc = fma(2.0, k, acc);
        return fma(h, k, v);
    }
    v = fma(h / 6.0, acc + k, v);
    return v;
}

// Lane N of each row of 16 lanes, broadcast to the row.
template <int N>
__device__ __forceinline__ double row_bcast(double x) {
    return __builtin_amdgcn_update_dpp(0.0, x, 0x150 + N, 0xf, 0xf, true);  // row_newbcast:N
}

// v of this lane plus v of the lane 32 (add_half) or 16 (add_row) away: the same
// two terms on both lanes, so values replicated over the four rows of 16 lanes
// stay equal bit for bit.
__device__ __forceinline__ double add_half(double v) {
    const uint2 w = __builtin_bit_cast(uint2, v);
    const auto lo = __builtin_amdgcn_permlane32_swap(w.x, w.x, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(w.y, w.y, false, false);
    return __builtin_bit_cast(double, make_uint2(lo[0], hi[0])) + __builtin_bit_cast(double, make_uint2(lo[1], hi[1]));
}
__device__ __forceinline__ double add_row(double v) {
    const uint2 w = __builtin_bit_cast(uint2, v);
    const auto lo = __builtin_amdgcn_permlane16_swap(w.x, w.x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(w.y, w.y, false, false);
    return __builtin_bit_cast(double, make_uint2(lo[0], hi[0])) + __builtin_bit_cast(double, make_uint2(lo[1], hi[1]));
}

// sum[t] += q[t][n] x[n] over the 16 columns of a chunk, x[n] in lane n of each row of 16.
template <int N, int RR>
__device__ __forceinline__ void lanes_chunk(const double (&q)[RR][16], double x, double (&sum)[RR][2]) {
    if constexpr (N < 16) {
        const double xn = row_bcast<N>(x);
#pragma unroll
        for (int t = 0; t < RR; ++t) sum[t][N & 1] = fma(q[t][N], xn, sum[t][N & 1]);
        lanes_chunk<N + 1, RR>(q, x, sum);
    }
}

// The same for one row tile whose columns come from LDS (column stride 64).
template <int N>
__device__ __forceinline__ void lanes_tail(const double* q, double x, double (&sum)[2]) {
    if constexpr (N < 16) {
        sum[N & 1] = fma(q[N * 64], row_bcast<N>(x), sum[N & 1]);
        lanes_tail<N + 1>(q, x, sum);
    }
}

// Workgroup (system, state). Wave w holds CH chunks of 16 columns (16 CH w ..)
// of all rows, lane = row within each row tile of 64: RR tiles in registers and,
// with TAIL, one more in LDS (a 255 x 255 Q is the whole register file). The x
// values of a chunk sit one per lane (replicated over the four rows of 16
// lanes) and are broadcast by the DPP unit. The waves' partial sums meet in
// LDS, double-buffered (one barrier per stage), and wave w sums, combines and
// keeps the elements of its own columns, so x never passes through LDS.
template <int RR, bool TAIL, int CH>
struct Lanes {
    static constexpr int RT = RR + (TAIL ? 1 : 0);
    static constexpr int W = (4 * RT + CH - 1) / CH;  // waves that cover 64 RT columns
};

template <int RR, bool TAIL, int CH>
__global__ __launch_bounds__((64 * Lanes<RR, TAIL, CH>::W)) void k_rk4_lanes(const double* const* Qs,
                                                                            const double* const* Ks, double* const* Vs,
                                                                            int M, int64_t ldq, double h,
                                                                            int64_t steps) {
    constexpr int W = Lanes<RR, TAIL, CH>::W, RT = Lanes<RR, TAIL, CH>::RT;
    __shared__ double part[2][W][RT * 64];
    __shared__ double tail[TAIL ? 64 * RT : 1][64];  // [column][row - 64 RR]
    const double* Q = Qs[blockIdx.x];
    double* V = Vs[blockIdx.x] + (int64_t)blockIdx.y * M;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double q[CH][RR][16];
#pragma unroll
    for (int u = 0; u < CH; ++u)
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int n = 0; n < 16; ++n) {
                const int row = 64 * t + lane, c = 16 * (CH * w + u) + n;
                const double a = row < M && c < M ? Q[row * ldq + c] : 0.0;
                if (t < RR) q[u][t][n] = a;
                else if (TAIL) tail[c][lane] = a;
            }
    // this lane's elements, one per chunk; those past M stay exactly zero
    bool mine[CH];
    double kc[CH], x[CH], v[CH], acc[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        const int e = 16 * (CH * w + u) + (lane & 15);
        mine[u] = e < M;
        kc[u] = mine[u] ? Ks[blockIdx.x][e] : 0.0;
        x[u] = v[u] = mine[u] ? V[e] : 0.0;
        acc[u] = 0.0;
    }
    // partials of waves that were not launched stay zero
    for (int i = threadIdx.x; i < 2 * W * RT * 64; i += blockDim.x) (&part[0][0][0])[i] = 0.0;
    __syncthreads();
    const int g = lane >> 4;
    for (int64_t st = 0; st < steps; ++st) {
#pragma unroll
        for (int stage = 1; stage <= 4; ++stage) {
            double (*pb)[RT * 64] = part[stage & 1];
            double sum[RR][2], tsum[2] = {0.0, 0.0};
#pragma unroll
            for (int t = 0; t < RR; ++t) sum[t][0] = sum[t][1] = 0.0;
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                lanes_chunk<0, RR>(q[u], x[u], sum);
                if (TAIL) lanes_tail<0>(&tail[16 * (CH * w + u)][lane], x[u], tsum);
            }
#pragma unroll
            for (int t = 0; t < RR; ++t) pb[w][64 * t + lane] = sum[t][0] + sum[t][1];
            if (TAIL) pb[w][64 * RR + lane] = tsum[0] + tsum[1];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                const int e = 16 * (CH * w + u) + (lane & 15);
                double k;
                if (W == 4) {
                    k = (pb[0][e] + pb[1][e]) + (pb[2][e] + pb[3][e]);
                } else {
                    // rows of 16 lanes take every fourth wave's partial and add up across the wavefront
                    k = pb[g][e];
#pragma unroll
                    for (int j = 4; j < W; j += 4) k += pb[j + g][e];
                    k = add_row(add_half(k));
                }
                const double xn = rk4_next(stage, h, k + kc[u], v[u], acc[u]);
                x[u] = mine[u] ? xn : 0.0;
            }
        }
    }
    if (g != 0) return;
#pragma unroll
    for (int u = 0; u < CH; ++u)
        if (mine[u]) V[16 * (CH * w + u) + lane] = v[u];
}

typedef void (*rk4_small_fn)(const double* const*, const double* const*, double* const*, int, int64_t, double, int64_t);

struct Rk4Small {
    rk4_small_fn fn;
    unsigned threads;
};

// Kernel and workgroup size for M <= 256: as many row tiles of 64 as M needs,
// one wave per 16 columns up to the 12 waves whose share of Q (96 registers a
// lane) fits; beyond, 8 waves of 32 columns (192) and the last row tile in LDS.
static Rk4Small rk4_small_pick(int M) {
    const unsigned th = 64u * (unsigned)((M + 15) / 16);
    if (M <= 64) return Rk4Small{k_rk4_lanes<1, false, 1>, th};
    if (M <= 128) return Rk4Small{k_rk4_lanes<2, false, 1>, th};
    if (M <= 192) return Rk4Small{k_rk4_lanes<3, false, 1>, th};
    return Rk4Small{k_rk4_lanes<3, true, 2>, 64u * (unsigned)((M + 31) / 32)};
}

}  // namespace
