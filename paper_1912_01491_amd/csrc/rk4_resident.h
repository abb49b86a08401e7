// RK4 of one dense system and one state with Q resident on the chip (256 < M <=
// 4096): a cooperative launch of one workgroup per compute unit holds Q in
// registers and LDS for all steps and exchanges only the stage vector.
//
// One launch per stage reads Q again from the last-level cache: 22.9 us for the
// 134 MB of N = 64, of which 19 are the read, and 4 to 6 us for systems of a few
// MB, most of it the launch. Resident, a stage is the exchange of M doubles
// through memory (a write and a poll, about 2 us) and M multiply-adds per row: us
// a stage, before and now, N = 20: 4.2 / 2.1, N = 37: 5.7 / 2.9, N = 50: 11.3 / 4.2,
// N = 64: 22.3 / 5.9. Registers and LDS hold 4096 x 4096 doubles (134 MB of 168);
// larger systems stream.
#pragma once

#include "lb_internal.h"
#include "rk4_small.h"
#include "rowdot.h"

namespace {

// The exchange: X is written and read with agent-scope accesses, so it passes
// the XCDs' separate L2s. A value not yet written reads as kPending, a signalling
// NaN, which no arithmetic result is (the vector unit returns quiet NaNs).
// Stage vector j lives in buffer j % 3. A workgroup that has read all of vector j
// knows that everyone has read vector j - 1 (vector j depends on all of it), and
// puts kPending back into its rows of that buffer, two exchanges before they are
// written again.
constexpr uint64_t kPending = 0x7ff0000000000001ull;

__device__ __forceinline__ uint64_t xchg_load(const double* p) {
    return __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void xchg_store(double* p, uint64_t v) {
    __hip_atomic_store(reinterpret_cast<uint64_t*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint2 w = __builtin_bit_cast(uint2, v);
    const uint2 o = make_uint2((unsigned)__builtin_amdgcn_update_dpp(0, (int)w.x, CTRL, 0xf, 0xf, true),
                               (unsigned)__builtin_amdgcn_update_dpp(0, (int)w.y, CTRL, 0xf, 0xf, true));
    return v + __builtin_bit_cast(double, o);
}

// Sum over the wavefront in the order of xor-shuffles by 32, 16, 8, 4, 2, 1, without LDS.
__device__ __forceinline__ double wave_sum_dpp(double v) {
    v = add_row(add_half(v));
    v = dpp_add<0x128>(v);  // row_ror:8
    v = dpp_add<0x124>(v);  // row_ror:4 (lanes 8 apart are equal by now)
    v = dpp_add<0x4e>(v);   // quad_perm:[2,3,0,1]
    return dpp_add<0xb1>(v);  // quad_perm:[1,0,3,2]
}

__global__ void k_resident_init(double* W, int64_t n) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) reinterpret_cast<uint64_t*>(W)[e] = kPending;
}

// Four rows per wave, RL of them in LDS; U column steps of 128 (M <= 128 U). Lane
// l holds columns 128 u + 2 l and the next one and sums them in the order of u,
// then the lanes are added by xor-shuffles: the order, and the bits, of k_gemv.
// The stage vector is polled once per workgroup and passed on through LDS (each
// wave polling all of it for itself, without barriers, was 1.6 times slower).
// Every wait ends: a wave whose exchange is not complete after `spins` polls
// (seconds; the cooperative launch has all of them resident, so none waits for
// one that cannot run) leaves NaN in its rows of V.
constexpr int kResRows = 4;

template <int RL, int U>
__global__ __launch_bounds__(256, 1) void k_rk4_resident(const double* const* Qs, const double* const* Ks,
                                                         double* const* Vs, int M, int64_t ldq, double* W,
                                                         int64_t wstride, double h, int64_t steps, int spins) {
    constexpr int R = kResRows, RR = R - RL, XB = RL ? 1 : 2;
    static_assert(U % 2 == 0, "whole rounds of 256 threads");
    __shared__ double xs[XB][128 * U];
    __shared__ double ql[RL ? 4 * RL : 1][RL ? 128 * U : 2];
    const double* Q = Qs[0];
    double* V = Vs[0];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row0 = ((int)blockIdx.x * 4 + wave) * R;
    lb_double2v q[RR][U];
#pragma unroll
    for (int t = 0; t < R; ++t) {
        const int row = row0 + t;
        const double* qr = Q + (int64_t)(row < M ? row : M - 1) * ldq;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = 2 * lane + 128 * u;
            const double a = row < M && c < M ? qr[c] : 0.0, b = row < M && c + 1 < M ? qr[c + 1] : 0.0;
            if (t < RR) q[t][u] = lb_double2v{a, b};
            else *reinterpret_cast<lb_double2v*>(&ql[wave * RL + t - RR][c]) = lb_double2v{a, b};
        }
    }
    const int mrow = row0 + lane;  // lanes 0 .. R - 1 keep a row's state
    const bool mine = lane < R && mrow < M;
    const double kc = mine ? Ks[0][mrow] : 0.0;
    double v = mine ? V[mrow] : 0.0, acc = 0.0;
    for (int c = threadIdx.x; c < 128 * U; c += 256)
        for (int b = 0; b < XB; ++b) xs[b][c] = b == 0 && c < M ? V[c] : 0.0;
    __syncthreads();
    // every wave has read V before any row of it is written (the end is an exchange away, or steps are none)
    // elements per thread of an exchange, and at a time (16 at once spill next to four rows of 32 steps)
    constexpr int NE = U / 2, NG = NE <= 8 ? NE : NE % 8 == 0 ? 8 : NE % 7 == 0 ? 7 : NE % 6 == 0 ? 6 : 5;
    static_assert(NE % NG == 0, "whole groups");
    int64_t j = 0;             // stage vectors exchanged so far
    for (int64_t st = 0; st < steps; ++st) {
#pragma unroll
        for (int stage = 1; stage <= 4; ++stage) {
            const double* x = xs[XB == 2 ? (stage & 1) ^ 1 : 0];
            double s[R];
#pragma unroll
            for (int t = 0; t < R; ++t) s[t] = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const lb_double2v xv = *reinterpret_cast<const lb_double2v*>(x + 2 * lane + 128 * u);
#pragma unroll
                for (int t = 0; t < R; ++t) {
                    const lb_double2v qv = t < RR ? q[t < RR ? t : 0][u]
                                                  : *reinterpret_cast<const lb_double2v*>(
                                                        &ql[wave * RL + t - RR][2 * lane + 128 * u]);
                    s[t] = fma(qv.x, xv.x, s[t]);
                    s[t] = fma(qv.y, xv.y, s[t]);
                }
            }
            double k = 0.0;
#pragma unroll
            for (int t = 0; t < R; ++t) {
                const double r = wave_sum_dpp(s[t]);
                if (lane == t) k = r;
            }
            const double xn = rk4_next(stage, h, k + kc, v, acc);
            if (stage == 4 && st + 1 == steps) break;
            // exchange vector j; its buffer, and the one to clear (vector j - 1, read by all once j is complete)
            double* buf = W + (j % 3) * wstride;
            double* old = W + ((j + 2) % 3) * wstride;
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): the last clearing is out before this vector is
            if (mine) xchg_store(buf + mrow, __builtin_bit_cast(uint64_t, xn));
            double* xw = xs[XB == 2 ? stage & 1 : 0];
            if (XB == 1) __syncthreads();  // the one buffer is still being read
#pragma unroll
            for (int i0 = 0; i0 < NE; i0 += NG) {
                uint64_t got[NG];
                bool all = true;
#pragma unroll
                for (int i = 0; i < NG; ++i) {
                    const int e = threadIdx.x + 256 * (i0 + i);
                    got[i] = e < M ? xchg_load(buf + e) : 0;
                }
#pragma unroll
                for (int i = 0; i < NG; ++i) all &= got[i] != kPending;
                for (int n = 0; !all; ++n) {
                    if (n > spins) {
                        if (mine) V[mrow] = __builtin_nan("");
                        return;
                    }
                    all = true;
#pragma unroll
                    for (int i = 0; i < NG; ++i) {
                        if (got[i] == kPending) got[i] = xchg_load(buf + threadIdx.x + 256 * (i0 + i));
                        all &= got[i] != kPending;
                    }
                }
#pragma unroll
                for (int i = 0; i < NG; ++i) xw[threadIdx.x + 256 * (i0 + i)] = __builtin_bit_cast(double, got[i]);
            }
            __syncthreads();
            if (j > 0 && mine) xchg_store(old + mrow, kPending);
            ++j;
        }
    }
    if (mine) V[mrow] = v;
}

typedef void (*rk4_resident_fn)(const double* const*, const double* const*, double* const*, int, int64_t, double*,
                                int64_t, double, int64_t, int);

struct Rk4Resident {
    rk4_resident_fn fn = nullptr;
    unsigned grid = 0;
};

// Kernel and grid for one system and one state, or none. Four rows per wave, so
// that a workgroup's 16 rows are one line of the exchange (with 1, 2 and 3 rows
// per wave N = 32 took 4.4, 3.0 and 2.9 us a stage; with 4, 2.5).
static Rk4Resident rk4_resident_pick(int64_t M) {
    Rk4Resident r;
    if (M <= 256 || M > 4096) return r;
    r.grid = (unsigned)((M + 4 * kResRows - 1) / (4 * kResRows));
    r.fn = M <= 512    ? k_rk4_resident<0, 4>
           : M <= 768  ? k_rk4_resident<0, 6>
           : M <= 1024 ? k_rk4_resident<0, 8>
           : M <= 1536 ? k_rk4_resident<0, 12>
           : M <= 2048 ? k_rk4_resident<0, 16>
           : M <= 2560 ? k_rk4_resident<0, 20>
           : M <= 3072 ? k_rk4_resident<0, 24>
           : M <= 3584 ? k_rk4_resident<1, 28>
                       : k_rk4_resident<1, 32>;
    return r;
}

// Whether a cooperative launch of `grid` workgroups, one per compute unit, fits the current device.
static bool rk4_resident_fits(int device, unsigned grid) {
    int coop = 0, cus = 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, device) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return coop && grid <= (unsigned)cus;
}

}  // namespace
