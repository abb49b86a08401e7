// RK4 of one dense system and one state with Q resident on the chip (256 < M <=
// 4096): a launch of one workgroup per 16 rows holds Q in registers and LDS for all
// steps and exchanges only the stage vector.
//
// One launch per stage reads Q again from the last-level cache: 22.1 us for the
// 134 MB of N = 64, of which 19 are the read, and 4 to 6 us for systems of a few
// MB, most of it the launch. Resident, a stage is the exchange of M doubles
// through memory (a write and a poll, about 2 us) and M multiply-adds per row: us
// a stage of 100 steps, launches and resident, N = 20: 4.4 / 2.0, N = 37: 5.1 / 2.8,
// N = 50: 11.1 / 4.2, N = 64: 22.1 / 5.9. As a cooperative launch, which HIP runs one
// at a time, N = 37 took 3.0, and 8 threads with N = 17 each 18.1 between them,
// now 4.4. Registers and LDS hold 4096 x 4096 doubles (134 MB of 168);
// larger systems stream.
//
// The workgroups wait for each other, so all of them have to be on the chip at
// once. Other streams and processes may hold a part of it for any time, and no
// launch keeps them off, so the workgroups first count themselves in: the last one
// to arrive decides that they go; one that has waited for `start` decides that they
// leave, whichever comes first. From then on each wait is for a workgroup that
// runs. A wait beyond `run` all the same (a process put aside) ends the attempt.
// V is written by the kernel behind it, k_resident_end: with the attempt's result
// where no wave left, else by integrating from the untouched V in a form that is
// right with any number of workgroups on the chip.
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

// What the workgroups of a run share besides the vectors, cleared by k_resident_init.
struct ResidentCtl {
    unsigned decision;  // 0: open, else one of the two below
    unsigned arrived;   // workgroups that have started
    unsigned long long ticket, done;  // k_resident_end: pieces of work taken, and finished
};
constexpr unsigned kGo = 1, kLeave = 2;

template <typename T>
__device__ __forceinline__ T agent_load(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T agent_add(T* p, T v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Settles an open decision; one that is settled stays.
__device__ __forceinline__ void decide(ResidentCtl* c, unsigned d) {
    unsigned open = 0;
    __hip_atomic_compare_exchange_strong(&c->decision, &open, d, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void k_resident_init(double* W, int64_t n, ResidentCtl* ctl) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) reinterpret_cast<uint64_t*>(W)[e] = kPending;
    if (e == 0) *ctl = ResidentCtl{};
}

// Four rows per wave, RL of them in LDS; U column steps of 128 (M <= 128 U). Lane
// l holds columns 128 u + 2 l and the next one and sums them in the order of u,
// then the lanes are added by xor-shuffles: the order, and the bits, of k_gemv.
// The stage vector is polled once per workgroup and passed on through LDS (each
// wave polling all of it for itself, without barriers, was 1.6 times slower).
// start, run: ticks of the constant 100 MHz clock. A wave that leaves has settled the
// decision to that, or found it so, and a decision that still is to go when the
// kernel has ended means that every wave came to its end. The other waves of its
// workgroup (a barrier does not wait for one that has ended) and the other workgroups
// may go on with a stage vector that lacks its part, up to their next wait for one of
// its rows: nothing they write is used then.
constexpr int kResRows = 4;

template <int RL, int U>
__global__ __launch_bounds__(256, 1) void k_rk4_resident(const double* const* Qs, const double* const* Ks,
                                                         double* const* Vs, int M, int64_t ldq, double* W,
                                                         int64_t wstride, double h, int64_t steps, double* out,
                                                         ResidentCtl* ctl, int64_t start, int64_t run) {
    constexpr int R = kResRows, RR = R - RL, XB = RL ? 1 : 2;
    static_assert(U % 2 == 0, "whole rounds of 256 threads");
    __shared__ double xs[XB][128 * U];
    __shared__ double ql[RL ? 4 * RL : 1][RL ? 128 * U : 2];
    const int64_t since = wall_clock64();
    // arrives before it loads Q, waits after
    if (threadIdx.x == 0) {
        if (start == 0) decide(ctl, kLeave);
        if (agent_add(&ctl->arrived, 1u) + 1 == gridDim.x) decide(ctl, kGo);
    }
    const double* Q = Qs[0];
    const double* V = Vs[0];
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
    unsigned d;
    while ((d = agent_load(&ctl->decision)) == 0)
        if (lane == 0 && wall_clock64() - since >= start) decide(ctl, kLeave);
    if (d != kGo) return;
    __syncthreads();
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
                int64_t from = 0;
                for (unsigned n = 1; !all; ++n) {
                    if (run == 0 || n % 256 == 0) {
                        const int64_t now = wall_clock64();
                        if (from == 0) from = now;
                        if (now - from >= run || agent_load(&ctl->decision) != kGo) {
                            __hip_atomic_store(&ctl->decision, kLeave, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            break;
                        }
                    }
                    all = true;
#pragma unroll
                    for (int i = 0; i < NG; ++i) {
                        if (got[i] == kPending) got[i] = xchg_load(buf + threadIdx.x + 256 * (i0 + i));
                        all &= got[i] != kPending;
                    }
                }
                if (__any(!all)) return;
#pragma unroll
                for (int i = 0; i < NG; ++i) xw[threadIdx.x + 256 * (i0 + i)] = __builtin_bit_cast(double, got[i]);
            }
            __syncthreads();
            if (j > 0 && mine) xchg_store(old + mrow, kPending);
            ++j;
        }
    }
    if (mine) out[mrow] = v;
}

__device__ __forceinline__ unsigned long long first_lane(unsigned long long v) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
    return (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 | lo;
}

// Behind the attempt: its result into V, or, where it was left, the integration from
// the start. The pieces (stage by stage, 16 rows each, a row per wave) are handed out
// in order, and a workgroup waits only for pieces handed out before its own, which
// running workgroups hold: it ends with any number of them on the chip. V, the
// accumulators and the stage vectors pass between workgroups as above. A row's sum is
// k_gemv's (wave_rowdots), so the bits are the same on every way. On a free chip, in
// us a stage, a launch per stage / this: N = 17 4.1 / 4.2, N = 37 5.0 / 9.0, N = 50
// 11.0 / 16.8, N = 64 22 / 31 (pieces of 32 and 64 rows: 34 and 39 at N = 64): the two
// counters, 8 to 10 us for the 256 workgroups of N = 64, and x read by each of them.
template <bool ALIGNED>
__global__ __launch_bounds__(1024) void k_resident_end(const double* const* Qs, const double* const* Ks,
                                                       double* const* Vs, int M, int64_t ldq, double* W,
                                                       int64_t wstride, double h, int64_t steps, const double* out,
                                                       ResidentCtl* ctl) {
    __shared__ __align__(16) double xs[4096];
    __shared__ unsigned long long piece;
    double* V = Vs[0];
    if (ctl->decision == kGo) {
        const int e = (int)(blockIdx.x * blockDim.x + threadIdx.x);
        if (e < M) V[e] = out[e];
        return;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const unsigned long long tiles = (unsigned)(M + 15) / 16, total = 4 * (unsigned long long)steps * tiles;
    double *Acc = W, *Xa = W + wstride, *Xb = W + 2 * wstride;
    unsigned long long next = 0, mine = 0;
    if (threadIdx.x == 0) next = agent_add(&ctl->ticket, 1ull);
    // One thread's work per round in one place and every branch around a barrier on wave-uniform
    // values: with the first thread's additions at the round's end as well, the compiler let its
    // wave's other lanes run on into the next round's barriers without it.
    for (;; mine = 1) {
        if (wave == 0) {
            if (lane == 0) {
                agent_add(&ctl->done, mine);
                piece = next;
            }
            const unsigned long long t = first_lane(next);
            if (t < total)
                while (agent_load(&ctl->done) < t / tiles * tiles) __builtin_amdgcn_s_sleep(1);
            if (lane == 0) next = agent_add(&ctl->ticket, 1ull);  // on its way during this piece
        }
        __syncthreads();
        const unsigned long long t = first_lane(piece);
        if (t >= total) return;
        const int stage = (int)(t / tiles % 4) + 1;
        const double* x = stage == 1 ? V : stage == 3 ? Xb : Xa;
        double* xn = stage == 4 ? V : stage == 2 ? Xb : Xa;
        for (int e = threadIdx.x; e < M; e += 1024) xs[e] = __builtin_bit_cast(double, xchg_load(x + e));
        __syncthreads();
        const int row = (int)(t % tiles) * 16 + wave;
        if (row < M) {
            const double* q = Qs[0] + (int64_t)row * ldq;
            double k;
            wave_rowdots<1, ALIGNED, false>(&q, xs, M, lane, &k);
            if (lane == 0) {
                double v = __builtin_bit_cast(double, xchg_load(V + row));
                double acc = stage > 1 ? __builtin_bit_cast(double, xchg_load(Acc + row)) : 0.0;
                const double n = rk4_next(stage, h, k + Ks[0][row], v, acc);
                xchg_store(xn + row, __builtin_bit_cast(uint64_t, n));
                if (stage < 4) xchg_store(Acc + row, __builtin_bit_cast(uint64_t, acc));
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): these rows are out before the piece counts as done
        __syncthreads();
    }
}

typedef void (*rk4_resident_fn)(const double* const*, const double* const*, double* const*, int, int64_t, double*,
                                int64_t, double, int64_t, double*, ResidentCtl*, int64_t, int64_t);

struct Rk4Resident {
    rk4_resident_fn fn = nullptr;
    unsigned grid = 0;
    bool wide = false;  // takes more than half of the chip
    int64_t start = 0, run = 0;
    int device = 0;
};

// Doubles of one of the run's vectors, and the bytes it needs behind k_gemv's three: its
// result and the shared words.
static int64_t rk4_resident_stride(int64_t M) { return (int64_t)lb_align(M, 32); }
static size_t rk4_resident_bytes(int64_t M) { return sizeof(double) * rk4_resident_stride(M) + sizeof(ResidentCtl); }
static bool rk4_resident_range(int64_t M) { return M > 256 && M <= 4096; }

// Kernel and grid for one system and one state, or none. Four rows per wave, so
// that a workgroup's 16 rows are one line of the exchange (with 1, 2 and 3 rows
// per wave N = 32 took 4.4, 3.0 and 2.9 us a stage; with 4, 2.5).
static Rk4Resident rk4_resident_pick(int64_t M) {
    Rk4Resident r;
    if (!rk4_resident_range(M)) return r;
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

static int rk4_compute_units(int device) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess) return cus;
    (void)hipGetLastError();
    return 0;
}

}  // namespace
