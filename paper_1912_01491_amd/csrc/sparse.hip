// Sparse data preparation: Q in CSR form and K for a Hamiltonian H and jump
// operators L_p with rates g_p, i.e. a Kossakowski matrix given through its
// spectral form gamma = sum_p g_p l_p l_p^+ (Sec. 2) with sparse l_p, as in the
// dimer model of Sec. 3 (P = 1).
//
// With L(X) = -i[H, X] + sum_p g_p (L_p X L_p^+ - 1/2 {L_p^+ L_p, X}) and its
// adjoint L^+(Y) = i[H, Y] + sum_p g_p (L_p^+ Y L_p - 1/2 {L_p^+ L_p, Y}),
//     Q_sn = Tr(F_s L(F_n)) = Tr(L^+(F_s) F_n),  K_s = Tr(L^+(F_s)) / N,
// so row s of Q is the expansion of the sparse matrix L^+(F_s) over the basis:
// off-diagonal entries give the S/J columns, the diagonal gives the D columns
// through prefix sums (w_m(x) = 1/sqrt(m(m+1)) for x < m, -m/sqrt(m(m+1)) at
// x = m). Rows of the diagonal generators are built column-wise instead:
// Q[D^m][n] = sum_x w_m(x) (L(F_n))_xx, and column n contributes to every
// row m >= the first position where diag(L(F_n)) is nonzero.
//
// The identity part c = Tr(L_p)/N of each jump operator is moved into the
// Hamiltonian (H += (i g_p/2)(conj(c) L0 - c L0^+), L0 = L_p - c 1), because
// the generator basis has no identity element.
//
// Pipeline (a count ends before the last step, where a fill knows the number of
// entries and asks for the arrays, then writes columns and values):
//   densify H, L_p -> trace shift -> G = sum_p g_p L0^+ L0, A = i H - G/2
//   column lists of A and L0_p, row lists of L0_p (ELL, width = max degree)
//   pair rows:   one thread per row, the entries of L^+(F_s) in LDS, sorted in
//                registers, merged and expanded
//   diag lists:  diag(L(F_n)) per column n (count, scan, fill), then their
//                exclusive prefix sums
//   D rows:      one block per row over the columns that carry a diagonal
// The stored entries (7.5 M for the N = 1000 dimer) are written in a fraction
// of a millisecond; what the phases cost is the latency of many small steps, so
// every loop over N or M runs across lanes and the scans stay on the device.
// N = 1000 dimer: 14.9 ms before, 0.97 ms as two calls (a count, and a fill that
// has to count again), 0.58 ms as one, 0.47 ms with the pair rows' counts beside the
// diagonals' lists and the two fills beside each other on a second stream. Below
// N = 400 launches and read-backs are all of it: 0.24 ms at N = 100 with 30 launches and three
// read-backs, 0.16 ms with 22 and two.
// Rows are written with sorted column indices (S block, J block, D block);
// entries whose value is exactly zero are not stored.
#include "lb_internal.h"
#include "scan.h"

#include <string.h>

#include <algorithm>

namespace {

constexpr double kR = 0.70710678118654752440;
constexpr int kMaxRowEntries = 64;  // entries of L^+(F_s) held per pair row
constexpr int64_t kListEntries = 10 << 20;  // of the diagonals' lists, reserved unseen (28 bytes each)
constexpr int kValueEntries = 24;   // up to which their values are held too

struct Ell {
    int* idx;     // N x W
    double* val;  // N x W complex
    const int* cnt;  // N
    int W;
};

__device__ __forceinline__ cd ell_val(const Ell& e, int i, int t) { return cload(e.val, (int64_t)i * e.W + t); }
__device__ __forceinline__ int ell_idx(const Ell& e, int i, int t) { return e.idx[(int64_t)i * e.W + t]; }

// ---------------------------------------------------------------------------
// Dense set-up kernels
// ---------------------------------------------------------------------------

// One wavefront per row. Entries go in parallel when the row's columns are
// strictly increasing; otherwise (repeated columns add up) one lane adds them
// in their order. Columns outside 0..N-1 are ignored.
struct DenseJobs {
    lb_csr_c128 m[8];
    double* D[8];
};

__global__ __launch_bounds__(64) void k_densify(int N, DenseJobs jobs) {
    const int64_t *rowptr = jobs.m[blockIdx.y].rowptr, *col = jobs.m[blockIdx.y].col;
    const double* val = jobs.m[blockIdx.y].val;
    double* D = jobs.D[blockIdx.y];
    const int r = blockIdx.x, lane = threadIdx.x;
    double* row = D + 2 * (int64_t)r * N;
    for (int c = lane; c < N; c += 64) cstore(row, c, cmk(0, 0));
    const int64_t e0 = rowptr[r], e1 = rowptr[r + 1];
    bool bad = false;
    for (int64_t e = e0 + lane; e + 1 < e1; e += 64) bad |= col[e + 1] <= col[e];
    __syncthreads();
    if (__ballot(bad) == 0) {
        for (int64_t e = e0 + lane; e < e1; e += 64) {
            const int64_t c = col[e];
            if (c >= 0 && c < N) cstore(row, c, cadd(cmk(0, 0), cload(val, e)));
        }
    } else if (lane == 0) {
        for (int64_t e = e0; e < e1; ++e) {
            const int64_t c = col[e];
            if (c < 0 || c >= N) continue;
            cstore(row, c, cadd(cload(row, c), cload(val, e)));
        }
    }
}

// single block: c_p = Tr(L_p)/N for all p, and L0_p = L_p - c_p 1 in place
__global__ void k_shift_l(int N, int P, double* Ld, double* c) {
    __shared__ double sr[256], si[256];
    for (int p = 0; p < P; ++p) {
        double r = 0, i = 0;
        for (int x = threadIdx.x; x < N; x += blockDim.x) {
            const cd v = cload(Ld + 2 * (int64_t)p * N * N, (int64_t)x * N + x);
            r += v.re;
            i += v.im;
        }
        sr[threadIdx.x] = r;
        si[threadIdx.x] = i;
        __syncthreads();
        for (int s = blockDim.x / 2; s > 0; s >>= 1) {
            if ((int)threadIdx.x < s) {
                sr[threadIdx.x] += sr[threadIdx.x + s];
                si[threadIdx.x] += si[threadIdx.x + s];
            }
            __syncthreads();
        }
        const cd t = cmk(sr[0] / N, si[0] / N);
        if (threadIdx.x == 0) cstore(c, p, t);
        double* L = Ld + 2 * (int64_t)p * N * N;
        for (int x = threadIdx.x; x < N; x += blockDim.x)
            cstore(L, (int64_t)x * N + x, csub(cload(L, (int64_t)x * N + x), t));
        __syncthreads();
    }
}

// H += sum_p (i g_p / 2)(conj(c_p) L0 - c_p L0^+);  G = sum_p g_p L0^+ L0;  A = i H - G/2.
// One block per row a: column a of L0_p (a strided read) goes to LDS once, with
// the list of its nonzeros in increasing x; then threads take b, so G_ab costs
// the column's degree and not N.
__global__ __launch_bounds__(256) void k_heff_a(int N, int P, const double* rates, const double* c, const double* Ld,
                                                const double* Hd, double* A) {
    extern __shared__ double2 lcol[];  // N values, then N indices
    int* xl = reinterpret_cast<int*>(lcol + N);
    __shared__ int wcnt[4];
    const int a = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int b0 = 0; b0 < N; b0 += 4 * 256) {
        // four b per thread at a time
        cd h[4], g[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = b0 + 256 * u + threadIdx.x;
            h[u] = b < N ? cload(Hd, (int64_t)a * N + b) : cmk(0, 0);
            g[u] = cmk(0, 0);
        }
        for (int p = 0; p < P; ++p) {
            const double* L = Ld + 2 * (int64_t)p * N * N;
            int n = 0;
            for (int x0 = 0; x0 < N; x0 += 256) {
                const int x = x0 + threadIdx.x;
                const cd v = x < N ? cload(L, (int64_t)x * N + a) : cmk(0, 0);
                const bool nz = !(v.re == 0.0 && v.im == 0.0);
                const unsigned long long m = __ballot(nz);
                __syncthreads();
                if (lane == 0) wcnt[w] = __popcll(m);
                __syncthreads();
                int o = n + __popcll(m & ((1ull << lane) - 1ull));
                for (int i = 0; i < 4; ++i) {
                    if (i < w) o += wcnt[i];
                    n += wcnt[i];
                }
                if (nz) xl[o] = x;
                if (x < N) lcol[x] = make_double2(v.re, v.im);
            }
            __syncthreads();
            const cd cp = cmk(c[2 * p], c[2 * p + 1]);
            const double gp = rates[p];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int b = b0 + 256 * u + threadIdx.x;
                if (b >= N) continue;
                const cd l_ab = cload(L, (int64_t)a * N + b);
                const cd ldag_ab = cmk(lcol[b].x, -lcol[b].y);
                const cd d = csub(cmul(cconj(cp), l_ab), cmul(cp, ldag_ab));
                h[u] = cadd(h[u], cscale(cmk(-d.im, d.re), 0.5 * gp));  // (i g/2) d
                cd s = cmk(0, 0);
                for (int t = 0; t < n; ++t) {
                    const int x = xl[t];
                    s = cadd(s, cmul(cmk(lcol[x].x, -lcol[x].y), cload(L, (int64_t)x * N + b)));
                }
                g[u] = cadd(g[u], cscale(s, gp));
            }
            __syncthreads();
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = b0 + 256 * u + threadIdx.x;
            // A = i h - g/2
            if (b < N)
                cstore(A, (int64_t)a * N + b, cmk(-h[u].im - 0.5 * g[u].re, h[u].re - 0.5 * g[u].im));
        }
    }
}

// Nonzeros of the N x N complex matrices in ELL lists, one wavefront per list.
// List set 0 is A by column; 1 + 2p and 2 + 2p are L0_p by row and by column.
__device__ __forceinline__ cd ell_src(int N, const double* A, const double* Ld, int set, int i, int j) {
    const double* D = set == 0 ? A : Ld + 2 * (int64_t)((set - 1) >> 1) * N * N;
    return set == 0 || !(set & 1) ? cload(D, (int64_t)j * N + i) : cload(D, (int64_t)i * N + j);
}

__global__ __launch_bounds__(256) void k_ell_count(int N, const double* A, const double* Ld, int* cnt) {
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, set = blockIdx.y;
    if (i >= N) return;
    int n = 0;
    for (int j0 = 0; j0 < N; j0 += 64) {
        const int j = j0 + lane;
        const cd v = j < N ? ell_src(N, A, Ld, set, i, j) : cmk(0, 0);
        n += __popcll(__ballot(v.re != 0.0 || v.im != 0.0));
    }
    if (lane == 0) cnt[(int64_t)set * N + i] = n;
}

// Widest list of each set, one wavefront per set.
__global__ __launch_bounds__(64) void k_ell_width(int N, const int* cnt, int* wmax) {
    int m = 0;
    for (int i = threadIdx.x; i < N; i += 64) m = max(m, cnt[(int64_t)blockIdx.x * N + i]);
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
    if (threadIdx.x == 0) wmax[blockIdx.x] = m;
}

__global__ __launch_bounds__(256) void k_ell_fill(int N, const double* A, const double* Ld, const Ell* ells) {
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, set = blockIdx.y;
    if (i >= N) return;
    const Ell e = ells[set];
    int n = 0;
    for (int j0 = 0; j0 < N; j0 += 64) {
        const int j = j0 + lane;
        const cd v = j < N ? ell_src(N, A, Ld, set, i, j) : cmk(0, 0);
        const bool nz = v.re != 0.0 || v.im != 0.0;
        const unsigned long long m = __ballot(nz);
        if (nz) {
            const int64_t o = (int64_t)i * e.W + n + __popcll(m & ((1ull << lane) - 1ull));
            e.idx[o] = j;
            cstore(e.val, o, v);
        }
        n += __popcll(m);
    }
}

// ---------------------------------------------------------------------------
// Pair rows: Y = L^+(F_s), F_s = al E_uv + be E_vu (u < v)
// ---------------------------------------------------------------------------

struct PairArgs {
    int N, P, bound;  // bound: largest number of entries of a row of L^+(F_s)
    int64_t Pp;       // number of pairs
    const Ell* ells;  // set 0: columns of A = iH - G/2; 1 + 2p: rows of L0_p
    const double* rates;
    const int* act;   // the nact jump operators with a nonzero rate and an entry, in order
    int nact;
    // outputs
    int64_t* cnt;          // count phase: entries per row
    int* ns;               // entries in the S block, from the count to the fill
    const int64_t* rowptr; // fill phase
    int64_t* col;
    double* val;
    double* K;
    int* overflow;
};

// Sorts the first n of at most NB keys (stride 64 in LDS) by Batcher's odd-even
// merge network on registers: no data-dependent step, NB (log NB)^2 / 4 exchanges.
template <int NB>
__device__ __forceinline__ void sort_keys(uint32_t* key, int n) {
    uint32_t k[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) k[i] = i < n ? key[i * 64] : 0xffffffffu;
#pragma unroll
    for (int p = 1; p < NB; p <<= 1)
#pragma unroll
        for (int q = p; q >= 1; q >>= 1)
#pragma unroll
            for (int j = q % p; j + q < NB; j += 2 * q)
#pragma unroll
                for (int i = 0; i < q; ++i)
                    if (i + j + q < NB && (i + j) / (2 * p) == (i + j + q) / (2 * p)) {
                        const uint32_t lo = min(k[i + j], k[i + j + q]), hi = max(k[i + j], k[i + j + q]);
                        k[i + j] = lo;
                        k[i + j + q] = hi;
                    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
        if (i < n) key[i * 64] = k[i];
}

__device__ __forceinline__ uint32_t row_pos(int N, int64_t Pp, int a, int c) {
    if (a == c) return (uint32_t)(2 * Pp + a);
    return (uint32_t)(2 * lb_upair(N, a, c) + (a > c ? 1 : 0));
}

// Entries of a row on their way to col and val, two at a time where the arrays are
// 16-byte aligned: lanes write different rows, so a store is a request per lane, and
// half as many of them take the rocked dimer's fill from 516 to 406 us at N = 1000.
struct RowOut {
    int64_t* col;
    double* val;
    bool pairs, held = false;
    int64_t c0 = 0;
    double q0 = 0;
    __device__ __forceinline__ void put(int64_t o, int64_t c, double q) {
        if (pairs && !(o & 1)) {
            held = true;
            c0 = c;
            q0 = q;
        } else if (held) {
            *reinterpret_cast<longlong2*>(col + o - 1) = longlong2{c0, c};
            *reinterpret_cast<double2*>(val + o - 1) = make_double2(q0, q);
            held = false;
        } else {
            col[o] = c;
            val[o] = q;
        }
    }
    // o: where the next entry would go
    __device__ __forceinline__ void flush(int64_t o) {
        if (!held) return;
        col[o - 1] = c0;
        val[o - 1] = q0;
        held = false;
    }
};

// One thread per row, one wavefront per block. The same arithmetic in the count and
// the fill phase, so they agree on which entries are exactly zero and not stored.
//
// A row's entries while it is formed: [entry][lane] in LDS, a sort key (position
// << 6 | entry; position = pair * 2 + (a > c) for the off-diagonal entry (a, c),
// 2 P + a for the diagonal, below 2^23 for N <= 2048, so keys are unique and
// sorting keeps the order of equal positions) and either its value (VALS, 20 bytes
// an entry) or the term it comes from (6 bytes), its value being formed from the
// lists when it is summed. A row of few entries is fastest with its values at hand;
// one of many then leaves three wavefronts on a CU, too few to hide the lists'
// latency. A whole preparation at N = 1000 with values / with terms: dimer (14
// entries) 0.51 / 0.56 ms, rocked dimer (38) 1.42 / 1.06 ms.
// Terms: kind | t1 << 3 | t2 << 7 | operator << 10, where an entry bound of 64
// keeps t1 below 16 (4 lists of A), t1 and t2 below 6 (2 W^2) and operators below 32.
template <int NB, bool VALS>
__global__ __launch_bounds__(64) void k_pair_rows(PairArgs g, int fill) {
    extern __shared__ double2 rowmem[];
    const int64_t s = (int64_t)blockIdx.x * 64 + threadIdx.x;
    const int N = g.N;
    const int64_t Pp = g.Pp;
    const bool live = s < 2 * Pp;
    double2* vals = rowmem + threadIdx.x;
    uint32_t* key = reinterpret_cast<uint32_t*>(rowmem + (VALS ? 64 * g.bound : 0)) + threadIdx.x;
    uint16_t* terms = reinterpret_cast<uint16_t*>(key - threadIdx.x + 64 * g.bound) + threadIdx.x;
    const int cls = s >= Pp ? 1 : 0;
    int u = 0, v = 1;
    if (live) {
        int cc;
        lb_decode(N, s - cls * Pp, cc, u, v);
    }
    const double fre = cls == 0 ? kR : 0.0, fim = cls == 0 ? 0.0 : -kR;  // al = (F_s)_uv; (F_s)_vu = be = conj(al)
    const int* aidx = g.ells[0].idx;
    const double* aval = g.ells[0].val;
    const int aw = g.ells[0].W;
    auto value = [&](int term) __attribute__((always_inline)) {
        const int kind = term & 7, t1 = term >> 3 & 15;
        const cd f = cmk(fre, kind & 1 ? -fim : fim);  // al for even kinds, be for odd ones
        if (kind < 4) {
            cd w = cload(aval, (int64_t)(kind == 1 || kind == 2 ? v : u) * aw + t1);
            if (kind >= 2) w.im = -w.im;
            return cmul(f, w);
        }
        const int t2 = term >> 7 & 7, p = g.act[term >> 10];
        const Ell* e = g.ells + 1 + 2 * p;
        const int64_t x = kind == 4 ? u : v, y = u + v - x;
        const cd l1 = cload(e->val, x * e->W + t1), l2 = cload(e->val, y * e->W + t2);
        return cscale(cmul(f, cmul(cconj(l1), l2)), g.rates[p]);
    };
    int n = 0;
    auto push = [&](uint32_t pos, int term) __attribute__((always_inline)) {
        if (n >= g.bound) {
            *g.overflow = 1;
            return;
        }
        if (VALS) {
            const cd y = value(term);
            vals[n * 64] = make_double2(y.re, y.im);
        } else {
            terms[n * 64] = (uint16_t)term;
        }
        key[n * 64] = (pos << 6) | (uint32_t)n;
        ++n;
    };
    if (live) {
        const int nu = g.ells[0].cnt[u], nv = g.ells[0].cnt[v];
        const int *iu = aidx + (int64_t)u * aw, *iv = aidx + (int64_t)v * aw;
        // i H F_s - G F_s / 2 = A F_s: (a, v) += al A_au, (a, u) += be A_av
        for (int t = 0; t < nu; ++t) push(row_pos(N, Pp, iu[t], v), 0 | t << 3);
        for (int t = 0; t < nv; ++t) push(row_pos(N, Pp, iv[t], u), 1 | t << 3);
        // -i F_s H - F_s G / 2 = F_s A^+: (u, c) += al conj(A_cv), (v, c) += be conj(A_cu)
        for (int t = 0; t < nv; ++t) push(row_pos(N, Pp, u, iv[t]), 2 | t << 3);
        for (int t = 0; t < nu; ++t) push(row_pos(N, Pp, v, iu[t]), 3 | t << 3);
        // g_p L0^+ F_s L0: (a, c) += g al conj(L0_ua) L0_vc + g be conj(L0_va) L0_uc
        for (int p = 0; p < g.nact; ++p) {
            const Ell* e = g.ells + 1 + 2 * g.act[p];
            const int lu = e->cnt[u], lv = e->cnt[v];
            const int *ju = e->idx + (int64_t)u * e->W, *jv = e->idx + (int64_t)v * e->W;
            for (int t1 = 0; t1 < lu; ++t1)
                for (int t2 = 0; t2 < lv; ++t2) push(row_pos(N, Pp, ju[t1], jv[t2]), 4 | t1 << 3 | t2 << 7 | p << 10);
            for (int t1 = 0; t1 < lv; ++t1)
                for (int t2 = 0; t2 < lu; ++t2) push(row_pos(N, Pp, jv[t1], ju[t2]), 5 | t1 << 3 | t2 << 7 | p << 10);
        }
    }
    auto val_of = [&](uint32_t k) __attribute__((always_inline)) {
        if (!VALS) return value(terms[(k & 63u) * 64]);
        const double2 y = vals[(k & 63u) * 64];
        return cmk(y.x, y.y);
    };
    sort_keys<NB>(key, n);
    const uint32_t diag0 = (uint32_t)(2 * Pp);
    // Off-diagonal entries come first, pair by pair: Y_pq (p < q) and Y_qp, each
    // the sum of its entries in the order they were formed. Tr(Y S_pq) =
    // r (Y_pq + Y_qp); Tr(Y J_pq) = i r (Y_pq - Y_qp). The S block of the row
    // is followed by the J block; the count's number of S entries lets the fill write
    // both in one pass over the pairs.
    constexpr uint32_t kEnd = 0xffffffffu;
    auto key_at = [&](int i) { return i < n ? key[i * 64] : kEnd; };
    const uint32_t dkey = diag0 << 6;  // keys of diagonal entries start here
    int64_t o = fill && live ? g.rowptr[s] : 0, oj = fill && live ? o + g.ns[s] : 0;
    int nd0 = 0;  // first diagonal entry
    uint32_t k = key_at(0), kn = key_at(1);
    cd e = k < dkey ? val_of(k) : cmk(0, 0);
    const bool pairs = (((uintptr_t)g.col | (uintptr_t)g.val) & 15) == 0;
    RowOut outs{g.col, g.val, pairs}, outj{g.col, g.val, pairs};
    while (k < dkey) {
        const uint32_t pr = k >> 7;
        cd y0 = cmk(0, 0), y1 = cmk(0, 0);
        do {
            const cd en = kn < dkey ? val_of(kn) : cmk(0, 0);  // the next entry's on its way
            if (k & 64u) y1 = cadd(y1, e);
            else y0 = cadd(y0, e);
            e = en;
            k = kn;
            ++nd0;
            kn = key_at(nd0 + 1);
        } while ((k >> 7) == pr && k < dkey);
        const double qs = kR * (y0.re + y1.re), qj = -kR * (y0.im - y1.im);
        if (qs != 0.0) {
            if (fill) outs.put(o, pr, qs);
            ++o;
        }
        if (qj != 0.0) {
            if (fill) outj.put(oj, Pp + pr, qj);
            ++oj;
        }
    }
    if (fill) outs.flush(o);
    else if (live) g.ns[s] = (int)o;
    o = fill ? oj : o + oj;
    // Diagonal entries (merged by position): Tr Y, and the D columns m from
    // max(1, first position) to the last position, or to N-1 when Tr(Y) != 0:
    // beyond the last position the value is Tr(Y)/sqrt(m(m+1)).
    auto merged = [&](int& i) __attribute__((always_inline)) {  // sum of the entries at entry i's position; i moves past them
        const uint32_t ps = key_at(i) >> 6;
        cd y = val_of(key_at(i++));
        while (i < n && key_at(i) >> 6 == ps) y = cadd(y, val_of(key_at(i++)));
        return y;
    };
    cd tr = cmk(0, 0);
    double asum = 0;
    int xmin = N, xlast = -1;
    for (int i = nd0; i < n;) {
        const int x = (int)((key_at(i) >> 6) - diag0);
        if (xlast < 0) xmin = x;
        xlast = x;
        const cd y = merged(i);
        tr = cadd(tr, y);
        asum += fabs(y.re) + fabs(y.im);
    }
    const bool traced = xlast >= 0 && fabs(tr.re) > 1e-13 * asum;
    if (fill && live) g.K[s] = tr.re / N;
    double pre = 0.0;
    int di = nd0;
    for (int x = xmin; x <= xlast; ++x) {
        cd y = cmk(0, 0);
        if (key_at(di) >> 6 == diag0 + (uint32_t)x) y = merged(di);
        if (x >= 1) {
            const double q = (pre - (double)x * y.re) / sqrt((double)x * (x + 1));
            if (q != 0.0) {
                if (fill) outj.put(o, 2 * Pp + x - 1, q);  // the D block follows the J block
                ++o;
            }
        }
        pre += y.re;
    }
    if (fill) outj.flush(o);
    // The tail beyond the last position, one row of the wavefront at a time
    // across its lanes. |q| falls with m, so all of it is nonzero if the last is.
    int t0 = xlast + 1 > 1 ? xlast + 1 : 1;
    int len = live && traced && t0 < N ? N - t0 : 0;
    if (len > 0 && !(pre / sqrt((double)(N - 1) * N) != 0.0)) {
        int keep = 0;
        for (int x = t0; x < N; ++x) keep += pre / sqrt((double)x * (x + 1)) != 0.0;
        len = keep;
    }
    if (!fill) {
        if (live) g.cnt[s] = o + len;
        return;
    }
    unsigned long long todo = __ballot(len > 0);
    while (todo) {
        const int src = __ffsll(todo) - 1;
        todo &= todo - 1;
        const int x0 = __shfl(t0, src, 64), cnt = __shfl(len, src, 64);
        const double p = __shfl(pre, src, 64);
        const int64_t o0 = __shfl(o, src, 64);
        for (int i = threadIdx.x; i < cnt; i += 64) {
            const int x = x0 + i;
            g.col[o0 + i] = 2 * Pp + x - 1;
            g.val[o0 + i] = p / sqrt((double)x * (x + 1));
        }
    }
}

// ---------------------------------------------------------------------------
// Diagonal of L(F_n) for every column n (carrying lists for the D rows)
// ---------------------------------------------------------------------------

struct DiagArgs {
    int N, P;
    int64_t Pp, M;
    const double* A;   // dense N x N, Z = A^+
    const Ell* ells;   // 1 + 2p: rows of L0_p, 2 + 2p: its columns
    const double* rates;
    int64_t* cnt;
    const int64_t* off;
    int* pos;
    double* val;   // complex
};

__device__ __forceinline__ cd zel(const double* A, int N, int i, int j) { return cconj(cload(A, (int64_t)j * N + i)); }

// small sorted accumulator
struct DAcc {
    int x[kMaxRowEntries];
    cd v[kMaxRowEntries];
    int n;
    __device__ void add(int p, cd val, int* ovf) {
        for (int i = 0; i < n; ++i)
            if (x[i] == p) {
                v[i] = cadd(v[i], val);
                return;
            }
        if (n >= kMaxRowEntries) {
            *ovf = 1;
            return;
        }
        int i = n++;
        while (i > 0 && x[i - 1] > p) {
            x[i] = x[i - 1];
            v[i] = v[i - 1];
            --i;
        }
        x[i] = p;
        v[i] = val;
    }
};

__device__ __forceinline__ void diag_pair(const DiagArgs& g, int64_t nidx, int fill, int* ovf) {
    if (nidx >= 2 * g.Pp) return;
    const int N = g.N;
    const int cls = nidx >= g.Pp ? 1 : 0;
    int cc, x, y;
    lb_decode(N, nidx - cls * g.Pp, cc, x, y);
    const cd al = cls == 0 ? cmk(kR, 0) : cmk(0, -kR);  // (F_n)_xy
    const cd be = cls == 0 ? cmk(kR, 0) : cmk(0, kR);   // (F_n)_yx
    DAcc acc;
    acc.n = 0;
    // (Z F_n + F_n Z^+)_aa: a = y: Z_yx al + be conj(Z_yx); a = x: Z_xy be + al conj(Z_xy)
    const cd zyx = zel(g.A, N, y, x), zxy = zel(g.A, N, x, y);
    const cd dy = cadd(cmul(zyx, al), cmul(be, cconj(zyx)));
    const cd dx = cadd(cmul(zxy, be), cmul(al, cconj(zxy)));
    if (dx.re != 0.0 || dx.im != 0.0) acc.add(x, dx, ovf);
    if (dy.re != 0.0 || dy.im != 0.0) acc.add(y, dy, ovf);
    // g_p (L0 F_n L0^+)_aa = g_p (L0_ax al conj(L0_ay) + L0_ay be conj(L0_ax))
    for (int p = 0; p < g.P; ++p) {
        const Ell Lc = g.ells[2 + 2 * p];
        const double gp = g.rates[p];
        if (gp == 0.0) continue;
        for (int t1 = 0; t1 < Lc.cnt[x]; ++t1) {
            const int a = ell_idx(Lc, x, t1);
            for (int t2 = 0; t2 < Lc.cnt[y]; ++t2) {
                if (ell_idx(Lc, y, t2) != a) continue;
                const cd lax = ell_val(Lc, x, t1), lay = ell_val(Lc, y, t2);
                const cd d = cadd(cmul(lax, cmul(al, cconj(lay))), cmul(lay, cmul(be, cconj(lax))));
                acc.add(a, cscale(d, gp), ovf);
            }
        }
    }
    if (!fill) {
        g.cnt[nidx] = acc.n;
        return;
    }
    const int64_t o = g.off[nidx];
    for (int i = 0; i < acc.n; ++i) {
        g.pos[o + i] = acc.x[i];
        cstore(g.val, o + i, acc.v[i]);
    }
}

// D columns n = D^m': diag_a = w_m'(a) 2 Re Z_aa + sum_p g_p sum_{y <= m'} w_m'(y) |L0_p,ay|^2,
// one wavefront per column, lanes along a (a ballot keeps the positions in order).
__device__ __forceinline__ void diag_dcol(const DiagArgs& g, int mm, int lane, int fill) {
    const int N = g.N;
    if (mm >= N) return;
    const int64_t nidx = 2 * g.Pp + mm - 1;
    const int64_t o = fill ? g.off[nidx] : 0;
    const double nrm = 1.0 / sqrt((double)mm * (mm + 1));
    auto wd = [&](int x) { return x < mm ? nrm : (x == mm ? -(double)mm * nrm : 0.0); };  // lb_wdiag(mm, x)
    int64_t n = 0;
    for (int a0 = 0; a0 < N; a0 += 64) {
        const int a = a0 + lane;
        bool nz = false;
        cd d = cmk(0, 0);
        if (a < N) {
            nz = a <= mm;
            d = cmk(wd(a) * 2.0 * cload(g.A, (int64_t)a * N + a).re, 0.0);
            for (int p = 0; p < g.P; ++p) {
                const Ell Lr = g.ells[1 + 2 * p];
                double s = 0;
                for (int t = 0; t < Lr.cnt[a]; ++t) {
                    const int yy = ell_idx(Lr, a, t);
                    if (yy > mm) continue;
                    const cd l = ell_val(Lr, a, t);
                    s += wd(yy) * (l.re * l.re + l.im * l.im);
                    nz = true;
                }
                d.re += g.rates[p] * s;
            }
        }
        const unsigned long long m = __ballot(nz);
        if (nz && fill) {
            const int64_t r = o + n + __popcll(m & ((1ull << lane) - 1ull));
            g.pos[r] = a;
            cstore(g.val, r, d);
        }
        n += __popcll(m);
    }
    if (!fill && lane == 0) g.cnt[nidx] = n;
}

// diag(L(1))_x = 2 Re Z_xx + sum_p g_p sum_b |L0_p,xb|^2, with Z = A^+ (Re Z_xx = Re A_xx)
__device__ __forceinline__ void l1diag(int N, int P, const double* rates, const double* A, const Ell* Lrow, double* out,
                                       int x) {
    if (x >= N) return;
    double s = 2.0 * cload(A, (int64_t)x * N + x).re;
    for (int p = 0; p < P; ++p) {
        const Ell Lr = Lrow[2 * p];
        double q = 0;
        for (int t = 0; t < Lr.cnt[x]; ++t) {
            const cd v = ell_val(Lr, x, t);
            q += v.re * v.re + v.im * v.im;
        }
        s += rates[p] * q;
    }
    out[x] = s;
}

// The N - 1 columns of diagonal generators, four to a block, then those of the
// pairs, 256 to a block, then (to count) diag(L(1)): two independent chains of latency side by side (one
// after the other 43 us at N = 1000).
__global__ __launch_bounds__(256) void k_diag(DiagArgs g, unsigned nd, unsigned np, int fill, double* l1, int* ovf) {
    const unsigned b = blockIdx.x;
    if (b < nd) diag_dcol(g, (int)(b * 4 + (threadIdx.x >> 6)) + 1, threadIdx.x & 63, fill);
    else if (b < nd + np) diag_pair(g, (int64_t)(b - nd) * 256 + threadIdx.x, fill, ovf);
    else l1diag(g.N, g.P, g.rates, g.A, g.ells + 1, l1, (int)((b - nd - np) * 256 + threadIdx.x));
}

// D rows: Q[D^m][n] = sum_x w_m(x) diag_n(x) = (pre_n(m) - m diag_n(m)) / sqrt(m(m+1)),
// pre_n(m) = sum_{x<m} diag_n(x), over carrying columns n with key(n) <= m.
struct DRowArgs {
    int N;
    int64_t Pp, M;
    const int64_t* carrying;  // how many columns carry
    const int64_t* carry;   // carrying column indices, increasing
    const int64_t* off;     // per column offsets into pos/val (M+1)
    const int* pos;
    const double* val;
    const double* pref;     // exclusive prefix of Re val within each column's list
    const double* l1diag;
    int64_t* cnt;
    const int64_t* rowptr;
    int64_t* col;
    double* qv;
    double* K;
};

// Exclusive prefix sums of the diagonal lists, added one by one in the lists'
// order. Columns of pairs (a few entries each) take a thread, columns of
// diagonal generators (up to N entries, the last ncarry - npair of the carrying
// ones) a wavefront: it loads 64 entries at once, the next 64 ahead, and passes
// the running sum along the lanes.
__global__ __launch_bounds__(64) void k_diag_prefix(int N, const int64_t* carrying, unsigned pair_blocks,
                                                    const int64_t* carry, const int64_t* off, const double* val,
                                                    double* pref) {
    const int lane = threadIdx.x;
    // every diagonal generator's column carries (its list starts at position 0), after those of the pairs
    const int64_t ncarry = *carrying, npair = ncarry - (N - 1);
    if (blockIdx.x < pair_blocks) {
        const int64_t t = (int64_t)blockIdx.x * 64 + lane;
        if (t >= npair) return;
        const int64_t c = carry[t];
        double run = 0;
        for (int64_t e = off[c]; e < off[c + 1]; ++e) {
            pref[e] = run;
            run += val[2 * e];
        }
        return;
    }
    const int64_t t = npair + (blockIdx.x - pair_blocks);
    if (t >= ncarry) return;
    const int64_t c = carry[t];
    const int64_t e0 = off[c], e1 = off[c + 1];
    double run = 0, next = e0 + lane < e1 ? val[2 * (e0 + lane)] : 0.0;
    for (int64_t e = e0; e < e1; e += 64) {
        const uint2 w = __builtin_bit_cast(uint2, next);
        if (e + 64 + lane < e1) next = val[2 * (e + 64 + lane)];
        double mine = 0;
#pragma unroll
        for (int l = 0; l < 64; ++l) {
            if (l == lane) mine = run;
            run += __builtin_bit_cast(double, make_uint2((unsigned)__builtin_amdgcn_readlane((int)w.x, l),
                                                         (unsigned)__builtin_amdgcn_readlane((int)w.y, l)));
        }
        if (e + lane < e1) pref[e + lane] = mine;
    }
}

// One block of 16 wavefronts per D row, each over a contiguous sixteenth of the
// carrying columns, 64 at a time: a column contributes when its list reaches
// row m (key <= m <= last position: the list sums to Tr L(F_n) = 0, so rows
// beyond its last position vanish) and the value is not exactly zero. Ballots
// and the wavefronts' counts keep the columns in increasing order.
constexpr int kDrowWaves = 16;

__device__ __forceinline__ bool drow_value(const DRowArgs& g, int64_t t, int64_t t1, int m, double nrm, int64_t& c,
                                           double& q) {
    if (t >= t1) return false;
    c = g.carry[t];
    int64_t lo = g.off[c], hi = g.off[c + 1] - 1;
    const int key = g.pos[lo] > 1 ? g.pos[lo] : 1;
    if (key > m || g.pos[hi] < m) return false;
    // first entry at position >= m; positions increase, so it is at most m - pos[lo] entries on, and
    // exactly there in a list without gaps (those of the diagonal generators)
    const int64_t at0 = lo + (m - g.pos[lo]);
    if (at0 >= lo && at0 < hi) hi = at0;
    if (g.pos[hi] == m) lo = hi;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (g.pos[mid] < m) lo = mid + 1;
        else hi = mid;
    }
    const double at = g.pos[lo] == m ? g.val[2 * lo] : 0.0;
    q = (g.pref[lo] - (double)m * at) * nrm;
    return q != 0.0;
}

__global__ __launch_bounds__(64 * kDrowWaves) void k_drows_sparse(DRowArgs g, int fill) {
    __shared__ int64_t wcnt[kDrowWaves];
    extern __shared__ double l1[];  // fill phase: diag(L(1)), N entries
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m = blockIdx.x + 1;
    const int N = g.N;
    if (fill)
        for (int x = threadIdx.x; x <= m; x += 64 * kDrowWaves) l1[x] = g.l1diag[x];
    const int64_t row = 2 * g.Pp + m - 1;
    const double nrm = 1.0 / sqrt((double)m * (m + 1));
    const int64_t ncarry = *g.carrying;
    const int64_t per = ((ncarry + kDrowWaves - 1) / kDrowWaves + 63) / 64 * 64;
    const int64_t t0 = w * per, t1 = t0 + per < ncarry ? t0 + per : ncarry;
    int64_t n = 0, c = 0;
    double q = 0.0;
    for (int64_t t = t0; t < t1; t += 64) n += __popcll(__ballot(drow_value(g, t + lane, t1, m, nrm, c, q)));
    if (lane == 0) wcnt[w] = n;
    __syncthreads();
    int64_t o = 0, tot = 0;
    for (int i = 0; i < kDrowWaves; ++i) {
        if (i < w) o += wcnt[i];
        tot += wcnt[i];
    }
    if (!fill) {
        if (threadIdx.x == 0) g.cnt[row] = tot;
        return;
    }
    o += g.rowptr[row];
    for (int64_t t = t0; t < t1; t += 64) {
        const bool keep = drow_value(g, t + lane, t1, m, nrm, c, q);
        const unsigned long long mask = __ballot(keep);
        if (keep) {
            const int64_t r = o + __popcll(mask & ((1ull << lane) - 1ull));
            g.col[r] = c;
            g.qv[r] = q;
        }
        o += __popcll(mask);
    }
    if (threadIdx.x == 64 * (kDrowWaves - 1)) {
        double k = 0;
#pragma unroll 8
        for (int x = 0; x < m; ++x) k += nrm * l1[x];  // lb_wdiag(m, x), its root taken once
        k += -(double)m * nrm * l1[m];
        g.K[row] = k / N;
    }
}

}  // namespace

// Work on the context's second stream between fork() and join(). A return in
// between (an error, a workspace to be grown) waits for it: it uses the workspace.
struct AuxWork {
    lb_ctx* c;
    bool open = false;
    explicit AuxWork(lb_ctx* c) : c(c) {}
    AuxWork(const AuxWork&) = delete;
    ~AuxWork() {
        if (open) (void)hipStreamSynchronize(c->aux);
    }
    int fork() {
        LB_HIP(hipEventRecord(c->ev_fork, c->stream));
        LB_HIP(hipStreamWaitEvent(c->aux, c->ev_fork, 0));
        open = true;
        return LB_OK;
    }
    int join() {
        LB_HIP(hipEventRecord(c->ev_join, c->aux));
        LB_HIP(hipStreamWaitEvent(c->stream, c->ev_join, 0));
        open = false;
        return LB_OK;
    }
};

// exact: read the length of the diagonals' lists back in any case.
// Returns LB_OK, a negative status, or 1 when the workspace must grow to *want
// bytes first (growing reallocates it, so the caller restarts from the top).
static int sparse_body(lb_ctx* c, int N, const lb_csr_c128* H, int P, const double* rates, const lb_csr_c128* L,
                       lb_sparse_alloc alloc, void* user, int64_t* nnz, bool exact, size_t* want) {
    hipStream_t s = c->stream;
    const int64_t M = (int64_t)N * N - 1;
    const int64_t Pp = lb_npairs(N);
    const int64_t NN = (int64_t)N * N;
    const int nsets = 1 + 2 * P;
    // workspace layout
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = lb_align(off + bytes, 256);
        return o;
    };
    const size_t o_h = take(sizeof(double) * 2 * NN);
    const size_t o_l = take(sizeof(double) * 2 * NN * (P > 0 ? P : 1));
    const size_t o_a = take(sizeof(double) * 2 * NN);
    const size_t o_c = take(sizeof(double) * 2 * (P + 1));
    const size_t o_l1 = take(sizeof(double) * N);
    const size_t o_cnt = take(sizeof(int) * (size_t)N * nsets);
    const size_t o_ells = take(sizeof(Ell) * nsets + sizeof(int) * kMaxRowEntries);  // then the pair rows' operators
    const size_t o_rowcnt = take(sizeof(int64_t) * (M + 1));
    const size_t o_dcnt = take(sizeof(int64_t) * (M + 1));
    const size_t o_ns = take(sizeof(int) * 2 * (size_t)Pp);
    const size_t o_carry = take(sizeof(int64_t) * (M + 1));
    const size_t o_scan = take(sizeof(int64_t) * scan_scratch(M));
    // read back: scan totals (diagonal entries, carrying columns; stored entries, -), overflow flags, ELL widths
    const size_t info_bytes = sizeof(int64_t) * 4 + sizeof(int) * (2 + nsets), h_rates = lb_align(info_bytes, 64);
    const size_t o_info = take(h_rates + sizeof(double) * (P + 1));  // then the rates
    const size_t fixed = off;
    int rc = lb_ws_reserve(c, fixed);
    if (rc) return rc;
    char* ws = (char*)c->ws;
    double* Hd = (double*)(ws + o_h);
    double* Ld = (double*)(ws + o_l);
    double* A = (double*)(ws + o_a);
    double* cvec = (double*)(ws + o_c);
    double* drates = (double*)(ws + o_info + h_rates);
    double* l1 = (double*)(ws + o_l1);
    int* cnts = (int*)(ws + o_cnt);
    Ell* dells = (Ell*)(ws + o_ells);
    int64_t* rowcnt = (int64_t*)(ws + o_rowcnt);
    int64_t* dcnt = (int64_t*)(ws + o_dcnt);
    int64_t* carry = (int64_t*)(ws + o_carry);
    int64_t* scratch = (int64_t*)(ws + o_scan);
    int64_t* tot = (int64_t*)(ws + o_info);
    int* ovf = (int*)(tot + 4);
    int* wmax = ovf + 2;

    // pinned staging: [info read back | rates | ELL descriptors, operators of the pair rows]
    const size_t h_ells = h_rates + lb_align(sizeof(double) * (P + 1), 64);
    rc = lb_host_reserve(c, h_ells + sizeof(Ell) * nsets + sizeof(int) * kMaxRowEntries);
    if (rc) return rc;
    LB_HIP(hipStreamSynchronize(s));  // an earlier copy on this stream may still read the staging buffer
    char* host = (char*)c->host;
    const int64_t* htot = (const int64_t*)host;
    const int* hovf = (const int*)(htot + 4);
    const int* hw = hovf + 2;
    memset(host, 0, info_bytes);
    for (int p = 0; p < P; ++p) ((double*)(host + h_rates))[p] = rates[p];
    LB_HIP(hipMemcpyAsync(tot, host, h_rates + sizeof(double) * P, hipMemcpyHostToDevice, s));

    // dense set-up
    for (int p0 = -1; p0 < P; p0 += 8) {
        DenseJobs jobs = {};
        const int n = std::min(8, P - p0);
        for (int i = 0; i < n; ++i) {
            jobs.m[i] = p0 + i < 0 ? *H : L[p0 + i];
            jobs.D[i] = p0 + i < 0 ? Hd : Ld + 2 * NN * (p0 + i);
        }
        hipLaunchKernelGGL(k_densify, dim3(N, n), dim3(64), 0, s, N, jobs);
        LB_CHECK_LAUNCH();
    }
    if (P > 0) {
        hipLaunchKernelGGL(k_shift_l, dim3(1), dim3(256), 0, s, N, P, Ld, cvec);
        LB_CHECK_LAUNCH();
    }
    hipLaunchKernelGGL(k_heff_a, dim3(N), dim3(256), (sizeof(double2) + sizeof(int)) * N, s, N, P,
                       (const double*)drates,
                       (const double*)cvec, (const double*)Ld, (const double*)Hd, A);
    LB_CHECK_LAUNCH();

    // ELL lists: A by column, L0_p by row and by column
    const dim3 egrid(lb_blocks(N, 4), nsets);
    hipLaunchKernelGGL(k_ell_count, egrid, dim3(256), 0, s, N, (const double*)A, (const double*)Ld, cnts);
    LB_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_ell_width, dim3(nsets), dim3(64), 0, s, N, (const int*)cnts, wmax);
    LB_CHECK_LAUNCH();
    LB_HIP(hipMemcpyAsync(host, tot, info_bytes, hipMemcpyDeviceToHost, s));
    LB_HIP(hipStreamSynchronize(s));
    // 64-bit: a width squared may exceed int
    int64_t bound = 4 * (int64_t)hw[0];
    for (int p = 0; p < P; ++p) bound += 2 * (int64_t)hw[1 + 2 * p] * hw[1 + 2 * p];
    if (bound > kMaxRowEntries)
        return lb_fail(LB_ERR_UNSUPPORTED,
                       "sparse path needs bounded degrees: up to %lld entries per row of L^+(F_s) (limit %d); use "
                       "lindblad_prepare for dense operators",
                       (long long)bound, kMaxRowEntries);
    // ELL storage after the fixed part
    size_t o2 = fixed;
    auto take2 = [&](size_t bytes) {
        size_t o = o2;
        o2 = lb_align(o2 + bytes, 256);
        return o;
    };
    Ell* hl = (Ell*)(host + h_ells);
    for (int i = 0; i < nsets; ++i) {
        const int W = std::max(hw[i], 1);
        const size_t o_i = take2(sizeof(int) * (size_t)N * W);
        const size_t o_v = take2(sizeof(double) * 2 * (size_t)N * W);
        hl[i] = Ell{(int*)(ws + o_i), (double*)(ws + o_v), cnts + (size_t)N * i, W};
    }
    const size_t before_lists = o2;
    if (o2 > c->ws_bytes) {
        *want = o2 + (o2 >> 2);
        return 1;
    }
    int nact = 0;  // at most kMaxRowEntries / 2, as each adds at least 2 to the bound
    int* hact = (int*)(hl + nsets);
    for (int p = 0; p < P; ++p)
        if (rates[p] != 0.0 && hw[1 + 2 * p] > 0) hact[nact++] = p;
    LB_HIP(hipMemcpyAsync(dells, hl, sizeof(Ell) * nsets + sizeof(int) * nact, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_ell_fill, egrid, dim3(256), 0, s, N, (const double*)A, (const double*)Ld, (const Ell*)dells);
    LB_CHECK_LAUNCH();
    // carrying lists: diag(L(F_n)) for every column n
    DiagArgs da;
    da.N = N;
    da.P = P;
    da.Pp = Pp;
    da.M = M;
    da.A = A;
    da.ells = dells;
    da.rates = drates;
    da.cnt = dcnt;
    da.off = dcnt;
    da.pos = nullptr;
    da.val = nullptr;
    // row counts of the pair rows, which do not need the diagonals' lists, beside
    // the lists' set-up
    PairArgs pa;
    pa.N = N;
    pa.P = P;
    pa.bound = std::max((int)bound, 1);
    pa.Pp = Pp;
    pa.ells = dells;
    pa.rates = drates;
    pa.act = (const int*)(dells + nsets);
    pa.nact = nact;
    pa.cnt = rowcnt;
    pa.ns = (int*)(ws + o_ns);
    pa.rowptr = nullptr;
    pa.col = nullptr;
    pa.val = nullptr;
    pa.K = nullptr;
    pa.overflow = ovf;
    const bool vals = bound <= kValueEntries;
    void (*pair_rows)(PairArgs, int) = bound <= 16   ? k_pair_rows<16, true>
                                         : bound <= 24 ? k_pair_rows<24, true>
                                         : bound <= 40 ? k_pair_rows<40, false>
                                                       : k_pair_rows<64, false>;
    const size_t pair_lds =
        (size_t)64 * pa.bound * (sizeof(uint32_t) + (vals ? sizeof(double2) : sizeof(uint16_t)));
    rc = lb_aux_stream(c);
    if (rc) return rc;
    AuxWork aux(c);
    rc = aux.fork();
    if (rc) return rc;
    hipLaunchKernelGGL(pair_rows, dim3(lb_blocks(2 * Pp, 64)), dim3(64), pair_lds, c->aux, pa, 0);
    LB_CHECK_LAUNCH();

    const unsigned nd = lb_blocks(N - 1, 4), np = lb_blocks(2 * Pp, 256);
    hipLaunchKernelGGL(k_diag, dim3(nd + np + lb_blocks(N, 256)), dim3(256), 0, s, da, nd, np, 0, l1, ovf + 1);
    LB_CHECK_LAUNCH();
    rc = scan_counts(s, M, dcnt, dcnt, carry, scratch, tot);
    if (rc) return rc;
    // The lists hold at most this many entries: a pair's column its two positions and
    // those where the operators' columns meet, a diagonal generator's column N. Where
    // that much is affordable the host does not wait for the exact number (35 us).
    int64_t wide = 2;
    for (int p = 0; p < P; ++p) wide += rates[p] != 0.0 ? hw[2 + 2 * p] : 0;
    int64_t dtotal = 2 * Pp * std::min<int64_t>(wide, kMaxRowEntries) + (int64_t)(N - 1) * N;
    unsigned pb = lb_blocks(2 * Pp, 64);
    if (exact || dtotal > kListEntries) {
        LB_HIP(hipMemcpyAsync(host, tot, info_bytes, hipMemcpyDeviceToHost, s));
        LB_HIP(hipStreamSynchronize(s));
        dtotal = htot[0];
        pb = lb_blocks(htot[1] - (N - 1), 64);
    }
    size_t o3 = before_lists;
    auto take3 = [&](size_t bytes) {
        size_t o = o3;
        o3 = lb_align(o3 + bytes, 256);
        return o;
    };
    const size_t o_pos = take3(sizeof(int) * (size_t)std::max<int64_t>(dtotal, 1));
    const size_t o_dval = take3(sizeof(double) * 2 * (size_t)std::max<int64_t>(dtotal, 1));
    const size_t o_pref = take3(sizeof(double) * (size_t)std::max<int64_t>(dtotal, 1));
    if (o3 > c->ws_bytes) {
        *want = o3 + (o3 >> 3);
        return 1;
    }
    da.pos = (int*)(ws + o_pos);
    da.val = (double*)(ws + o_dval);
    hipLaunchKernelGGL(k_diag, dim3(nd + np), dim3(256), 0, s, da, nd, np, 1, l1, ovf + 1);
    LB_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_diag_prefix, dim3(pb + (unsigned)(N - 1)), dim3(64), 0, s, N, (const int64_t*)(tot + 1), pb,
                       (const int64_t*)carry, (const int64_t*)dcnt, (const double*)da.val, (double*)(ws + o_pref));
    LB_CHECK_LAUNCH();
    DRowArgs dr;
    dr.N = N;
    dr.Pp = Pp;
    dr.M = M;
    dr.carrying = tot + 1;
    dr.carry = carry;
    dr.off = dcnt;
    dr.pos = da.pos;
    dr.val = da.val;
    dr.pref = (const double*)(ws + o_pref);
    dr.l1diag = l1;
    dr.cnt = rowcnt;
    dr.rowptr = nullptr;
    dr.col = nullptr;
    dr.qv = nullptr;
    dr.K = nullptr;
    hipLaunchKernelGGL(k_drows_sparse, dim3(N - 1), dim3(64 * kDrowWaves), 0, s, dr, 0);
    LB_CHECK_LAUNCH();
    rc = aux.join();
    if (rc) return rc;
    rc = scan_counts(s, M, rowcnt, rowcnt, nullptr, scratch, tot + 2);
    if (rc) return rc;
    LB_HIP(hipMemcpyAsync(host, tot, info_bytes, hipMemcpyDeviceToHost, s));
    LB_HIP(hipStreamSynchronize(s));
    if (hovf[0] || hovf[1]) return lb_fail(LB_ERR_UNSUPPORTED, "sparse row buffer overflow (degrees too large)");
    *nnz = htot[2];
    if (!alloc) return LB_OK;
    lb_sparse_out out = {};
    rc = alloc(user, *nnz, &out);
    if (rc) return rc;
    dr.rowptr = pa.rowptr = out.rowptr;
    dr.col = pa.col = out.col;
    dr.qv = pa.val = out.val;
    dr.K = pa.K = out.K;
    LB_HIP(hipMemcpyAsync(out.rowptr, rowcnt, sizeof(int64_t) * (M + 1), hipMemcpyDeviceToDevice, s));
    rc = aux.fork();
    if (rc) return rc;
    hipLaunchKernelGGL(k_drows_sparse, dim3(N - 1), dim3(64 * kDrowWaves), sizeof(double) * N, c->aux, dr, 1);
    LB_CHECK_LAUNCH();
    hipLaunchKernelGGL(pair_rows, dim3(lb_blocks(2 * Pp, 64)), dim3(64), pair_lds, s, pa, 1);
    LB_CHECK_LAUNCH();
    return aux.join();
}

int lb_impl_sparse(lb_ctx* c, int N, const lb_csr_c128* H, int P, const double* rates, const lb_csr_c128* L,
                   lb_sparse_alloc alloc, void* user, int64_t* nnz) {
    size_t want = 0;
    bool exact = false;  // the diagonals' lists at their own size: where their bound's does not fit
    for (int attempt = 0; attempt < 8; ++attempt) {
        if (want) {
            int rc = lb_ws_reserve(c, want);
            want = 0;
            if (rc == LB_ERR_OOM && !exact) exact = true;
            else if (rc) return rc;
        }
        int rc = sparse_body(c, N, H, P, rates, L, alloc, user, nnz, exact, &want);
        if (rc != 1) return rc;
    }
    return lb_fail(LB_ERR_OOM, "sparse workspace sizing did not converge");
}
