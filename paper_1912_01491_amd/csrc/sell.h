// Sparse matrices in the slice layout used by the sparse RK4 stage and the
// steady-state operator.
//
// The CSR rows a caller passes are regrouped once per call into slices of 64
// consecutive rows (one wavefront, one row per lane), each slice stored entry-
// major: entry k of the slice's rows sits at [k * 64 + lane], padded to the
// slice's longest row with zero values whose column is the lane's own row. A
// wavefront's column and value loads are then full contiguous lines, no
// cross-lane reduction is needed, and entry k of neighbouring rows, which in
// the pair ordering are neighbouring pairs, tends to gather neighbouring x.
// Rows with more than kLongRow entries (the diagonal-generator rows and the
// rows coupled to them, ~N entries) are left out of the slices and take one
// block of 256 threads each, with a fixed-order block reduction.
//
// In the pair ordering most entries k of a slice have consecutive columns (row
// (u, v) couples to (u, v + d), (u + d, v), ... with v one more per lane): those
// groups keep one column for the slice, the lanes' columns follow from it, and
// the per-entry columns are neither written nor read. 8 bytes per entry instead
// of 12 (94 % of the groups of the N = 1000 rocked dimer).
//
// A second matrix (the drive term Q1 of a time-dependent system) can be
// regrouped alongside; its long rows are those of the first matrix.
#pragma once

#include "lb_internal.h"
#include "scan.h"

#include <algorithm>

namespace {

constexpr int kLongRow = 32;
constexpr int kSlice = 64;
// Slice entries per lane loaded before their products. 6, 8 and 9 measured 39.4,
// 39.9 and 39.6 us a stage on the rocked dimer (18 entries a row), 21.5, 21.0 and
// 21.0 us on the static one (7 entries).
constexpr int kChunk = 9;

// A row left out of the slices: its entries in the CSR arrays of the matrix and
// of the second one.
struct LongRow {
    int64_t row, e0, e1, f0, f1;
};
typedef const LongRow __attribute__((address_space(4)))* LongRowPtr;

// Slice widths (as 64 * entries, later scanned into offsets), the long-row
// mask of each slice and the list of long rows. One wavefront per slice.
__global__ __launch_bounds__(256) void k_sell_widths(int64_t M, int64_t S, const int64_t* rowptr,
                                                     const int64_t* rowptr1, int64_t* off0, int64_t* off1,
                                                     uint64_t* lmask, LongRow* longrows, int* nlong) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t sl = r / kSlice;
    if (sl >= S) return;  // whole wavefronts
    int64_t len0 = 0, len1 = 0;
    if (r < M) {
        len0 = rowptr[r + 1] - rowptr[r];
        if (rowptr1) len1 = rowptr1[r + 1] - rowptr1[r];
    }
    const bool lng = len0 > kLongRow;
    if (lng) {
        len0 = 0;
        len1 = 0;
        LongRow& lr = longrows[atomicAdd(nlong, 1)];
        lr.row = r;
        lr.e0 = rowptr[r];
        lr.e1 = rowptr[r + 1];
        if (rowptr1) {
            lr.f0 = rowptr1[r];
            lr.f1 = rowptr1[r + 1];
        }
    }
    for (int o = kSlice / 2; o > 0; o >>= 1) {
        len0 = max(len0, (int64_t)__shfl_xor(len0, o, kSlice));
        len1 = max(len1, (int64_t)__shfl_xor(len1, o, kSlice));
    }
    const uint64_t mask = __ballot(lng);
    if ((r & (kSlice - 1)) == 0) {
        off0[sl] = kSlice * len0;
        off1[sl] = kSlice * len1;
        lmask[sl] = mask;
    }
}

// What a wavefront needs to know about its slice, read with scalar loads in one
// go: every dependent read before the loads of values and x costs the stage a
// memory latency (7 entries per row leave only about three of them).
struct SellHead {
    int64_t off;     // first value of the slice
    uint64_t lmask;  // lanes whose row is long
    int64_t w;       // entries per row
    int64_t unused;
    // first lane's column of entry k if the lanes' columns are consecutive, else -1; from w on: 0.
    // Not set where w > kLongRow (rows of the second matrix whose row in the first is short).
    int base[(kLongRow + kChunk - 1) / kChunk * kChunk];
};

// One matrix of one slice into the slice layout, by a wavefront: the rows' runs
// of CSR entries are read 8 lanes to a row, turned in LDS (row stride odd) and
// written entry by entry. Rows past M and long rows are all padding. An entry
// that all 64 rows have, at consecutive columns, gets the first column in the
// slice's header and no per-lane columns.
constexpr int kSellLds = kSlice * (kLongRow + 1);

__device__ __forceinline__ void sell_put(int64_t r, int64_t M, int64_t sl, bool lng, const int64_t* rowptr,
                                         const int64_t* col, const double* val, const int64_t* off, int* scol,
                                         double* sval, uint64_t lmask, SellHead* head, double* lv, int* lc) {
    const int64_t o = off[sl];
    const int w = (int)((off[sl + 1] - o) / kSlice);
    const int lane = threadIdx.x, stride = w | 1;
    int64_t e0 = 0;
    int len = 0;
    if (r < M && !lng) {
        e0 = rowptr[r];
        len = (int)(rowptr[r + 1] - e0);
    }
    const int pad = (int)(r < M ? r : M - 1);
    if (lane == 0) {
        head[sl].off = o;
        head[sl].lmask = lmask;
        head[sl].w = w;
    }
    if (w > kLongRow) {  // wider than the header and the LDS tile: straight from the rows, all columns kept
        for (int k = 0; k < w; ++k) {
            const int64_t d = o + (int64_t)k * kSlice + lane;
            scol[d] = k < len ? (int)col[e0 + k] : pad;
            sval[d] = k < len ? val[e0 + k] : 0.0;
        }
        return;
    }
    for (int r0 = 0; r0 < kSlice; r0 += 8) {
        const int row = r0 + (lane >> 3);
        const int64_t re = __shfl(e0, row, kSlice);
        const int rl = __shfl(len, row, kSlice);
        int64_t c[kLongRow / 8];
        double v[kLongRow / 8];
#pragma unroll
        for (int u = 0; u < kLongRow / 8; ++u) {
            const int k = (lane & 7) + 8 * u;
            if (k < rl) {
                c[u] = col[re + k];
                v[u] = val[re + k];
            }
        }
#pragma unroll
        for (int u = 0; u < kLongRow / 8; ++u) {
            const int k = (lane & 7) + 8 * u;
            if (k < rl) {
                lc[row * stride + k] = (int)c[u];
                lv[row * stride + k] = v[u];
            }
        }
    }
    __syncthreads();
    for (int k = 0; k < w; ++k) {
        const bool have = k < len;
        const int c = have ? lc[lane * stride + k] : pad;
        const int c0 = __builtin_amdgcn_readfirstlane(c);
        const bool run = __ballot(have && c == c0 + lane) == ~0ull;
        const int64_t d = o + (int64_t)k * kSlice + lane;
        sval[d] = have ? lv[lane * stride + k] : 0.0;
        if (!run) scol[d] = c;
        if (lane == 0) head[sl].base[k] = run ? c0 : -1;
    }
    if (lane >= w && lane < (int)(sizeof(head->base) / sizeof(int))) head[sl].base[lane] = 0;
    __syncthreads();
}

// One wavefront per slice (with a thread per row reading its run of entries
// directly, N = 1000 rocked took 505 us; this 190).
__global__ __launch_bounds__(64) void k_sell_fill(int64_t M, const uint64_t* lmask, const int64_t* rowptr,
                                                  const int64_t* col, const double* val, const int64_t* off0,
                                                  int* scol0, double* sval0, SellHead* head0, const int64_t* rowptr1,
                                                  const int64_t* col1, const double* val1, const int64_t* off1,
                                                  int* scol1, double* sval1, SellHead* head1) {
    __shared__ double lv[kSellLds];
    __shared__ int lc[kSellLds];
    const int64_t sl = blockIdx.x;
    const int64_t r = sl * kSlice + threadIdx.x;
    const uint64_t lm = lmask[sl];
    const bool lng = (lm >> threadIdx.x) & 1;
    sell_put(r, M, sl, lng, rowptr, col, val, off0, scol0, sval0, lm, head0, lv, lc);
    if (rowptr1) sell_put(r, M, sl, lng, rowptr1, col1, val1, off1, scol1, sval1, lm, head1, lv, lc);
}

// A matrix (and optionally a second one) in the slice layout, with the CSR it
// came from (read by the long rows).
struct SellMat {
    int64_t M, S;
    const int64_t* col;  // CSR entries, for the long rows
    const double* val;
    const int64_t* col1;
    const double* val1;
    const SellHead* head0;
    const int* scol0;  // columns, of the entries without a base
    const double* sval0;
    const SellHead* head1;
    const int* scol1;
    const double* sval1;
    const LongRow* longrows;
    int nlong;
    int nlong8;   // long-row blocks padded to a multiple of 8
    int per_xcd;  // slice groups (of four slices) per XCD; launch nlong8 + 8 * per_xcd blocks
    int ngroups;  // slice groups
    int contig;   // slice groups in one contiguous range per XCD (sell_work)
};

// Work item of this block: a long row (w < nlong) or the slice group
// w - nlong; -1 for padding. Workgroups go to the 8 XCDs round robin by block
// id. The long rows keep that order (they are the heavy items, spread over
// all XCDs). With contig the slice groups are remapped so that each XCD
// walks one contiguous range of rows, whose gathers of x fall in three
// windows of about M/8 doubles (the rows' own pairs, the partner block, the
// diagonal part); that pays while those fit in the XCD's 4 MB L2 (M up to
// about 1.4 million) and costs beyond, where the natural order, with all
// XCDs on neighbouring rows at a time, shares one moving window instead.
__device__ __forceinline__ int sell_work(const SellMat& m) {
    const int b = blockIdx.x;
    if (b < m.nlong8) return b < m.nlong ? b : -1;
    const int sb = b - m.nlong8;
    const int g = m.contig ? (sb & 7) * m.per_xcd + (sb >> 3) : sb;
    return g < m.ngroups ? m.nlong + g : -1;
}

typedef const SellHead __attribute__((address_space(4)))* SellHeadPtr;  // read through the scalar cache

// acc[j] += sum over entries k .. k + n - 1 of value * x_j[column], in entry
// order, for the first nb of SB states; base: the entries' header columns. The n
// values (and x, or columns and then x) are loaded together before the products.
template <int SB, int n>
__device__ __forceinline__ void sell_chunk(const int* base, const double* v, const int* c, int lane,
                                           const double* Xin, int64_t M, int nb, double* acc) {
    double vv[n];
    int cc[n], any = 0;
#pragma unroll
    for (int u = 0; u < n; ++u) {
        vv[u] = v[u * kSlice];
        cc[u] = base[u];
        any |= cc[u];
    }
    if (any >= 0) {  // consecutive columns throughout: x is read as 512-byte runs
#pragma unroll
        for (int j = 0; j < SB; ++j)
            if (j < nb) {
                const double* x = Xin + (int64_t)j * M;
                double xx[n];
#pragma unroll
                for (int u = 0; u < n; ++u) xx[u] = (x + cc[u])[lane];
#pragma unroll
                for (int u = 0; u < n; ++u) acc[j] = fma(vv[u], xx[u], acc[j]);
            }
    } else {
#pragma unroll
        for (int u = 0; u < n; ++u) cc[u] = cc[u] >= 0 ? cc[u] + lane : c[u * kSlice];
#pragma unroll
        for (int j = 0; j < SB; ++j)
            if (j < nb) {
                const double* x = Xin + (int64_t)j * M;
                double xx[n];
#pragma unroll
                for (int u = 0; u < n; ++u) xx[u] = x[cc[u]];
#pragma unroll
                for (int u = 0; u < n; ++u) acc[j] = fma(vv[u], xx[u], acc[j]);
            }
    }
}

// The last r < n + 1 entries of a row as one chunk of exactly that many.
template <int SB, int n>
__device__ __forceinline__ void sell_rest(int r, const int* base, const double* v, const int* c, int lane,
                                          const double* Xin, int64_t M, int nb, double* acc) {
    if constexpr (n > 0) {
        if (r == n) sell_chunk<SB, n>(base, v, c, lane, Xin, M, nb, acc);
        else sell_rest<SB, n - 1>(r, base, v, c, lane, Xin, M, nb, acc);
    }
}

// The header up to the first chunk's columns.
struct SellFirst {
    int64_t off;
    uint64_t lmask;
    int w;
    int base[kChunk];
};

// All of it in one go: left to where each field is used, the compiler reads the mask, the
// offset and the columns one behind the other, and the static dimers of N = 40 to 160, whose
// slices have few runs of consecutive columns to make up for it, took 4.4 us a stage (3.9 so,
// with the rest of k_sell_stage's start; 4.2 with per-lane columns only). Where w > kLongRow
// the columns are not set and not used.
__device__ __forceinline__ SellFirst sell_first(SellHeadPtr head) {
    SellFirst f;
    f.off = head->off;
    f.lmask = head->lmask;
    f.w = (int)head->w;
#pragma unroll
    for (int u = 0; u < kChunk; ++u) f.base[u] = head->base[u];
    asm volatile("" ::"s"(f.off), "s"(f.lmask), "s"(f.w), "s"(f.base[0]), "s"(f.base[kChunk - 1]));
    return f;
}

template <int SB>
__device__ __forceinline__ void sell_row(const SellFirst& f, SellHeadPtr head, const int* scol, const double* sval,
                                         int lane, const double* Xin, int64_t M, int nb, double* acc) {
    const int w = f.w;
    const int* c = scol + f.off + lane;
    const double* v = sval + f.off + lane;
    if (w > kLongRow) {
        const int none = -1;
        for (int k = 0; k < w; ++k, c += kSlice, v += kSlice) sell_chunk<SB, 1>(&none, v, c, lane, Xin, M, nb, acc);
        return;
    }
    int base[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) base[u] = f.base[u];
    int k = 0;
    while (k + kChunk <= w) {
        sell_chunk<SB, kChunk>(base, v, c, lane, Xin, M, nb, acc);
        k += kChunk;
        c += kChunk * kSlice;
        v += kChunk * kSlice;
        if (k >= w) return;
#pragma unroll
        for (int u = 0; u < kChunk; ++u) base[u] = head->base[k + u];
    }
    sell_rest<SB, kChunk - 1>(w - k, base, v, c, lane, Xin, M, nb, acc);
}

// Sums of one long row of the matrix (s0) and of the second matrix (s1, when
// TWO) against x, by a block of 256 threads in a fixed order; every thread
// receives both.
template <bool TWO>
__device__ __forceinline__ void block_row_dots(const SellMat& m, LongRowPtr lr, const double* x, double& s0out,
                                               double& s1out) {
    __shared__ double red[4], red1[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t e1 = lr->e1;
    double s0 = 0.0, s1 = 0.0;
    int64_t e = lr->e0 + threadIdx.x;
    for (; e + 256 < e1; e += 512) {
        s0 = fma(m.val[e], x[m.col[e]], s0);
        s1 = fma(m.val[e + 256], x[m.col[e + 256]], s1);
    }
    if (e < e1) s0 = fma(m.val[e], x[m.col[e]], s0);
    double sum = s0 + s1;
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    double sd = 0.0;
    if (TWO) {
        for (int64_t f = lr->f0 + threadIdx.x; f < lr->f1; f += 256) sd = fma(m.val1[f], x[m.col1[f]], sd);
        for (int o = 32; o > 0; o >>= 1) sd += __shfl_xor(sd, o, 64);
    }
    if (lane == 0) {
        red[wave] = sum;
        red1[wave] = sd;
    }
    __syncthreads();
    s0out = (red[0] + red[1]) + (red[2] + red[3]);
    s1out = (red1[0] + red1[1]) + (red1[2] + red1[3]);
    __syncthreads();
}

// Regroups the CSR matrix (and the second one, if rowptr1 is not null) into
// the slice layout inside the context workspace, which is laid out as
// [slice offsets, masks, long rows | caller's region of extra_bytes | slices].
// On return c->ws + *extra_off is the caller's region (the workspace may have
// been reallocated, so pointers into it must be taken afterwards). Enqueued on
// the context stream; synchronises twice to learn the sizes.
static int sell_build(lb_ctx* c, int64_t M, const int64_t* rowptr, const int64_t* col, const double* val,
                      const int64_t* rowptr1, const int64_t* col1, const double* val1, size_t extra_bytes,
                      SellMat* out, size_t* extra_off) {
    hipStream_t s = c->stream;
    const bool two = rowptr1 != nullptr;
    // numbers of stored entries: 32-bit slice columns
    int64_t nnz = 0, nnz1 = 0;
    LB_HIP(hipMemcpyAsync(&nnz, rowptr + M, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    if (two) LB_HIP(hipMemcpyAsync(&nnz1, rowptr1 + M, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    LB_HIP(hipStreamSynchronize(s));
    if (nnz < 0 || nnz >= ((int64_t)1 << 31) || nnz1 < 0 || nnz1 >= ((int64_t)1 << 31))
        return lb_fail(LB_ERR_UNSUPPORTED, "nnz=%lld / %lld out of range", (long long)nnz, (long long)nnz1);
    const int64_t S = (M + kSlice - 1) / kSlice;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = lb_align(off + (bytes > 0 ? bytes : 1), 256);
        return o;
    };
    // phase 1 (sizes known from M): slice offsets, long-row masks and list
    const size_t o_off0 = take(sizeof(int64_t) * (size_t)(S + 1));
    const size_t o_off1 = take(sizeof(int64_t) * (size_t)(S + 1));
    const size_t o_mask = take(sizeof(uint64_t) * (size_t)S);
    const size_t o_long = take(sizeof(LongRow) * (size_t)std::min<int64_t>(M, nnz / (kLongRow + 1) + 1));
    const size_t o_nl = take(sizeof(int));
    const size_t o_head = take(sizeof(SellHead) * (size_t)S * (two ? 2 : 1));
    const size_t o_scan = take(sizeof(int64_t) * (scan_scratch(S) + 2));
    const size_t o_extra = take(extra_bytes);
    const size_t fixed = off;
    int rc = lb_ws_reserve(c, fixed);
    if (rc) return rc;
    int hl = 0;
    int64_t tot0 = 0, tot1 = 0;
    const unsigned rgrid = (unsigned)lb_blocks(S * kSlice, 256);
    for (int pass = 0; pass < 2; ++pass) {
        char* ws = (char*)c->ws;
        int64_t* off0 = (int64_t*)(ws + o_off0);
        int64_t* off1 = (int64_t*)(ws + o_off1);
        int* nlong = (int*)(ws + o_nl);
        LB_HIP(hipMemsetAsync(nlong, 0, sizeof(int), s));
        hipLaunchKernelGGL(k_sell_widths, dim3(rgrid), dim3(256), 0, s, M, S, rowptr, two ? rowptr1 : nullptr, off0,
                           off1, (uint64_t*)(ws + o_mask), (LongRow*)(ws + o_long), nlong);
        LB_CHECK_LAUNCH();
        int64_t* scratch = (int64_t*)(ws + o_scan);
        rc = scan_counts(s, S, off0, off0, nullptr, scratch, scratch + scan_scratch(S));
        if (!rc && two) rc = scan_counts(s, S, off1, off1, nullptr, scratch, scratch + scan_scratch(S));
        if (rc) return rc;
        LB_HIP(hipMemcpyAsync(&hl, nlong, sizeof(int), hipMemcpyDeviceToHost, s));
        LB_HIP(hipMemcpyAsync(&tot0, off0 + S, sizeof(int64_t), hipMemcpyDeviceToHost, s));
        if (two) LB_HIP(hipMemcpyAsync(&tot1, off1 + S, sizeof(int64_t), hipMemcpyDeviceToHost, s));
        LB_HIP(hipStreamSynchronize(s));
        off = fixed;
        take(sizeof(int) * (size_t)tot0);
        take(sizeof(double) * (size_t)tot0);
        take(sizeof(int) * (size_t)tot1);
        take(sizeof(double) * (size_t)tot1);
        if (off <= c->ws_bytes) break;
        // the workspace grows: its contents go, so the offsets are formed again
        rc = lb_ws_reserve(c, off);
        if (rc) return rc;
    }
    off = fixed;
    const size_t o_sc0 = take(sizeof(int) * (size_t)tot0);
    const size_t o_sv0 = take(sizeof(double) * (size_t)tot0);
    const size_t o_sc1 = take(sizeof(int) * (size_t)tot1);
    const size_t o_sv1 = take(sizeof(double) * (size_t)tot1);
    if (off > c->ws_bytes) return lb_fail(LB_ERR_DEVICE, "slice layout exceeds the workspace");
    char* ws = (char*)c->ws;
    SellMat m;
    m.M = M;
    m.S = S;
    m.col = col;
    m.val = val;
    m.col1 = col1;
    m.val1 = val1;
    SellHead* head0 = (SellHead*)(ws + o_head);
    SellHead* head1 = two ? head0 + S : nullptr;
    m.head0 = head0;
    m.scol0 = (const int*)(ws + o_sc0);
    m.sval0 = (const double*)(ws + o_sv0);
    m.head1 = head1;
    m.scol1 = (const int*)(ws + o_sc1);
    m.sval1 = (const double*)(ws + o_sv1);
    m.longrows = (const LongRow*)(ws + o_long);
    m.nlong = hl;
    m.nlong8 = (hl + 7) / 8 * 8;
    m.ngroups = (int)((S + 3) / 4);
    m.per_xcd = (m.ngroups + 7) / 8;
    m.contig = 3 * 8 * (M / 8) <= ((int64_t)4 << 20);  // three windows of M/8 doubles within 4 MB
    hipLaunchKernelGGL(k_sell_fill, dim3((unsigned)S), dim3(64), 0, s, M, (const uint64_t*)(ws + o_mask), rowptr, col,
                       val, (const int64_t*)(ws + o_off0), (int*)(ws + o_sc0), (double*)(ws + o_sv0), head0,
                       two ? rowptr1 : nullptr, col1, val1, (const int64_t*)(ws + o_off1), (int*)(ws + o_sc1),
                       (double*)(ws + o_sv1), head1);
    LB_CHECK_LAUNCH();
    *out = m;
    *extra_off = o_extra;
    return LB_OK;
}

}  // namespace
