// Exclusive scan of int64 counts on the device: per-tile sums, one block over
// the tiles, then the offsets of each tile. It replaces scans on the host,
// whose two PCIe copies and serial loop took 1.3 ms for 10^6 counts; the three
// launches here take 15 us. Up to kScanOne counts one workgroup walks all of them
// (10^4: 10 us), which is less than three launches one after the other.
#pragma once

#include "lb_internal.h"
#include "scan_pack.h"

namespace {

constexpr int kScanTile = 2048;  // counts per block (8 per thread)
constexpr int64_t kScanOne = 32768;

// A block's sum over the values of its W wavefronts in thread order; *before is the
// sum over earlier threads. Every thread must call it.
template <int W>
__device__ __forceinline__ int64_t block_scan(int64_t v, int64_t* before) {
    __shared__ int64_t wsum[W];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t inc = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t u = __shfl_up(inc, o, 64);
        if (lane >= o) inc += u;
    }
    __syncthreads();  // earlier readers of wsum
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    int64_t base = 0, tot = 0;
#pragma unroll 4
    for (int i = 0; i < W; ++i) {
        if (i < w) base += wsum[i];
        tot += wsum[i];
    }
    *before = base + inc - v;
    return tot;
}

// Per tile: sum of the counts and number of nonzero ones.
__global__ __launch_bounds__(256) void k_scan_tiles(int64_t n, const int64_t* src, int64_t* tsum, int64_t* tnz) {
    int64_t s = 0, z = 0, before;
    for (int64_t i = (int64_t)blockIdx.x * kScanTile + threadIdx.x, j = 0; j < kScanTile / 256; ++j, i += 256)
        if (i < n) {
            s += src[i];
            z += src[i] != 0;
        }
    s = block_scan<4>(s, &before);
    z = block_scan<4>(z, &before);
    if (threadIdx.x == 0) {
        tsum[blockIdx.x] = s;
        tnz[blockIdx.x] = z;
    }
}

// One block: exclusive scans of the tiles' sums and nonzero counts in place,
// totals to tot[0] and tot[1].
__global__ __launch_bounds__(256) void k_scan_mid(int64_t nt, int64_t* tsum, int64_t* tnz, int64_t* tot) {
    int64_t rs = 0, rz = 0;
    for (int64_t i0 = 0; i0 < nt; i0 += 256) {
        const int64_t i = i0 + threadIdx.x;
        const int64_t s = i < nt ? tsum[i] : 0, z = i < nt ? tnz[i] : 0;
        int64_t bs, bz;
        const int64_t ts = block_scan<4>(s, &bs);
        const int64_t tz = block_scan<4>(z, &bz);
        if (i < nt) {
            tsum[i] = rs + bs;
            tnz[i] = rz + bz;
        }
        rs += ts;
        rz += tz;
    }
    if (threadIdx.x == 0) {
        tot[0] = rs;
        tot[1] = rz;
    }
}

// Offsets of 8 counts per thread from start on, after bs counted and bz nonzero
// ones; both move on by the block's.
template <int W>
__device__ __forceinline__ void scan_eight(int64_t start, int64_t n, const int64_t* src, int64_t* dst, int64_t* list,
                                           int64_t& bs, int64_t& bz) {
    const int64_t i0 = start + 8 * threadIdx.x;
    int64_t v[8], s = 0, z = 0, os, oz;
    if (i0 + 8 <= n) {
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
            const longlong2 a = *reinterpret_cast<const longlong2*>(src + i0 + j);
            v[j] = a.x;
            v[j + 1] = a.y;
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = i0 + j < n ? src[i0 + j] : 0;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        s += v[j];
        z += v[j] != 0;
    }
    // both in one pass
    static_assert(8 * 64 * W <= kScanPackCounts, "counts of a workgroup");
    s = block_scan<W>(scan_pack(s, z), &os);
    oz = bz + scan_packed_nonzero(os);
    os = bs + scan_packed_sum(os);
    bs += scan_packed_sum(s);
    bz += scan_packed_nonzero(s);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (list && v[j] != 0) list[oz++] = i0 + j;
        const int64_t c = v[j];
        v[j] = os;
        os += c;
        if (i0 + j == n - 1) dst[n] = os;
    }
    if (i0 + 8 <= n) {
#pragma unroll
        for (int j = 0; j < 8; j += 2) *reinterpret_cast<longlong2*>(dst + i0 + j) = longlong2{v[j], v[j + 1]};
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (i0 + j < n) dst[i0 + j] = v[j];
    }
}

// Offsets dst[0..n] (dst[n] the total; dst may be src; both 16-byte aligned) and, when list is not
// null, the positions of the nonzero counts in increasing order.
__global__ __launch_bounds__(256) void k_scan_fin(int64_t n, const int64_t* src, const int64_t* tsum,
                                                  const int64_t* tnz, int64_t* dst, int64_t* list) {
    int64_t bs = tsum[blockIdx.x], bz = tnz[blockIdx.x];
    scan_eight<4>((int64_t)blockIdx.x * kScanTile, n, src, dst, list, bs, bz);
}

// The whole scan by one workgroup.
__global__ __launch_bounds__(1024) void k_scan_one(int64_t n, const int64_t* src, int64_t* dst, int64_t* list,
                                                   int64_t* tot) {
    int64_t bs = 0, bz = 0;
    for (int64_t i = 0; i < n; i += 8 * 1024) scan_eight<16>(i, n, src, dst, list, bs, bz);
    if (threadIdx.x == 0) {
        tot[0] = bs;
        tot[1] = bz;
    }
}

// int64 values of device scratch the scan of n counts needs.
static inline size_t scan_scratch(int64_t n) { return 2 * (size_t)((n + kScanTile - 1) / kScanTile); }

// Enqueues the scan of n >= 1 counts; tot[0] = their sum, tot[1] = how many are nonzero (device).
static int scan_counts(hipStream_t s, int64_t n, const int64_t* src, int64_t* dst, int64_t* list, int64_t* scratch,
                       int64_t* tot) {
    if (n <= kScanOne) {
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(1024), 0, s, n, src, dst, list, tot);
        LB_CHECK_LAUNCH();
        return LB_OK;
    }
    const unsigned nt = lb_blocks(n, kScanTile);
    int64_t *tsum = scratch, *tnz = scratch + nt;
    hipLaunchKernelGGL(k_scan_tiles, dim3(nt), dim3(256), 0, s, n, src, tsum, tnz);
    LB_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_scan_mid, dim3(1), dim3(256), 0, s, (int64_t)nt, tsum, tnz, tot);
    LB_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_scan_fin, dim3(nt), dim3(256), 0, s, n, src, (const int64_t*)tsum, (const int64_t*)tnz, dst,
                       list);
    LB_CHECK_LAUNCH();
    return LB_OK;
}

}  // namespace
