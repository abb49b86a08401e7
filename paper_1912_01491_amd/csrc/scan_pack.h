// A sum of counts and the number of nonzero ones in one 64-bit word, so that a
// workgroup's scan passes both at once. Up to 2^13 counts (a workgroup of 1024
// threads with eight each), all of them nonzero if need be, and a sum below 2^49: the
// number takes 14 bits, from bit 49 on, and the word stays positive.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define LB_HD __host__ __device__ __forceinline__
#else
#define LB_HD inline
#endif

constexpr int kScanPackBits = 49;
constexpr int64_t kScanPackCounts = 8 * 1024;  // of a workgroup at most

LB_HD int64_t scan_pack(int64_t sum, int64_t nonzero) { return sum | nonzero << kScanPackBits; }
LB_HD int64_t scan_packed_sum(int64_t v) { return v & (((int64_t)1 << kScanPackBits) - 1); }
LB_HD int64_t scan_packed_nonzero(int64_t v) { return v >> kScanPackBits; }
