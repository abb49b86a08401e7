// The scan of counts in steps of 1024 threads with eight each, its offsets and its list
// of nonzero counts, with a workgroup's sums and numbers of nonzero counts packed as the
// device code packs them, against a plain loop.
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "scan_pack.h"

static int check(const char* name, const std::vector<int64_t>& src) {
    const int64_t n = (int64_t)src.size();
    std::vector<int64_t> dst(n + 1), list;
    int64_t bs = 0, bz = 0;
    for (int64_t start = 0; start < n; start += kScanPackCounts) {
        std::vector<int64_t> word(kScanPackCounts / 8);
        for (size_t t = 0; t < word.size(); ++t) {
            int64_t s = 0, z = 0;
            for (int j = 0; j < 8; ++j) {
                const int64_t i = start + 8 * (int64_t)t + j;
                const int64_t v = i < n ? src[i] : 0;
                s += v;
                z += v != 0;
            }
            word[t] = scan_pack(s, z);
        }
        int64_t total = 0;
        for (size_t t = 0; t < word.size(); ++t) {
            int64_t os = bs + scan_packed_sum(total), oz = bz + scan_packed_nonzero(total);
            for (int j = 0; j < 8; ++j) {
                const int64_t i = start + 8 * (int64_t)t + j;
                if (i >= n) break;
                dst[i] = os;
                if (src[i] != 0) {
                    if (oz != (int64_t)list.size()) {
                        printf("%s: count %lld lists at %lld, not %zu\n", name, (long long)i, (long long)oz, list.size());
                        return 1;
                    }
                    list.push_back(i);
                    ++oz;
                }
                os += src[i];
                if (i == n - 1) dst[n] = os;
            }
            total += word[t];
        }
        bs += scan_packed_sum(total);
        bz += scan_packed_nonzero(total);
    }
    int64_t sum = 0;
    for (int64_t i = 0; i < n; ++i) {
        if (dst[i] != sum) {
            printf("%s: offset %lld is %lld, not %lld\n", name, (long long)i, (long long)dst[i], (long long)sum);
            return 1;
        }
        sum += src[i];
    }
    if (dst[n] != sum || bs != sum || bz != (int64_t)list.size()) {
        printf("%s: totals %lld %lld %lld, not %lld %zu\n", name, (long long)dst[n], (long long)bs, (long long)bz,
               (long long)sum, list.size());
        return 1;
    }
    return 0;
}

int main() {
    int bad = 0;
    for (int64_t n : {1, 8, 8191, 8192, 8193, 16384, 32768})
        for (int64_t v : {(int64_t)1, (int64_t)64, ((int64_t)1 << 49) / 32769}) {
            std::vector<int64_t> all(n, v), some(n), one(n, 0);
            for (int64_t i = 0; i < n; ++i) some[i] = (i * 2654435761u >> 7) % 3 ? v : 0;
            one[n - 1] = v;
            char name[96];
            snprintf(name, sizeof name, "n=%lld v=%lld", (long long)n, (long long)v);
            bad |= check(name, all) | check(name, some) | check(name, one);
        }
    if (!bad) printf("OK\n");
    return bad;
}
