// The position of column boundaries inside CSR rows.
#pragma once

#include "common.hpp"

namespace l1csr {

// seg[row][t] = first position p of the row with idx[p] >= t << shift
// (t = 0..ntiles), so seg[row][0] = ptr[row] and seg[row][ntiles] = ptr[row+1].
// One wave per row.
__device__ __forceinline__ void seg_row(int row, int ntiles, int shift, const int *__restrict__ ptr,
                                        const int *__restrict__ idx, int *__restrict__ seg) {
    const int lane = threadIdx.x & 63;
    const int s = ptr[row], e = ptr[row + 1];
    int *sr = seg + (int64_t)row * (ntiles + 1);
    // one search per tile boundary (lanes over tiles): 8-ary steps (seven
    // probes loaded together) while the interval is long, then binary.  The
    // answer stays in [lo, hi] ⊆ [s, e], also for a malformed row.
    for (int t = lane; t <= ntiles; t += kWave) {
        int lo = s, hi = e;
        if (t == 0) {
            hi = s;
        } else if (t < ntiles) {
            const int key = t << shift;
            while (hi - lo >= 8) {
                const int step = (hi - lo) >> 3;
                int v[7];
#pragma unroll
                for (int u = 0; u < 7; ++u) v[u] = idx[lo + (u + 1) * step];
                int c = 0;
#pragma unroll
                for (int u = 0; u < 7; ++u) c += v[u] < key ? 1 : 0;
                // probes 1..c lie before the answer, probe c + 1 (if any) at or after it
                const int nlo = c > 0 ? lo + c * step + 1 : lo;
                hi = c < 7 ? lo + (c + 1) * step : hi;
                lo = nlo;
            }
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (idx[mid] < key) lo = mid + 1; else hi = mid;
            }
        } else {
            lo = e;
        }
        sr[t] = lo;
    }
}

}  // namespace l1csr
