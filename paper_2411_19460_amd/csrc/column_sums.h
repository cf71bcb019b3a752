// Sums of a few hundred partial rows column by column in a fixed order: the last step of a parameter gradient.  Bound by
// memory latency (a few MB at most), so a workgroup of sixteen waves takes 64 columns, every wave each sixteenth row with
// eight loads in flight.  768 rows of 5120 columns: 5.7 us, 13.6 with four waves of four loads; 256 rows of 80 columns 5.5,
// 17.7 with four waves of one load.
#pragma once
#include "ssd_internal.h"

namespace ssdk {

constexpr int COLSUM_WAVES = 16, COLSUM_THREADS = 64 * COLSUM_WAVES;

struct ColsumLds {
    float red[COLSUM_WAVES][64];
};

// The sum of column `col` of part [nparts][stride] in the lanes of wave 0 (lane = the workgroup's column); every thread of
// the workgroup calls it.
static __device__ __forceinline__ float column_sum(ColsumLds& L, const float* part, int64_t nparts, int64_t stride, int64_t col, bool live) {
    constexpr int U = 8;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    float s = 0.f;
    if (live) {
        const float* src = part + col;
        int64_t p = wv;
        for (; p + (U - 1) * COLSUM_WAVES < nparts; p += U * COLSUM_WAVES) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = src[(p + u * COLSUM_WAVES) * stride];
#pragma unroll
            for (int u = 0; u < U; ++u) s += v[u];
        }
        for (; p < nparts; p += COLSUM_WAVES) s += src[p * stride];
    }
    L.red[wv][lane] = s;
    __syncthreads();
    s = 0.f;
    if (wv == 0)
#pragma unroll
        for (int q = 0; q < COLSUM_WAVES; ++q) s += L.red[q][lane];
    return s;
}

}  // namespace ssdk
