// Finalize of the one-frame Gram pass, shared by its own kernel and by the
// fused finalize + tridiagonal solve of single pushes.
#pragma once

#include "dmd_internal.h"

namespace dmd {

// Sums the per-workgroup partials in a fixed order (lane-strided partial sums,
// then a fixed butterfly), rejects a snapshot whose inner products are not
// finite, otherwise writes the new Gram row and column and advances the
// window: the oldest snapshot leaves a full window (the shift of Algorithm 1).
// Every lane issues its loads independently so that the reduction is bound by
// memory-level parallelism, not latency.
constexpr int kFinThreads = 1024;
constexpr int kFinLanes = 16;  // lanes per column

template <int NT>
__device__ inline void gram_finalize_body(double* __restrict__ G, const double* __restrict__ partials, int nblk, int m,
                                   int slots, DevState* __restrict__ st) {
    const int count = st->count;
    const int oldest = st->oldest;
    const int spare = slot_of(oldest, count, slots);
    const int keep0 = (count == m + 1) ? 1 : 0;
    const int nkept = count - keep0;

    __shared__ double g[kMaxM + 2];
    __shared__ int bad;
    if (threadIdx.x == 0) bad = 0;
    const int sub = threadIdx.x % kFinLanes;
    const int grp = threadIdx.x / kFinLanes;
    constexpr int kGroups = NT / kFinLanes;
    // four columns at a time, so that a workgroup of few threads keeps as many
    // loads in flight; each column's sum has the same order for every NT
    for (int j = grp; j <= nkept; j += 4 * kGroups) {
        double a[4][4];
        const double* pj[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ju = j + u * kGroups;
            pj[u] = partials + (int64_t)(ju <= nkept ? ju : j) * nblk;
            a[u][0] = a[u][1] = a[u][2] = a[u][3] = 0.0;
        }
        int b = sub;
        for (; b + 3 * kFinLanes < nblk; b += 4 * kFinLanes) {
            double p[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) p[u][q] = pj[u][b + q * kFinLanes];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) a[u][q] += p[u][q];
        }
        for (; b < nblk; b += kFinLanes)
#pragma unroll
            for (int u = 0; u < 4; ++u) a[u][0] += pj[u][b];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            double v = (a[u][0] + a[u][1]) + (a[u][2] + a[u][3]);
#pragma unroll
            for (int off = kFinLanes / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
            const int ju = j + u * kGroups;
            if (sub == 0 && ju <= nkept) g[ju] = v;
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j <= nkept; j += NT)
        if (!isfinite(g[j])) bad = 1;
    __syncthreads();
    if (bad) {
        if (threadIdx.x == 0) st->rejected_nonfinite += 1;
        return;
    }
    for (int j = threadIdx.x; j < nkept; j += NT) {
        const int sj = slot_of(oldest, keep0 + j, slots);
        G[sj + (int64_t)spare * slots] = g[j];  // <x_j, x_new>
        G[spare + (int64_t)sj * slots] = g[j];  // real data: symmetric
    }
    if (threadIdx.x == 0) {
        G[spare + (int64_t)spare * slots] = g[nkept];
        if (count == m + 1) st->oldest = slot_of(oldest, 1, slots);
        else st->count = count + 1;
        st->pushes += 1;
    }
}

}  // namespace dmd
