// Inverse of the k x k ADMM matrix, by one work-group of 256 threads.
#pragma once
#include "common.h"

namespace symnmf {

// minv = (2 gram + rho I)^-1, FP64 Gauss-Jordan in place; the matrix is
// symmetric positive definite, so no pivoting.  k <= 16 BS.
// A chain of k dependent pivots, bound by the latency of one: 16 x 16 threads
// hold BS x BS blocks of the matrix in registers (padded with the identity),
// the pivot's row and column go through LDS (rc: 4 KMAX doubles), in two
// buffers so that a pivot has one barrier.  The form with [M | I] in LDS, four
// barriers and two divisions by index per pivot took 441 / 63 / 11.3 us at k =
// 64 / 32 / 16; this takes 42 / 13.5 / 5.0 us.
template <typename HT, int BS>
__device__ inline void admm_inverse(const double* __restrict__ gram, int k, double rho, HT* __restrict__ minv,
                                    double* rc) {
    double* row[2] = {rc, rc + KMAX};
    double* col[2] = {rc + 2 * KMAX, rc + 3 * KMAX};
    const int t = threadIdx.x, ti = t >> 4, tj = t & 15;
    double a[BS][BS];
#pragma unroll
    for (int x = 0; x < BS; ++x)
#pragma unroll
        for (int y = 0; y < BS; ++y) {
            const int i = BS * ti + x, j = BS * tj + y;
            const double m = i < k && j < k ? 2.0 * gram[i * k + j] : 0.0;
            a[x][y] = i == j ? (i < k ? m + rho : 1.0) : m;
        }
#pragma unroll
    for (int y = 0; y < BS; ++y) {
        if (ti == 0) row[0][BS * tj + y] = a[0][y];
        if (tj == 0) col[0][BS * ti + y] = a[y][0];
    }
    for (int pb = 0; pb * BS < k; ++pb) {
#pragma unroll
        for (int e = 0; e < BS; ++e) {
            const int p = pb * BS + e;                       // identity past k: nothing changes
            const int buf = p & 1;
            __syncthreads();
            const double d = 1.0 / row[buf][p];
            double rj[BS], ci[BS];
#pragma unroll
            for (int y = 0; y < BS; ++y) {
                rj[y] = row[buf][BS * tj + y] * d;
                ci[y] = col[buf][BS * ti + y];
            }
#pragma unroll
            for (int x = 0; x < BS; ++x)
#pragma unroll
                for (int y = 0; y < BS; ++y) {
                    const bool pi = x == e && ti == pb, pj = y == e && tj == pb;
                    a[x][y] = pi ? (pj ? d : rj[y]) : (pj ? -ci[x] * d : a[x][y] - ci[x] * rj[y]);
                }
            // the next pivot's row and column
            const int nb = e + 1 < BS ? pb : pb + 1, ne = (e + 1) % BS;
#pragma unroll
            for (int y = 0; y < BS; ++y) {
                if (ti == nb) row[buf ^ 1][BS * tj + y] = a[ne][y];
                if (tj == nb) col[buf ^ 1][BS * ti + y] = a[y][ne];
            }
        }
    }
#pragma unroll
    for (int x = 0; x < BS; ++x)
#pragma unroll
        for (int y = 0; y < BS; ++y) {
            const int i = BS * ti + x, j = BS * tj + y;
            if (i < k && j < k) minv[i * k + j] = (HT)a[x][y];
        }
}

}  // namespace symnmf
