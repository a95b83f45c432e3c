// Shifted symmetric tridiagonal solve of the P-space preconditioner.
#pragma once
#include "smalleig.h"

namespace mbefci {

// LDS of tri_solve: per unknown the row's two off-diagonals, the reciprocal of
// its diagonal and its right-hand side, in two alternating buffers.
struct TriShared {
    double l[2][kPsp], u[2][kPsp], r[2][kPsp], w[2][kPsp];
};

// u = (theta - T)^-1 w for T with diagonal d and subdiagonal e, n <= kPsp
// unknowns, element i in thread i (threads past n return 0; every thread of
// the block calls this, thread i < n with its d_i, e_i, e_{i-1} and w_i).
//
// Parallel cyclic reduction: log2 n steps, each unknown eliminating its
// neighbours at distance 1, 2, 4 ..; a chain of n pivots (Thomas) is bound by
// the latency of its n divisions.  theta is at or below the spectrum of T but
// for the first iterations, where theta - T is definite and the reduction is
// stable without pivoting; diagonals are kept at |.| >= 1e-8.
__device__ __forceinline__ double tri_solve(TriShared &q, int n, double theta, double d, double e, double ep, double w) {
    const int i = threadIdx.x;
    const bool mine = i < n;
    double b = theta - d, l = i > 0 ? -ep : 0.0, u = i + 1 < n ? -e : 0.0;
    auto inv = [](double p) { return fast_rcp(fabs(p) < 1e-8 ? (p >= 0.0 ? 1e-8 : -1e-8) : p); };
    int k = 0;
    for (int s = 1; s < n; s <<= 1, k ^= 1) {
        if (mine) {
            q.l[k][i] = l;
            q.u[k][i] = u;
            q.r[k][i] = inv(b);
            q.w[k][i] = w;
        }
        __syncthreads();
        if (mine) {
            if (i >= s) {
                const int j = i - s;
                const double a = -l * q.r[k][j];
                b = fma(a, q.u[k][j], b);
                w = fma(a, q.w[k][j], w);
                l = a * q.l[k][j];
            }
            if (i + s < n) {
                const int j = i + s;
                const double a = -u * q.r[k][j];
                b = fma(a, q.l[k][j], b);
                w = fma(a, q.w[k][j], w);
                u = a * q.u[k][j];
            }
        }
    }
    return mine ? w * inv(b) : 0.0;
}

}  // namespace mbefci
