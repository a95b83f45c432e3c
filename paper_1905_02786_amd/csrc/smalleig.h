// Lowest eigenpair of the projected matrix of a Davidson iteration (at most
// kMaxSpace rows), by one wave.
#pragma once
#include "device.h"

namespace mbefci {

// Ordering point between the phases of a single wave's work in LDS: a wave
// executes its LDS operations in order, so only the compiler has to be kept
// from moving LDS accesses across this point.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Reciprocal and reciprocal square root: the hardware approximations refined
// by two Newton steps (to a few ulps).
__device__ __forceinline__ double fast_rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ double fast_rsq(double x) {
    double r = __builtin_amdgcn_rsq(x);
    r = r * fma(-0.5 * x * r, r, 1.5);
    return r * fma(-0.5 * x * r, r, 1.5);
}

template <int N> __device__ __forceinline__ double row_ror(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x120 + N, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x120 + N, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// x of the lane 16 (32) lanes further on, within the 32-lane half (the wave):
// row swaps on the vector ALU.
__device__ __forceinline__ double add_row16(double x) {
    const unsigned lo = __double2loint(x), hi = __double2hiint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double(b[0], a[0]) + __hiloint2double(b[1], a[1]);
}
__device__ __forceinline__ double add_row32(double x) {
    const unsigned lo = __double2loint(x), hi = __double2hiint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double(b[0], a[0]) + __hiloint2double(b[1], a[1]);
}

// Sum over the 16 lanes of a row, in every lane of it.
__device__ __forceinline__ double sum_row16(double x) {
    x += row_ror<8>(x);
    x += row_ror<4>(x);
    x += row_ror<2>(x);
    return x + row_ror<1>(x);
}

// Sum over the wave, in every lane.
__device__ __forceinline__ double sum_wave(double x) { return add_row32(add_row16(sum_row16(x))); }

template <int MS> struct SmallEig {
    static constexpr int IW = MS <= 16 ? 16 : 32;   // lanes of a row group: lane i & (IW - 1) owns row i
    static constexpr int NG = 64 / IW;              // row groups, which share the columns
    static constexpr int LD = IW + 1;
    double A[IW][LD];       // the matrix, destroyed
    double v[IW][IW];       // Householder vectors
    double w[IW], d[IW], e[IW], z[IW];
};

// Lowest eigenvalue and eigenvector of the symmetric m x m matrix in q.A
// (rows and columns >= m are not read), m <= MS, by one wave (64 lanes, all
// active); the vector's element i in every lane whose (lane & (IW - 1)) is i
// (zero for i >= m).
//
// A dense symmetric eigensolver for one pair: Householder tridiagonalisation
// T = Q^T A Q, the lowest eigenvalue of T by multisection (every lane tests
// one point with the leading minors of T - x, 65 subintervals a round), its
// vector by inverse iteration, y = Q z.  The work is a serial chain of a few
// thousand operations, so the layout serves latency: a row per lane, sums by
// row rotations and swaps on the vector ALU, the recurrences in registers.
// Against the cyclic Jacobi (all pairs, 64 lanes) it replaced: k_small_eig with
// the new column's sums 42-53 us per launch before, 11-13 us now (12 vectors,
// batches of 1 to 680 tuples); k_whole 6 us less per iteration.
template <int MS> __device__ double lowest_eig(SmallEig<MS> &q, int m, double &y) {
    constexpr int IW = SmallEig<MS>::IW, NG = SmallEig<MS>::NG;
    const int lane = threadIdx.x & 63, i = lane & (IW - 1), g = lane / IW;
    auto over_rows = [](double x) {   // sum over the IW rows
        x = sum_row16(x);
        return IW == 16 ? x : add_row16(x);
    };
    auto over_groups = [](double x) {   // sum over the NG groups
        if (NG == 4) x = add_row16(x);
        return add_row32(x);
    };
    for (int k = 0; k + 2 < m; ++k) {
        const double x = (i > k && i < m) ? q.A[i][k] : 0.0;
        const double s2 = over_rows(x * x), x0 = q.A[k + 1][k];
        const double nx = sqrt(s2), alpha = x0 > 0.0 ? -nx : nx, v0 = x0 - alpha;
        const double vn2 = 2.0 * fma(-x0, alpha, s2);   // |x - alpha e|^2: both terms positive
        if (!(vn2 > 1e-300)) {   // column already reduced: no reflection
            if (lane == 0) q.e[k] = x0;
            if (g == 0) q.v[k][i] = 0.0;
            wave_sync();
            continue;
        }
        const double vi = (i == k + 1 ? v0 : x) * (1.0 / sqrt(vn2));
        if (lane == 0) q.e[k] = alpha;
        if (g == 0) q.v[k][i] = vi;
        wave_sync();
        double p = 0.0;
        if (i > k && i < m)
            for (int j = k + 1 + g; j < m; j += NG) p += q.A[i][j] * q.v[k][j];
        p = over_groups(p);
        const double K = over_rows(vi * p), wi = 2.0 * (p - K * vi);
        if (g == 0) q.w[i] = wi;
        wave_sync();
        if (i > k && i < m)
            for (int j = k + 1 + g; j < m; j += NG) q.A[i][j] -= vi * q.w[j] + wi * q.v[k][j];
        wave_sync();
    }
    if (g == 0) {
        q.d[i] = i < m ? q.A[i][i] : 0.0;
        if (i + 2 == m) q.e[i] = q.A[i + 1][i];
        if (i + 1 >= m) q.e[i] = 0.0;
    }
    wave_sync();
    // Gershgorin bounds
    double lo, hi;
    {
        const double r = (i > 0 && i < m ? fabs(q.e[i - 1]) : 0.0) + fabs(q.e[i]);
        lo = i < m ? q.d[i] - r : 1e300;
        hi = i < m ? q.d[i] + r : -1e300;
#pragma unroll
        for (int o = IW / 2; o > 0; o >>= 1) {
            lo = fmin(lo, __shfl_xor(lo, o, 64));
            hi = fmax(hi, __shfl_xor(hi, o, 64));
        }
    }
    const double scale = fmax(hi - lo + fabs(lo), 1e-30);
    // T in registers, in units of scale; the rows past m decouple, above the spectrum
    const double sc = 1.0 / scale;
    double d[MS], e2[MS], e[MS];
#pragma unroll
    for (int k = 0; k < MS; ++k) {
        d[k] = k < m ? q.d[k] * sc : (lo * sc + 2.0);
        e[k] = k + 1 < m ? q.e[k] * sc : 0.0;
        e2[k] = e[k] * e[k];
    }
    double a = lo * sc, b = hi * sc;
    for (int round = 0; round < 10 && b - a > 2e-16; ++round) {
        const double x = a + (b - a) * ((lane + 1) / 65.0);
        // T - x is positive definite iff every leading minor is positive
        double p0 = 1.0, p1 = d[0] - x;
        bool pos = p1 > 0.0;
#pragma unroll
        for (int k = 1; k < MS; ++k) {
            const double p2 = fma(d[k] - x, p1, -e2[k - 1] * p0);
            p0 = p1;
            p1 = p2;
            pos = pos && p2 > 0.0;
        }
        const int n = __popcll(__ballot(pos));   // points below the lowest eigenvalue
        const double na = n > 0 ? a + (b - a) * (n / 65.0) : a;
        const double nb = n < 64 ? a + (b - a) * ((n + 1) / 65.0) : b;
        a = na;
        b = nb;
    }
    // inverse iteration just below the eigenvalue (T - sigma is positive
    // definite up to rounding, pivots kept at 1e-16)
    const double sigma = a - 4e-16;
    double ip[MS], z[MS];
    ip[0] = fast_rcp(fmax(d[0] - sigma, 1e-16));
#pragma unroll
    for (int k = 1; k < MS; ++k) ip[k] = fast_rcp(fmax(fma(-e2[k - 1], ip[k - 1], d[k] - sigma), 1e-16));
#pragma unroll
    for (int k = 0; k < MS; ++k) z[k] = k < m ? 1.0 + 0.11 * k : 0.0;
#pragma unroll 1
    for (int rep = 0; rep < 3; ++rep) {
#pragma unroll
        for (int k = 1; k < MS; ++k) z[k] = fma(-e[k - 1] * ip[k - 1], z[k - 1], z[k]);
        z[MS - 1] *= ip[MS - 1];
#pragma unroll
        for (int k = MS - 2; k >= 0; --k) z[k] = fma(-e[k], z[k + 1], z[k]) * ip[k];
    }
    double mine = 0.0;
#pragma unroll
    for (int k = 0; k < MS; ++k)
        if (i == k) mine = z[k];
    // y = H_0 ... H_{m-3} z, normalised (scaled by its largest element first)
    double big = fabs(mine);
#pragma unroll
    for (int o = IW / 2; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o, 64));
    mine *= 1.0 / big;
    for (int k = m - 3; k >= 0; --k) {
        const double vi = q.v[k][i];
        mine -= 2.0 * over_rows(vi * mine) * vi;
    }
    y = mine * (1.0 / sqrt(over_rows(mine * mine)));
    if (i >= m) y = 0.0;
    return 0.5 * (a + b) * scale;
}

}  // namespace mbefci
