// Kernels of the CASSCF expansion reference (Sec. 2: the orbitals of the
// reference space chosen to minimise its CASCI energy): the integrals in
// rotated orbitals phi'_j = sum_i phi_i U_ij, and the Fock matrices that give
// the orbital gradient and the canonical orbitals.
#include "device.h"

namespace mbefci {

// h' = U^T h U, one block per row i: t = U_i^T h in LDS, then t U (n <= 64).
__global__ __launch_bounds__(64) void k_rot_h(const double *h, const double *U, double *out, int n) {
    __shared__ double t[kMaxOrb];
    const int i = blockIdx.x, l = threadIdx.x;
    if (l < n) {
        double s = 0.0;
#pragma unroll 8
        for (int p = 0; p < n; ++p) s += U[p * n + i] * h[p * n + l];
        t[l] = s;
    }
    __syncthreads();
    if (l < n) {
        double s = 0.0;
#pragma unroll 8
        for (int q = 0; q < n; ++q) s += t[q] * U[q * n + l];
        out[i * n + l] = s;
    }
}

// One quarter of the four-index transformation: out[j][a] = sum_s in[a][s]
// U[s][j] for the n^3 leading indices a, i.e. the last index is contracted
// with U and the new index moves to the front.  Four passes turn (pq|rs) into
// (ij|kl)'.  A block takes 32 consecutive a and every j: the 32 x n tile of
// `in` and U sit in LDS, each half-wave owns an eighth of the j (U reads are
// broadcasts), each lane one a (writes coalesced along a).
constexpr int kQuarterRows = 32;

__global__ __launch_bounds__(256) void k_quarter(const double *in, const double *U, double *out, int n) {
    __shared__ double X[kQuarterRows][kMaxOrb + 1];
    __shared__ double Us[kMaxOrb][kMaxOrb + 1];
    const int64_t n3 = (int64_t)n * n * n;
    const int64_t a0 = (int64_t)blockIdx.x * kQuarterRows;
    const int tid = threadIdx.x;
    for (int i = tid; i < n * n; i += 256) Us[i / n][i % n] = U[i];
    for (int i = tid; i < kQuarterRows * n; i += 256) {
        const int r = i / n, s = i % n;
        X[r][s] = (a0 + r < n3) ? in[(a0 + r) * n + s] : 0.0;
    }
    __syncthreads();
    const int a = tid & (kQuarterRows - 1), jg = tid / kQuarterRows;   // 8 groups of j
    constexpr int JW = kMaxOrb / 8;
    double acc[JW];
#pragma unroll
    for (int k = 0; k < JW; ++k) acc[k] = 0.0;
    for (int s = 0; s < n; ++s) {
        const double x = X[a][s];
#pragma unroll
        for (int k = 0; k < JW; ++k) {
            const int j = jg + 8 * k;
            if (j < n) acc[k] += x * Us[s][j];
        }
    }
    if (a0 + a < n3) {
#pragma unroll
        for (int k = 0; k < JW; ++k) {
            const int j = jg + 8 * k;
            if (j < n) out[(int64_t)j * n3 + a0 + a] = acc[k];
        }
    }
}

hipError_t launch_rotate_integrals(const double *h0, const double *eri0, const double *U, double *h, double *eri,
                                   double *tmp, int n, hipStream_t s) {
    if (n < 1 || n > kMaxOrb) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_rot_h, dim3(n), dim3(64), 0, s, h0, U, h, n);
    const int64_t n3 = (int64_t)n * n * n;
    const dim3 grid((unsigned)((n3 + kQuarterRows - 1) / kQuarterRows));
    hipLaunchKernelGGL(k_quarter, grid, dim3(256), 0, s, eri0, U, tmp, n);
    hipLaunchKernelGGL(k_quarter, grid, dim3(256), 0, s, (const double *)tmp, U, eri, n);
    hipLaunchKernelGGL(k_quarter, grid, dim3(256), 0, s, (const double *)eri, U, tmp, n);
    hipLaunchKernelGGL(k_quarter, grid, dim3(256), 0, s, (const double *)tmp, U, eri, n);
    return hipGetLastError();
}

// Fock matrix f_pq = h_pq + sum_rs gamma_rs [(pq|rs) - 1/2 (pr|sq)], one
// block per pair p >= q (both triangles written).  It reads two n x n slices
// of the integrals per pair, (pq|..) and (pr|qs) over r, s, both along s; the
// whole is 8 n^4 bytes from L2 and a block-wide sum.  One thread per entry,
// as before, put 576 threads on the chip at n = 24: 143 us, now 4.3 us.
__global__ __launch_bounds__(256) void k_fock(const double *h, const double *eri, const double *g1, int n, double *f) {
    int p, q;
    pair_of(blockIdx.x, p, q);
    const int n2 = n * n;
    const int64_t n3 = (int64_t)n2 * n;
    const double *J = eri + p * n3 + (int64_t)q * n2, *K = eri + p * n3 + q * n;
    double acc = 0.0;
    for (int i = threadIdx.x; i < n2; i += 256) {
        const int r = i / n, s = i - r * n;
        acc += g1[i] * (J[i] - 0.5 * K[(int64_t)r * n2 + s]);
    }
    __shared__ double sh[16];
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) {
        f[p * n + q] = h[p * n + q] + acc;
        if (p != q) f[q * n + p] = h[q * n + p] + acc;
    }
}

// Generalised Fock matrix F_pq = sum_r gamma_pr h_qr + sum_rst Gamma_prst
// (qr|st), one block per entry (rows p without density are zero: Gamma
// vanishes unless all its indices are among the frozen, core and active
// orbitals `occ`).  g2h holds Gamma / 2 (the gradient accumulators' convention).
__global__ __launch_bounds__(256) void k_fock_gen(const double *h, const double *eri, const double *g1,
                                                  const double *g2h, const int32_t *occ, int no, int n, double *F) {
    const int p = blockIdx.x / n, q = blockIdx.x % n;
    const int64_t n2 = (int64_t)n * n, n3 = n2 * n;
    __shared__ int o[kMaxOrb];
    __shared__ double sh[16];
    if ((int)threadIdx.x < no) o[threadIdx.x] = occ[threadIdx.x];
    __syncthreads();
    bool has = false;
    for (int i = 0; i < no; ++i) has |= o[i] == p;
    double acc = 0.0;
    if (has) {
        for (int i = threadIdx.x; i < no * no * no; i += 256) {
            const int64_t x = o[i / (no * no)] * n2 + o[i / no % no] * n + o[i % no];
            acc += 2.0 * g2h[p * n3 + x] * eri[q * n3 + x];
        }
        for (int i = threadIdx.x; i < no; i += 256) acc += g1[p * n + o[i]] * h[q * n + o[i]];
    }
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) F[p * n + q] = acc;
}

hipError_t launch_fock(const double *h, const double *eri, const double *g1, const double *g2h, const int32_t *occ,
                       int no, int n, double *F, double *f, hipStream_t s) {
    hipLaunchKernelGGL(k_fock, dim3(n * (n + 1) / 2), dim3(256), 0, s, h, eri, g1, n, f);
    if (g2h) hipLaunchKernelGGL(k_fock_gen, dim3(n * n), dim3(256), 0, s, h, eri, g1, g2h, occ, no, n, F);
    return hipGetLastError();
}

// Hessian of the closed-shell energy in the occupied-virtual rotations of the
// orbitals that `eri` and the Fock matrix f are given in (the first no
// occupied), derivative of the gradient 4 f_ai in the rotated frame:
//   H_ai,bj = 4 [ d_ij f_ab - d_ab f_ij + 4 (ai|bj) - (ab|ij) - (aj|ib) ],
// row and column index a * no + i.
__global__ __launch_bounds__(256) void k_hf_hessian(const double *eri, const double *f, int no, int n, double *H) {
    const int nv = n - no, np = no * nv;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)np * np) return;
    const int k = (int)(idx / np), l = (int)(idx % np);
    const int a = no + k / no, i = k % no, b = no + l / no, j = l % no;
    double x = 4.0 * ERI_AT(eri, n, a, i, b, j) - ERI_AT(eri, n, a, b, i, j) - ERI_AT(eri, n, a, j, b, i);
    if (i == j) x += f[a * n + b];
    if (a == b) x -= f[i * n + j];
    H[idx] = 4.0 * x;
}

hipError_t launch_hf_hessian(const double *eri, const double *f, int no, int n, double *H, hipStream_t s) {
    const int64_t np = (int64_t)no * (n - no);
    if (np > 0) hipLaunchKernelGGL(k_hf_hessian, dim3((unsigned)((np * np + 255) / 256)), dim3(256), 0, s, eri, f, no, n, H);
    return hipGetLastError();
}

}  // namespace mbefci
