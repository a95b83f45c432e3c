// Whole-tuple mode: one workgroup runs the complete Davidson solve of one
// small CASCI (Sec. 2: each increment needs the lowest eigenvalue of H over
// the tuple's CAS) in a single launch.  The per-iteration work of a small
// tuple is a few microseconds, far below the cost of the dozen launches of
// one batched iteration, so here the iteration loop itself runs on the
// device: Ritz pair of the projected matrix, residual and correction, two
// classical Gram-Schmidt passes and sigma, separated by workgroup barriers.
//
// The per-batch set-up is the batched path's: integral gather, string
// Hamiltonians, diagonal, P space and guess (V_0, normalised).  The basis V is
// kept orthonormal, so the projected matrix G = V^T H V is symmetric and is
// diagonalised directly.  Sigma is formed per determinant from the vector in
// LDS:
//   sigma(I_a, I_b) = sum_J_a H_a[I_a][J_a] c(J_a, I_b) + sum_J_b H_b[I_b][J_b] c(I_a, J_b)
//                   + sum over alpha links (J_a, P, s_a) of I_a and beta links (J_b, Q, s_b) of I_b
//                     of s_a s_b (P|Q) c(J_a, J_b)
// (plus lambda S_- S_+ c with a spin shift), the same operator the batched
// kernels apply.  On exit theta, status, iteration count, m and the Ritz
// coefficients y on V are written as the batched iteration leaves them.
#include "device.h"
#include "smalleig.h"
#include "symmetry.h"
#include "tridiag.h"

namespace mbefci {

constexpr int kWholeThreads = 512;
constexpr int kWholeWaves = kWholeThreads / 64;
constexpr int kWholeLd = kMaxSpace + 1;   // row stride of the small LDS matrices
constexpr int kWholeRed = kMaxSpace + 2;
constexpr int kWholeMaxLds = 160 * 1024;

struct WholeShared {
    double G[kMaxSpace][kWholeLd];      // projected matrix on the orthonormal basis
    double red[kWholeWaves][kWholeRed];
    double sum[kWholeRed];
    double y[kMaxSpace], yp[kMaxSpace], z[kMaxSpace];
    double pr[kPsp], pw[kPsp];
    double pd[kPsp], pe[kPsp];   // diagonal and subdiagonal of the P-space tridiagonal factor
    double pp[kWholeThreads / kPsp][kPsp];   // partial sums of the P-space products
    double theta, mu;
    int done, keep, cur;
};

// LDS set aside for the static part of k_whole
constexpr size_t kWholeStatic = 55952;
static_assert(sizeof(WholeShared) + sizeof(SmallEig<kMaxSpace>) + sizeof(TriShared) <= kWholeStatic, "static LDS of k_whole");

// Dynamic LDS: the vector of the current sigma, the pair integrals, the
// string Hamiltonians (one when both spins have the same electron count) and
// the two link tables.
size_t whole_lds_bytes(const ParamLayout &pl, int64_t dim, int64_t Na, int64_t Nb, int nentA, int nentB, bool same) {
    return 8 * (size_t)((dim + 1) & ~int64_t(1)) + 8 * (size_t)pl.P * pl.Kpad + 8 * (size_t)Nb * Nb +
           (same ? 0 : 8 * (size_t)Na * Na) + 4 * (size_t)(Na * nentA + Nb * nentB);
}

// The same with the diagonal links summed (k_whole<MS, true>): pair integrals
// extended by a row per alpha string and a column per beta string, shorter
// link tables.
static size_t whole_lds_bytes_diag(const Batch &b) {
    const int64_t rows = b.pl.P + b.Na, ld = (b.pl.P + b.Nb) | 1;
    if (b.na < 1 || b.nb < 1 || rows > 1023 || b.pl.P + b.Nb > 1023) return (size_t)-1;   // (10-bit row fields)
    return 8 * (size_t)((b.dim + 1) & ~int64_t(1)) + 8 * (size_t)((rows * ld + 1) & ~int64_t(1)) + 8 * (size_t)b.Nb * b.Nb +
           (b.Ha == b.Hb ? 0 : 8 * (size_t)b.Na * b.Na) +
           4 * (size_t)(b.Na * (b.nentA - b.na + 1) + b.Nb * (b.nentB - b.nb + 1));
}

bool whole_fits(const ParamLayout &pl, int64_t dim, int64_t Na, int64_t Nb, int nentA, int nentB, bool same) {
    return pl.nA <= kWholeMaxActive && dim <= kWholeMaxDim && nentB <= kWholeMaxNent && nentA <= kWholeMaxNent &&
           whole_lds_bytes(pl, dim, Na, Nb, nentA, nentB, same) + kWholeStatic <= (size_t)kWholeMaxLds;
}

// Sums over the workgroup of acc[0 .. n-1] into w.sum[0 .. n-1] and, with
// `ext`, of x into w.sum[n] (n uniform); every thread may read w.sum after
// the call.
template <int N>
__device__ __forceinline__ void wg_sums(WholeShared &w, const double (&acc)[N], int n, bool ext = false,
                                        double x = 0.0) {
    const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        if (k < n) {
            const double v = wave_sum(acc[k]);
            if (l == 0) w.red[wv][k] = v;
        }
    }
    if (ext) {
        const double v = wave_sum(x);
        if (l == 0) w.red[wv][n] = v;
        ++n;
    }
    __syncthreads();
    if ((int)threadIdx.x < n) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < kWholeWaves; ++i) s += w.red[i][threadIdx.x];
        w.sum[threadIdx.x] = s;
    }
    __syncthreads();
}

// Lowest eigenpair of the symmetric m x m matrix w.G, by the first wave (the
// others wait at the workgroup barrier at the end): w.theta, and w.y (zero
// past m).
template <int MS>
__device__ __forceinline__ void wg_lowest_eig(WholeShared &w, SmallEig<MS> &q, int m) {
    constexpr int IW = SmallEig<MS>::IW;
    const int tid = threadIdx.x;
    if (tid < 64) {
        for (int k = tid; k < m * IW; k += 64) {
            const int r = k / IW, c = k & (IW - 1);
            if (c < m) q.A[r][c] = w.G[r][c];
        }
        wave_sync();
        double y;
        const double th = lowest_eig<MS>(q, m, y);
        if (tid < kMaxSpace) w.y[tid] = tid < m ? y : 0.0;
        if (tid == 0) w.theta = th;
    }
    __syncthreads();
}

// DIAG: the diagonal links of a string (p, p), p occupied, all lead back to
// the string, so their integrals are summed once per solve, sum_p (pp|Q) as an
// extra row (column) of the pair table, and one link stands for them: 1 + n
// (n_A - n) links per string instead of n (n_A - n + 1).  Sigma is bound by
// the LDS gathers of its link pairs (about 9 cycles each per wave), whose
// number falls by a third (11 orbitals, doublet: 533 -> 385 us per launch).
// Without it where the table does not fit.
template <int MS, bool DIAG>
__global__ __launch_bounds__(kWholeThreads) void k_whole(Batch b) {
    const int t = blockIdx.x, tid = threadIdx.x;
    const int64_t dim = b.dim;
    const int Na = (int)b.Na, Nb = (int)b.Nb;
    const int nentA = DIAG ? b.nentA - b.na + 1 : b.nentA, nentB = DIAG ? b.nentB - b.nb + 1 : b.nentB;
    const ParamLayout &pl = b.pl;
    const int P = pl.P, ldE = DIAG ? (P + Nb) | 1 : pl.Kpad, rowsE = DIAG ? P + Na : P;
    const bool same = b.Ha == b.Hb;
    __shared__ WholeShared w;
    __shared__ SmallEig<MS> eig;
    __shared__ TriShared tri;
    extern __shared__ double wlds[];
    double *cL = wlds;                                    // [dim] vector of the current sigma
    double *eri = cL + ((dim + 1) & ~int64_t(1));         // [rowsE][ldE] (P|Q) / 2
    double *hB = eri + ((rowsE * ldE + 1) & ~1);          // [Nb][Nb] beta string Hamiltonian
    double *hA = same ? hB : hB + Nb * Nb;                // [Na][Na] alpha string Hamiltonian
    uint32_t *lkA = reinterpret_cast<uint32_t *>(same ? hB + Nb * Nb : hA + Na * Na);   // [Na][nentA]
    uint32_t *lkB = lkA + Na * nentA;                     // [Nb][nentB]
    const double *prm = b.params + (int64_t)t * pl.stride;
    const double *Ha = b.Ha + (int64_t)t * Na * Na, *Hb = b.Hb + (int64_t)t * Nb * Nb;
    for (int i = tid; i < P * P; i += kWholeThreads) eri[(i / P) * ldE + i % P] = prm[pl.off_eri + (i / P) * pl.Kpad + i % P];
    for (int i = tid; i < Nb * Nb; i += kWholeThreads) hB[i] = Hb[i];
    if (!same)
        for (int i = tid; i < Na * Na; i += kWholeThreads) hA[i] = Ha[i];
    // (a string's diagonal links come first in the tables)
    auto links = [&](uint32_t *dst, const uint32_t *src, int N, int nel, int nent) {
        for (int i = tid; i < N * nent; i += kWholeThreads) {
            const int I = i / nent, e = i % nent;
            if (!DIAG) dst[i] = src[i];
            else dst[i] = e == 0 ? (uint32_t)I | ((uint32_t)(P + I) << 20) : src[I * (nent + nel - 1) + nel - 1 + e];
        }
    };
    links(lkA, b.linkA, Na, b.na, nentA);
    links(lkB, b.linkB, Nb, b.nb, nentB);
    if (DIAG) {
        __syncthreads();
        for (int i = tid; i < P * Nb; i += kWholeThreads) {   // columns: sum over the orbitals of I_b
            double *row = eri + (i / Nb) * ldE;
            double s = 0.0;
            for (uint32_t x = b.strB[i % Nb]; x; x &= x - 1) {
                const int q = __ffs(x) - 1;
                s += row[q * (q + 3) / 2];
            }
            row[P + i % Nb] = s;
        }
        __syncthreads();
        for (int i = tid; i < Na * (P + Nb); i += kWholeThreads) {   // rows: over those of I_a
            const int I = i / (P + Nb), c = i % (P + Nb);
            double s = 0.0;
            for (uint32_t x = b.strA[I]; x; x &= x - 1) {
                const int q = __ffs(x) - 1;
                s += eri[(q * (q + 3) / 2) * ldE + c];
            }
            eri[(P + I) * ldE + c] = s;
        }
    }
    if (b.psp > 0 && tid < b.psp) {
        w.pd[tid] = b.pT[(int64_t)t * 3 * kPsp + tid];
        w.pe[tid] = b.pT[(int64_t)t * 3 * kPsp + kPsp + tid];
    }
    double *V = b.V + (int64_t)t * b.max_space * dim;
    double *S = b.S + (int64_t)t * b.max_space * dim;
    const double *hd = b.Hd + (int64_t)t * dim;
    const int maxs = b.max_space;
    const double lam = b.spin_shift;
    // V_i and S_i, i < m, through buffer resources that end after vector
    // m - 1: loads past it read zero, so all loads of a determinant are issued
    // at once (the coefficients there are zero too)
    const uint32_t vstride = (uint32_t)dim * (uint32_t)sizeof(double);
    auto rsrc = [&](double *base, int nvec) {
        return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, (int)(nvec * vstride), 0x00020000);
    };
    auto ld = [&](__amdgpu_buffer_rsrc_t r, int64_t d, int i) {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (uint32_t)d * 8u, (uint32_t)i * vstride, 0));
    };

    // out[i] = sum_k M[k][i] u[k], i < n (M row-major with stride kPsp; u,
    // out in LDS), the k range split over the workgroup's threads in
    // kWholeThreads / kPsp parts; ends with a barrier
    auto psp_product = [&](const double *Mx, const double *u, double *out) {
        constexpr int NP = kWholeThreads / kPsp;
        const int n = b.psp, i = tid % kPsp, part = tid / kPsp;
        const int k0 = part * n / NP, k1 = (part + 1) * n / NP;
        double s = 0.0;
        if (i < n) {
#pragma unroll 8
            for (int k = k0; k < k1; ++k) s += Mx[k * kPsp + i] * u[k];
        }
        w.pp[part][i] = s;
        __syncthreads();
        if (tid < n) {
            double v = 0.0;
#pragma unroll
            for (int q = 0; q < NP; ++q) v += w.pp[q][tid];
            out[tid] = v;
        }
        __syncthreads();
    };

    // sigma of the vector in cL at determinant d
    auto sigma_det = [&](int64_t d) -> double {
        const int Ia = (int)(d / Nb), Ib = (int)(d - (int64_t)Ia * Nb);
        double acc = 0.0;
        const double *ha = hA + Ia * Na;
        for (int Ja = 0; Ja < Na; ++Ja) acc += ha[Ja] * cL[Ja * Nb + Ib];
        const double *crow = cL + Ia * Nb;
        for (int Jb = 0; Jb < Nb; ++Jb) acc += hB[Jb * Nb + Ib] * crow[Jb];   // H_b symmetric
        uint32_t lb[kWholeMaxNent];
#pragma unroll
        for (int e = 0; e < kWholeMaxNent; ++e) lb[e] = e < nentB ? lkB[Ib * nentB + e] : 0u;
        double ab = 0.0;
        const uint32_t *la = lkA + Ia * nentA;
        for (int ea = 0; ea < nentA; ++ea) {
            const uint32_t L = la[ea];
            const double *er = eri + (int)((L >> 20) & 0x3FFu) * ldE;
            const double *cr = cL + (int)(L & 0xFFFFFu) * Nb;
            double s = 0.0;
#pragma unroll
            for (int e = 0; e < kWholeMaxNent; ++e) {
                if (e < nentB) {
                    const uint32_t M = lb[e];
                    const double v = er[(M >> 20) & 0x3FFu] * cr[M & 0xFFFFFu];
                    s += (M >> 31) ? -v : v;
                }
            }
            ab += (L >> 31) ? -s : s;
        }
        acc += 2.0 * ab;   // the table holds (P|Q) / 2
        if (lam != 0.0) acc += lam * spin_ss(b, cL, Ia, Ib);
        if (b.sym_shift != 0.0) acc += sym_pen(b, t, b.strA[Ia], b.strB[Ib]) * cL[d];
        return acc;
    };

    // first basis vector: the guess, normalised by the set-up
    for (int64_t d = tid; d < dim; d += kWholeThreads) cL[d] = V[d];
    __syncthreads();
    {
        double acc[1] = {0.0};
        for (int64_t d = tid; d < dim; d += kWholeThreads) {
            const double s = sigma_det(d);
            S[d] = s;
            acc[0] += cL[d] * s;
        }
        wg_sums(w, acc, 1);
        if (tid == 0) {
            w.G[0][0] = w.sum[0];
            for (int i = 0; i < kMaxSpace; ++i) w.yp[i] = i == 0 ? 1.0 : 0.0;
        }
        __syncthreads();
    }
    int m = 1, iter = 0, status = ST_RUNNING, force = 0;
    double theta_prev = 1e300, theta = 0.0;
    while (true) {
        wg_lowest_eig<MS>(w, eig, m);
        theta = w.theta;
        const bool restart = m >= maxs || force;
        force = 0;
        if (tid == 0) {
            int keep = restart ? 1 : 0;
            if (restart && b.restart_keep > 1) {
                // the previous Ritz vector (coordinates yp, zero past its
                // length) made orthogonal to this one by two passes
                for (int i = 0; i < m; ++i) w.z[i] = w.yp[i];
                for (int pass = 0; pass < 2; ++pass) {
                    double dd = 0.0;
                    for (int i = 0; i < m; ++i) dd += w.z[i] * w.y[i];
                    for (int i = 0; i < m; ++i) w.z[i] -= dd * w.y[i];
                }
                double nz = 0.0;
                for (int i = 0; i < m; ++i) nz += w.z[i] * w.z[i];
                if (nz > 1e-12) {
                    const double sc = 1.0 / sqrt(nz);
                    double mu = 0.0;
                    for (int i = 0; i < m; ++i) w.z[i] *= sc;
                    for (int i = 0; i < m; ++i)
                        for (int j = 0; j < m; ++j) mu += w.z[i] * w.G[i][j] * w.z[j];
                    w.mu = mu;
                    keep = 2;
                }
            }
            for (int i = m; i < kMaxSpace; ++i) w.z[i] = 0.0;
            w.keep = keep;
            if (!restart)
                for (int i = 0; i < kMaxSpace; ++i) w.yp[i] = w.y[i];
        }
        __syncthreads();
        const int keep = w.keep;
        // Ritz vector x = V y, residual r = S y - theta x, correction
        // r / (theta - H_II) (clamped) into the next basis slot; on restart x,
        // S x (and the kept direction) replace V_0, S_0 (V_1, S_1) in place
        const int slot = restart ? keep : m;
        {
            double acc[1] = {0.0};
            double *T = V + (int64_t)slot * dim;
            const __amdgpu_buffer_rsrc_t rV = rsrc(V, m), rS = rsrc(S, m);
            double yy[MS], zz[MS];
#pragma unroll
            for (int i = 0; i < MS; ++i) {
                yy[i] = w.y[i];
                zz[i] = w.z[i];
            }
            for (int64_t d = tid; d < dim; d += kWholeThreads) {
                double x = 0.0, ax = 0.0, x2 = 0.0, a2 = 0.0;
#pragma unroll
                for (int i = 0; i < MS; ++i) {
                    const double v = ld(rV, d, i), s = ld(rS, d, i);
                    x += yy[i] * v;
                    ax += yy[i] * s;
                    if (keep == 2) {
                        x2 += zz[i] * v;
                        a2 += zz[i] * s;
                    }
                }
                const double r = ax - theta * x;
                acc[0] += r * r;
                double den = theta - hd[d];
                if (fabs(den) < 1e-8) den = den >= 0.0 ? 1e-8 : -1e-8;
                if (restart) {
                    V[d] = x;
                    S[d] = ax;
                    if (keep == 2) {
                        V[dim + d] = x2;
                        S[dim + d] = a2;
                    }
                }
                T[d] = r / den;
            }
            wg_sums(w, acc, 1);
        }
        const double rn = sqrt(w.sum[0]);
        if (restart) {
            m = keep;
            if (tid == 0) {
                for (int i = 0; i < kMaxSpace; ++i) {
                    w.y[i] = i == 0 ? 1.0 : 0.0;
                    w.yp[i] = w.y[i];
                }
                w.G[0][0] = theta;
                if (keep == 2) {
                    w.G[0][1] = w.G[1][0] = 0.0;
                    w.G[1][1] = w.mu;
                }
            }
            __syncthreads();
        }
        ++iter;
        if (!isfinite(rn) || !isfinite(theta)) status = ST_NONFINITE;
        // (a P space that is the whole space holds the exact eigenvector: the
        // correction's equation is singular there, and a small residual is enough)
        else if (rn < b.r_tol && (b.psp >= dim || fabs(theta - theta_prev) < b.e_tol)) status = ST_DONE;
        else if (iter >= b.max_iter) status = ST_MAXITER;
        theta_prev = theta;
        if (status != ST_RUNNING) break;
        double *T = V + (int64_t)m * dim;
        // P space: the correction there is the exact (theta - H_PP)^-1 r_P,
        // H_PP = Q Tr Q^T with Tr tridiagonal
        if (b.psp > 0) {
            const int n = b.psp;
            const int32_t *pidx = b.pidx + (int64_t)t * kPsp;
            const double *Q = b.pQ + (int64_t)t * kPsp * kPsp, *Qt = b.pQt + (int64_t)t * kPsp * kPsp;
            const double *dT = w.pd, *eT = w.pe;
            if (tid < n) {
                const int64_t d = pidx[tid];
                const __amdgpu_buffer_rsrc_t rV = rsrc(V, m), rS = rsrc(S, m);
                double r = 0.0;
#pragma unroll
                for (int i = 0; i < MS; ++i) r += w.y[i] * (ld(rS, d, i) - theta * ld(rV, d, i));
                w.pr[tid] = r;
            }
            __syncthreads();
            psp_product(Q, w.pr, w.pw);
            {
                const bool own = tid < n;
                const double u = tri_solve(tri, n, theta, own ? dT[tid] : 0.0, own ? eT[tid] : 0.0,
                                           own && tid > 0 ? eT[tid - 1] : 0.0, own ? w.pw[tid] : 0.0);
                __syncthreads();
                if (own) w.pw[tid] = u;
            }
            __syncthreads();
            psp_product(Qt, w.pw, w.pr);
            if (tid < n) T[pidx[tid]] = w.pr[tid];
            __syncthreads();
        }
        // two classical Gram-Schmidt passes of T against V_0 .. V_{m-1}
        double t0, tn;
        {
            const __amdgpu_buffer_rsrc_t rV = rsrc(V, m);
            double acc[MS], tt = 0.0;
#pragma unroll
            for (int i = 0; i < MS; ++i) acc[i] = 0.0;
            for (int64_t d = tid; d < dim; d += kWholeThreads) {
                const double tv = T[d];
#pragma unroll
                for (int i = 0; i < MS; ++i) acc[i] += ld(rV, d, i) * tv;
                tt += tv * tv;
            }
            wg_sums(w, acc, m, true, tt);
            t0 = sqrt(w.sum[m]);
            double cf[MS];
#pragma unroll
            for (int i = 0; i < MS; ++i) cf[i] = i < m ? w.sum[i] : 0.0;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < MS; ++i) acc[i] = 0.0;
            for (int64_t d = tid; d < dim; d += kWholeThreads) {
                double vv[MS], tv = T[d];
#pragma unroll
                for (int i = 0; i < MS; ++i) vv[i] = ld(rV, d, i);
#pragma unroll
                for (int i = 0; i < MS; ++i) tv -= cf[i] * vv[i];
                T[d] = tv;
#pragma unroll
                for (int i = 0; i < MS; ++i) acc[i] += vv[i] * tv;
            }
            wg_sums(w, acc, m);
#pragma unroll
            for (int i = 0; i < MS; ++i) cf[i] = i < m ? w.sum[i] : 0.0;
            __syncthreads();
            double a2[1] = {0.0};
            for (int64_t d = tid; d < dim; d += kWholeThreads) {
                double tv = T[d];
#pragma unroll
                for (int i = 0; i < MS; ++i) tv -= cf[i] * ld(rV, d, i);
                T[d] = tv;
                a2[0] += tv * tv;
            }
            wg_sums(w, a2, 1);
            tn = sqrt(w.sum[0]);
        }
        if (!(tn > 1e-8 * t0) || !(tn > 1e-300)) {
            // the correction lies in the subspace: converged if the residual
            // is small (an invariant subspace), else restart from the Ritz
            // vector, or stalled when the subspace is that vector already
            if (rn < b.r_tol) {
                status = ST_DONE;
                break;
            }
            if (m > 1) {
                force = 1;
                continue;
            }
            status = ST_STALLED;
            break;
        }
        // V_m = T / |T|, also into LDS for its sigma
        {
            const double sc = 1.0 / tn;
            for (int64_t d = tid; d < dim; d += kWholeThreads) {
                const double v = T[d] * sc;
                T[d] = v;
                cL[d] = v;
            }
            __syncthreads();
        }
        // S_m = H V_m and the new column of G
        {
            const __amdgpu_buffer_rsrc_t rV = rsrc(V, m);
            double acc[MS], dm = 0.0;
#pragma unroll
            for (int i = 0; i < MS; ++i) acc[i] = 0.0;
            double *Sm = S + (int64_t)m * dim;
            for (int64_t d = tid; d < dim; d += kWholeThreads) {
                const double s = sigma_det(d);
                Sm[d] = s;
#pragma unroll
                for (int i = 0; i < MS; ++i) acc[i] += ld(rV, d, i) * s;
                dm += cL[d] * s;
            }
            wg_sums(w, acc, m, true, dm);
            if (tid <= m) {
                w.G[tid][m] = w.sum[tid];
                w.G[m][tid] = w.sum[tid];
            }
            __syncthreads();
            ++m;
        }
    }
    if (tid == 0) {
        b.theta[t] = theta;
        b.status[t] = status;
        b.iter[t] = iter;
        b.m[t] = m;
        double *y = b.y + (int64_t)t * kMaxSpace;
        for (int i = 0; i < kMaxSpace; ++i) y[i] = i < m ? w.y[i] : 0.0;
    }
}

template <int MS> static void launch_whole_ms(const Batch &b, hipStream_t s) {
    const size_t diag = whole_lds_bytes_diag(b);
    if (diag <= (size_t)kWholeMaxLds - kWholeStatic)
        hipLaunchKernelGGL((k_whole<MS, true>), dim3(b.B), dim3(kWholeThreads), diag, s, b);
    else
        hipLaunchKernelGGL((k_whole<MS, false>), dim3(b.B), dim3(kWholeThreads),
                           whole_lds_bytes(b.pl, b.dim, b.Na, b.Nb, b.nentA, b.nentB, b.Ha == b.Hb), s, b);
}

hipError_t launch_whole(const Batch &b, hipStream_t s) {
    if (b.max_space <= 12) launch_whole_ms<12>(b, s);
    else launch_whole_ms<kMaxSpace>(b, s);
    return hipGetLastError();
}

hipError_t init_whole_kernels() {
    const int dyn = kWholeMaxLds - (int)kWholeStatic;
    for (const void *f : {(const void *)k_whole<12, false>, (const void *)k_whole<12, true>,
                          (const void *)k_whole<kMaxSpace, false>, (const void *)k_whole<kMaxSpace, true>}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace mbefci
