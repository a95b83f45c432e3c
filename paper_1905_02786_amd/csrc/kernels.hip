// HIP kernels (gfx950 / CDNA4, FP64) of the batched CASCI solver.
//
// Every kernel works on a batch of tuples of one shape class (same active
// orbital count and active electron counts, hence the same determinant space
// and string tables); blockIdx.y (or blockIdx.x for per-tuple kernels) selects
// the tuple.  Reductions are block partial sums followed by a fixed-order sum,
// so results do not depend on scheduling.
//
// The active-space Hamiltonian (CASCI of Sec. 2 with a frozen core) is
//   H = E_core + sum_pq k_pq E_pq + 1/2 sum_pqrs (pq|rs) E_pq E_rs,
//   k_pq = h^eff_pq - 1/2 sum_r (pr|rq),  h^eff_pq = h_pq + sum_c [2(pq|cc) - (pc|cq)],
//   E_core = E_const + sum_c 2 h_cc + sum_cd [2(cc|dd) - (cd|dc)],
// over p, q, r, s in A and c in the core C.
#include <type_traits>

#include "device.h"
#include "smalleig.h"
#include "symmetry.h"
#include "tridiag.h"

namespace mbefci {

// ---------------------------------------------------------------- gather --
// One block per tuple: E_core, k (pair-packed), diagonal helpers and the
// half-scaled pair matrix 1/2 (pq|rs) zero-padded for the MFMA tiles.
__global__ __launch_bounds__(256) void k_gather(Batch b) {
    const int t = blockIdx.x, tid = threadIdx.x, nth = blockDim.x;
    const ParamLayout &pl = b.pl;
    const int nA = b.nA, nC = b.nC, n = b.norb;
    double *prm = b.params + (int64_t)t * pl.stride;
    __shared__ int sA[kMaxActive], sC[64];
    __shared__ int pp[kMaxActive * (kMaxActive + 1) / 2], qq[kMaxActive * (kMaxActive + 1) / 2];
    __shared__ double heff[kMaxActive * kMaxActive];
    __shared__ double red[16];
    if (tid < nA) sA[tid] = b.act[(int64_t)t * nA + tid];
    if (tid < nC) sC[tid] = b.core[(int64_t)t * nC + tid];
    if (tid < pl.P) {
        int p, q;
        pair_of(tid, p, q);
        pp[tid] = p;
        qq[tid] = q;
    }
    __syncthreads();
    const double *h = b.h, *eri = b.eri;

    double part = 0.0;
    for (int idx = tid; idx < nC + nC * nC; idx += nth) {
        if (idx < nC) {
            const int c = sC[idx];
            part += 2.0 * h[c * n + c];
        } else {
            const int u = idx - nC, c = sC[u / nC], d = sC[u % nC];
            part += 2.0 * ERI_AT(eri, n, c, c, d, d) - ERI_AT(eri, n, c, d, d, c);
        }
    }
    const double ec = block_sum(part, red);
    if (tid == 0) prm[pl.off_ecore] = b.e_const + ec;

    for (int idx = tid; idx < nA * nA; idx += nth) {
        const int ap = sA[idx / nA], aq = sA[idx % nA];
        double v = h[ap * n + aq];
        for (int k = 0; k < nC; ++k) {
            const int c = sC[k];
            v += 2.0 * ERI_AT(eri, n, ap, aq, c, c) - ERI_AT(eri, n, ap, c, c, aq);
        }
        heff[idx] = v;
    }
    __syncthreads();
    for (int idx = tid; idx < pl.P; idx += nth) {
        const int p = pp[idx], q = qq[idx], ap = sA[p], aq = sA[q];
        double v = heff[p * nA + q];
        for (int r = 0; r < nA; ++r) v -= 0.5 * ERI_AT(eri, n, ap, sA[r], sA[r], aq);
        prm[pl.off_k + idx] = v;
    }
    for (int idx = tid; idx < nA; idx += nth) prm[pl.off_hd1 + idx] = heff[idx * nA + idx];
    for (int idx = tid; idx < nA * nA; idx += nth) {
        const int ap = sA[idx / nA], aq = sA[idx % nA];
        prm[pl.off_J + idx] = ERI_AT(eri, n, ap, ap, aq, aq);
        prm[pl.off_K + idx] = ERI_AT(eri, n, ap, aq, aq, ap);
    }
    for (int idx = tid; idx < pl.Ppad * pl.Kpad; idx += nth) {
        const int R = idx / pl.Kpad, Q = idx % pl.Kpad;
        double v = 0.0;
        if (R < pl.P && Q < pl.P)
            v = 0.5 * ERI_AT(eri, n, sA[pp[R]], sA[qq[R]], sA[pp[Q]], sA[qq[Q]]);
        prm[pl.off_eri + idx] = v;
    }
}

hipError_t launch_gather(const Batch &b, hipStream_t s) {
    hipLaunchKernelGGL(k_gather, dim3(b.B), dim3(256), 0, s, b);
    return hipGetLastError();
}

// ----------------------------------------------------------------- hdiag --
// H_II = E_a(Ia) + E_b(Ib) + sum_{i in Ia, j in Ib} (ii|jj), with
// E_s(I) = sum_{i in I} h^eff_ii + 1/2 sum_{i,j in I} [(ii|jj) - (ij|ji)].
__global__ __launch_bounds__(256) void k_hdiag(Batch b, double *out, int64_t ostride, int add_ecore) {
    const int t = blockIdx.y;
    const ParamLayout &pl = b.pl;
    const double *prm = b.params + (int64_t)t * pl.stride;
    __shared__ double hd[kMaxActive], J[kMaxActive * kMaxActive], K[kMaxActive * kMaxActive];
    const int nA = b.nA;
    for (int i = threadIdx.x; i < nA; i += blockDim.x) hd[i] = prm[pl.off_hd1 + i];
    for (int i = threadIdx.x; i < nA * nA; i += blockDim.x) {
        J[i] = prm[pl.off_J + i];
        K[i] = prm[pl.off_K + i];
    }
    __syncthreads();
    const double ec = add_ecore ? prm[pl.off_ecore] : 0.0;
    for (int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; d < b.dim;
         d += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t ma = b.strA[d / b.Nb], mb = b.strB[d % b.Nb];
        double e = 0.0;
        for (uint32_t x = ma; x; x &= x - 1) {
            const int i = __ffs(x) - 1;
            e += hd[i];
            for (uint32_t y = ma; y; y &= y - 1) {
                const int j = __ffs(y) - 1;
                e += 0.5 * (J[i * nA + j] - K[i * nA + j]);
            }
            for (uint32_t y = mb; y; y &= y - 1) e += J[i * nA + __ffs(y) - 1];
        }
        for (uint32_t x = mb; x; x &= x - 1) {
            const int i = __ffs(x) - 1;
            e += hd[i];
            for (uint32_t y = mb; y; y &= y - 1) {
                const int j = __ffs(y) - 1;
                e += 0.5 * (J[i * nA + j] - K[i * nA + j]);
            }
        }
        // level shift toward the lowest spin of the sector: lambda times the
        // diagonal of S_- S_+, n_b - (orbitals holding both spins)
        if (b.spin_shift != 0.0) e += b.spin_shift * (double)(b.nb - __popc(ma & mb));
        // level shift away from the other irreps (spatial symmetry targeting)
        if (b.sym_shift != 0.0) e += sym_pen(b, t, ma, mb);
        out[(int64_t)t * ostride + d] = e + ec;
    }
}

hipError_t launch_hdiag(const Batch &b, double *out, int64_t ostride, int add_ecore, hipStream_t s) {
    dim3 grid(grid_for(b.dim, 256, 4096), b.B);
    hipLaunchKernelGGL(k_hdiag, grid, dim3(256), 0, s, b, out, ostride, add_ecore);
    return hipGetLastError();
}

// -------------------------------------------------------------- Davidson --
// Per-tuple state lives in the Batch arrays.  Vector kernels use grid
// (nblk, B) and write block partials to part[t][blk][*]; per-tuple kernels
// (one block of 64 threads per tuple) sum them in block order.

// column sums of the partials for i < nx (thread i), fixed block order
__device__ double sum_parts(const Batch &b, int t, int i) {
    double s = 0.0;
    for (int blk = 0; blk < b.nblk; ++blk) s += parts(b, t, blk)[i];
    return s;
}

// the same plus the P-space correction block (guess norm)
__device__ double sum_parts_x(const Batch &b, int t, int i) {
    const double s = sum_parts(b, t, i);
    return b.psp > 0 ? s + parts(b, t, b.nblk)[i] : s;
}

// Block-reduce up to NP (<= kParts) per-thread accumulators into partials.
template <int NP = kParts>
__device__ void store_block_partials(const Batch &b, int t, const double *acc, int nx) {
    __shared__ double sh[4][NP];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        if (i < nx) {
            const double v = wave_sum(acc[i]);
            if (lane == 0) sh[w][i] = v;
        }
    }
    __syncthreads();
    if (threadIdx.x < nx) {
        double s = 0.0;
        for (int k = 0; k < 4; ++k) s += sh[k][threadIdx.x];
        parts(b, t, blockIdx.x)[threadIdx.x] = s;
    }
}

// ------------------------------------------------------- P-space ----------
// Davidson preconditioner on the P space of the psp determinants with the
// lowest diagonal energies: the correction there solves (theta - H_PP) t_P =
// r_P exactly (H_PP = Q T Q^T, T tridiagonal, both computed once per tuple),
// elsewhere t = r / (theta - H_II).  The initial guess is the lowest
// eigenvector of H_PP plus the same 1e-3 admixture as the determinant guess
// (none when P is the whole space, where that eigenvector is exact).

// P selection, one block per tuple: histogram of H_II over [min, max] in 1024
// bins, then the determinants of the bins below the one holding the psp-th
// smallest value, and from that bin the lowest indices up to psp, in index
// order (deterministic, ties broken by index).  Bound by the latency of one
// workgroup's loads: sixteen waves, and for the last two passes a contiguous
// range each, so that the places come from one prefix sum over the waves
// (waves without a determinant of P skip the last pass).  245 025 to 853 776
// determinants 4.0 -> 1.1 ms, 3136 to 15 876 39 -> 14 us, 120 to 1225 12 ->
// 4 us a launch, against four waves and two barriers per 256 determinants.
__global__ __launch_bounds__(1024) void k_psp_select(Batch b) {
    constexpr int NW = 16, NT = 64 * NW;
    const int t = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int n = b.psp;
    const double *hd = b.Hd + (int64_t)t * b.dim;
    int32_t *out = b.pidx + (int64_t)t * kPsp;
    __shared__ double rmin[NW], rmax[NW];
    __shared__ int hist[1024], sum[1024 / 64];
    __shared__ int sB, sC0, sNeed, wc1[NW], wc2[NW];
    if (b.dim <= n) {
        for (int i = tid; i < n; i += NT) out[i] = i;
        return;
    }
    double mn = 1e300, mx = -1e300;
#pragma unroll 4
    for (int64_t d = tid; d < b.dim; d += NT) {
        mn = fmin(mn, hd[d]);
        mx = fmax(mx, hd[d]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mn = fmin(mn, __shfl_xor(mn, o, 64));
        mx = fmax(mx, __shfl_xor(mx, o, 64));
    }
    if (lane == 0) {
        rmin[wv] = mn;
        rmax[wv] = mx;
    }
    hist[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        mn = fmin(mn, rmin[q]);
        mx = fmax(mx, rmax[q]);
    }
    const double scale = mx > mn ? 1024.0 / (mx - mn) : 0.0;
    auto bin = [&](double v) -> int {
        const int k = (int)((v - mn) * scale);
        return k < 0 ? 0 : (k > 1023 ? 1023 : k);
    };
#pragma unroll 4
    for (int64_t d = tid; d < b.dim; d += NT) atomicAdd(&hist[bin(hd[d])], 1);
    __syncthreads();
    // the first bin where the running count reaches n
    int inc = hist[tid];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) sum[wv] = inc;
    __syncthreads();
    for (int q = 0; q < wv; ++q) inc += sum[q];
    if (inc >= n && inc - hist[tid] < n) {
        sB = tid;
        sC0 = inc - hist[tid];
        sNeed = n - (inc - hist[tid]);
    }
    __syncthreads();
    const int B = sB, C0 = sC0, need = sNeed;
    const int64_t len = ((b.dim + NT - 1) / NT) * 64, d0 = wv * len, d1 = d0 + len < b.dim ? d0 + len : b.dim;
    int c1 = 0, c2 = 0;
#pragma unroll 4
    for (int64_t d = d0 + lane; d < d1; d += 64) {
        const int k = bin(hd[d]);
        c1 += k < B;
        c2 += k == B;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        c1 += __shfl_xor(c1, o, 64);
        c2 += __shfl_xor(c2, o, 64);
    }
    if (lane == 0) {
        wc1[wv] = c1;
        wc2[wv] = c2;
    }
    __syncthreads();
    int o1 = 0, o2 = 0;
    for (int q = 0; q < wv; ++q) {
        o1 += wc1[q];
        o2 += wc2[q];
    }
    if (c1 == 0 && (c2 == 0 || o2 >= need)) return;
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    for (int64_t e = d0; e < d1; e += 64) {
        const int64_t d = e + lane;
        const int k = d < d1 ? bin(hd[d]) : 2048;
        const bool f1 = k < B, f2 = k == B;
        const uint64_t m1 = __ballot(f1), m2 = __ballot(f2);
        const int p2 = o2 + __popcll(m2 & below);
        if (f1) out[o1 + __popcll(m1 & below)] = (int32_t)d;
        if (f2 && p2 < need) out[C0 + p2] = (int32_t)d;
        o1 += __popcll(m1);
        o2 += __popcll(m2);
    }
}

// Pair index of the single excitation between two strings.
__device__ __forceinline__ int single_pair(uint32_t mi, uint32_t mj) {
    const int p = __ffs(mi & ~mj) - 1, q = __ffs(mj & ~mi) - 1;
    const int lo = p < q ? p : q, hi = p < q ? q : p;
    return hi * (hi + 1) / 2 + lo;
}

// Sign of the single excitation that turns string J into string I (one
// orbital created in I, one annihilated from J): the parity of J's occupied
// orbitals strictly between the two.
__device__ __forceinline__ double excitation_sign(uint32_t mi, uint32_t mj) {
    const uint32_t diff = mi ^ mj;
    return odd_between(mj, __ffs(mi & diff) - 1, __ffs(mj & diff) - 1) ? -1.0 : 1.0;
}

// H_PP[i][j] = H_a[Ia][Ja] d(Ib,Jb) + H_b[Ib][Jb] d(Ia,Ja)
//            + sum_PQ (P|Q) <Ia|E+_P|Ja> <Ib|E+_Q|Jb>  (upper triangle, mirrored)
// plus, with a spin level shift, lambda <I|S_- S_+|J>: n_b - (orbitals
// holding both spins) on the diagonal, -s_a s_b where an alpha electron
// moves q <- p and a beta electron p <- q (I = E^a_qp E^b_pq J).
__global__ __launch_bounds__(256) void k_psp_build(Batch b) {
    const int t = blockIdx.x, n = b.psp;
    const ParamLayout &pl = b.pl;
    const double *prm = b.params + (int64_t)t * pl.stride;
    const int32_t *pi = b.pidx + (int64_t)t * kPsp;
    const double *Ha = b.Ha + (int64_t)t * b.Na * b.Na, *Hb = b.Hb + (int64_t)t * b.Nb * b.Nb;
    double *H = b.pQ + (int64_t)t * kPsp * kPsp;
    for (int idx = blockIdx.y * 256 + threadIdx.x; idx < n * n; idx += gridDim.y * 256) {
        const int i = idx / n, j = idx % n;
        if (j < i) continue;
        const int64_t I = pi[i], J = pi[j];
        const int64_t ia = I / b.Nb, ib = I % b.Nb, ja = J / b.Nb, jb = J % b.Nb;
        double v = 0.0;
        if (ib == jb) v += Ha[ia * b.Na + ja];
        if (ia == ja) v += Hb[ib * b.Nb + jb];
        const uint32_t mia = b.strA[ia], mja = b.strA[ja], mib = b.strB[ib], mjb = b.strB[jb];
        const int da = __popc(mia ^ mja), db = __popc(mib ^ mjb);
        double x = 0.0;
        if (da <= 2 && db <= 2) {
            const double *e = prm + pl.off_eri;
            const int P = da ? single_pair(mia, mja) : 0, Q = db ? single_pair(mib, mjb) : 0;
            if (da && db) {
                x = e[P * pl.Kpad + Q];
            } else if (da) {
                for (uint32_t y = mib; y; y &= y - 1) {
                    const int q = __ffs(y) - 1;
                    x += e[P * pl.Kpad + q * (q + 3) / 2];
                }
            } else {
                for (uint32_t z = mia; z; z &= z - 1) {
                    const int p = __ffs(z) - 1;
                    const double *ep = e + p * (p + 3) / 2 * pl.Kpad;
                    if (db) x += ep[Q];
                    else
                        for (uint32_t y = mib; y; y &= y - 1) {
                            const int q = __ffs(y) - 1;
                            x += ep[q * (q + 3) / 2];
                        }
                }
            }
            if (da) x *= excitation_sign(mia, mja);
            if (db) x *= excitation_sign(mib, mjb);
        }
        v += 2.0 * x;   // stored as 1/2 (P|Q)
        if (b.sym_shift != 0.0 && I == J) v += sym_pen(b, t, b.strA[ia], b.strB[ib]);
        if (b.spin_shift != 0.0) {
            if (I == J) {
                v += b.spin_shift * (double)(b.nb - __popc(mia & mib));
            } else {
                const uint32_t xa = mia ^ mja, xb = mib ^ mjb;
                if (da == 2 && db == 2 && (mia & xa) == (mjb & xb) && (mja & xa) == (mib & xb))
                    v -= b.spin_shift * excitation_sign(mia, mja) * excitation_sign(mib, mjb);
            }
        }
        H[i * kPsp + j] = v;
        H[j * kPsp + i] = v;
    }
}

// Factorisation of H_PP = Q T Q^T (T tridiagonal) and the lowest eigenvector
// y of H_PP, one block per tuple, n <= NP determinants.
//
// n^3 operations in a chain of n - 2 reflections: bound by the latency of one
// workgroup's steps, so the matrix stays in registers, a 4 x 4 patch per
// thread (all of it, both triangles), and a step is three barriers: the
// column's wave makes the reflector (sums and broadcasts on the vector ALU)
// and leaves it in LDS, where it stays; the partial products A v of the waves;
// their sums and v . A v.  Waves whose columns are finished only keep the
// barriers.  The steps are unrolled by four, so that a column's place in the
// patches is a constant.  Q = H_0 ... H_{n-3} is then accumulated backwards,
// column by column without barriers (16 rows per lane, NP / 16 lanes per
// column), the rows above each reflector left out.  NP = 32, 64 and 128 (64,
// 256 and 1024 threads) keep small P spaces from paying for the large one's
// barriers.
// Meanwhile the first wave finds the lowest eigenvalue of T by multisection on
// the leading minors (one point per lane and round), its vector from the
// twisted factorisation at that eigenvalue (Fernando; Dhillon and Parlett):
// pivots downwards and upwards by two lanes, joined at the row of the smallest
// |gamma|.
// At 128 determinants 170-211 us a launch (up to one tuple per CU), 73 us at
// 64, 38-43 us at 32; 315-406, 103 and 58-68 us with the reflector made by
// every wave for itself from a column in LDS, a branch per patch element, and
// the eigenvalue found by all threads before Q; 1050 us and 190 us with the
// matrix in LDS and nine barriers a step.  Of the 128-determinant launch the
// reflections take 145 us, Q 24 us.
template <int N> __device__ __forceinline__ double dpp_move(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), N, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), N, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

template <int NP> struct PspFactor {
    static constexpr int G = NP / 4;          // patches per side
    static constexpr int NT = G * G;          // threads
    static constexpr int NW = NT / 64;
    static constexpr int LPC = NP / 16;       // lanes per column of Q
    static constexpr size_t lds = sizeof(double) * ((size_t)NP * NP + (size_t)NW * NP + 9 * (size_t)NP + 8);
    static constexpr int CW = 4 * 64 / G;     // columns per wave
};

template <int NP>
__global__ __launch_bounds__(PspFactor<NP>::NT) void k_psp_factor(Batch b) {
    constexpr int G = PspFactor<NP>::G, NT = PspFactor<NP>::NT, NW = PspFactor<NP>::NW, LPC = PspFactor<NP>::LPC,
                  CW = PspFactor<NP>::CW;
    const int t = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, n = b.psp;
    const int r = tid % G, c = tid / G;
    extern __shared__ __attribute__((aligned(16))) double lds[];
    double *V = lds;                    // [NP][NP] reflectors
    double *part = V + NP * NP;         // [NW][NP] the waves' shares of A v
    double *x = part + NW * NP;         // [2][NP]
    double *p = x + 2 * NP;             // [NP] A v
    double *sd = p + NP, *se = sd + NP; // [NP] T
    double *pu = se + NP, *pl = pu + NP;   // [NP] pivots downwards and upwards, then e / pivot
    double *z = pl + NP;                // [NP] eigenvector of T
    double *sh = z + NP;                // [2] shares of v . A v
    double *gQ = b.pQ + (int64_t)t * kPsp * kPsp;
    double *dT = b.pT + (int64_t)t * 3 * kPsp, *eT = dT + kPsp, *yv = eT + kPsp;
    double a[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            a[i][j] = (4 * r + i < n && 4 * c + j < n) ? gQ[(4 * r + i) * kPsp + 4 * c + j] : 0.0;
    for (int i = tid; i < NP; i += NT) se[i] = 0.0;
    for (int i = tid; i < NW * NP; i += NT) part[i] = 0.0;
    if (tid < 2) sh[tid] = 0.0;
    __syncthreads();
    const int wc0 = wv * CW;   // the wave's first column
    for (int kb = 0; 4 * kb + 2 < n; ++kb) {
#pragma unroll
        for (int kj = 0; kj < 4; ++kj) {   // (unrolled: the column's place in the patches is a constant)
            const int k = 4 * kb + kj;
            if (k + 2 >= n) break;
            double *vk = V + k * NP;
            if (wv == k / CW) {   // the column's wave makes the reflector
                double xi[4], s2 = 0.0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    xi[i] = 4 * r + i > k ? a[i][kj] : 0.0;
                    s2 = fma(xi[i], xi[i], s2);
                }
                if (G == 8) {
                    s2 += dpp_move<0xB1>(s2);
                    s2 += dpp_move<0x4E>(s2);
                    s2 += dpp_move<0x141>(s2);
                } else {
                    s2 = sum_row16(s2);
                    if (G == 32) s2 = add_row16(s2);
                }
                const double xs = xi[(kj + 1) & 3];
                const int l0 = (kb * G & 63) + kb + (kj == 3);   // row k + 1 of the column
                const double x0 = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(xs), l0),
                                                   __builtin_amdgcn_readlane(__double2loint(xs), l0));
                // a column already reduced has no reflection (v = 0)
                const bool red = !(s2 > 1e-300);
                const double nx = s2 * fast_rsq(s2), alpha = x0 > 0.0 ? -nx : nx;
                const double inv = red ? 0.0 : fast_rsq(2.0 * fma(-x0, alpha, s2));
                if (c == kb) {
                    dbl2v *o = reinterpret_cast<dbl2v *>(vk + 4 * r);
                    double v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = red ? 0.0 : (4 * r + i == k + 1 ? x0 - alpha : xi[i]) * inv;
                    o[0] = dbl2v{v[0], v[1]};
                    o[1] = dbl2v{v[2], v[3]};
                    if (r == 0) se[k] = red ? x0 : alpha;
                }
            }
            __syncthreads();
            const bool act = wc0 + CW > k + 1;   // (columns up to k are finished)
            double vr[4], vc[4];
            if (act) {
                const dbl2v *qr = reinterpret_cast<const dbl2v *>(vk + 4 * r);
                const dbl2v *qc = reinterpret_cast<const dbl2v *>(vk + 4 * c);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const dbl2v u = qr[i], w = qc[i];
                    vr[2 * i] = u.x;
                    vr[2 * i + 1] = u.y;
                    vc[2 * i] = w.x;
                    vc[2 * i + 1] = w.y;
                }
                double pr[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    double q = a[i][0] * vc[0];
                    q = fma(a[i][1], vc[1], q);
                    q = fma(a[i][2], vc[2], q);
                    q = fma(a[i][3], vc[3], q);
                    if (G == 8) q += row_ror<8>(q);
                    if (G <= 16) q = add_row16(q);
                    pr[i] = add_row32(q);
                }
                if (lane < G) {
                    dbl2v *o = reinterpret_cast<dbl2v *>(part + wv * NP + 4 * r);
                    o[0] = dbl2v{pr[0], pr[1]};
                    o[1] = dbl2v{pr[2], pr[3]};
                }
            } else if (wc0 + CW == k + 1 && lane < G) {   // no share any more
                dbl2v *o = reinterpret_cast<dbl2v *>(part + wv * NP + 4 * r);
                o[0] = o[1] = dbl2v{0.0, 0.0};
            }
            __syncthreads();
            if (tid < (NP > 64 ? NP : 64)) {
                double K = 0.0;
                if (NP >= 64 || tid < NP) {
                    double q[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int w = 0; w < NW; ++w) q[w & 3] += part[w * NP + tid];
                    const double pi = (q[0] + q[1]) + (q[2] + q[3]);
                    p[tid] = pi;
                    K = vk[tid] * pi;
                }
                K = sum_wave(K);
                if (lane == 0) sh[wv] = K;
            }
            __syncthreads();
            if (act) {
                const double K = NP > 64 ? sh[0] + sh[1] : sh[0];
                const dbl2v *qr = reinterpret_cast<const dbl2v *>(p + 4 * r);
                const dbl2v *qc = reinterpret_cast<const dbl2v *>(p + 4 * c);
                double wr[4], wc[4];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const dbl2v u = qr[i], w = qc[i];
                    wr[2 * i] = 2.0 * fma(-K, vr[2 * i], u.x);
                    wr[2 * i + 1] = 2.0 * fma(-K, vr[2 * i + 1], u.y);
                    wc[2 * i] = 2.0 * fma(-K, vc[2 * i], w.x);
                    wc[2 * i + 1] = 2.0 * fma(-K, vc[2 * i + 1], w.y);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) a[i][j] = fma(-vr[i], wc[j], fma(-wr[i], vc[j], a[i][j]));
            }
        }
    }
    if (r == c) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sd[4 * r + i] = a[i][i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (4 * r + i == n - 1 && 4 * c + j == n - 2) se[n - 2] = a[i][j];
    __syncthreads();
    for (int i = tid; i < n; i += NT) {
        dT[i] = sd[i];
        eT[i] = se[i];
    }
    // The lowest eigenpair of T by the first wave (the others go on to Q):
    // Gershgorin bounds, multisection, twisted factorisation.  The chains
    // read their operands eight steps at a time, ahead of the arithmetic.
    if (tid < 64) {
        __builtin_amdgcn_s_setprio(3);
        double lo = 1e300, hi = -1e300;
        for (int i = lane; i < n; i += 64) {
            const double q = (i > 0 ? fabs(se[i - 1]) : 0.0) + fabs(se[i]);
            lo = fmin(lo, sd[i] - q);
            hi = fmax(hi, sd[i] + q);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo = fmin(lo, __shfl_xor(lo, o, 64));
            hi = fmax(hi, __shfl_xor(hi, o, 64));
        }
        // T in units of scale (p: diagonal, x: subdiagonal, x2: its square,
        // one row later); the rows past n decouple, above the spectrum
        double *x2 = x + NP;
        const double scale = fmax(hi - lo + fabs(lo), 1e-30);
        lo /= scale;
        hi /= scale;
        for (int i = lane; i < NP; i += 64) {
            p[i] = i < n ? sd[i] / scale : lo + 2.0;
            x[i] = i + 1 < n ? se[i] / scale : 0.0;
            const double em = i > 0 && i < n ? se[i - 1] / scale : 0.0;
            x2[i] = em * em;
        }
        wave_sync();
        for (int round = 0; round < 10 && hi - lo > 2e-16; ++round) {
            const double y = lo + (hi - lo) * ((lane + 1) / 65.0);
            // T - y is positive definite iff every leading minor is positive; the
            // pair of minors is scaled back every eight rows
            double p0 = 0.0, p1 = 1.0;
            int neg = 0;   // sign bits
            for (int i0 = 0; i0 < n; i0 += 8) {
                double dd[8], ee[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    dd[u] = p[i0 + u];
                    ee[u] = x2[i0 + u];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const double p2 = fma(dd[u] - y, p1, -ee[u] * p0);
                    p0 = p1;
                    p1 = p2;
                    neg |= __double2hiint(p2);
                }
                const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
                p0 = __builtin_amdgcn_ldexp(p0, ex);
                p1 = __builtin_amdgcn_ldexp(p1, ex);
            }
            const int idx = __popcll(__ballot(neg >= 0));   // points below the lowest eigenvalue
            const double nlo = idx > 0 ? lo + (hi - lo) * (idx / 65.0) : lo;
            const double nhi = idx < 64 ? lo + (hi - lo) * ((idx + 1) / 65.0) : hi;
            lo = nlo;
            hi = nhi;
        }
        // twisted factorisation of T - lo
        auto keep = [](double q) { return fabs(q) < 1e-18 ? (q >= 0.0 ? 1e-18 : -1e-18) : q; };
        if (lane < 2) {
            // lane 0: pu_i = d_i - e_{i-1}^2 / pu_{i-1}; lane 1: pl_i = d_i - e_i^2 / pl_{i+1}
            const int st = lane ? -1 : 1, i0 = lane ? n - 1 : 0;
            double *out = lane ? pl : pu;
            double q = keep(p[i0] - lo);
            out[i0] = q;
            for (int s0 = 1; s0 < n; s0 += 8) {
                double dd[8], ee[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int i = i0 + st * min(s0 + u, n - 1);
                    dd[u] = p[i] - lo;
                    ee[u] = x2[i + lane];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    q = keep(fma(-ee[u], fast_rcp(q), dd[u]));
                    if (s0 + u < n) out[i0 + st * (s0 + u)] = q;
                }
            }
        }
        wave_sync();
        double best = 1e300;
        int kb = 0;
        for (int i = lane; i < n; i += 64) {
            const double gam = fabs(pu[i] + pl[i] - (p[i] - lo));
            if (gam < best) {
                best = gam;
                kb = i;
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double q = __shfl_xor(best, o, 64);
            const int kq = __shfl_xor(kb, o, 64);
            if (q < best || (q == best && kq < kb)) {
                best = q;
                kb = kq;
            }
        }
        wave_sync();
        // reciprocals, and multipliers towards the ends (x2: downwards pivots, pl: upwards)
        for (int i = lane; i < n; i += 64) {
            pu[i] = fast_rcp(pu[i]);
            x2[i] = -x[i] * pu[i];
            pl[i] = i > 0 ? -x[i - 1] * fast_rcp(pl[i]) : 0.0;
        }
        wave_sync();
        if (lane < 2) {   // lane 0: rows above kb, upwards; lane 1: rows below, downwards
            const int st = lane ? 1 : -1, len = lane ? n - 1 - kb : kb, top = max(kb, n - 1 - kb);
            const double *f = lane ? pl : x2;
            double q = 1.0;
            if (lane == 0) z[kb] = q;
            for (int s0 = 1; s0 <= top; s0 += 8) {
                double ff[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) ff[u] = f[kb + st * min(s0 + u, len)];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    q *= ff[u];
                    if (s0 + u <= len) z[kb + st * (s0 + u)] = q;
                }
            }
        }
        wave_sync();
        // one step of inverse iteration on it: the twisted vector still holds
        // the other eigenvectors to |lambda - lo| / gap
        if (lane == 0) {
            double q = 0.0;
            for (int i0 = 0; i0 < n; i0 += 8) {   // (1 - x2 S) z, scaled by the pivots
                double ff[8], zz[8], rr[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int i = min(i0 + u, n - 1);
                    ff[u] = i > 0 ? x2[i - 1] : 0.0;
                    zz[u] = z[i];
                    rr[u] = pu[i];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    q = fma(ff[u], q, zz[u]);
                    if (i0 + u < n) z[i0 + u] = q * rr[u];
                }
            }
            q = 0.0;
            for (int s0 = 0; s0 < n; s0 += 8) {
                double ff[8], zz[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int i = max(n - 1 - s0 - u, 0);
                    ff[u] = x2[i];
                    zz[u] = z[i];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    q = fma(ff[u], q, zz[u]);
                    if (s0 + u < n) z[n - 1 - s0 - u] = q;
                }
            }
        }
        wave_sync();
        double big = 0.0;
        for (int i = lane; i < n; i += 64) big = fmax(big, fabs(z[i]));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o, 64));
        // the sign is fixed (positive sum in T's basis): the admixture of the
        // guess has one of its own
        double zs = 0.0;
        for (int i = lane; i < n; i += 64) zs += z[i] / big;
        const double sb = sum_wave(zs) < 0.0 ? -1.0 / big : 1.0 / big;
        for (int i = lane; i < n; i += 64) z[i] *= sb;
        double nz = 0.0;
        for (int i = lane; i < n; i += 64) nz += z[i] * z[i];
        nz = 1.0 / sqrt(sum_wave(nz));
        for (int i = lane; i < n; i += 64) z[i] *= nz;
        __builtin_amdgcn_s_setprio(0);
    }
    // Q, column cq: H_k applied for k = n - 3 .. 0 to the unit vector; lane j
    // of the column's LPC lanes holds the row pairs 2 (j + LPC m), 2 (j + LPC m) + 1
    const int cq = tid / LPC, j = tid % LPC;
    double q0[8], q1[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        q0[m] = 2 * (j + LPC * m) == cq ? 1.0 : 0.0;
        q1[m] = 2 * (j + LPC * m) + 1 == cq ? 1.0 : 0.0;
    }
    // (columns up to k of the product are still unit vectors orthogonal to v_k)
    const int ctop = ((wv << 6) + 63) / LPC;   // the wave's last column
    // (v_k is zero up to row k: the rows go in eight chunks, those of the
    // reflections of one range of k start at chunk MB)
    auto apply = [&](auto mb) {
        constexpr int MB = decltype(mb)::value, CH = 2 * LPC;
        for (int k = min(min(n - 3, ctop - 1), (MB + 1) * CH - 2); k >= 0 && k >= MB * CH - 1; --k) {
            const dbl2v *v = reinterpret_cast<const dbl2v *>(V + k * NP) + j;
            dbl2v vv[8];
            double s = 0.0, s1 = 0.0;
#pragma unroll
            for (int m = MB; m < 8; ++m) {
                vv[m] = v[LPC * m];
                s = fma(vv[m].x, q0[m], s);
                s1 = fma(vv[m].y, q1[m], s1);
            }
            s += s1;
            s += dpp_move<0xB1>(s);                    // lane ^ 1
            if (LPC >= 4) s += dpp_move<0x4E>(s);      // lane ^ 2
            if (LPC >= 8) s += dpp_move<0x141>(s);     // the other half of eight lanes
            s *= -2.0;
#pragma unroll
            for (int m = MB; m < 8; ++m) {
                q0[m] = fma(s, vv[m].x, q0[m]);
                q1[m] = fma(s, vv[m].y, q1[m]);
            }
        }
    };
    apply(std::integral_constant<int, 7>{});
    apply(std::integral_constant<int, 6>{});
    apply(std::integral_constant<int, 5>{});
    apply(std::integral_constant<int, 4>{});
    apply(std::integral_constant<int, 3>{});
    apply(std::integral_constant<int, 2>{});
    apply(std::integral_constant<int, 1>{});
    apply(std::integral_constant<int, 0>{});
    double *gQt = b.pQt + (int64_t)t * kPsp * kPsp;
    if (cq < n) {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int i = 2 * (j + LPC * m);
            if (i < n) {
                gQ[i * kPsp + cq] = q0[m];
                gQt[cq * kPsp + i] = q0[m];
            }
            if (i + 1 < n) {
                gQ[(i + 1) * kPsp + cq] = q1[m];
                gQt[cq * kPsp + i + 1] = q1[m];
            }
        }
    }
    __syncthreads();   // z complete, V no longer read
    // y = Q z: every column's lanes leave z_c Q[:, c] in V (row i, column c), summed by rows
    const double zc = cq < n ? z[cq] : 0.0;
    constexpr int LD = NP + 1;
    static_assert((size_t)NP * LD <= (size_t)NP * NP + PspFactor<NP>::NW * NP, "y sums");
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const int i = 2 * (j + LPC * m);
        V[cq * LD + i] = zc * q0[m];
        V[cq * LD + i + 1] = zc * q1[m];
    }
    __syncthreads();
    for (int i = tid; i < n; i += NT) {
        double s = 0.0;
#pragma unroll 8
        for (int q = 0; q < n; ++q) s += V[q * LD + i];
        yv[i] = s;
    }
}

template <int NP> static void launch_psp_factor(const Batch &b, hipStream_t s) {
    hipLaunchKernelGGL(k_psp_factor<NP>, dim3(b.B), dim3(PspFactor<NP>::NT), PspFactor<NP>::lds, s, b);
}

hipError_t launch_pspace(const Batch &b, hipStream_t s) {
    if (b.psp <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_psp_select, dim3(b.B), dim3(1024), 0, s, b);
    const int per = b.B > 64 ? 2048 : 512;   // elements per block: one block per CU or so for few tuples
    hipLaunchKernelGGL(k_psp_build, dim3(b.B, (b.psp * b.psp + per - 1) / per), dim3(256), 0, s, b);
    if (b.psp <= 32) launch_psp_factor<32>(b, s);
    else if (b.psp <= 64) launch_psp_factor<64>(b, s);
    else launch_psp_factor<128>(b, s);
    return hipGetLastError();
}

// V_0 += lowest eigenvector of H_PP on the P determinants; the change of
// |V_0|^2 into the extra partial block.
__global__ __launch_bounds__(kPsp) void k_psp_guess(Batch b) {
    const int t = blockIdx.x, i = threadIdx.x, n = b.psp;
    double *v0 = b.V + (int64_t)t * b.max_space * b.dim;
    const double *yv = b.pT + (int64_t)t * 3 * kPsp + 2 * kPsp;
    double dn = 0.0;
    if (i < n) {
        const int64_t d = b.pidx[(int64_t)t * kPsp + i];
        const double o = v0[d], nv = o + yv[i];
        v0[d] = nv;
        dn = nv * nv - o * o;
    }
    __shared__ double sh[2];
    dn = wave_sum(dn);
    if ((i & 63) == 0) sh[i >> 6] = dn;
    __syncthreads();
    if (i == 0) {
        double *px = parts(b, t, b.nblk);
        px[0] = sh[0] + (kPsp > 64 ? sh[1] : 0.0);
    }
}

__device__ __forceinline__ double guess_noise(int64_t d) {
    uint64_t z = (uint64_t)d + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

// block-local minimum of Hd: value and index into partials 0 and 1
__global__ __launch_bounds__(256) void k_guess_min(Batch b) {
    const int t = blockIdx.y;
    const double *hd = b.Hd + (int64_t)t * b.dim;
    double best = 1e300;
    int64_t bi = INT64_MAX;
    for (int64_t d = (int64_t)blockIdx.x * 256 + threadIdx.x; d < b.dim; d += (int64_t)gridDim.x * 256) {
        const double v = hd[d];
        if (v < best || (v == best && d < bi)) { best = v; bi = d; }
    }
    __shared__ double sv[256];
    __shared__ int64_t si[256];
    sv[threadIdx.x] = best;
    si[threadIdx.x] = bi;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            const double v2 = sv[threadIdx.x + o];
            const int64_t i2 = si[threadIdx.x + o];
            if (v2 < sv[threadIdx.x] || (v2 == sv[threadIdx.x] && i2 < si[threadIdx.x])) {
                sv[threadIdx.x] = v2;
                si[threadIdx.x] = i2;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        parts(b, t, blockIdx.x)[0] = sv[0];
        parts(b, t, blockIdx.x)[1] = (double)si[0];
    }
}

__global__ void k_guess_pick(Batch b) {
    const int t = blockIdx.x;
    if (threadIdx.x != 0) return;
    double best = 1e300, bi = 1e300;
    for (int blk = 0; blk < b.nblk; ++blk) {
        const double v = parts(b, t, blk)[0], i = parts(b, t, blk)[1];
        if (v < best || (v == best && i < bi)) { best = v; bi = i; }
    }
    b.coef[(int64_t)t * kMaxSpace] = bi;
}

// V_0 = e_imin + 1e-3 * noise(d) (with a P space: the noise alone, the P
// eigenvector follows), partial norm^2
__global__ __launch_bounds__(256) void k_guess_fill(Batch b) {
    const int t = blockIdx.y;
    const int64_t imin = b.psp <= 0 ? (int64_t)b.coef[(int64_t)t * kMaxSpace] : -1;
    double *v0 = b.V + (int64_t)t * b.max_space * b.dim;
    // a P space that is the whole space gives the exact eigenvector: no admixture
    const double amp = (b.psp > 0 && b.psp >= b.dim) ? 0.0 : 1e-3;
    double acc[kParts];
    acc[0] = 0.0;
    for (int64_t d = (int64_t)blockIdx.x * 256 + threadIdx.x; d < b.dim; d += (int64_t)gridDim.x * 256) {
        const double v = (d == imin ? 1.0 : 0.0) + amp * guess_noise(d);
        v0[d] = v;
        acc[0] += v * v;
    }
    store_block_partials(b, t, acc, 1);
}

__global__ void k_guess_norm(Batch b) {
    const int t = blockIdx.x;
    if (threadIdx.x == 0) b.coef[(int64_t)t * kMaxSpace] = 1.0 / sqrt(sum_parts_x(b, t, 0));
}

__global__ __launch_bounds__(256) void k_scale_v0(Batch b) {
    const int t = blockIdx.y;
    const double s = b.coef[(int64_t)t * kMaxSpace];
    double *v0 = b.V + (int64_t)t * b.max_space * b.dim;
    for (int64_t d = (int64_t)blockIdx.x * 256 + threadIdx.x; d < b.dim; d += (int64_t)gridDim.x * 256)
        v0[d] *= s;
}

// The whole guess with a P space, one workgroup per tuple: admixture, P
// eigenvector, norm, scaling.  One launch instead of four for spaces that a
// workgroup passes over in a few steps (each launch costs a small class about
// 4 us; the passes of kGuessOne determinants take that long).
constexpr int64_t kGuessOne = 16384;

__global__ __launch_bounds__(1024) void k_guess_one(Batch b) {
    const int t = blockIdx.x, tid = threadIdx.x;
    __shared__ double sh[16];
    double *v0 = b.V + (int64_t)t * b.max_space * b.dim;
    const double *yv = b.pT + (int64_t)t * 3 * kPsp + 2 * kPsp;
    const double amp = b.psp >= b.dim ? 0.0 : 1e-3;   // (as in k_guess_fill)
    double acc = 0.0;
    for (int64_t d = tid; d < b.dim; d += 1024) {
        const double v = amp * guess_noise(d);
        v0[d] = v;
        acc += v * v;
    }
    __syncthreads();
    if (tid < b.psp) {
        const int64_t d = b.pidx[(int64_t)t * kPsp + tid];
        const double o = v0[d], nv = o + yv[tid];
        v0[d] = nv;
        acc += nv * nv - o * o;
    }
    const double s = 1.0 / sqrt(block_sum(acc, sh));
    __syncthreads();
    for (int64_t d = tid; d < b.dim; d += 1024) v0[d] *= s;
}

hipError_t launch_guess(const Batch &b, hipStream_t s) {
    if (b.psp > 0 && b.dim <= kGuessOne) {
        hipLaunchKernelGGL(k_guess_one, dim3(b.B), dim3(1024), 0, s, b);
        return hipGetLastError();
    }
    dim3 grid(b.nblk, b.B);
    if (b.psp <= 0) {   // the determinant of lowest diagonal (with a P space its eigenvector instead)
        hipLaunchKernelGGL(k_guess_min, grid, dim3(256), 0, s, b);
        hipLaunchKernelGGL(k_guess_pick, dim3(b.B), dim3(64), 0, s, b);
    }
    hipLaunchKernelGGL(k_guess_fill, grid, dim3(256), 0, s, b);
    if (b.psp > 0) hipLaunchKernelGGL(k_psp_guess, dim3(b.B), dim3(kPsp), 0, s, b);
    hipLaunchKernelGGL(k_guess_norm, dim3(b.B), dim3(64), 0, s, b);
    hipLaunchKernelGGL(k_scale_v0, grid, dim3(256), 0, s, b);
    return hipGetLastError();
}

__global__ void k_init_state(Batch b) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= b.B) return;
    b.status[t] = ST_RUNNING;
    b.m[t] = 0;              // V_0 holds the guess; its sigma follows, then m = 1
    b.iter[t] = 0;
    b.restart[t] = 0;
    b.theta[t] = 0.0;
    b.theta_prev[t] = 1e300;
    b.R[(int64_t)t * kMaxSpace * kMaxSpace] = 1.0;   // V_0 is normalised: Q_0 = V_0
    double *zp = b.zp + (int64_t)t * kMaxSpace;
    for (int i = 0; i < kMaxSpace; ++i) zp[i] = i == 0 ? 1.0 : 0.0;
    b.run[t] = t;
    if (t == 0) {
        b.counter[0] = b.B;
        b.counter[2] = 0;   // explicit Gram-Schmidt passes of the batch
    }
}

hipError_t launch_init_state(const Batch &b, hipStream_t s) {
    hipLaunchKernelGGL(k_init_state, dim3((b.B + 255) / 256), dim3(256), 0, s, b);
    return hipGetLastError();
}

// partial dots V_i . y for i <= m[t] (running tuples only)
template <int MS>
__global__ __launch_bounds__(256) void k_dots(Batch b, VecRef yref) {
    const int t = blockIdx.y;
    if (b.status[t] != ST_RUNNING) return;
    const int nx = b.m[t] + 1;
    const double *V = b.V + (int64_t)t * b.max_space * b.dim;
    const double *y = vref(yref, t, b.dim);
    double acc[MS + 1];
#pragma unroll
    for (int i = 0; i < MS + 1; ++i) acc[i] = 0.0;
    for (int64_t d = (int64_t)blockIdx.x * 256 + threadIdx.x; d < b.dim; d += (int64_t)gridDim.x * 256) {
        const double yv = y[d];
#pragma unroll
        for (int i = 0; i < MS + 1; ++i)
            if (i < nx) acc[i] += V[(int64_t)i * b.dim + d] * yv;
    }
    store_block_partials<MS + 1>(b, t, acc, nx);
}

hipError_t launch_dots(const Batch &b, VecRef y, hipStream_t s) {
    if (b.max_space <= 12) hipLaunchKernelGGL(k_dots<12>, dim3(b.nblk, b.B), dim3(256), 0, s, b, y);
    else hipLaunchKernelGGL(k_dots<kMaxSpace>, dim3(b.nblk, b.B), dim3(256), 0, s, b, y);
    return hipGetLastError();
}

constexpr int kNormPart = kParts - 1;   // partial column of |T|^2 after the explicit passes (k_cgs)

// Start of an iteration, one wave per tuple: the projected matrix gains the
// column of the vector whose sigma was formed last, and its lowest eigenpair
// gives the Ritz vector's coefficients.
//
// b.G holds the projection B = R^T (V^T H V) R on the orthonormal basis Q =
// V R.  With g_i = V_i . S_m (partial blocks 0 .. nsum-1; with `sd` the
// entries i < gemm_dot_first from the S-dots of k_ritz instead), c and s of
// k_step (column m of R is (-R c, 1) s; c = 0 after the explicit passes):
//   B_im = s ((R^T g)_i - (B c)_i),  B_mm = s^2 (c . B c - 2 c . R^T g + g_m).
// Block 0 also clears the iteration's counters (running tuples, explicit
// Gram-Schmidt passes), which k_step counts after it: no
// memset node in the iteration's launches.
template <int MS>
__global__ __launch_bounds__(64) void k_small_eig(Batch b, int nsum, int sd) {
    const int t = blockIdx.x, lane = threadIdx.x;
    if (t == 0 && lane < 2) b.counter[lane] = 0;
    const int32_t st0 = b.status[t];
    if (st0 != ST_RUNNING && st0 != ST_RESTART) return;
    __shared__ SmallEig<MS> q;
    __shared__ double B[kMaxSpace][kMaxSpace + 1], R[kMaxSpace][kMaxSpace + 1];
    __shared__ double gv[kMaxSpace], cv[kMaxSpace], wv[kMaxSpace];
    constexpr int IW = SmallEig<MS>::IW;
    double *Gg = b.G + (int64_t)t * kMaxSpace * kMaxSpace;
    const double *Rg = b.R + (int64_t)t * kMaxSpace * kMaxSpace;
    int m = b.m[t];
    bool grow = st0 == ST_RUNNING;   // the basis has a new vector, V_m
    const bool two = grow && m > 0 && b.cgs2[t];
    double sn = 0.0;   // after the explicit passes: 1 / |V_m|
    if (two) {
        // A correction that lies inside the subspace (its projection kept less
        // than 1e-8 of its norm) adds nothing: the Ritz pair is converged if
        // the residual is below r_tol (an invariant subspace, e.g. a
        // one-determinant space); otherwise the tuple restarts from its Ritz
        // vector now, or has stalled when the subspace already is that one
        // vector.
        double x = 0.0;
        for (int blk = lane; blk < b.nblk; blk += 64) x += parts(b, t, blk)[kNormPart];
        const double tn = sqrt(sum_wave(x));
        if (!(tn > 1e-8 * b.tnorm0[t]) || !(tn > 1e-300) || m >= b.max_space) {
            if (b.rnorm[t] < b.r_tol || m <= 1) {
                if (lane == 0) b.status[t] = b.rnorm[t] < b.r_tol ? ST_DONE : ST_STALLED;
                return;
            }
            grow = false;
        }
        sn = 1.0 / tn;
    }
    const int n = grow ? m + 1 : m;   // columns of the basis
    for (int k = lane; k < n * IW; k += 64) {
        const int r = k / IW, c = k & (IW - 1);
        if (c < m && r < m) B[r][c] = Gg[r * kMaxSpace + c];
        if (c < n && r <= c) R[r][c] = two && c == m ? (r == m ? sn : 0.0) : Rg[r * kMaxSpace + c];
    }
    if (grow) {
        const int i0 = sd ? gemm_dot_first(b, t, m) : 0;
        if (two && lane <= m) b.R[(int64_t)t * kMaxSpace * kMaxSpace + lane * kMaxSpace + m] = lane == m ? sn : 0.0;
        if (lane < i0) gv[lane] = b.sdot[(int64_t)t * kMaxSpace + lane];
        for (int c = i0; c <= m; ++c) {
            double x = 0.0;
            for (int blk = lane; blk < nsum; blk += 64) x += parts(b, t, blk)[c];
            x = wave_sum(x);
            if (lane == 0) gv[c] = x;
        }
        if (lane < m) cv[lane] = two ? 0.0 : b.coef[(int64_t)t * kMaxSpace + lane];
        wave_sync();
        const double s = R[m][m];
        double rg = 0.0, bc = 0.0;
        if (lane < m) {
            for (int j = 0; j <= lane; ++j) rg += R[j][lane] * gv[j];
            for (int j = 0; j < m; ++j) bc += B[lane][j] * cv[j];
        }
        const double cc = wave_sum(lane < m ? cv[lane] * (bc - 2.0 * rg) : 0.0);
        wave_sync();
        const double v = lane < m ? s * (rg - bc) : s * s * (cc + gv[m]);
        if (lane <= m) {
            B[lane][m] = B[m][lane] = v;
            Gg[lane * kMaxSpace + m] = Gg[m * kMaxSpace + lane] = v;
        }
        ++m;
        if (lane == 0) b.m[t] = m;
    } else if (st0 == ST_RESTART && lane == 0) {
        b.status[t] = ST_RUNNING;
    }
    wave_sync();
    for (int k = lane; k < m * IW; k += 64) {
        const int r = k / IW, c = k & (IW - 1);
        if (c < m) q.A[r][c] = B[r][c];
    }
    wave_sync();
    double z;
    const double th = lowest_eig<MS>(q, m, z);
    // coefficients R z on the stored basis
    if (lane < m) gv[lane] = z;
    wave_sync();
    if (lane < m) {
        double v = 0.0;
        for (int j = lane; j < m; ++j) v += R[lane][j] * gv[j];
        b.y[(int64_t)t * kMaxSpace + lane] = v;
    }
    // A restart keeps the Ritz vector and, with restart_keep 2, the previous
    // iteration's Ritz vector (zp, coordinates of Q, zero past its length)
    // made orthogonal to it by two passes in these coordinates; kept when that
    // leaves a norm above 1e-6.  Its coefficients on the stored basis are R w,
    // its Rayleigh quotient w . B w.  The two are orthonormal and the projected
    // matrix on them is diag(theta, mu).
    const bool rs = m >= b.max_space || !grow;
    double *zp = b.zp + (int64_t)t * kMaxSpace;
    const double zl = lane < m ? z : 0.0;
    int keep = rs ? 1 : 0;
    if (rs && b.restart_keep > 1) {
        double w = lane < m ? zp[lane] : 0.0;
        for (int pass = 0; pass < 2; ++pass) w -= wave_sum(zl * w) * zl;
        const double nw = wave_sum(w * w);
        if (nw > 1e-12) {
            w *= 1.0 / sqrt(nw);
            if (lane < m) wv[lane] = w;
            wave_sync();
            double bw = 0.0, y2 = 0.0;
            if (lane < m) {
                for (int j = 0; j < m; ++j) bw += B[lane][j] * wv[j];
                for (int j = lane; j < m; ++j) y2 += R[lane][j] * wv[j];
                b.y2[(int64_t)t * kMaxSpace + lane] = y2;
            }
            const double mu = wave_sum(w * bw);
            if (lane == 0) b.mu[t] = mu;
            keep = 2;
        }
    }
    if (!rs && lane < kMaxSpace) zp[lane] = zl;
    if (lane == 0) {
        b.theta[t] = th;
        b.restart[t] = keep;
    }
}

template <int MS, bool V2, bool K2>
__device__ __forceinline__ void ritz_body(const Batch &b, int t, int m, int rs) {
    const double th = b.theta[t];
    const double *yv = b.y + (int64_t)t * kMaxSpace, *zv = b.y2 + (int64_t)t * kMaxSpace;
    double yy[MS], zz[MS];
#pragma unroll
    for (int i = 0; i < MS; ++i) {
        yy[i] = (i < m) ? yv[i] : 0.0;
        zz[i] = (K2 && i < m) ? zv[i] : 0.0;
    }
    double *V = b.V + (int64_t)t * b.max_space * b.dim;
    double *S = b.S + (int64_t)t * b.max_space * b.dim;
    const double *hd = b.Hd + (int64_t)t * b.dim;
    double *T = V + (int64_t)(rs ? rs : m) * b.dim;
    constexpr bool SD = MS <= kSdMax;
    constexpr int NACC = SD ? kSdOff + MS : 2 + MS;
    double acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = 0.0;
    // one determinant: Ritz vector, residual, preconditioned correction, its
    // projections on the basis and its dots with the basis' sigma vectors
    auto one = [&](const double (&vd)[MS], const double (&sd)[MS], double x, double ax, double x2, double a2,
                   double h) -> double {
        const double r = ax - th * x;
        acc[0] += r * r;
        double den = th - h;
        if (fabs(den) < 1e-8) den = (den >= 0.0) ? 1e-8 : -1e-8;
        const double tv = r / den;
        acc[1] += tv * tv;
        if (rs) {
            acc[2] += x * tv;
            if (SD) acc[kSdOff] += ax * tv;
            if (K2) {
                acc[3] += x2 * tv;
                if (SD) acc[kSdOff + 1] += a2 * tv;
            }
        } else {
            // (vd[i] = sd[i] = 0 for i >= m: those sums stay unused)
#pragma unroll
            for (int i = 0; i < MS; ++i) {
                acc[2 + i] += vd[i] * tv;
                if (SD) acc[kSdOff + i] += sd[i] * tv;
            }
        }
        return tv;
    };
    // V_i and S_i, i < m, through buffer resources that end after vector m - 1:
    // the loads of vectors past m read zero, so every load of a determinant is
    // issued at once (no branch on m between them); the added terms are
    // exact zeros (yy[i] = 0 there)
    const int vbytes = (int)((int64_t)m * b.dim * (int64_t)sizeof(double));
    const __amdgpu_buffer_rsrc_t rV = __builtin_amdgcn_make_buffer_rsrc(V, (short)0, vbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rS = __builtin_amdgcn_make_buffer_rsrc(S, (short)0, vbytes, 0x00020000);
    const uint32_t vstride = (uint32_t)b.dim * (uint32_t)sizeof(double);
    if (V2) {
        // pairs of determinants with 16-byte loads (dim even: every vector 16-byte aligned)
        typedef double dbl2 __attribute__((ext_vector_type(2)));
        const int64_t n2 = b.dim >> 1;
        for (int64_t d2 = (int64_t)blockIdx.x * 256 + threadIdx.x; d2 < n2; d2 += (int64_t)gridDim.x * 256) {
            const int64_t d = d2 << 1;
            const uint32_t vo = (uint32_t)d * (uint32_t)sizeof(double);
            double v0[MS], v1[MS], s0[MS], s1[MS];
            double x0 = 0.0, x1 = 0.0, a0 = 0.0, a1 = 0.0, z0 = 0.0, z1 = 0.0, c0 = 0.0, c1 = 0.0;
            dbl2 vv[MS], ss[MS];
#pragma unroll
            for (int i = 0; i < MS; ++i) {
                vv[i] = __builtin_bit_cast(dbl2, __builtin_amdgcn_raw_buffer_load_b128(rV, vo, (uint32_t)i * vstride, 0));
                ss[i] = __builtin_bit_cast(dbl2, __builtin_amdgcn_raw_buffer_load_b128(rS, vo, (uint32_t)i * vstride, 0));
            }
#pragma unroll
            for (int i = 0; i < MS; ++i) {
                v0[i] = vv[i].x;
                v1[i] = vv[i].y;
                s0[i] = ss[i].x;
                s1[i] = ss[i].y;
                x0 += yy[i] * vv[i].x;
                x1 += yy[i] * vv[i].y;
                a0 += yy[i] * ss[i].x;
                a1 += yy[i] * ss[i].y;
                if (K2) {
                    z0 += zz[i] * vv[i].x;
                    z1 += zz[i] * vv[i].y;
                    c0 += zz[i] * ss[i].x;
                    c1 += zz[i] * ss[i].y;
                }
            }
            const dbl2 h = *reinterpret_cast<const dbl2 *>(hd + d);
            const double t0 = one(v0, s0, x0, a0, z0, c0, h.x);
            const double t1 = one(v1, s1, x1, a1, z1, c1, h.y);
            *reinterpret_cast<dbl2 *>(T + d) = dbl2{t0, t1};
            if (rs) {
                *reinterpret_cast<dbl2 *>(V + d) = dbl2{x0, x1};
                *reinterpret_cast<dbl2 *>(S + d) = dbl2{a0, a1};
                if (K2) {
                    *reinterpret_cast<dbl2 *>(V + b.dim + d) = dbl2{z0, z1};
                    *reinterpret_cast<dbl2 *>(S + b.dim + d) = dbl2{c0, c1};
                }
            }
        }
    } else {
        for (int64_t d = (int64_t)blockIdx.x * 256 + threadIdx.x; d < b.dim; d += (int64_t)gridDim.x * 256) {
            const uint32_t vo = (uint32_t)d * (uint32_t)sizeof(double);
            double x = 0.0, ax = 0.0, x2 = 0.0, a2 = 0.0, vd[MS], sd[MS];
#pragma unroll
            for (int i = 0; i < MS; ++i) {
                vd[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rV, vo, (uint32_t)i * vstride, 0));
                sd[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rS, vo, (uint32_t)i * vstride, 0));
            }
#pragma unroll
            for (int i = 0; i < MS; ++i) {
                x += yy[i] * vd[i];
                ax += yy[i] * sd[i];
                if (K2) {
                    x2 += zz[i] * vd[i];
                    a2 += zz[i] * sd[i];
                }
            }
            T[d] = one(vd, sd, x, ax, x2, a2, hd[d]);
            if (rs) {
                V[d] = x;
                S[d] = ax;
                if (K2) {
                    V[b.dim + d] = x2;
                    S[b.dim + d] = a2;
                }
            }
        }
    }
    store_block_partials<NACC>(b, t, acc, (SD ? kSdOff : 2) + (rs ? rs : m));
}

// x = V y, Ax = S y, r = Ax - theta x, T = r / (theta - Hd) (clamped);
// partials |r|^2, |T|^2 and the projections V_i . T on the subspace the
// correction is added to (V_i, i < m, or on restart the kept vectors: x, and
// x2 = V y2 when restart = 2), and for MS <= kSdMax the dots S_i . T (Ax . T,
// A x2 . T on restart) from partial kSdOff.  T is stored as the next basis
// vector itself: V_m, or V_restart on restart, where V_0 <- x, S_0 <- Ax (and
// V_1 <- x2, S_1 <- A x2) in place (each thread owns its d and reads every
// vector there before it writes).
template <int MS, bool V2>
__global__ __launch_bounds__(256) void k_ritz(Batch b) {
    const int t = blockIdx.y;
    if (b.status[t] != ST_RUNNING) return;
    const int m = b.m[t], rs = b.restart[t];
    if (rs == 2) ritz_body<MS, V2, true>(b, t, m, rs);
    else ritz_body<MS, V2, false>(b, t, m, rs);
}

// After k_ritz, one block of 512 threads per tuple: the column sums of its
// partials, the P-space part of the correction, the convergence test, restart
// bookkeeping and the running count, and what becomes of the correction.
//
// P space: T on the P determinants <- (theta - H_PP)^-1 r_P = Q (theta - T)^-1
// Q^T r_P (tri_solve), with the changes of |T|^2, of the projections V_i . T
// (on restart the kept vectors' x . T and x2 . T) and of the dots S_i . T
// (Ax . T, A x2 . T) added to the sums.  T is the vector k_ritz wrote, V_m
// (V_restart on restart).
//
// The correction on the orthonormal basis: c = Q^T T = R^T d with d the
// projections V_i . T, and the norm outside the subspace, kept = |T|^2 -
// |c|^2.  When that keeps at least half of |T|^2 (Kahan's criterion for one
// classical Gram-Schmidt pass; the difference of squares is then accurate to a
// few ulps) T joins the basis unchanged: V = Q U gains the column (c,
// sqrt(kept)), so R = U^-1 gains (-R c, 1) / sqrt(kept), and no vector pass is
// needed.  Otherwise cgs2 is set, coef = R c (T - V R c is T's part outside
// the subspace) and the explicit passes follow.
//
// Every item is latency: 8 waves share the sums over blocks (16 lanes per
// column) and the two 128 x 128 products (32 rows each), and the tridiagonal
// solve takes log2 n steps.  Before, in three launches (128 threads, a serial
// solve, one lane per column sum): 52-63 us on the 24-orbital expansion's
// batches and up to 200 us at 200 blocks per tuple; now 10-20 us.
constexpr int kStepThreads = 512;

template <int MS>
__global__ __launch_bounds__(kStepThreads) void k_step(Batch b) {
    const int t = blockIdx.x, tid = threadIdx.x;
    if (b.status[t] != ST_RUNNING) return;
    const int m0 = b.m[t], rs = b.restart[t], nk = rs ? rs : m0;
    const double th = b.theta[t];
    constexpr bool SD = MS <= kSdMax;
    constexpr int NACC = SD ? kSdOff + MS : 2 + MS;
    constexpr int NPART = kStepThreads / kPsp;   // threads per P determinant
    __shared__ double sum[NACC], px[NACC], r[kPsp], w[kPsp], red[NPART][kPsp], red2[NPART][kPsp];
    __shared__ double wsum[NPART][2][MS], ssum[NPART][2][MS], nsum[2];
    __shared__ TriShared tri;
    // column sums, 16 lanes a column, in a fixed order
    for (int c = tid >> 4; c < NACC; c += kStepThreads / 16) {
        const int l = tid & 15, j = c < 2 ? -1 : (SD && c >= kSdOff ? c - kSdOff : c - 2);
        double x = 0.0;
        if (j < nk && !(SD && c < kSdOff && c >= 2 + MS))
            for (int blk = l; blk < b.nblk; blk += 16) x += parts(b, t, blk)[c];
        x = sum_row16(x);
        if (l == 0) {
            sum[c] = x;
            px[c] = 0.0;
        }
    }
    if (b.psp > 0) {
        const int n = b.psp, i = tid & (kPsp - 1), part = tid / kPsp;
        const double *V = b.V + (int64_t)t * b.max_space * b.dim;
        const double *S = b.S + (int64_t)t * b.max_space * b.dim;
        const double *Q = b.pQ + (int64_t)t * kPsp * kPsp, *Qt = b.pQt + (int64_t)t * kPsp * kPsp;
        const double *dT = b.pT + (int64_t)t * 3 * kPsp, *eT = dT + kPsp;
        const double *yy = b.y + (int64_t)t * kMaxSpace;
        double *T = b.V + ((int64_t)t * b.max_space + nk) * b.dim;
        // this thread's vectors k = part + NPART u at determinant i
        constexpr int NU = (MS + NPART - 1) / NPART;
        double vv[NU], ss[NU], x = 0.0, ax = 0.0, told = 0.0;
        int64_t d = 0;
        if (i < n) {
            d = b.pidx[(int64_t)t * kPsp + i];
            if (part == 0) told = T[d];
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int k = part + NPART * u;
            vv[u] = ss[u] = 0.0;
            if (i < n && k < nk) {
                vv[u] = V[(int64_t)k * b.dim + d];
                ss[u] = S[(int64_t)k * b.dim + d];
            }
            const double yk = rs ? (k == 0 ? 1.0 : 0.0) : (k < nk ? yy[k] : 0.0);   // (restart: V_0 = x, S_0 = A x)
            x += yk * vv[u];
            ax += yk * ss[u];
        }
        red[part][i] = ax - th * x;
        __syncthreads();
        if (tid < kPsp) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < NPART; ++q) s += red[q][i];
            r[i] = s;
        }
        __syncthreads();
        // out_i = sum_k M[k][i] u_k over this part's rows
        const int k0 = part * n / NPART, k1 = (part + 1) * n / NPART;
        auto product = [&](const double *M, const double *u) {
            double s = 0.0;
            if (i < n) {
#pragma unroll 16
                for (int k = k0; k < k1; ++k) s += M[k * kPsp + i] * u[k];
            }
            return s;
        };
        red2[part][i] = product(Q, r);
        __syncthreads();
        double wv = 0.0, di = 0.0, ei = 0.0, ep = 0.0;
        if (tid < n) {
#pragma unroll
            for (int q = 0; q < NPART; ++q) wv += red2[q][i];
            di = dT[i];
            ei = eT[i];
            ep = i > 0 ? eT[i - 1] : 0.0;
        }
        const double uv = tri_solve(tri, n, th, di, ei, ep, wv);
        if (tid < kPsp) w[i] = uv;
        __syncthreads();
        red[part][i] = product(Qt, w);
        __syncthreads();
        double tv = 0.0;
#pragma unroll
        for (int q = 0; q < NPART; ++q) tv += red[q][i];
        if (part == 0) {
            r[i] = i < n ? tv - told : 0.0;
            if (i < n) T[d] = tv;
            const double s = sum_wave(i < n ? tv * tv - told * told : 0.0);
            if ((tid & 63) == 0) nsum[tid >> 6] = s;
        }
        __syncthreads();
        const double dt = r[i];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int k = part + NPART * u;
            if (k >= nk) break;   // the same in every lane of the part
            const double a = sum_wave(vv[u] * dt);
            if ((tid & 63) == 0) wsum[part][(tid >> 6) & 1][u] = a;
            if (SD) {
                const double c = sum_wave(ss[u] * dt);
                if ((tid & 63) == 0) ssum[part][(tid >> 6) & 1][u] = c;
            }
        }
        __syncthreads();
        if (tid < nk) {
            const int p = tid % NPART, u = tid / NPART;
            px[2 + tid] = wsum[p][0][u] + wsum[p][1][u];
            if (SD) px[kSdOff + tid] = ssum[p][0][u] + ssum[p][1][u];
        }
        if (tid == 0) px[1] = nsum[0] + nsum[1];
    }
    __syncthreads();
    if (tid >= 64) return;
    // convergence and restart bookkeeping (every lane takes the same decisions)
    const int lane = tid;
    const double rn = sqrt(sum[0]), t2 = sum[1] + px[1];
    int st = ST_RUNNING;
    if (!isfinite(rn) || !isfinite(th)) st = ST_NONFINITE;
    // (a P space that is the whole space holds the exact eigenvector: the
    // correction's equation is singular there, and a small residual is enough)
    else if (rn < b.r_tol && (b.psp >= b.dim || fabs(th - b.theta_prev[t]) < b.e_tol)) st = ST_DONE;
    const int it = b.iter[t] + 1;
    if (st == ST_RUNNING && it >= b.max_iter) st = ST_MAXITER;
    double *R = b.R + (int64_t)t * kMaxSpace * kMaxSpace;
    const int m = nk;
    if (rs) {   // V_0 = x, S_0 = A x (and V_1, S_1 the kept direction) already written
        double *G = b.G + (int64_t)t * kMaxSpace * kMaxSpace;
        double *y = b.y + (int64_t)t * kMaxSpace, *zp = b.zp + (int64_t)t * kMaxSpace;
        if (lane < kMaxSpace) zp[lane] = lane == 0 ? 1.0 : 0.0;   // x, in the new coordinates
        if (lane == 0) {
            b.m[t] = rs;
            G[0] = th;
            R[0] = 1.0;   // x = Q y has unit norm
            y[0] = 1.0;
            if (rs == 2) {
                G[1] = G[kMaxSpace] = 0.0;
                G[kMaxSpace + 1] = b.mu[t];
                R[1] = 0.0;
                R[kMaxSpace + 1] = 1.0;
                y[1] = 0.0;
            }
        }
    }
    // (before theta_prev is replaced: every lane has read it)
    wave_sync();
    if (lane == 0) {
        b.rnorm[t] = rn;
        b.tnorm0[t] = sqrt(t2);
        b.iter[t] = it;
        b.theta_prev[t] = th;
        b.status[t] = st;
    }
    if (st != ST_RUNNING) return;
    if (lane == 0) b.run[atomicAdd(b.counter, 1)] = t;   // (in any order: sigma takes the tuples from this list)
    // the correction on the basis (R of a restart: the identity)
    if (lane < m) {
        r[lane] = sum[2 + lane] + px[2 + lane];
        if (SD) b.sdot[(int64_t)t * kMaxSpace + lane] = sum[kSdOff + lane] + px[kSdOff + lane];
    }
    wave_sync();
    double c = 0.0;
    if (lane < m) {
        if (rs) c = r[lane];
        else
            for (int j = 0; j <= lane; ++j) c += R[j * kMaxSpace + lane] * r[j];
        w[lane] = c;
    }
    const double c2 = sum_wave(c * c);
    wave_sync();
    double a = 0.0;   // (R c)_i
    if (lane < m) {
        if (rs) a = c;
        else
            for (int j = lane; j < m; ++j) a += R[lane * kMaxSpace + j] * w[j];
    }
    const double kept = t2 - c2;
    const int two = !(kept >= 0.5 * t2);
    if (lane == 0) b.cgs2[t] = two;
    if (two) {
        if (lane < m) b.coef[(int64_t)t * kMaxSpace + lane] = a;
        if (lane == 0) {
            atomicAdd(b.counter + 1, 1);   // this iteration (the profiled loop launches the passes only then)
            atomicAdd(b.counter + 2, 1);   // the whole batch
        }
        return;
    }
    if (!(kept > 1e-300) || m >= b.max_space) {
        if (lane == 0) b.status[t] = rn < b.r_tol ? ST_DONE : (m > 1 ? ST_RESTART : ST_STALLED);
        return;
    }
    const double s = 1.0 / sqrt(kept);
    if (lane < m) b.coef[(int64_t)t * kMaxSpace + lane] = c;   // for the new column of the projected matrix
    if (lane < m) R[lane * kMaxSpace + m] = -a * s;
    if (lane == m) R[m * kMaxSpace + m] = s;
}

hipError_t launch_iter_head(const Batch &b, int nsum, bool sd, hipStream_t s) {
    if (b.max_space <= 12) hipLaunchKernelGGL(k_small_eig<12>, dim3(b.B), dim3(64), 0, s, b, nsum, sd ? 1 : 0);
    else hipLaunchKernelGGL(k_small_eig<kMaxSpace>, dim3(b.B), dim3(64), 0, s, b, nsum, sd ? 1 : 0);
    const bool v2 = (b.dim & 1) == 0;
    if (b.max_space <= 12) {
        if (v2) hipLaunchKernelGGL((k_ritz<12, true>), dim3(b.nblk, b.B), dim3(256), 0, s, b);
        else hipLaunchKernelGGL((k_ritz<12, false>), dim3(b.nblk, b.B), dim3(256), 0, s, b);
    } else {
        if (v2) hipLaunchKernelGGL((k_ritz<kMaxSpace, true>), dim3(b.nblk, b.B), dim3(256), 0, s, b);
        else hipLaunchKernelGGL((k_ritz<kMaxSpace, false>), dim3(b.nblk, b.B), dim3(256), 0, s, b);
    }
    if (b.max_space <= 12) hipLaunchKernelGGL(k_step<12>, dim3(b.B), dim3(kStepThreads), 0, s, b);
    else hipLaunchKernelGGL(k_step<kMaxSpace>, dim3(b.B), dim3(kStepThreads), 0, s, b);
    return hipGetLastError();
}

// Tuples whose correction T = V_m lies too close to the subspace: two passes
// of classical Gram-Schmidt of T against V_0 .. V_{m-1} (coefficients on the
// stored basis), each one pass over the basis vectors.  Every other tuple
// returns at once.  The first pass (coefficients from k_step) also forms the
// projections of the result, the second sums them (every workgroup for
// itself, coef = R R^T d) and forms |T|^2; V_m is left unnormalised and
// 1 / |T| goes into R (k_small_eig, which also decides whether T adds
// anything).  Two launches an iteration instead of six, most of them empty for
// most tuples: 14 instead of 37 us an iteration on the 24-orbital expansion.
template <int MS, bool V2, bool SECOND>
__global__ __launch_bounds__(256) void k_cgs(Batch b) {
    const int t = blockIdx.y;
    if (b.status[t] != ST_RUNNING || !b.cgs2[t]) return;
    const int m = b.m[t], tid = threadIdx.x;
    double cf[MS];
    if (SECOND) {
        __shared__ double d[MS], c[MS], a[MS];
        const double *R = b.R + (int64_t)t * kMaxSpace * kMaxSpace;
        for (int i = tid >> 4; i < MS; i += 16) {
            double x = 0.0;
            if (i < m)
                for (int blk = tid & 15; blk < b.nblk; blk += 16) x += parts(b, t, blk)[i];
            x = sum_row16(x);
            if ((tid & 15) == 0) d[i] = x;
        }
        __syncthreads();
        if (tid < m) {
            double x = 0.0;
            for (int j = 0; j <= tid; ++j) x += R[j * kMaxSpace + tid] * d[j];
            c[tid] = x;
        }
        __syncthreads();
        if (tid < MS) {
            double x = 0.0;
            if (tid < m)
                for (int j = tid; j < m; ++j) x += R[tid * kMaxSpace + j] * c[j];
            a[tid] = x;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MS; ++i) cf[i] = a[i];
    } else {
        const double *cp = b.coef + (int64_t)t * kMaxSpace;
#pragma unroll
        for (int i = 0; i < MS; ++i) cf[i] = (i < m) ? cp[i] : 0.0;
    }
    const double *V = b.V + (int64_t)t * b.max_space * b.dim;
    double *T = b.V + ((int64_t)t * b.max_space + m) * b.dim;
    constexpr int NACC = SECOND ? 1 : MS;
    double acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = 0.0;
    // V_i, i < m, through a buffer resource that ends after vector m - 1 (the
    // loads past it read zero, and cf[i] = 0 there): all loads at once
    const __amdgpu_buffer_rsrc_t rV = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double *>(V), (short)0, (int)((int64_t)m * b.dim * (int64_t)sizeof(double)), 0x00020000);
    const uint32_t vstride = (uint32_t)b.dim * (uint32_t)sizeof(double);
    if (V2) {
        // pairs of determinants with 16-byte loads (dim even)
        const int64_t n2 = b.dim >> 1;
        for (int64_t d2 = (int64_t)blockIdx.x * 256 + tid; d2 < n2; d2 += (int64_t)gridDim.x * 256) {
            const int64_t d = d2 << 1;
            const uint32_t vo = (uint32_t)d * (uint32_t)sizeof(double);
            dbl2v vv[MS];
#pragma unroll
            for (int i = 0; i < MS; ++i)
                vv[i] = __builtin_bit_cast(dbl2v, __builtin_amdgcn_raw_buffer_load_b128(rV, vo, (uint32_t)i * vstride, 0));
            dbl2v v = *reinterpret_cast<const dbl2v *>(T + d);
#pragma unroll
            for (int i = 0; i < MS; ++i) {
                v.x -= cf[i] * vv[i].x;
                v.y -= cf[i] * vv[i].y;
            }
            *reinterpret_cast<dbl2v *>(T + d) = v;
            if (SECOND) {
                acc[0] += v.x * v.x;
                acc[0] += v.y * v.y;
            } else {
#pragma unroll
                for (int i = 0; i < NACC; ++i) {
                    acc[i] += vv[i].x * v.x;
                    acc[i] += vv[i].y * v.y;
                }
            }
        }
    } else {
        for (int64_t d = (int64_t)blockIdx.x * 256 + tid; d < b.dim; d += (int64_t)gridDim.x * 256) {
            const uint32_t vo = (uint32_t)d * (uint32_t)sizeof(double);
            double vd[MS];
#pragma unroll
            for (int i = 0; i < MS; ++i)
                vd[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rV, vo, (uint32_t)i * vstride, 0));
            double v = T[d];
#pragma unroll
            for (int i = 0; i < MS; ++i) v -= cf[i] * vd[i];
            T[d] = v;
            if (SECOND) {
                acc[0] += v * v;
            } else {
#pragma unroll
                for (int i = 0; i < NACC; ++i) acc[i] += vd[i] * v;
            }
        }
    }
    if (!SECOND) {
        store_block_partials<NACC>(b, t, acc, m);
        return;
    }
    __shared__ double sh[4];
    const double x = sum_wave(acc[0]);
    if ((tid & 63) == 0) sh[tid >> 6] = x;
    __syncthreads();
    if (tid == 0) parts(b, t, blockIdx.x)[kNormPart] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

template <int MS, bool V2> static void launch_cgs(const Batch &b, hipStream_t s) {
    const dim3 grid(b.nblk, b.B);
    hipLaunchKernelGGL((k_cgs<MS, V2, false>), grid, dim3(256), 0, s, b);
    hipLaunchKernelGGL((k_cgs<MS, V2, true>), grid, dim3(256), 0, s, b);
}

hipError_t launch_orthonormalize(const Batch &b, hipStream_t s) {
    const bool v2 = (b.dim & 1) == 0;
    if (b.max_space <= 12) {
        if (v2) launch_cgs<12, true>(b, s);
        else launch_cgs<12, false>(b, s);
    } else {
        if (v2) launch_cgs<kMaxSpace, true>(b, s);
        else launch_cgs<kMaxSpace, false>(b, s);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------- RDMs ------
// Ritz vector x = sum_i y_i V_i (normalised) into T, for every tuple.
__global__ __launch_bounds__(256) void k_form_x(Batch b) {
    const int t = blockIdx.y;
    const int m = b.m[t];
    const double *yv = b.y + (int64_t)t * kMaxSpace;
    double yy[kMaxSpace];
#pragma unroll
    for (int i = 0; i < kMaxSpace; ++i) yy[i] = (i < m) ? yv[i] : 0.0;
    const double *V = b.V + (int64_t)t * b.max_space * b.dim;
    double *T = b.T + (int64_t)t * b.dim;
    for (int64_t d = (int64_t)blockIdx.x * 256 + threadIdx.x; d < b.dim; d += (int64_t)gridDim.x * 256) {
        double x = 0.0;
#pragma unroll
        for (int i = 0; i < kMaxSpace; ++i)
            if (i < m) x += yy[i] * V[(int64_t)i * b.dim + d];
        T[d] = x;
    }
}

hipError_t launch_form_x(const Batch &b, hipStream_t s) {
    hipLaunchKernelGGL(k_form_x, dim3(b.nblk, b.B), dim3(256), 0, s, b);
    return hipGetLastError();
}

// Gram matrix of the transition vectors: column i = p * nA + q holds
// D_pq(I) = <I|E_pq|x> (a link E_ab|I'> = s|I> of string I' adds s x_{I'} to
// D_ba(I') ... written here from the ket side: the link (a created, b
// annihilated) of string I moving I to J gives <I|E_ba|J> = s, so
// D_ba(I) += s x_J), column nA^2 holds x itself.  G = D^T D over the
// determinants, accumulated with FP64 MFMA on 32-determinant tiles staged in
// LDS; every block writes its upper tile pairs to part[t][blk][NP*NP].
constexpr int kRdmTile = 32;

__global__ __launch_bounds__(256) void k_rdm_gram(Batch b, VecRef xref, double *part, int NP, int nblk_r) {
    const int t = blockIdx.y;
    const int nA = b.nA, nn = nA * nA;
    const int ld = NP + 1;
    extern __shared__ double Dt[];                       // [32][NP+1]
    __shared__ int pp[kMaxActive * (kMaxActive + 1) / 2], qq[kMaxActive * (kMaxActive + 1) / 2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ar = lane & 15, kr = lane >> 4;
    if (tid < b.pl.P) {
        int p, q;
        pair_of(tid, p, q);
        pp[tid] = p;
        qq[tid] = q;
    }
    const double *x = vref(xref, t, b.dim);
    const int NT = NP / 16, npairs = NT * (NT + 1) / 2;
    dbl4 acc[kRdmMaxPairs];
#pragma unroll
    for (int u = 0; u < kRdmMaxPairs; ++u) acc[u] = dbl4{0.0, 0.0, 0.0, 0.0};
    const int64_t ntiles = (b.dim + kRdmTile - 1) / kRdmTile;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += nblk_r) {
        __syncthreads();
        for (int i = tid; i < kRdmTile * ld; i += 256) Dt[i] = 0.0;
        __syncthreads();
        const int j = tid & 31, part8 = tid >> 5;
        const int64_t d = tile * kRdmTile + j;
        if (d < b.dim) {
            const int64_t Ka = d / b.Nb, Kb = d % b.Nb;
            const uint32_t ma = b.strA[Ka], mb = b.strB[Kb];
            for (int e = part8; e < b.nentA + b.nentB; e += 8) {
                const bool alpha = e < b.nentA;
                const uint32_t L = alpha ? b.linkA[Ka * b.nentA + e] : b.linkB[Kb * b.nentB + (e - b.nentA)];
                int J, Q;
                double s;
                link_decode(L, J, Q, s);
                const int p = pp[Q], q = qq[Q];
                const uint32_t m = alpha ? ma : mb;
                // the annihilated orbital of the link is the one occupied in the string
                const int an = (m >> p & 1u) ? p : q;
                const int cr = (an == p) ? q : p;
                const double xv = alpha ? x[(int64_t)J * b.Nb + Kb] : x[Ka * b.Nb + J];
                atomicAdd(&Dt[j * ld + an * nA + cr], s * xv);
            }
            if (part8 == 0) Dt[j * ld + nn] = x[d];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kRdmMaxPairs; ++u) {
            const int uu = wave + 4 * u;
            if (uu < npairs) {
                int ti = 0, rem = uu;
                while (rem >= NT - ti) { rem -= NT - ti; ++ti; }
                const int tj = ti + rem;
#pragma unroll
                for (int ks = 0; ks < kRdmTile / 4; ++ks) {
                    const double a = Dt[(ks * 4 + kr) * ld + ti * 16 + ar];
                    const double bb = Dt[(ks * 4 + kr) * ld + tj * 16 + ar];
                    acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bb, acc[u], 0, 0, 0);
                }
            }
        }
    }
    double *out = part + ((int64_t)t * nblk_r + blockIdx.x) * NP * NP;
#pragma unroll
    for (int u = 0; u < kRdmMaxPairs; ++u) {
        const int uu = wave + 4 * u;
        if (uu < npairs) {
            int ti = 0, rem = uu;
            while (rem >= NT - ti) { rem -= NT - ti; ++ti; }
            const int tj = ti + rem;
#pragma unroll
            for (int v = 0; v < 4; ++v) out[(int64_t)(ti * 16 + kr + 4 * v) * NP + tj * 16 + ar] = acc[u][v];
        }
    }
}

// G[t] (NP x NP, symmetric) = sum over blocks of the upper tile pairs
__global__ __launch_bounds__(256) void k_rdm_reduce(const double *part, double *G, int NP, int nblk_r) {
    const int t = blockIdx.y;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)NP * NP) return;
    int i = (int)(idx / NP), j = (int)(idx % NP);
    if (i / 16 > j / 16) { const int x = i; i = j; j = x; }
    double s = 0.0;
    for (int blk = 0; blk < nblk_r; ++blk) s += part[((int64_t)t * nblk_r + blk) * NP * NP + (int64_t)i * NP + j];
    G[(int64_t)t * NP * NP + idx] = s;
}

int rdm_np(int nA) { return round_up(nA * nA + 1, 16); }

size_t rdm_lds_bytes(int NP) { return sizeof(double) * (size_t)kRdmTile * (NP + 1); }

hipError_t launch_rdm(const Batch &b, VecRef x, double *part, double *G, int nblk_r, hipStream_t s) {
    const int NP = rdm_np(b.nA);
    hipLaunchKernelGGL(k_rdm_gram, dim3(nblk_r, b.B), dim3(256), rdm_lds_bytes(NP), s, b, x, part, NP, nblk_r);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_rdm_reduce, dim3((unsigned)(((int64_t)NP * NP + 255) / 256), b.B), dim3(256), 0, s, part, G,
                       NP, nblk_r);
    return hipGetLastError();
}

// Weighted embedding of the batch's density matrices into the full-space
// gradient (n x n and n^4 doubles, row-major), w[t] the weight of tuple t:
//   grad_h[o_p, o_q] += w gamma_pq,  grad_eri[o_p, o_q, o_r, o_s] += w/2 Gamma_pqrs
// with gamma_pq = G[pq, x] and Gamma_pqrs = G[qp, rs] - d_qr gamma_ps over the
// active orbitals o, and for the doubly occupied core c, d: gamma_cc = 2,
// Gamma_cccc = 2, Gamma_ccdd = 4 and Gamma_cddc = -2 (c != d), Gamma_pqcc =
// Gamma_ccpq = 2 gamma_pq, Gamma_pccq = Gamma_cqpc = -gamma_pq.  Tuples share
// full-space entries, so the adds are atomic (their order, and the last bits
// of the sums, are not fixed).
__device__ __forceinline__ void grad_add(double *a, double v) { unsafeAtomicAdd(a, v); }

__global__ __launch_bounds__(256) void k_rdm_embed_act(Batch b, const double *w, double *ge) {
    const int t = blockIdx.y;
    const double wt = w[t];
    if (wt == 0.0 || b.status[t] != ST_DONE) return;   // unconverged: solved again, embedded then
    const int nA = b.nA, nn = nA * nA, NP = round_up(nn + 1, 16), n = b.norb;
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= nn * nn) return;
    const int p = idx / (nA * nn), q = (idx / nn) % nA, r = (idx / nA) % nA, s = idx % nA;
    const double *G = b.rdm_G + (int64_t)t * NP * NP;
    const int32_t *o = b.act + (int64_t)t * nA;
    double v = G[(int64_t)(q * nA + p) * NP + r * nA + s];
    if (q == r) v -= G[(int64_t)(p * nA + s) * NP + nn];
    grad_add(ge + (((int64_t)o[p] * n + o[q]) * n + o[r]) * n + o[s], 0.5 * wt * v);
}

__global__ __launch_bounds__(256) void k_rdm_embed_core(Batch b, const double *w, double *gh, double *ge) {
    const int t = blockIdx.x;
    const double wt = w[t];
    if (wt == 0.0 || b.status[t] != ST_DONE) return;
    const int nA = b.nA, nn = nA * nA, NP = round_up(nn + 1, 16), n = b.norb, nC = b.nC;
    const double *G = b.rdm_G + (int64_t)t * NP * NP;
    const int32_t *o = b.act + (int64_t)t * nA, *C = b.core + (int64_t)t * nC;
    const double hw = 0.5 * wt;
    auto E = [&](int p, int q, int r, int s) { return ge + (((int64_t)p * n + q) * n + r) * n + s; };
    for (int i = threadIdx.x; i < nn; i += 256) {
        const int p = i / nA, q = i % nA;
        grad_add(gh + (int64_t)o[p] * n + o[q], wt * G[(int64_t)i * NP + nn]);
    }
    for (int i = threadIdx.x; i < nC * nC; i += 256) {
        const int c = C[i / nC], d = C[i % nC];
        if (c == d) {
            grad_add(gh + (int64_t)c * n + c, 2.0 * wt);
            grad_add(E(c, c, c, c), hw * 2.0);
        } else {
            grad_add(E(c, c, d, d), hw * 4.0);
            grad_add(E(c, d, d, c), hw * -2.0);
        }
    }
    for (int i = threadIdx.x; i < nC * nn; i += 256) {
        const int c = C[i / nn], pq = i % nn, p = pq / nA, q = pq % nA;
        const double g = G[(int64_t)pq * NP + nn];
        grad_add(E(o[p], o[q], c, c), hw * 2.0 * g);
        grad_add(E(c, c, o[p], o[q]), hw * 2.0 * g);
        grad_add(E(o[p], c, c, o[q]), -hw * g);
        grad_add(E(c, o[q], o[p], c), -hw * g);
    }
}

hipError_t launch_rdm_embed(const Batch &b, const double *w, double *gh, double *ge, hipStream_t s) {
    const int n4 = b.nA * b.nA * b.nA * b.nA;
    hipLaunchKernelGGL(k_rdm_embed_act, dim3((n4 + 255) / 256, b.B), dim3(256), 0, s, b, w, ge);
    hipLaunchKernelGGL(k_rdm_embed_core, dim3(b.B), dim3(256), 0, s, b, w, gh, ge);
    return hipGetLastError();
}

__global__ void k_finalize(Batch b) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= b.B) return;
    b.out_e[t] = b.params[(int64_t)t * b.pl.stride + b.pl.off_ecore] + b.theta[t];
    b.out_status[t] = b.status[t];
}

hipError_t launch_finalize(const Batch &b, hipStream_t s) {
    hipLaunchKernelGGL(k_finalize, dim3((b.B + 255) / 256), dim3(256), 0, s, b);
    return hipGetLastError();
}

// The workspace of the allocation-free entry point: a file-scope device array
// that the code object brings (each GPU the library runs on holds its own
// copy until the process ends).  Host code never passes its name to a kernel
// or a copy: scratch_address() resolves it once per device, with that device
// current, and callers use the returned pointer.
static __device__ __align__(256) char scratch[kScratchBytes];

hipError_t scratch_address(void **ptr) {
    *ptr = nullptr;
    return hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch));
}

hipError_t init_kernels() {
    hipError_t e = init_sigma_kernels();
    if (e != hipSuccess) return e;
    if ((e = init_whole_kernels()) != hipSuccess) return e;
    if ((e = init_ccs_kernels()) != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)k_psp_factor<128>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)PspFactor<128>::lds);
}

}  // namespace mbefci
