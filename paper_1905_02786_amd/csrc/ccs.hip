// Coupled-cluster base energies (CCSD and CCSD(T), equations as in cc.hip) of
// tuples small enough for LDS: one workgroup per tuple, everything but the
// DIIS history on chip.
//
// A tuple of 9 active orbitals has 450 independent amplitudes and about 2e5
// multiply-adds per iteration once spin and antisymmetry are used; the
// spin-orbital loops over L2-resident N^4 arrays that this replaces did thirty
// times that and waited for a load at every term (680 order-3 tuples of 24
// orbitals: 70 ms; now 7.0 ms).  So:
//  * T2 is kept for i < j, a < b and the spin classes aa, ab, bb only: a
//    matrix (occupied pair) x (virtual pair) per class.  The ladder terms are
//    products of such matrices with W_abef and W_mnij, class by class.
//  * The ring terms use particle-hole matrices over (i, a): K0 (same spin), K+
//    (i alpha, a beta), K- (i beta, a alpha).  t_ij^ab couples K0 with K0 and
//    K+ with K-; W_mbej couples each set with itself.
//  * Integrals come from one table (pq|rs) over active pairs, P x P.
//  * t_i^e t_m^a <mb||ej> is folded into H_mb,ij = <mb||ij> + P(ij) sum_e t_i^e
//    <mb||ej>, contracted with t_m^a like <mb||ij> itself.
// W_abef, W_mnij and H are done with before W_mbej is formed in their place.
#include "smalleig.h"

namespace mbefci {

constexpr int kCcsThreads = 512;
constexpr int kCcDiis = 6;

// Sizes of one tuple: nA orbitals, oa (ob) occupied and va (vb) virtual ones
// of each spin; offsets (doubles) of its arrays in LDS.
struct CcsShape {
    int nA, oa, ob, va, vb;
    int P, n0, np, nm, ldm;          // pairs; sizes of K0, K+, K-; row length of the (+,-) matrix
    int nO[3], nV[3], oT[3], nT2, L; // pairs of a class, its offset in T2, all of T2, T1 and T2
    int oG, oX, oXpm, o2, oTc, oTn, oTau, oF, oFae, oFmi, oFme, oFbe2, oFmj2, oTab, total;
    int oWv[3], oWo[3], oH[3], oWp, oWm;   // within region 2: W_abef, W_mnij, H, then W_mbej (K0 first)
    int nHb[3];

    __host__ __device__ void init(int nA_, int oa_, int ob_) {
        nA = nA_;
        oa = oa_;
        ob = ob_;
        va = nA - oa;
        vb = nA - ob;
        P = nA * (nA + 1) / 2;
        n0 = oa * va + ob * vb;
        np = oa * vb;
        nm = ob * va;
        ldm = nm | 1;
        nO[0] = oa * (oa - 1) / 2;
        nO[1] = oa * ob;
        nO[2] = ob * (ob - 1) / 2;
        nV[0] = va * (va - 1) / 2;
        nV[1] = va * vb;
        nV[2] = vb * (vb - 1) / 2;
        nT2 = 0;
        for (int c = 0; c < 3; ++c) {
            oT[c] = nT2;
            nT2 += nO[c] * nV[c];
        }
        L = n0 + nT2;
        int o = 0;
        auto take = [&](int n) {
            const int at = o;
            o += (n + 1) & ~1;
            return at;
        };
        oG = take(P * P);
        oX = take(n0 * n0);
        oXpm = take(np * ldm);
        nHb[0] = oa * va;
        nHb[1] = np + nm;
        nHb[2] = ob * vb;
        int r = 0;
        for (int c = 0; c < 3; ++c) {
            oWv[c] = r;
            r += nV[c] * nV[c];
            oWo[c] = r;
            r += nO[c] * nO[c];
            oH[c] = r;
            r += nO[c] * nHb[c];
        }
        oWp = n0 * n0;
        oWm = oWp + np * np;
        const int ring = oWm + nm * nm;
        o2 = take(r > ring ? r : ring);
        oTc = take(L);
        oTn = take(L);
        oTau = take(nT2);
        oF = take(2 * nA * nA);
        oFae = take(va * va + vb * vb);
        oFmi = take(oa * oa + ob * ob);
        oFme = take(n0);
        oFbe2 = take(va * va + vb * vb);
        oFmj2 = take(oa * oa + ob * ob);
        // index tables (16 bits): pair of two orbitals, pairs of each class, K0, K+, K-
        oTab = take((nA * nA + nO[0] + nO[1] + nO[2] + nV[0] + nV[1] + nV[2] + n0 + np + nm + 3) / 4);
        total = o;
    }
};

size_t ccs_lds_bytes(int nA, int oa, int ob) {
    CcsShape s;
    s.init(nA, oa, ob);
    return sizeof(double) * (size_t)s.total;
}

int64_t ccs_history_doubles(int nA, int oa, int ob) {
    CcsShape s;
    s.init(nA, oa, ob);
    return 2 * (int64_t)kCcDiis * s.L;
}

struct CcsArgs {
    const double *h, *eri;
    int n;
    const int32_t *act, *nact, *core, *ncore;
    int stride, nalpha, nbeta;
    double e_const;
    double *work;          // DIIS history per tuple
    int64_t slice;
    int triples, max_iter;
    double tol;
    double *out;
    int32_t *status;
};

__global__ __launch_bounds__(kCcsThreads, 4) void k_ccsd_lds(CcsArgs A) {
    constexpr int NT = kCcsThreads;
    const int t = blockIdx.x, tid = threadIdx.x;
    const int n = A.n, nA = A.nact[t], nC = A.ncore[t];
    const int32_t *act = A.act + (int64_t)t * A.stride, *core = A.core + (int64_t)t * A.stride;
    const double *eri = A.eri, *h = A.h;
    const int64_t n2 = (int64_t)n * n, n3 = n2 * n;
    auto E = [&](int p, int q, int r, int s) { return eri[p * n3 + q * n2 + r * n + s]; };
    __shared__ int sact[kMaxOrb], score[kMaxOrb];
    __shared__ double sh[16];
    __shared__ double Bm[kCcDiis][kCcDiis], Mm[8][8], xs[8], coef[kCcDiis];
    static_assert(kCcDiis + 1 < 8, "DIIS system");
    __shared__ int bad_sh;
    extern __shared__ double lds[];
    int oa = 0, ob = 0;
    for (int k = 0; k < nA; ++k) {
        oa += act[k] < A.nalpha;
        ob += act[k] < A.nbeta;
    }
    __shared__ CcsShape S;   // (in LDS: its arrays are indexed by the spin class)
    static_assert(sizeof(sact) + sizeof(score) + sizeof(sh) + sizeof(Bm) + sizeof(Mm) + sizeof(xs) + sizeof(coef) +
                      sizeof(bad_sh) + sizeof(S) + 16 <= kCcsStaticLds && kCcsMaxLds + kCcsStaticLds <= 160 * 1024,
                  "static LDS of k_ccsd_lds");
    if (tid == 0) S.init(nA, oa, ob);
    __syncthreads();
    const int va = S.va, vb = S.vb, o = oa + ob, v = va + vb, P = S.P, n0 = S.n0;
    double *G = lds + S.oG, *X = lds + S.oX, *Xpm = lds + S.oXpm, *R2 = lds + S.o2;
    double *T1 = lds + S.oTc, *T2 = T1 + n0, *N1 = lds + S.oTn, *N2 = N1 + n0, *tau = lds + S.oTau;
    double *F = lds + S.oF, *Fae = lds + S.oFae, *Fmi = lds + S.oFmi, *Fme = lds + S.oFme;
    double *Fbe2 = lds + S.oFbe2, *Fmj2 = lds + S.oFmj2;
    uint16_t *PI = reinterpret_cast<uint16_t *>(lds + S.oTab);
    uint16_t *ol = PI + nA * nA, *vl = ol + S.nO[0] + S.nO[1] + S.nO[2];
    uint16_t *kl = vl + S.nV[0] + S.nV[1] + S.nV[2], *kp = kl + n0, *km = kp + S.np;
    for (int i = tid; i < nA; i += NT) sact[i] = act[i];
    for (int i = tid; i < nC; i += NT) score[i] = core[i];
    if (tid == 0) bad_sh = 0;
    for (int i = tid; i < nA * nA; i += NT) {
        const int p = i / nA, q = i % nA, hi = p > q ? p : q, lo = p > q ? q : p;
        PI[i] = (uint16_t)(hi * (hi + 1) / 2 + lo);
    }
    // index lists: spin-orbitals i < oa alpha, the others beta (virtual ones likewise)
    for (int i = tid; i < o * o; i += NT) {
        const int x = i / o, y = i % o;
        if (x >= y) continue;
        const uint16_t e = (uint16_t)(x | (y << 8));
        if (y < oa) ol[y * (y - 1) / 2 + x] = e;
        else if (x < oa) ol[S.nO[0] + x * ob + y - oa] = e;
        else ol[S.nO[0] + S.nO[1] + (y - oa) * (y - oa - 1) / 2 + x - oa] = e;
    }
    for (int i = tid; i < v * v; i += NT) {
        const int x = i / v, y = i % v;
        if (x >= y) continue;
        const uint16_t e = (uint16_t)(x | (y << 8));
        if (y < va) vl[y * (y - 1) / 2 + x] = e;
        else if (x < va) vl[S.nV[0] + x * vb + y - va] = e;
        else vl[S.nV[0] + S.nV[1] + (y - va) * (y - va - 1) / 2 + x - va] = e;
    }
    for (int i = tid; i < o * v; i += NT) {
        const int x = i / v, a = i % v;
        const uint16_t e = (uint16_t)(x | (a << 8));
        if (x < oa && a < va) kl[x * va + a] = e;
        else if (x >= oa && a >= va) kl[oa * va + (x - oa) * vb + a - va] = e;
        else if (x < oa) kp[x * vb + a - va] = e;
        else km[(x - oa) * va + a] = e;
    }
    __syncthreads();
    // the occupied active orbitals of a spin are its first ones (the active list ascends)
    auto so = [&](int i) { return i >= oa ? 1 : 0; };
    auto sv = [&](int a) { return a >= va ? 1 : 0; };
    auto xo = [&](int i) { return i >= oa ? i - oa : i; };                  // active position of an occupied one
    auto xv = [&](int a) { return a >= va ? ob + a - va : oa + a; };        // and of a virtual one
    auto g = [&](int p, int q, int r, int s) { return G[PI[p * nA + q] * P + PI[r * nA + s]]; };
    // <PQ||RS> of active positions x and spins s
    auto asy = [&](int xP, int sP, int xQ, int sQ, int xR, int sR, int xS, int sS) {
        double w = 0.0;
        if (sP == sR && sQ == sS) w = g(xP, xR, xQ, xS);
        if (sP == sS && sQ == sR) w -= g(xP, xS, xQ, xR);
        return w;
    };
    for (int i = tid; i < P * P; i += NT) {
        int p, q, r, s;
        pair_of(i / P, p, q);
        pair_of(i % P, r, s);
        G[i] = E(sact[p], sact[q], sact[r], sact[s]);
    }
    __syncthreads();
    // Fock operator of Phi on the active orbitals, per spin
    for (int i = tid; i < 2 * nA * nA; i += NT) {
        const int s = i / (nA * nA), p = i / nA % nA, q = i % nA, op = sact[p], oq = sact[q];
        double x = h[op * n + oq];
        for (int c = 0; c < nC; ++c) x += 2.0 * E(op, oq, score[c], score[c]) - E(op, score[c], score[c], oq);
        for (int m = 0; m < oa; ++m) x += g(p, q, m, m) - (s == 0 ? g(p, m, m, q) : 0.0);
        for (int m = 0; m < ob; ++m) x += g(p, q, m, m) - (s == 1 ? g(p, m, m, q) : 0.0);
        F[i] = x;
    }
    // reference energy <Phi|H|Phi>
    double eref = 0.0;
    {
        const int nocc = 2 * nC + o;   // core spin-orbitals (both spins), then the active occupied ones
        auto orb = [&](int k, int &p, int &s) {
            if (k < 2 * nC) {
                p = score[k >> 1];
                s = k & 1;
            } else {
                p = sact[xo(k - 2 * nC)];
                s = so(k - 2 * nC);
            }
        };
        for (int k = tid; k < nocc; k += NT) {
            int p, s;
            orb(k, p, s);
            eref += h[p * n + p];
        }
        for (int kk = tid; kk < nocc * nocc; kk += NT) {
            int p, s, q, s2;
            orb(kk / nocc, p, s);
            orb(kk % nocc, q, s2);
            eref += 0.5 * (E(p, p, q, q) - (s == s2 ? E(p, q, q, p) : 0.0));
        }
    }
    eref = block_sum(eref, sh);
    __syncthreads();
    auto f = [&](int s, int p, int q) { return F[(s * nA + p) * nA + q]; };
    auto foo = [&](int i) { return f(so(i), xo(i), xo(i)); };
    auto fvv = [&](int a) { return f(sv(a), xv(a), xv(a)); };
    for (int k = tid; k < n0; k += NT)
        if (!(foo(kl[k] & 255) - fvv(kl[k] >> 8) < 0.0)) bad_sh = 1;
    __syncthreads();
    if (bad_sh) {
        if (tid == 0) {
            A.out[t] = __builtin_nan("");
            A.status[t] = 1;
        }
        return;
    }
    double *Hist = A.work + (int64_t)t * A.slice, *Err = Hist + (int64_t)kCcDiis * S.L;
    // T1 (and any K0 vector) of i, a of the same spin
    auto k0 = [&](int i, int a) { return i < oa ? i * va + a : oa * va + (i - oa) * vb + a - va; };
    auto t1 = [&](int i, int a) { return so(i) == sv(a) ? T1[k0(i, a)] : 0.0; };
    // antisymmetric T2 element; i, j, a, b any
    auto t2 = [&](int i, int j, int a, int b) -> double {
        const int c = so(i) + so(j);
        if (c != sv(a) + sv(b)) return 0.0;
        bool neg = false;
        if (i > j) {
            const int x = i;
            i = j;
            j = x;
            neg = !neg;
        }
        if (a > b) {
            const int x = a;
            a = b;
            b = x;
            neg = !neg;
        }
        int io, iv;
        if (c == 1) {
            io = i * ob + j - oa;
            iv = a * vb + b - va;
        } else {
            if (i == j || a == b) return 0.0;
            const int di = c ? oa : 0, da = c ? va : 0;
            io = (j - di) * (j - di - 1) / 2 + i - di;
            iv = (b - da) * (b - da - 1) / 2 + a - da;
        }
        const double w = T2[S.oT[c] + io * S.nV[c] + iv];
        return neg ? -w : w;
    };
    auto o_of = [&](int c) { return c == 0 ? 0 : (c == 1 ? S.nO[0] : S.nO[0] + S.nO[1]); };
    auto v_of = [&](int c) { return c == 0 ? 0 : (c == 1 ? S.nV[0] : S.nV[0] + S.nV[1]); };
    // T2 element k: class, pairs and orbitals
    auto decode = [&](int k, int &c, int &io, int &iv, int &i, int &j, int &a, int &b) {
        c = k < S.oT[1] ? 0 : (k < S.oT[2] ? 1 : 2);
        const int r = k - S.oT[c];
        io = r / S.nV[c];
        iv = r % S.nV[c];
        const int eo = ol[o_of(c) + io], ev = vl[v_of(c) + iv];
        i = eo & 255;
        j = eo >> 8;
        a = ev & 255;
        b = ev >> 8;
    };
    // occupied (virtual) spin-orbitals of spin s: o0(s) .. o0(s + 1)
    auto o0 = [&](int s) { return s == 0 ? 0 : (s == 1 ? oa : o); };
    auto v0 = [&](int s) { return s == 0 ? 0 : (s == 1 ? va : v); };
    for (int k = tid; k < S.L; k += NT) T1[k] = 0.0;
    __syncthreads();

    const int l16 = tid & 15, row = tid >> 4;   // 16 lanes per output of the long sums
    double e_cc = 0.0, e_old = 0.0;
    int it = 0, nh = 0, conv = 0;
    for (; it < A.max_iter && S.L > 0; ++it) {
        // tau, and T2 in particle-hole form
        for (int k = tid; k < S.nT2; k += NT) {
            int c, io, iv, i, j, a, b;
            decode(k, c, io, iv, i, j, a, b);
            tau[k] = T2[k] + t1(i, a) * t1(j, b) - t1(i, b) * t1(j, a);
        }
        for (int k = tid; k < n0 * n0; k += NT) {
            const int x = kl[k / n0], y = kl[k % n0];
            X[k] = t2(x & 255, y & 255, x >> 8, y >> 8);
        }
        for (int k = tid; k < S.np * S.nm; k += NT) {
            const int r = k / S.nm, q = k % S.nm, x = kp[r], y = km[q];
            Xpm[r * S.ldm + q] = t2(x & 255, y & 255, x >> 8, y >> 8);
        }
        __syncthreads();
        // one-body intermediates, 16 lanes each
        const int nae = va * va + vb * vb, nmi = oa * oa + ob * ob, nOall = S.nO[0] + S.nO[1] + S.nO[2];
        for (int k0_ = row; k0_ < nae + nmi + n0; k0_ += NT / 16) {
            double x = 0.0;
            if (k0_ < nae) {
                const int s = k0_ >= va * va ? 1 : 0, r = s ? k0_ - va * va : k0_, nv = s ? vb : va;
                const int a = v0(s) + r / nv, e = v0(s) + r % nv;
                if (l16 == 0 && a != e) x = f(s, xv(a), xv(e));
                for (int m = o0(s) + l16; m < o0(s + 1); m += 16) x -= 0.5 * f(s, xo(m), xv(e)) * t1(m, a);
                for (int q = l16; q < n0; q += 16) {
                    const int m = kl[q] & 255, ff = kl[q] >> 8;
                    x += T1[q] * asy(xo(m), so(m), xv(a), s, xv(ff), so(m), xv(e), s);
                }
                for (int q = l16; q < nOall * v; q += 16) {
                    const int pr = ol[q / v], m = pr & 255, nn = pr >> 8, ff = q % v;
                    if (so(m) + so(nn) != s + sv(ff)) continue;
                    const double ta = t2(m, nn, a, ff) + 0.5 * (t1(m, a) * t1(nn, ff) - t1(m, ff) * t1(nn, a));
                    x -= ta * asy(xo(m), so(m), xo(nn), so(nn), xv(e), s, xv(ff), sv(ff));
                }
            } else if (k0_ < nae + nmi) {
                const int kk = k0_ - nae, s = kk >= oa * oa ? 1 : 0, r = s ? kk - oa * oa : kk, ns = s ? ob : oa;
                const int m = o0(s) + r / ns, i = o0(s) + r % ns;
                if (l16 == 0 && m != i) x = f(s, xo(m), xo(i));
                for (int e = v0(s) + l16; e < v0(s + 1); e += 16) x += 0.5 * t1(i, e) * f(s, xo(m), xv(e));
                for (int q = l16; q < n0; q += 16) {
                    const int nn = kl[q] & 255, e = kl[q] >> 8;
                    x += T1[q] * asy(xo(m), s, xo(nn), so(nn), xo(i), s, xv(e), so(nn));
                }
                for (int nn = 0; nn < o; ++nn) {
                    const int c = s + so(nn);
                    for (int q = l16; q < S.nV[c]; q += 16) {
                        const int pr = vl[v_of(c) + q], e = pr & 255, ff = pr >> 8;
                        const double ta = t2(i, nn, e, ff) + 0.5 * (t1(i, e) * t1(nn, ff) - t1(i, ff) * t1(nn, e));
                        x += ta * asy(xo(m), s, xo(nn), so(nn), xv(e), sv(e), xv(ff), sv(ff));
                    }
                }
            } else {
                const int pr = kl[k0_ - nae - nmi], m = pr & 255, e = pr >> 8, s = so(m);
                if (l16 == 0) x = f(s, xo(m), xv(e));
                for (int q = l16; q < n0; q += 16) {
                    const int nn = kl[q] & 255, ff = kl[q] >> 8;
                    x += T1[q] * asy(xo(m), s, xo(nn), so(nn), xv(e), s, xv(ff), so(nn));
                }
            }
            x = sum_row16(x);
            if (l16 == 0) {
                if (k0_ < nae) Fae[k0_] = x;
                else if (k0_ < nae + nmi) Fmi[k0_ - nae] = x;
                else Fme[k0_ - nae - nmi] = x;
            }
        }
        __syncthreads();
        auto fme = [&](int m, int e) { return Fme[k0(m, e)]; };   // (same spin)
        for (int k = tid; k < nae + nmi; k += NT) {
            if (k < nae) {
                const int s = k >= va * va ? 1 : 0, r = s ? k - va * va : k, nv = s ? vb : va;
                const int b = v0(s) + r / nv, e = v0(s) + r % nv;
                double x = Fae[k];
                for (int m = o0(s); m < o0(s + 1); ++m) x -= 0.5 * t1(m, b) * fme(m, e);
                Fbe2[k] = x;
            } else {
                const int kk = k - nae, s = kk >= oa * oa ? 1 : 0, r = s ? kk - oa * oa : kk, ns = s ? ob : oa;
                const int m = o0(s) + r / ns, j = o0(s) + r % ns;
                double x = Fmi[kk];
                for (int e = v0(s); e < v0(s + 1); ++e) x += 0.5 * t1(j, e) * fme(m, e);
                Fmj2[kk] = x;
            }
        }
        auto at_vv = [&](int a, int e) {   // index of a same-spin virtual (occupied) pair in Fae (Fmi)
            return a < va ? a * va + e : va * va + (a - va) * vb + e - va;
        };
        auto at_oo = [&](int m, int i) { return m < oa ? m * oa + i : oa * oa + (m - oa) * ob + i - oa; };
        // W_abef, W_mnij and H, class by class
        for (int c = 0; c < 3; ++c) {
            const int nV = S.nV[c], nO = S.nO[c], nH = S.nHb[c];
            const double *tc = tau + S.oT[c];
            for (int k = tid; k < nV * nV; k += NT) {
                const int ab = k / nV, ef = k % nV, pa = vl[v_of(c) + ab], pe = vl[v_of(c) + ef];
                const int a = pa & 255, b = pa >> 8, e = pe & 255, ff = pe >> 8;
                const int sa = sv(a), sb = sv(b), se = sv(e), sf = sv(ff), xa = xv(a), xb = xv(b), xe = xv(e), xf = xv(ff);
                double x = asy(xa, sa, xb, sb, xe, se, xf, sf);
                for (int m = o0(sb); m < o0(sb + 1); ++m) x -= t1(m, b) * asy(xa, sa, xo(m), sb, xe, se, xf, sf);
                for (int m = o0(sa); m < o0(sa + 1); ++m) x += t1(m, a) * asy(xb, sb, xo(m), sa, xe, se, xf, sf);
                for (int q = 0; q < nO; ++q) {
                    const int pm = ol[o_of(c) + q], m = pm & 255, nn = pm >> 8;
                    x += 0.5 * tc[q * nV + ab] * asy(xo(m), so(m), xo(nn), so(nn), xe, se, xf, sf);
                }
                R2[S.oWv[c] + k] = x;
            }
            for (int k = tid; k < nO * nO; k += NT) {
                const int mn = k / nO, ij = k % nO, pm = ol[o_of(c) + mn], pi = ol[o_of(c) + ij];
                const int m = pm & 255, nn = pm >> 8, i = pi & 255, j = pi >> 8;
                const int sm = so(m), sn = so(nn), si = so(i), sj = so(j), xm = xo(m), xn = xo(nn), xi = xo(i), xj = xo(j);
                double x = asy(xm, sm, xn, sn, xi, si, xj, sj);
                for (int e = v0(sj); e < v0(sj + 1); ++e) x += t1(j, e) * asy(xm, sm, xn, sn, xi, si, xv(e), sj);
                for (int e = v0(si); e < v0(si + 1); ++e) x -= t1(i, e) * asy(xm, sm, xn, sn, xj, sj, xv(e), si);
                for (int q = 0; q < nV; ++q) {
                    const int pe = vl[v_of(c) + q], e = pe & 255, ff = pe >> 8;
                    x += 0.5 * tc[ij * nV + q] * asy(xm, sm, xn, sn, xv(e), sv(e), xv(ff), sv(ff));
                }
                R2[S.oWo[c] + k] = x;
            }
            // (m, b) of H: K0 of the spin for aa and bb, K+ then K- for ab
            for (int k = tid; k < nO * nH; k += NT) {
                const int ij = k / nH, mb = k % nH, pi = ol[o_of(c) + ij];
                const int pm = c == 0 ? kl[mb] : (c == 2 ? kl[oa * va + mb] : (mb < S.np ? kp[mb] : km[mb - S.np]));
                const int m = pm & 255, b = pm >> 8, i = pi & 255, j = pi >> 8;
                const int sm = so(m), sb = sv(b), si = so(i), sj = so(j), xm = xo(m), xb = xv(b), xi = xo(i), xj = xo(j);
                double x = asy(xm, sm, xb, sb, xi, si, xj, sj);
                for (int e = v0(si); e < v0(si + 1); ++e) x += t1(i, e) * asy(xm, sm, xb, sb, xv(e), si, xj, sj);
                for (int e = v0(sj); e < v0(sj + 1); ++e) x -= t1(j, e) * asy(xm, sm, xb, sb, xv(e), sj, xi, si);
                R2[S.oH[c] + k] = x;
            }
        }
        __syncthreads();
        // new T1, 16 lanes each
        for (int k = row; k < n0; k += NT / 16) {
            const int pr = kl[k], i = pr & 255, a = pr >> 8, s = so(i), xi = xo(i), xa = xv(a);
            double x = l16 == 0 ? f(s, xi, xa) : 0.0;
            for (int e = v0(s) + l16; e < v0(s + 1); e += 16) x += t1(i, e) * Fae[at_vv(a, e)];
            for (int m = o0(s) + l16; m < o0(s + 1); m += 16) x -= t1(m, a) * Fmi[at_oo(m, i)];
            for (int q = l16; q < n0; q += 16) {
                const int nn = kl[q] & 255, ff = kl[q] >> 8;
                x += X[q * n0 + k] * Fme[q];
                x -= T1[q] * asy(xo(nn), so(nn), xa, s, xi, s, xv(ff), so(nn));
            }
            for (int m = 0; m < o; ++m) {
                const int c = s + so(m);
                for (int q = l16; q < S.nV[c]; q += 16) {
                    const int pe = vl[v_of(c) + q], e = pe & 255, ff = pe >> 8;
                    x -= t2(i, m, e, ff) * asy(xo(m), so(m), xa, s, xv(e), sv(e), xv(ff), sv(ff));
                }
            }
            for (int q = l16; q < nOall * v; q += 16) {
                const int pm = ol[q / v], m = pm & 255, nn = pm >> 8, e = q % v;
                if (so(m) + so(nn) != s + sv(e)) continue;
                x -= t2(m, nn, a, e) * asy(xo(nn), so(nn), xo(m), so(m), xv(e), sv(e), xi, s);
            }
            x = sum_row16(x);
            if (l16 == 0) N1[k] = x / (foo(i) - fvv(a));
        }
        // new T2 but for the ring terms and the denominator
        for (int k = tid; k < S.nT2; k += NT) {
            int c, io, iv, i, j, a, b;
            decode(k, c, io, iv, i, j, a, b);
            const int si = so(i), sj = so(j), sa = sv(a), sb = sv(b), xi = xo(i), xj = xo(j), xa = xv(a), xb = xv(b);
            const int nV = S.nV[c], nO = S.nO[c], nH = S.nHb[c];
            const double *tc = tau + S.oT[c], *Wv = R2 + S.oWv[c] + iv * nV, *Wo = R2 + S.oWo[c] + io;
            double x = asy(xi, si, xj, sj, xa, sa, xb, sb);
            for (int e = v0(sb); e < v0(sb + 1); ++e) x += t2(i, j, a, e) * Fbe2[at_vv(b, e)];
            for (int e = v0(sa); e < v0(sa + 1); ++e) x -= t2(i, j, b, e) * Fbe2[at_vv(a, e)];
            for (int m = o0(sj); m < o0(sj + 1); ++m) x -= t2(i, m, a, b) * Fmj2[at_oo(m, j)];
            for (int m = o0(si); m < o0(si + 1); ++m) x += t2(j, m, a, b) * Fmj2[at_oo(m, i)];
#pragma unroll 4
            for (int q = 0; q < nO; ++q) x += tc[q * nV + iv] * Wo[q * nO];
#pragma unroll 4
            for (int q = 0; q < nV; ++q) x += tc[io * nV + q] * Wv[q];
            for (int e = v0(si); e < v0(si + 1); ++e) x += t1(i, e) * asy(xa, sa, xb, sb, xv(e), si, xj, sj);
            for (int e = v0(sj); e < v0(sj + 1); ++e) x -= t1(j, e) * asy(xa, sa, xb, sb, xv(e), sj, xi, si);
            const double *Hc = R2 + S.oH[c] + io * nH;
            // index of (m, b) in H's rows
            auto hb = [&](int m, int bb) {
                if (c == 0) return m * va + bb;
                if (c == 2) return (m - oa) * vb + bb - va;
                return m < oa ? m * vb + bb - va : S.np + (m - oa) * va + bb;
            };
            for (int m = o0(sa); m < o0(sa + 1); ++m) x -= t1(m, a) * Hc[hb(m, b)];
            for (int m = o0(sb); m < o0(sb + 1); ++m) x += t1(m, b) * Hc[hb(m, a)];
            N2[k] = x;
        }
        __syncthreads();
        // W_mbej as matrices [(m e)][(j b)] over K0, K+ and K-
        for (int blk = 0; blk < 3; ++blk) {
            const int nk = blk == 0 ? n0 : (blk == 1 ? S.np : S.nm);
            const uint16_t *kk = blk == 0 ? kl : (blk == 1 ? kp : km);
            double *W = R2 + (blk == 0 ? 0 : (blk == 1 ? S.oWp : S.oWm));
            for (int k = tid; k < nk * nk; k += NT) {
                const int rme = k / nk, rjb = k % nk;
                const int pm = kk[rme], pj = kk[rjb], m = pm & 255, e = pm >> 8, j = pj & 255, b = pj >> 8;
                const int sm = so(m), sj = so(j), sb = sv(b), xm = xo(m), xe = xv(e), xj = xo(j), xb = xv(b);
                const bool dj = blk == 0, dk = sm == sj;
                const double *Gme = G + PI[xm * nA + xe] * P;
                auto two = [&](int r, int s, int p, int q) {   // dj (me|rs) - dk (mp|qe)
                    double w = 0.0;
                    if (dj) w = Gme[PI[r * nA + s]];
                    if (dk) w -= g(xm, p, q, xe);
                    return w;
                };
                double x = two(xb, xj, xj, xb);
                for (int ff = v0(sj); ff < v0(sj + 1); ++ff) x += t1(j, ff) * two(xb, xv(ff), xv(ff), xb);
                for (int nn = o0(sb); nn < o0(sb + 1); ++nn) x -= t1(nn, b) * two(xo(nn), xj, xj, xo(nn));
                // - sum_nf (1/2 t_jn^fb + t_j^f t_n^b) <mn||ef>, t_jn^fb = -X[(jb)][(nf)]
                if (blk == 0) {
                    for (int s3 = 0; s3 < 2; ++s3) {
                        const bool ex = s3 == sm, tt = s3 == sj;
                        int q = s3 ? oa * va : 0;
                        for (int nn = o0(s3); nn < o0(s3 + 1); ++nn) {
                            const int xn = xo(nn);
                            const uint16_t *pn = PI + xn * nA;
                            const double tnb = tt ? t1(nn, b) : 0.0;
                            const double *Tj = T1 + k0(j, v0(sj));
                            const uint16_t pne = pn[xe];
                            const int xf0 = s3 ? ob : oa, nv = s3 ? vb : va;
                            for (int q2 = 0; q2 < nv; ++q2, ++q) {
                                double w = Gme[pn[xf0 + q2]];
                                if (ex) w -= G[PI[xm * nA + xf0 + q2] * P + pne];
                                double z = -0.5 * X[q * n0 + rjb];
                                if (tt) z += Tj[q2] * tnb;
                                x -= z * w;
                            }
                        }
                    }
                } else {
                    // (n f) of the other kind: n of b's spin, f of j's
                    for (int nn = o0(sb); nn < o0(sb + 1); ++nn) {
                        const double tnb = t1(nn, b);
                        const uint16_t pne = PI[xo(nn) * nA + xe];
                        const int nf = v0(sj + 1) - v0(sj);
                        for (int q2 = 0; q2 < nf; ++q2) {
                            const int r = (nn - o0(sb)) * nf + q2;
                            const double z = -0.5 * (blk == 1 ? Xpm[rjb * S.ldm + r] : Xpm[r * S.ldm + rjb]) +
                                             t1(j, v0(sj) + q2) * tnb;
                            x += z * G[PI[xm * nA + xv(v0(sj) + q2)] * P + pne];
                        }
                    }
                }
                W[k] = x;
            }
        }
        __syncthreads();
        // ring terms R(ia,jb) - R(ja,ib) - R(ib,ja) + R(jb,ia), R = X W, and the denominator
        for (int k = tid; k < S.nT2; k += NT) {
            int c, io, iv, i, j, a, b;
            decode(k, c, io, iv, i, j, a, b);
            double x = 0.0;
            if (c == 1) {
                const int ia = k0(i, a), jb = k0(j, b), ib = i * vb + b - va, ja = (j - oa) * va + a;
#pragma unroll 4
                for (int q = 0; q < n0; ++q)
                    x += X[q * n0 + ia] * R2[q * n0 + jb] + X[q * n0 + jb] * R2[q * n0 + ia];
                const double *Wp = R2 + S.oWp, *Wm = R2 + S.oWm;
#pragma unroll 4
                for (int q = 0; q < S.np; ++q) x -= Xpm[q * S.ldm + ja] * Wp[q * S.np + ib];
#pragma unroll 4
                for (int q = 0; q < S.nm; ++q) x -= Xpm[ib * S.ldm + q] * Wm[q * S.nm + ja];
            } else {
                const int ia = k0(i, a), jb = k0(j, b), ib = k0(i, b), ja = k0(j, a);
#pragma unroll 2
                for (int q = 0; q < n0; ++q) {
                    const double *Xq = X + q * n0, *Wq = R2 + q * n0;
                    x += Xq[ia] * Wq[jb] + Xq[jb] * Wq[ia];
                    x -= Xq[ja] * Wq[ib] + Xq[ib] * Wq[ja];
                }
            }
            N2[k] = (N2[k] + x) / (foo(i) + foo(j) - fvv(a) - fvv(b));
        }
        __syncthreads();
        // DIIS: store the update and its change, extrapolate (each T2 element
        // stands for four)
        const int slot = it % kCcDiis;
        double dmax = 0.0;
        for (int k = tid; k < S.L; k += NT) {
            const double d = N1[k] - T1[k];
            Hist[slot * S.L + k] = N1[k];
            Err[slot * S.L + k] = d;
            dmax = fmax(dmax, fabs(d));
        }
#pragma unroll
        for (int q = 32; q > 0; q >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, q, 64));
        if ((tid & 63) == 0) sh[tid >> 6] = dmax;
        __syncthreads();
        for (int q = 0; q < NT / 64; ++q) dmax = fmax(dmax, sh[q]);
        nh = nh < kCcDiis ? nh + 1 : kCcDiis;
        // one wave per history vector
        if ((tid >> 6) < nh) {
            const int q = tid >> 6;
            double d = 0.0;
            for (int k = tid & 63; k < S.L; k += 64)
                d += (k < n0 ? 1.0 : 4.0) * Err[slot * S.L + k] * Err[q * S.L + k];
            d = sum_wave(d);
            if ((tid & 63) == 0) {
                Bm[slot][q] = d;
                Bm[q][slot] = d;
            }
        }
        __syncthreads();
        if (tid < 64) {
            // (nh + 1) x (nh + 1) system [B -1; -1 0] c = [0; -1] by Gaussian
            // elimination with partial pivoting, one matrix element per lane
            const int m = nh, r = tid >> 3, c = tid & 7;
            double scale = 0.0;
            for (int i = 0; i < m; ++i) scale = fmax(scale, Bm[i][i]);
            scale = scale > 0.0 ? 1.0 / scale : 1.0;
            double w = 0.0;
            if (r <= m && c <= m) w = (r < m && c < m) ? Bm[r][c] * scale : (r == m && c == m ? 0.0 : -1.0);
            if (r <= m && c == 7) w = r < m ? 0.0 : -1.0;   // right-hand side
            Mm[r][c] = w;
            wave_sync();
            bool ok = true;
            for (int q = 0; q <= m && ok; ++q) {
                int piv = q;
                double big = fabs(Mm[q][q]);
                for (int i = q + 1; i <= m; ++i) {
                    const double y = fabs(Mm[i][q]);
                    if (y > big) {
                        big = y;
                        piv = i;
                    }
                }
                if (!(big > 1e-300)) {
                    ok = false;
                    break;
                }
                const int from = r == q ? piv : (r == piv ? q : r);   // rows q and piv swapped
                const double pr = Mm[piv][c], pv = Mm[piv][q], mine = Mm[from][c], lead = Mm[from][q];
                wave_sync();
                Mm[r][c] = r > q ? mine - lead / pv * pr : mine;
                wave_sync();
            }
            // back substitution (not Gauss-Jordan: with fewer amplitudes than
            // vectors the system is singular to rounding, and the solution has
            // to keep to its upper rows, the sum rule among them)
            if (ok) {
                for (int i = m; i >= 0; --i) {
                    double w2 = Mm[i][7];
                    for (int j = i + 1; j <= m; ++j) w2 -= Mm[i][j] * xs[j];
                    if (tid == 0) xs[i] = w2 / Mm[i][i];
                    wave_sync();
                }
            }
            if (tid < m) coef[tid] = ok ? xs[tid] : (tid == slot ? 1.0 : 0.0);
        }
        __syncthreads();
        for (int k = tid; k < S.L; k += NT) {
            double x = 0.0;
            for (int q = 0; q < nh; ++q) x += coef[q] * Hist[q * S.L + k];
            T1[k] = x;
        }
        __syncthreads();
        // correlation energy: f_ia t_i^a + sum over i < j, a < b of <ij||ab> tau_ij^ab
        double e = 0.0;
        for (int k = tid; k < S.nT2; k += NT) {
            int c, io, iv, i, j, a, b;
            decode(k, c, io, iv, i, j, a, b);
            e += asy(xo(i), so(i), xo(j), so(j), xv(a), sv(a), xv(b), sv(b)) *
                 (T2[k] + t1(i, a) * t1(j, b) - t1(i, b) * t1(j, a));
        }
        for (int k = tid; k < n0; k += NT) e += f(so(kl[k] & 255), xo(kl[k] & 255), xv(kl[k] >> 8)) * T1[k];
        e_cc = block_sum(e, sh);
        __syncthreads();
        if (dmax < A.tol && fabs(e_cc - e_old) < 1e-2 * A.tol) {
            conv = 1;
            break;
        }
        e_old = e_cc;
    }
    if (S.L == 0) conv = 1;
    double e_t = 0.0;
    if (conv && A.triples) {
        // unique triples i<j<k, a<b<c, ranked by combination index
        const int nocc3 = o * (o - 1) * (o - 2) / 6, nvir3 = v * (v - 1) * (v - 2) / 6;
        auto unrank3 = [](int r, int m, int &x, int &y, int &z) {
            // lexicographic: x < y < z < m
            for (x = 0;; ++x) {
                const int c = (m - x - 1) * (m - x - 2) / 2;
                if (r < c) break;
                r -= c;
            }
            for (y = x + 1;; ++y) {
                const int c = m - y - 1;
                if (r < c) break;
                r -= c;
            }
            z = y + 1 + r;
        };
        for (int k = tid; k < nocc3 * nvir3; k += NT) {
            int i, j, kk, a, b, c;
            unrank3(k / nvir3, o, i, j, kk);
            unrank3(k % nvir3, v, a, b, c);
            if (so(i) + so(j) + so(kk) != sv(a) + sv(b) + sv(c)) continue;   // spin-forbidden: no amplitude
            const int I[3] = {i, j, kk}, Av[3] = {a, b, c};
            double x = 0.0, y = 0.0;
            // P(i/jk): (i,j,k) +, (j,i,k) -, (k,j,i) -; the same for (a/bc)
            for (int pi = 0; pi < 3; ++pi) {
                const int p1 = I[pi], p2 = I[pi == 1 ? 0 : 1], p3 = I[pi == 2 ? 0 : 2];
                const double sg = pi == 0 ? 1.0 : -1.0;
                for (int pa = 0; pa < 3; ++pa) {
                    const int q1 = Av[pa], q2 = Av[pa == 1 ? 0 : 1], q3 = Av[pa == 2 ? 0 : 2];
                    const double s = sg * (pa == 0 ? 1.0 : -1.0);
                    double u = 0.0;
                    const int se = so(p2) + so(p3) - sv(q1), sm = sv(q2) + sv(q3) - so(p1);
                    if (se == 0 || se == 1)
                        for (int e = v0(se); e < v0(se + 1); ++e)
                            u += t2(p2, p3, q1, e) *
                                 asy(xv(e), se, xo(p1), so(p1), xv(q2), sv(q2), xv(q3), sv(q3));
                    if (sm == 0 || sm == 1)
                        for (int m = o0(sm); m < o0(sm + 1); ++m)
                            u -= t2(p1, m, q2, q3) * asy(xo(m), sm, xv(q1), sv(q1), xo(p2), so(p2), xo(p3), so(p3));
                    x += s * u;
                    y += s * t1(p1, q1) * asy(xo(p2), so(p2), xo(p3), so(p3), xv(q2), sv(q2), xv(q3), sv(q3));
                }
            }
            e_t += x * (x + y) / (foo(i) + foo(j) + foo(kk) - fvv(a) - fvv(b) - fvv(c));
        }
        e_t = block_sum(e_t, sh);
    }
    if (tid == 0) {
        A.out[t] = conv ? A.e_const + eref + e_cc + e_t : __builtin_nan("");
        A.status[t] = conv ? 0 : 2;
    }
}

hipError_t launch_ccsd_lds(const double *h, const double *eri, int n, const int32_t *act, const int32_t *nact,
                           const int32_t *core, const int32_t *ncore, int stride, int nalpha, int nbeta, double e_const,
                           int ntup, size_t lds, double *work, int64_t slice, int triples, int max_iter, double tol,
                           double *out, int32_t *status, hipStream_t s) {
    if (ntup <= 0) return hipSuccess;
    CcsArgs a{h, eri, n, act, nact, core, ncore, stride, nalpha, nbeta, e_const, work, slice, triples, max_iter, tol,
              out, status};
    hipLaunchKernelGGL(k_ccsd_lds, dim3(ntup), dim3(kCcsThreads), lds, s, a);
    return hipGetLastError();
}

hipError_t init_ccs_kernels() {
    return hipFuncSetAttribute((const void *)k_ccsd_lds, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kCcsMaxLds);
}

}  // namespace mbefci
