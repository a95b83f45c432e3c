"""Measured cases: what a program of this library spends its time on.

Every case is one call (or the few calls that belong together) through the
Python entry points of paper_1905_02786_amd, over the sizes that the library
is used at:

* sigma    H times a few vectors on one tuple's CAS (Context.tuple_sigma): the
           building block for a caller's own eigensolver or response solver;
* expand   a whole many-body expansion (Context.run), closed and open shell,
           with and without screening and spin targeting;
* tuples   CASCI energies of a list of tuples of one order
           (Context.solve_tuples): one worker's share of a large order;
* grad     summed energy and its gradient with respect to every integral
           (autograd.MBEFCIEnergy forward and backward);
* base     coupled-cluster base energies of a list of tuples
           (Context.tuple_base, CCSD and CCSD(T));
* hf       integrals in, Hartree-Fock orbitals and the transformed
           Hamiltonian out (Context.set_hamiltonian, hf, hamiltonian).

Hamiltonians are seeded random ones of the recipe of the 24-orbital order
sweep: orbital energies -1.3 .. -0.5 (occupied) and 0.2 .. 2.5 (virtual),
off-diagonal h of deviation 0.05, and (pq|rs) = sum_L B^L_pq B^L_rs with
2.5 n symmetric Gaussian B^L whose variances add up to `scale` (0.2 there).
The cases that need a mean-field reference (base, hf) use a weaker coupling,
at which the Hartree-Fock determinant is a sensible one.

Increments are not returned beside the energies: they are the energies' own
signed sums (Eq. 3), of the size of the solver's tolerance at high orders.
"""
import itertools
import math

import numpy as np
import torch

import paper_1905_02786_amd as M
from paper_1905_02786_amd.autograd import MBEFCIEnergy

BASE = dict(nalpha=6, nbeta=6, nfrozen=0, ref0=3, nref=6, order=0, count=1, scale=0.2, a=0.0, spin_shift=0.0)


def _case(kind, **kw):
    return {**BASE, "kind": kind, **kw}


def listed():
    return [
        # the smallest call: one product on the reference space of the 24-orbital
        # problem, 400 determinants; launches and host work count
        _case("sigma", name="sigma (6e,6o)", norb=24, nfrozen=1, nvec=1),
        # a block of three vectors on one of the largest spaces of the 60-orbital
        # problem, 627,264 determinants
        _case("sigma", name="sigma (10e,12o) x3", norb=60, ref0=2, nref=8, order=4, nvec=3, nocc=1),
        # a small molecule in a minimal basis, frozen core, full order: 32 tuples
        _case("expand", name="expand 8 orbitals", norb=8, nalpha=3, nbeta=3, nfrozen=1, ref0=2, nref=2, max_order=5,
              a=5.0),
        # full order and no screening on 10 orbitals: 256 tuples up to 44,100 determinants
        _case("expand", name="expand 10 orbitals", norb=10, nalpha=4, nbeta=4, ref0=3, nref=2, max_order=8),
        # open shell, the lowest doublet by the level shift, 11 orbitals, truncated order
        _case("expand", name="expand 11 orbitals doublet", norb=11, nalpha=5, nbeta=4, ref0=3, nref=3, max_order=4,
              spin_shift=1.0),
        # the order sweep of the 24-orbital problem through order 3: 834 tuples
        _case("expand", name="expand 24 orbitals", norb=24, nfrozen=1, max_order=3, a=5.0),
        # one worker's share of order 5 of the 24-orbital problem
        _case("tuples", name="tuples 24 orbitals order 5", norb=24, nfrozen=1, order=5, count=151),
        # one worker's share of order 4 of the 60-orbital problem, the largest spaces
        _case("tuples", name="tuples 60 orbitals order 4", norb=60, ref0=2, nref=8, order=4, count=61, scale=0.375),
        # energy and gradient of a truncated expansion, tuples solved again in the backward pass
        _case("grad", name="gradient 10 orbitals", norb=10, nalpha=4, nbeta=4, ref0=3, nref=2, max_order=3, formed=0),
        # energy and gradient formed together, 24 orbitals, order 2
        _case("grad", name="gradient 24 orbitals", norb=24, nfrozen=1, max_order=2, formed=1),
        # CCSD(T) bases of the order-3 tuples of the 24-orbital problem
        _case("base", name="CCSD(T) base order 3", norb=24, nfrozen=1, order=3, count=680, scale=0.1, model=3),
        # Hartree-Fock orbitals of the 24-orbital problem
        _case("hf", name="Hartree-Fock 24 orbitals", norb=24, nfrozen=1, scale=0.1),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same kinds, sizes over the whole range."""
    top = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["sigma", "expand", "tuples", "grad", "base", "hf"])
        if kind in ("sigma", "tuples", "base"):
            n = rng.randint(14, 60 if kind != "base" else 32)
            ne = rng.randint(4, 7)
            open_ = rng.choice([0, 0, 1]) if kind != "base" else 0
            nref = rng.randint(4, 8)
            ref0 = max(1, ne - open_ - rng.randint(2, 4))
            order = rng.randint(0, 5 if kind != "base" else 4)
            c = _case(kind, norb=n, nalpha=ne, nbeta=ne - open_, nfrozen=rng.randint(0, 1), ref0=ref0, nref=nref,
                      order=order)
            if kind == "sigma":
                c.update(nvec=_log_int(rng, 1, 8), nocc=rng.randint(0, 2))
            elif kind == "tuples":
                c.update(count=_log_int(rng, 4, 200))
            else:
                c.update(count=_log_int(rng, 4, 700), scale=0.1, model=rng.choice([2, 3, 3]))
        elif kind in ("expand", "grad"):
            small = rng.random() < 0.6
            n = rng.randint(7, 11) if small else rng.randint(12, 26)
            ne = rng.randint(3, 5) if small else rng.randint(4, 6)
            open_ = rng.choice([0, 0, 1])
            c = _case(kind, norb=n, nalpha=ne, nbeta=ne - open_, nfrozen=rng.randint(0, 1), ref0=ne - rng.randint(1, 2),
                      nref=rng.randint(2, 4) if small else rng.randint(3, 6),
                      max_order=rng.randint(3, 8) if small else rng.randint(1, 3), a=rng.choice([0.0, 2.5, 5.0]))
            if kind == "grad":
                c.update(a=0.0, max_order=min(c["max_order"], 4), formed=rng.randint(0, 1))
            elif rng.random() < 0.25:
                c.update(a=0.0, spin_shift=1.0)
        else:
            n = rng.randint(8, 40)
            ne = rng.randint(3, 6)
            c = _case(kind, norb=n, nalpha=ne, nbeta=ne, ref0=ne - 1, nref=2, scale=0.1 if n > 16 else 0.05)
        if _valid(c) and _cost(c) <= top:
            return c


def _valid(c):
    ref = range(c["ref0"], c["ref0"] + c["nref"])
    n, na, nb = c["norb"], c["nalpha"], c["nbeta"]
    if ref[0] < c["nfrozen"] or ref[-1] >= n - 1 or na > nb and not set(range(nb, na)) <= set(ref):
        return False
    if c["kind"] == "hf":
        return True
    x = _expansion(c)
    kmax = c["order"] if c["kind"] in ("sigma", "tuples", "base") else min(c["max_order"], len(x))
    if kmax > len(x) or c.get("nocc", 0) > min(c["order"], sum(p < nb for p in x)):
        return False
    if c["kind"] in ("sigma", "tuples", "base") and c.get("count", 1) > math.comb(len(x), c["order"]):
        return False
    if c["nref"] + kmax > 12 and c["kind"] != "base" or c["nref"] + kmax > 11 and c["kind"] == "base":
        return False
    if c["kind"] in ("sigma", "tuples"):
        worst = max(_dim(c, t) for t in _tuples(c))
        return worst >= 4 and worst * c.get("nvec", 1) <= 4_000_000 and worst * len(_tuples(c)) <= 60_000_000
    return sum(math.comb(len(x), k) for k in range(kmax + 1)) <= 2500


def _expansion(c):
    ref = set(range(c["ref0"], c["ref0"] + c["nref"]))
    return [p for p in range(c["nfrozen"], c["norb"]) if p not in ref]


def _space(c, tup):
    """(active orbitals, core orbitals, active alpha, active beta electrons) of a tuple."""
    act = sorted(set(range(c["ref0"], c["ref0"] + c["nref"])) | set(int(p) for p in tup))
    core = [p for p in range(c["nbeta"]) if p not in act]
    return act, core, sum(p < c["nalpha"] for p in act), sum(p < c["nbeta"] for p in act)


def _dim(c, tup):
    act, _, na, nb = _space(c, tup)
    return math.comb(len(act), na) * math.comb(len(act), nb)


def _tuples(c):
    """The tuples of a sigma, tuples or base case: a regular selection of the
    order's lexicographic list (sigma: one tuple of nocc occupied orbitals)."""
    x, k = _expansion(c), c["order"]
    if k == 0:
        return [()]
    if c["kind"] == "sigma":
        occ, vir = [p for p in x if p < c["nbeta"]], [p for p in x if p >= c["nbeta"]]
        m = min(c.get("nocc", 0), len(occ), k)
        return [tuple(sorted(occ[:m] + vir[2:2 + k - m]))]
    total, count = math.comb(len(x), k), c["count"]
    step = max(1, total // count)
    return list(itertools.islice(itertools.combinations(x, k), 0, step * (count - 1) + 1, step))


def _all_tuples(c):
    x = _expansion(c)
    return [t for k in range(min(c["max_order"], len(x)) + 1) for t in itertools.combinations(x, k)]


def _sigma_flops(c, tup):
    """One product: the pair rows that link each alpha string, times the pair
    matrix, and the two string Hamiltonians."""
    act, _, na, nb = _space(c, tup)
    n = len(act)
    p, s = n * (n + 1) // 2, math.comb(n, na) + math.comb(n, nb)
    return 2.0 * _dim(c, tup) * ((1 + na * (n - na)) * p + s)


def _cc_flops(c, tup):
    """One CCSD iteration: the ladder, hole-hole and ring contractions over
    the spin-conserving blocks."""
    act, _, na, nb = _space(c, tup)
    o, v = na + nb, 2 * len(act) - na - nb
    return o * o * v ** 4 / 4.0 + o ** 4 * v * v / 4.0 + 2.0 * (o * v) ** 3


APPLICATIONS = 12      # products that even a good start vector needs
CC_ITERATIONS = 12
FOCK_BUILDS = 12


def work(case):
    c, n = case, case["norb"]
    ints = 8.0 * (n * n + n ** 4 / 8)
    if c["kind"] == "sigma":
        t = _tuples(c)[0]
        return {"bytes": 16.0 * _dim(c, t) * c["nvec"], "flops": _sigma_flops(c, t) * c["nvec"]}
    if c["kind"] == "hf":
        return {"bytes": 8.0 * 2 * n ** 4, "flops": 4.0 * n ** 4 * FOCK_BUILDS + 8.0 * n ** 5}
    if c["kind"] == "base":
        return {"bytes": ints + 8.0 * c["count"], "flops": CC_ITERATIONS * sum(_cc_flops(c, t) for t in _tuples(c))}
    ts = _tuples(c) if c["kind"] == "tuples" else _all_tuples(c)
    flops = APPLICATIONS * sum(_sigma_flops(c, t) for t in ts)
    if c["kind"] == "grad":
        return {"bytes": ints + 8.0 * (n * n + n ** 4), "flops": 2.0 * flops}
    return {"bytes": ints + 8.0 * len(ts), "flops": flops}


def _cost(c):
    """Rough time of a pass, for draw()."""
    w = work(c)
    return w["flops"] / (2e12 if c["kind"] in ("sigma", "tuples") else 2e11) + w["bytes"] / 1e11


# ------------------------------------------------------------------ inputs --

def _hamiltonian(c, seed):
    n, no = c["norb"], c["nbeta"]
    rng = np.random.default_rng(seed)
    h = np.triu(rng.normal(0.0, 0.05, (n, n)), 1)
    h = h + h.T + np.diag(np.concatenate([np.linspace(-1.3, -0.5, no), np.linspace(0.2, 2.5, n - no)]))
    nvec = max(20, int(2.5 * n))
    b = rng.normal(0.0, math.sqrt(c["scale"] / nvec), (nvec, n, n))
    b = (np.triu(b) + np.triu(b, 1).transpose(0, 2, 1)).reshape(nvec, n * n)
    eri = b.T @ b
    return h, (0.5 * (eri + eri.T)).reshape(n, n, n, n)


def _fock(h, eri, dm):
    n = len(h)
    ex = np.ascontiguousarray(eri.transpose(0, 2, 1, 3)).reshape(n * n, n * n)
    d = dm.reshape(-1)
    return h + 2.0 * (eri.reshape(n * n, n * n) @ d).reshape(n, n) - (ex @ d).reshape(n, n)


def _scf(h, eri, no):
    """Closed-shell orbitals (columns, ascending, largest entry positive) and
    the energy, by DIIS on a level shift that is released."""
    n = len(h)
    orb = np.linalg.eigh(h)[1]
    fs, es = [], []
    for it in range(300):
        dm = orb[:, :no] @ orb[:, :no].T
        f = _fock(h, eri, dm)
        err = f @ dm - dm @ f
        if np.abs(err).max() < 2e-14 * n:
            break
        fs, es = (fs + [f])[-8:], (es + [err])[-8:]
        m = len(fs)
        a = -np.ones((m + 1, m + 1))
        a[m, m] = 0.0
        a[:m, :m] = [[np.sum(x * y) for y in es] for x in es]
        a[:m, :m] /= max(a[i, i] for i in range(m))
        w = np.linalg.lstsq(a, np.r_[np.zeros(m), -1.0], rcond=None)[0][:m]
        g = sum(x * y for x, y in zip(w, fs))
        orb = np.linalg.eigh(g + (np.eye(n) - dm if it < 12 else 0.0))[1]
    energy = float(np.sum(dm * (h + f)))
    # canonical within the occupied and within the virtual block
    cols = []
    for p in (orb[:, :no], orb[:, no:]):
        cols.append(p @ np.linalg.eigh(p.T @ f @ p)[1])
    orb = np.concatenate(cols, axis=1)
    big = np.abs(orb).argmax(axis=0)
    return orb * np.sign(orb[big, np.arange(n)]), energy


def _rotate(h, eri, u):
    n = len(h)
    for _ in range(4):   # contract the last index, move it to the front
        eri = (u.T @ eri.reshape(n ** 3, n).T).reshape(n, n, n, n)
    h, eri = u.T @ h @ u, eri.reshape(n * n, n * n)
    eri = 0.5 * (eri + eri.T)
    t = eri.reshape(n, n, n, n)
    t = 0.5 * (t + t.transpose(1, 0, 2, 3))
    return 0.5 * (h + h.T), 0.5 * (t + t.transpose(0, 1, 3, 2))


def _inputs(c, seed):
    h, eri = _hamiltonian(c, seed)
    if c["kind"] == "base":   # canonical orbitals, as the (T) correction needs
        h, eri = _rotate(h, eri, _scf(h, eri, c["nbeta"])[0])
    return h, eri


def _vectors(c, seed):
    dim = _dim(c, _tuples(c)[0])
    g = torch.Generator(device="cuda").manual_seed(seed)
    v = torch.randn(c["nvec"], dim, dtype=torch.float64, device="cuda", generator=g)
    return v / v.norm(dim=1, keepdim=True)


def prepare(case, seed):
    c = case
    h, eri = _inputs(c, seed)
    ref = list(range(c["ref0"], c["ref0"] + c["nref"]))
    st = {"case": c, "kind": c["kind"]}
    opts = dict(a=c["a"], max_order=c.get("max_order", 0), spin_shift=c["spin_shift"])
    if c["kind"] == "grad":
        st["h"], st["eri"] = (torch.tensor(x, device="cuda", requires_grad=True) for x in (h, eri))
        st["spec"] = dict(nalpha=c["nalpha"], nbeta=c["nbeta"], nfrozen=c["nfrozen"], ref=ref, gradient=c["formed"],
                          a=c["a"], max_order=c["max_order"])
        st["ws"] = M.workspace(4 << 30)
        return st
    ctx = M.Context(device=0)
    ctx.set_hamiltonian(h, eri)
    ctx.set_spaces(c["nalpha"], c["nbeta"], c["nfrozen"], ref)
    if c["kind"] == "base":
        opts["base_model"] = c["model"]
    ctx.set_options(**opts)
    st["ctx"] = ctx
    if c["kind"] == "hf":
        st.update(h=h, eri=eri, ref=ref, ws=M.workspace(1 << 30))
    elif c["kind"] == "expand":
        st["ws"] = M.workspace(8 << 30)
    else:
        st["tuples"] = _tuples(c)
        if c["kind"] == "sigma":
            st["c"] = _vectors(c, seed)
        st["ws"] = M.workspace((8 if c["kind"] == "tuples" else 4) << 30)
    return st


def run(state):
    kind, c, ws = state["kind"], state["case"], state["ws"]
    if kind == "sigma":
        return state["ctx"].tuple_sigma(c["order"], state["tuples"][0], state["c"], ws)
    if kind == "expand":
        res = state["ctx"].run(ws)
        return {"eps": [o.eps for o in res.orders], "status": [o.status for o in res.orders],
                "total": np.float64(res.total), "tuples": [o.tuples for o in res.orders]}
    if kind == "tuples":
        eps, status = state["ctx"].solve_tuples(c["order"], state["tuples"], ws)
        return {"eps": eps, "status": status}
    if kind == "grad":
        state["h"].grad = state["eri"].grad = None
        e = MBEFCIEnergy.apply(state["h"], state["eri"], state["spec"], ws)
        e.backward()
        return {"energy": e.detach(), "dh": state["h"].grad, "deri": state["eri"].grad}
    if kind == "base":
        return state["ctx"].tuple_base(c["order"], state["tuples"], ws)
    ctx = state["ctx"]
    ctx.set_hamiltonian(state["h"], state["eri"])
    out = ctx.hf(ws)
    h, eri, _ = ctx.hamiltonian()
    return {"energy": np.float64(out["energy"]), "U": out["U"], "h": h, "eri": eri}


# ------------------------------------------------- the same in plain torch --

def _dev():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _string_ops(n, k):
    """Dense E_pq on the strings of k electrons in n orbitals: [n, n, S, S]."""
    strs = [m for m in range(1 << n) if bin(m).count("1") == k]
    at = {m: i for i, m in enumerate(strs)}
    e = np.zeros((n, n, len(strs), len(strs)))
    for j, m in enumerate(strs):
        for q in range(n):
            if not m >> q & 1:
                continue
            r = m ^ (1 << q)
            s1 = bin(m & ((1 << q) - 1)).count("1")
            for p in range(n):
                if not r >> p & 1:
                    s2 = bin(r & ((1 << p) - 1)).count("1")
                    e[p, q, at[r | 1 << p], j] = -1.0 if (s1 + s2) & 1 else 1.0
    return torch.tensor(e, device=_dev())


class _Cas:
    """H = e_core + sum k_pq E_pq + 1/2 sum (pq|rs) E_pq E_rs of several tuples
    of one shape (the frozen core in h), applied to batches [B, Sa, Sb]."""

    def __init__(self, c, h, eri, tuples, ops):
        sp = [_space(c, t) for t in tuples]
        n, na, nb = len(sp[0][0]), sp[0][2], sp[0][3]
        hs, es, ec = [], [], []
        for act, core, _, _ in sp:
            ia = np.ix_(act, act)
            heff = h[ia].copy()
            e0 = 2.0 * sum(h[k, k] for k in core)
            for k in core:
                heff += 2.0 * eri[:, :, k, k][ia] - eri[:, k, k, :][ia]
                e0 += sum(2.0 * eri[k, k, j, j] - eri[k, j, j, k] for j in core)
            g = eri[np.ix_(act, act, act, act)]
            hs.append(heff - 0.5 * np.einsum("prrq->pq", g))
            es.append(g.reshape(n * n, n * n))
            ec.append(e0)
        dev = _dev()
        self.k, self.g = (torch.tensor(np.array(x), device=dev) for x in (hs, es))
        self.core = torch.tensor(np.array(ec), device=dev)
        for key in ((n, na), (n, nb)):
            if key not in ops:
                ops[key] = _string_ops(*key)
        self.ea, self.eb = ops[n, na], ops[n, nb]
        self.n, self.lam, self.nb = n, c["spin_shift"], nb
        self.shape = (len(tuples), self.ea.shape[2], self.eb.shape[2])
        self.dim = self.shape[1] * self.shape[2]

    def moved(self, x):
        """E_pq x, [B, n^2, Sa, Sb]."""
        b, sa, sb = x.shape
        n2 = self.n * self.n
        d = (self.ea.reshape(n2 * sa, sa) @ x).reshape(b, n2, sa, sb)
        r = x.reshape(b * sa, sb) @ self.eb.reshape(n2, sb, sb).transpose(1, 2).contiguous().permute(1, 0, 2).reshape(sb, n2 * sb)
        return d + r.reshape(b, sa, n2, sb).transpose(1, 2)

    def apply(self, x, core=False):
        b, sa, sb = x.shape
        n2 = self.n * self.n
        d = self.moved(x).reshape(b, n2, sa * sb)
        w = 0.5 * (self.g @ d) + self.k.reshape(b, n2, 1) * x.reshape(b, 1, sa * sb)
        w = w.reshape(b, n2, sa, sb)
        y = self.ea.permute(2, 0, 1, 3).reshape(sa, n2 * sa) @ w.reshape(b, n2 * sa, sb)
        y = y + w.transpose(1, 2).reshape(b * sa, n2 * sb).matmul(
            self.eb.reshape(n2, sb, sb).transpose(1, 2).reshape(n2 * sb, sb)).reshape(b, sa, sb)
        if self.lam:
            # S-S+ = N_beta - sum_pq Ea_qp Eb_pq
            s = torch.zeros_like(y)
            for p in range(self.n):
                for q in range(self.n):
                    s += self.ea[q, p] @ x @ self.eb[p, q].T
            y = y + self.lam * (self.nb * x - s)
        return y + self.core.reshape(b, 1, 1) * x if core else y

    def matrix(self, i):
        """H of tuple i, column by column."""
        k, g = self.k, self.g
        eye = torch.eye(self.dim, dtype=torch.float64, device=_dev()).reshape(self.dim, *self.shape[1:])
        cols = []
        for j in range(0, self.dim, 128):
            x = eye[j:j + 128]
            self.k, self.g = k[i:i + 1].expand(len(x), -1, -1), g[i:i + 1]
            cols.append(self.apply(x).reshape(len(x), self.dim))
        self.k, self.g = k, g
        h = torch.cat(cols)
        return (0.5 * (h + h.T)).cpu().numpy()

    def lowest(self):
        """Lowest eigenvalue (without e_core) and vector of every tuple."""
        b, sa, sb = self.shape
        if self.dim <= 900:
            vals, vecs = [], []
            for i in range(b):
                w, v = np.linalg.eigh(self.matrix(i))
                vals.append(w[0])
                vecs.append(v[:, 0])
            dev = _dev()
            return (torch.tensor(np.array(vals), device=dev),
                    torch.tensor(np.array(vecs), device=dev).reshape(b, sa, sb))
        g = torch.Generator(device=_dev()).manual_seed(1)
        x = torch.randn(b, self.dim, dtype=torch.float64, device=_dev(), generator=g)
        m = 70
        for _ in range(20):   # Lanczos with full orthogonalisation, restarted
            x = x / x.norm(dim=1, keepdim=True)
            q = torch.empty(b, m, self.dim, dtype=torch.float64, device=_dev())
            t = torch.zeros(b, m, m, dtype=torch.float64, device=_dev())
            q[:, 0] = x
            for j in range(m):
                r = self.apply(q[:, j].reshape(b, sa, sb)).reshape(b, self.dim)
                if j == 0:
                    th = (x * r).sum(1, keepdim=True)
                    res = (r - th * x).norm(dim=1).max()
                t[:, j, j] = (r * q[:, j]).sum(1)
                for _ in range(2):
                    r = r - ((q[:, :j + 1] @ r.unsqueeze(2)).transpose(1, 2) @ q[:, :j + 1]).squeeze(1)
                if j + 1 < m:
                    nr = r.norm(dim=1)
                    t[:, j, j + 1] = t[:, j + 1, j] = nr
                    q[:, j + 1] = r / nr.clamp_min(1e-300).unsqueeze(1)
            if res < 1e-11:
                return th.squeeze(1), x.reshape(b, sa, sb)
            y = torch.linalg.eigh(t.cpu())[1][:, :, 0].to(_dev())
            x = (y.unsqueeze(1) @ q).squeeze(1)
        raise RuntimeError("no convergence")


def _solve(c, h, eri, tuples, vectors=False):
    """{tuple: energy or (energy, vector, shape class)} of the tuples."""
    groups, ops, out = {}, {}, {}
    for t in tuples:
        act, core, na, nb = _space(c, t)
        groups.setdefault((len(act), na, nb), []).append(t)
    for (n, na, nb), ts in groups.items():
        dim = math.comb(n, na) * math.comb(n, nb)
        step = max(1, int(2e9 / (8.0 * dim * (2 * n * n + 80))))
        for i in range(0, len(ts), step):
            cas = _Cas(c, h, eri, ts[i:i + step], ops)
            e, x = cas.lowest()
            e = (e + cas.core).cpu().numpy()
            for j, t in enumerate(ts[i:i + step]):
                out[t] = float(e[j])
            if vectors:
                d = cas.moved(x).reshape(len(e), n * n, dim)
                gram = d @ d.transpose(1, 2).contiguous()
                gam = (d @ x.reshape(len(e), dim, 1)).squeeze(2)
                for j, t in enumerate(ts[i:i + step]):
                    out[t] = float(e[j]), gam[j].cpu().numpy().reshape(n, n), gram[j].cpu().numpy()
    return out


def _exact_seconds(c, tuples):
    s = 0.0
    for t in tuples:
        act, _, na, nb = _space(c, t)
        n, dim = len(act), _dim(c, t)
        if dim > 900:
            sa, sb = math.comb(n, na), math.comb(n, nb)
            s += 150 * (4.0 * n * n * dim * (sa + sb) / 3e13 + 1e-3 / 20) * (3 if c["spin_shift"] else 1)
        else:
            s += 2e-9 * dim ** 3 / 3 + 3e-3
    return s


def _exact_expand(c, h, eri):
    x = _expansion(c)
    eps, inc, orders, sums = {}, {}, [], []
    for k in range(min(c["max_order"], len(x)) + 1):
        ts = list(itertools.combinations(x, k))
        if k >= 2 and c["a"] > 0:
            tau = 1e-10 * c["a"] ** (k - 2)
            ts = [t for t in ts if any(abs(inc.get(s, 0.0)) >= tau for s in itertools.combinations(t, k - 1))]
        if not ts:
            break
        eps.update(_solve(c, h, eri, ts))
        for t in ts:
            inc[t] = eps[t] - sum(inc.get(s, 0.0) for j in range(k) for s in itertools.combinations(t, j))
        orders.append(ts)
        sums.append(sum(inc[t] for t in ts))
    return {"eps": [np.array([eps[t] for t in ts]) for ts in orders], "status": None, "total": np.float64(sum(sums)),
            "tuples": None}


def _exact_grad(c, h, eri):
    n, ts = c["norb"], _all_tuples(c)
    got = _solve(c, h, eri, ts, vectors=True)
    w = {}
    for t in reversed(ts):   # supersets come later in the list
        w.setdefault(t, 1)
        for j in range(len(t)):
            for s in itertools.combinations(t, j):
                w[s] = w.get(s, 1) - w[t]
    e, gh, ge = 0.0, np.zeros((n, n)), np.zeros((n, n, n, n))
    for t in ts:
        if w[t] == 0:
            continue
        act, core, _, _ = _space(c, t)
        m = len(act)
        en, gam, gram = got[t]
        e += w[t] * en
        # <E_pq E_rs> = (E_qp x, E_rs x)
        two = gram.reshape(m, m, m, m).transpose(1, 0, 2, 3).copy()
        for q in range(m):
            two[:, q, q, :] -= gam
        one = np.zeros((n, n))
        one[np.ix_(act, act)] = gam
        gh += w[t] * one
        ge[np.ix_(act, act, act, act)] += 0.5 * w[t] * two
        for k in core:
            gh[k, k] += 2.0 * w[t]
            ge[:, :, k, k] += w[t] * one
            ge[k, k, :, :] += w[t] * one
            ge[:, k, k, :] -= 0.5 * w[t] * one
            ge[k, :, :, k] -= 0.5 * w[t] * one.T
            for j in core:
                ge[k, k, j, j] += 2.0 * w[t]
                ge[k, j, j, k] -= 1.0 * w[t]
    return {"energy": torch.tensor(e, dtype=torch.float64), "dh": gh, "deri": ge}


def _exact_cc(c, h, eri, tuples):
    """Spin-orbital CCSD (and (T)) energies of tuples of one shape, batched."""
    act0, _, na, nb = _space(c, tuples[0])
    m, no = len(act0), na + nb
    nv, dev = 2 * m - no, _dev()
    so = [(i, 0) for i in range(na)] + [(i, 1) for i in range(nb)] + \
         [(i, 0) for i in range(na, m)] + [(i, 1) for i in range(nb, m)]   # active orbitals ascend: occupied first
    orb, spin = [s[0] for s in so], np.array([s[1] for s in so])
    same = torch.tensor((spin[:, None] == spin[None, :]).astype(float), device=dev)
    fs, vs, e0 = [], [], []
    for t in tuples:
        act, core, _, _ = _space(c, t)
        heff = h[np.ix_(act, act)].copy()
        ec = 2.0 * sum(h[k, k] for k in core)
        for k in core:
            heff += 2.0 * eri[:, :, k, k][np.ix_(act, act)] - eri[:, k, k, :][np.ix_(act, act)]
            ec += sum(2.0 * eri[k, k, j, j] - eri[k, j, j, k] for j in core)
        g = torch.tensor(eri[np.ix_(act, act, act, act)], device=dev)[orb][:, orb][:, :, orb][:, :, :, orb]
        g = g * same[:, :, None, None] * same[None, None]
        v = g.permute(0, 2, 1, 3)
        v = v - v.permute(0, 1, 3, 2)
        f = torch.tensor(heff, device=dev)[orb][:, orb] * same
        ec += float(torch.diagonal(f)[:no].sum())
        f = f + torch.einsum("pmqm->pq", v[:, :no, :, :no])
        ec += 0.5 * float(torch.einsum("mnmn->", v[:no, :no, :no, :no]))
        fs.append(f)
        vs.append(v)
        e0.append(ec)
    f, v = torch.stack(fs), torch.stack(vs)
    O, V = slice(0, no), slice(no, None)
    d = torch.diagonal(f, dim1=1, dim2=2)
    d1 = d[:, :no, None] - d[:, None, no:]
    d2 = d1[:, :, None, :, None] + d1[:, None, :, None, :]
    fo = f - torch.diag_embed(d)
    ein = torch.einsum
    oo, ov, vv = fo[:, O, O], fo[:, O, V], fo[:, V, V]
    oooo, ooov, oovv = v[:, O, O, O, O], v[:, O, O, O, V], v[:, O, O, V, V]
    ovov, ovvo, ovvv, vvvv = v[:, O, V, O, V], v[:, O, V, V, O], v[:, O, V, V, V], v[:, V, V, V, V]
    ovoo, oovo, vovv = v[:, O, V, O, O], v[:, O, O, V, O], v[:, V, O, V, V]
    t1, t2 = ov / d1, oovv / d2
    hist = []
    for _ in range(200):
        tt = ein("xia,xjb->xijab", t1, t1)
        tt = tt - tt.transpose(3, 4)
        tau, tau_ = t2 + tt, t2 + 0.5 * tt
        fae = vv - 0.5 * ein("xme,xma->xae", ov, t1) + ein("xmf,xmafe->xae", t1, ovvv) \
            - 0.5 * ein("xmnaf,xmnef->xae", tau_, oovv)
        fmi = oo + 0.5 * ein("xie,xme->xmi", t1, ov) + ein("xne,xmnie->xmi", t1, ooov) \
            + 0.5 * ein("xinef,xmnef->xmi", tau_, oovv)
        fme = ov + ein("xnf,xmnef->xme", t1, oovv)
        w = ein("xje,xmnie->xmnij", t1, ooov)
        wo = oooo + w - w.transpose(3, 4) + 0.25 * ein("xijef,xmnef->xmnij", tau, oovv)
        w = ein("xmb,xamef->xabef", t1, vovv)
        wv = vvvv - w + w.transpose(1, 2) + 0.25 * ein("xmnab,xmnef->xabef", tau, oovv)
        wr = ovvo + ein("xjf,xmbef->xmbej", t1, ovvv) - ein("xnb,xmnej->xmbej", t1, oovo) \
            - ein("xjnfb,xmnef->xmbej", 0.5 * t2 + ein("xjf,xnb->xjnfb", t1, t1), oovv)
        n1 = ov + ein("xie,xae->xia", t1, fae) - ein("xma,xmi->xia", t1, fmi) + ein("ximae,xme->xia", t2, fme) \
            - ein("xnf,xnaif->xia", t1, ovov) - 0.5 * ein("ximef,xmaef->xia", t2, ovvv) \
            - 0.5 * ein("xmnae,xnmei->xia", t2, oovo)
        pa = ein("xijae,xbe->xijab", t2, fae - 0.5 * ein("xmb,xme->xbe", t1, fme))
        pi = ein("ximab,xmj->xijab", t2, fmi + 0.5 * ein("xje,xme->xmj", t1, fme))
        r = ein("ximae,xmbej->xijab", t2, wr) - ein("xie,xma,xmbej->xijab", t1, t1, ovvo)
        r = r - r.transpose(1, 2)
        r = r - r.transpose(3, 4)
        s = ein("xie,xejab->xijab", t1, v[:, V, O, V, V])
        q = ein("xma,xmbij->xijab", t1, ovoo)
        n2 = oovv + pa - pa.transpose(3, 4) - pi + pi.transpose(1, 2) + 0.5 * ein("xmnab,xmnij->xijab", tau, wo) \
            + 0.5 * ein("xijef,xabef->xijab", tau, wv) + r + s - s.transpose(1, 2) - q + q.transpose(3, 4)
        n1, n2 = n1 / d1, n2 / d2
        b = len(n1)
        new = torch.cat([n1.reshape(b, -1), n2.reshape(b, -1)], 1)
        old = torch.cat([t1.reshape(b, -1), t2.reshape(b, -1)], 1)
        step = float((new - old).abs().max())
        hist = (hist + [(new, new - old)])[-6:]
        if len(hist) > 2 and step > 1e-13:   # DIIS per tuple
            es = torch.stack([x[1] for x in hist], 1)
            k = len(hist)
            a = -torch.ones(b, k + 1, k + 1, dtype=torch.float64)
            a[:, k, k] = 0.0
            a[:, :k, :k] = (es @ es.transpose(1, 2).contiguous()).cpu()
            sc = torch.diagonal(a[:, :k, :k], dim1=1, dim2=2).amax(1).clamp_min(1e-300)
            a[:, :k, :k] /= sc[:, None, None]
            rhs = torch.zeros(b, k + 1, 1, dtype=torch.float64)
            rhs[:, k] = -1.0
            co = (torch.linalg.pinv(a, rcond=1e-14) @ rhs)[:, :k].to(dev)
            new = (torch.stack([x[0] for x in hist], 1) * co).sum(1)
        t1, t2 = new[:, :no * nv].reshape(b, no, nv), new[:, no * nv:].reshape(b, no, no, nv, nv)
        if step < 1e-12:
            break
    else:
        raise RuntimeError("no convergence")
    e = ein("xia,xia->x", ov, t1) + 0.25 * ein("xijab,xijab->x", oovv, t2) \
        + 0.5 * ein("xijab,xia,xjb->x", oovv, t1, t1)
    if c["model"] == 3:
        for x in range(len(tuples)):
            con = torch.einsum("jkad,dibc->ijkabc", t2[x], v[x, V, O, V, V]) \
                - torch.einsum("imbc,majk->ijkabc", t2[x], v[x, O, V, O, O])
            dis = torch.einsum("ia,jkbc->ijkabc", t1[x], oovv[x])

            def anti(y):
                y = y - y.permute(1, 0, 2, 3, 4, 5) - y.permute(2, 1, 0, 3, 4, 5)
                return y - y.permute(0, 1, 2, 4, 3, 5) - y.permute(0, 1, 2, 5, 4, 3)
            con, dis = anti(con), anti(dis)
            dd = d1[x]
            d3 = dd[:, None, None, :, None, None] + dd[None, :, None, None, :, None] + dd[None, None, :, None, None, :]
            e[x] += (con * (con + dis) / d3).sum() / 36.0
    return (e.cpu().numpy() + np.array(e0)).tolist()


def exact(case, seed):
    """What run() returns, from dense string operators, restarted Lanczos,
    einsum coupled cluster and a plain SCF, all in 64 bits."""
    c = case
    h, eri = _inputs(c, seed)
    if c["kind"] == "hf":
        u, e = _scf(h, eri, c["nbeta"])
        h2, eri2 = _rotate(h, eri, u)
        return {"energy": np.float64(e), "U": u, "h": h2, "eri": eri2}
    if c["kind"] == "sigma":
        cas = _Cas(c, h, eri, _tuples(c), {})
        x = _vectors(c, seed)
        y = [cas.apply(v.reshape(1, *cas.shape[1:]), core=True).reshape(1, -1) for v in x]
        return torch.cat(y)
    if c["kind"] == "base":
        ts = _tuples(c)
        if sum(_cc_flops(c, t) for t in ts) > 1e11:
            return None
        groups, out = {}, {}
        for t in ts:
            groups.setdefault(_space(c, t)[2:], []).append(t)
        for g in groups.values():
            for i in range(0, len(g), 64):
                out.update(zip(g[i:i + 64], _exact_cc(c, h, eri, g[i:i + 64])))
        return np.array([out[t] for t in ts])
    ts = _tuples(c) if c["kind"] == "tuples" else _all_tuples(c)
    if _exact_seconds(c, ts) > 10.0:
        return None
    if c["kind"] == "tuples":
        got = _solve(c, h, eri, ts)
        return {"eps": np.array([got[t] for t in ts]), "status": None}
    return _exact_expand(c, h, eri) if c["kind"] == "expand" else _exact_grad(c, h, eri)
