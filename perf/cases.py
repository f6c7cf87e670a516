"""Timed work of the exact-diagonalisation library: what its users have it do, by entry point.

A case is a dict of plain values with a "kind" (the entry point) and its sizes. `prepare` makes what
a program holds before the call (states, model handles), `run` is one pass through the public entry
points, `work` the bytes and operations of a pass that no implementation can do without, and `exact`
the same outputs from plain torch / numpy in 64 bits. Every state is complex128.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_1802_10052_amd as P

DEV = "cuda:0"
SX = np.array([[0, 1], [1, 0]], np.complex128)
SZ = np.array([[1, 0], [0, -1]], np.complex128)
SMINUS = np.array([[0, 0], [1, 0]], np.complex128)
XX = np.kron(SX, SX)
YY = np.array([[0, 0, 0, -1], [0, 0, 1, 0], [0, 1, 0, 0], [-1, 0, 0, 0]], np.complex128)
ZZ = np.kron(SZ, SZ)


def listed():
    return [
        # the smallest product, one of thousands that a user's own iteration makes on a short chain:
        # launches and the host path count
        {"name": "apply_tfim_L14", "kind": "apply", "model": "tfim", "L": 14},
        # the library's headline: one product with the transverse-field Ising chain on 2^28 amplitudes
        {"name": "apply_tfim_L28", "kind": "apply", "model": "tfim", "L": 28},
        # the critical Ising chain's ground state, full reorthogonalisation, no restart
        {"name": "lanczos_tfim_L14", "kind": "lanczos", "model": "tfim", "L": 14, "reorth": "full", "basis": 0},
        # the ground state of the XXZ chain with random fields, restarted on 24 stored vectors
        {"name": "lanczos_xxz_L26", "kind": "lanczos", "model": "xxz", "L": 26, "reorth": "partial", "basis": 24},
        # a quench of a short chain with observables every step: ten Krylov steps, small states
        {"name": "quench_xxz_L12", "kind": "krylov", "model": "xxz", "L": 12, "steps": 10},
        # one step (with the observables before and after) of the quench on 2^28 amplitudes
        {"name": "quench_tfim_L28", "kind": "krylov", "model": "tfim", "L": 28, "steps": 1},
        # one fourth-order Suzuki-Trotter step of a long chain with an odd number of sites
        {"name": "trotter_tfim_L27", "kind": "trotter", "model": "tfim", "L": 27, "order": 4, "steps": 1},
        # an Arnoldi step of the dissipative chain's density matrix (2^26 entries)
        {"name": "liouville_L13", "kind": "liouville", "L": 13, "steps": 1},
        # the half-chain entropy and Schmidt spectrum of a complex state, a 2048 x 2048 reduction
        {"name": "entropy_L22", "kind": "entropy", "L": 22, "cut": 11, "real": False},
        # every single-site and two-site density matrix of a state
        {"name": "rdm_L26", "kind": "rdm", "L": 26, "two_site": True},
        # a batch of quantum trajectories of mixed chain lengths, the first ten time steps
        {"name": "traj_mixed_320", "kind": "traj", "n_traj": 320, "Lmin": 8, "Lmax": 16, "steps": 10},
        # the gradient of a final-time observable over the bond couplings of four time slices
        {"name": "adjoint_L20", "kind": "adjoint", "L": 20, "slices": 4},
    ]


def draw(rng):
    """One more case of the listed ranges; chain lengths (logarithms of the sizes) are uniform."""
    kind = rng.choice(["apply", "lanczos", "krylov", "trotter", "liouville", "entropy", "rdm", "traj", "adjoint"])
    if kind == "apply":
        model = rng.choice(["tfim", "xxz", "lrqi", "liouville"])
        return {"kind": kind, "model": model, "L": rng.randint(7, 14) if model == "liouville" else rng.randint(13, 28),
                "field": round(rng.uniform(0.3, 1.5), 3)}
    if kind == "lanczos":
        # ground states with a gap: the Ising chain off its ordered phase (field >= 1), the XXZ chain on an
        # even number of sites (an odd one has a nearly degenerate doublet, whose vectors are not comparable)
        reorth, model = rng.choice(["full", "partial"]), rng.choice(["tfim", "xxz"])
        L = rng.randint(10, 16) if reorth == "full" else rng.randint(17, 25)
        return {"kind": kind, "model": model, "reorth": reorth, "basis": 0 if reorth == "full" else 24,
                "L": L - L % 2 if model == "xxz" else L,
                "field": round(rng.uniform(1.0, 1.5) if model == "tfim" else rng.uniform(0.3, 0.8), 3)}
    if kind == "krylov":
        L = rng.randint(8, 27)
        return {"kind": kind, "model": rng.choice(["tfim", "xxz"]), "L": L, "field": round(rng.uniform(0.3, 1.5), 3),
                "steps": rng.randint(1, 20) if L < 22 else rng.randint(1, 3) if L < 25 else 1}
    if kind == "trotter":
        L = rng.randint(8, 27)
        return {"kind": kind, "model": rng.choice(["tfim", "xxz"]), "L": L, "order": rng.choice([2, 4]),
                "field": round(rng.uniform(0.3, 1.5), 3), "steps": rng.randint(1, 20) if L < 22 else 1}
    if kind == "liouville":
        L = rng.randint(4, 13)
        return {"kind": kind, "L": L, "steps": rng.randint(1, 10) if L < 11 else 1}
    if kind == "entropy":
        L = rng.randint(10, 24)
        return {"kind": kind, "L": L, "cut": rng.randint(max(4, L // 2 - 3), L // 2), "real": rng.random() < 0.5}
    if kind == "rdm":
        return {"kind": kind, "L": rng.randint(10, 28), "two_site": rng.random() < 0.6}
    if kind == "traj":
        hi = rng.randint(9, 16)
        return {"kind": kind, "n_traj": rng.randint(16, 320), "Lmin": rng.randint(6, hi), "Lmax": hi,
                "steps": rng.randint(4, 10)}
    return {"kind": "adjoint", "L": rng.randint(8, 20), "slices": rng.randint(2, 4)}


# ---- models ---------------------------------------------------------------------------------

def _desc(case, seed):
    """Rule-set description of the case's Hamiltonian (fields and couplings from the seed)."""
    L, model = case["L"], case.get("model", "xxz")
    rng = np.random.default_rng([seed, 2])
    f = case.get("field", 0.5)
    d = SimpleNamespace(L=L, site_ops=np.zeros((0, 2, 2)), site_coef=np.zeros((0, L)),
                        bond_ops=np.zeros((0, 4, 4)), bond_coef=np.zeros((0, L - 1)))
    if model == "tfim":
        d.site_ops, d.site_coef = np.array([SX]), np.full((1, L), -f)
        d.bond_ops, d.bond_coef = np.array([ZZ]), np.full((1, L - 1), -1.0)
    elif model == "lrqi":
        phi, r = math.pi / 4, np.arange(1, L, dtype=np.float64)
        d.site_ops, d.site_coef = np.array([SX]), np.full((1, L), -math.sin(phi))
        d.inf_ops, d.inf_ops2, d.inf_coef = np.array([SZ]), np.array([SZ]), np.full((1, L), -math.cos(phi))
        d.inf_f = (r ** -1.5).reshape(1, L - 1)
    else:
        if case["kind"] == "adjoint":  # bonds J_b (xx + yy + zz/2) with J_b = 1: the couplings come per slice
            d.bond_coef = np.stack([np.ones(L - 1), np.ones(L - 1), np.full(L - 1, 0.5)])
        elif case["kind"] in ("liouville", "traj") or model == "liouville":
            d.bond_coef = np.ones((3, L - 1))
        else:
            d.site_ops, d.site_coef = np.array([SZ]), rng.uniform(-f, f, (1, L))
            d.bond_coef = np.stack([np.ones(L - 1), np.ones(L - 1), np.full(L - 1, 0.5)])
        d.bond_ops = np.array([XX, YY, ZZ])
    return d


def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _random_state(L, seed, real=False):
    g = _gen(seed, 11)
    if real:
        v = torch.randn(1 << L, dtype=torch.float64, device=DEV, generator=g).to(torch.complex128)
    else:
        v = torch.randn(1 << L, dtype=torch.complex128, device=DEV, generator=g)
    v /= torch.linalg.vector_norm(v)
    return v


def _product_state(L, seed):
    """Spins near up, each tilted by its own angle: the usual start of a quench."""
    rng = np.random.default_rng([seed, 7])
    v = torch.ones(1, dtype=torch.complex128, device=DEV)
    for th, ph in zip(rng.normal(0.0, 0.4, L), rng.uniform(0, 2 * math.pi, L)):
        s = torch.tensor([math.cos(th / 2), math.sin(th / 2) * complex(math.cos(ph), math.sin(ph))],
                         dtype=torch.complex128, device=DEV)
        v = (v[:, None] * s[None, :]).reshape(-1)
    return v


def _neel(L):
    x = sum(1 << (L - 1 - k) for k in range(L) if k % 2)
    v = torch.zeros(1 << L, dtype=torch.complex128, device=DEV)
    v[x] = 1.0
    return v


GAMMA = 0.1


def _adjoint_args(case, seed):
    L = case["L"]
    J = np.random.default_rng([seed, 5]).uniform(0.5, 1.5, (case["slices"], L - 1))
    return J, np.array([(-1) ** k for k in range(L)], np.float64) / L


# ---- one pass -------------------------------------------------------------------------------

def prepare(case, seed):
    kind, s = case["kind"], SimpleNamespace(kind=case["kind"], case=case)
    if kind in ("apply", "lanczos", "krylov", "trotter"):
        desc = _desc(case, seed)
        if case["model"] == "liouville":
            s.model = P.Liouville(desc, [SMINUS], np.full((1, desc.L), GAMMA))
        else:
            s.model = P.Model(desc)
        s.psi = _product_state(case["L"], seed) if kind in ("krylov", "trotter") else \
            _random_state(s.model.L, seed, real=kind == "lanczos")
        if kind == "apply":
            s.out = torch.empty_like(s.psi)
    elif kind == "liouville":
        s.model = P.Liouville(_desc(case, seed), [SMINUS], np.full((1, case["L"]), GAMMA))
        p = _product_state(case["L"], seed)
        s.psi = (p[:, None] * p.conj()[None, :]).reshape(-1)
    elif kind in ("entropy", "rdm"):
        s.psi = _random_state(case["L"], seed, case.get("real", False))
    elif kind == "traj":
        ls = _lengths(case)
        s.models = [P.Model(_desc({**case, "L": L}, seed)) for L in ls]
        s.psi0 = [_neel(L) for L in ls]
        s.rates = [np.full(L, GAMMA) for L in ls]
        s.which = np.arange(case["n_traj"], dtype=np.int32) % len(ls)
        s.seed = seed
    else:
        s.model = P.Model(_desc(case, seed))
        s.J, s.w = _adjoint_args(case, seed)
        s.psi = _neel(case["L"])
    return s


def _lengths(case):
    return list(range(case["Lmin"], case["Lmax"] + 1, 2))


def run(s):
    c = s.case
    if s.kind == "apply":
        return P.apply_H(s.model, s.psi, s.out)
    if s.kind == "lanczos":
        if c["basis"]:
            e, psi, _ = P.lanczos_ground(s.model, s.psi, tol=1e-10, max_iter=1000, max_basis=c["basis"], n_keep=5,
                                         reorth=c["reorth"])
        else:
            e, psi, _ = P.lanczos_ground(s.model, s.psi, tol=1e-10, max_iter=300, reorth=c["reorth"])
        return [e, psi]
    if s.kind == "krylov":
        psi, obs, _ = P.krylov_evolve(s.model, s.psi, 0.05, c["steps"], m_max=20, tol=1e-10)
        return [psi, obs]
    if s.kind == "liouville":
        psi, obs, _ = P.krylov_evolve(s.model, s.psi, 0.05, c["steps"], m_max=30, tol=1e-10, hermitian=False)
        return [psi, obs]
    if s.kind == "trotter":
        psi, obs = P.trotter_evolve(s.model, s.psi, 0.05, c["steps"], order=c["order"])
        return [psi, obs]
    if s.kind == "entropy":
        return list(P.entropy(s.psi, c["L"], c["cut"], spectrum=True))
    if s.kind == "rdm":
        r1, r2 = P.rdm(s.psi, c["L"], two_site=c["two_site"])
        return [r1, r2] if c["two_site"] else [r1]
    if s.kind == "traj":
        r = P.trajectories(s.models, SMINUS, s.rates, s.psi0, s.which, 0.01, c["steps"], 2, s.seed, m_max=20, tol=1e-10)
        return [r["sz"], r["n_jumps"], r["jump_t"], r["jump_site"]]
    return list(P.evolve_adjoint(s.model, s.J, s.psi, 0.1, s.w, substeps=2, quad_nodes=8, m_fixed=20, m_max=30))


# ---- what a pass cannot do without ----------------------------------------------------------

def _product(L, model):
    """(bytes, flops) of one H psi: the state read once and written once; two real multiply-adds
    per off-diagonal entry with a real coefficient and two for the diagonal."""
    if model == "liouville":
        D = float(1 << (2 * L))
        return 32 * D, D * (4 * 0.5 * 2 * (L - 1) + 4 + 4 * 0.25 * L)
    D = float(1 << L)
    flips = L if model in ("tfim", "lrqi") else 0.5 * (L - 1)
    return 32 * D, D * (4 * flips + 4)


def work(case):
    kind, L = case["kind"], case.get("L", 0)
    if kind == "apply":
        b, f = _product(L, case["model"])
    elif kind == "lanczos":  # about as many products as these chains take to 1e-10
        b, f = _product(L, case["model"])
        n = 6 * L
        b, f = n * b, n * f
    elif kind == "krylov":  # about ten Krylov vectors a step
        b, f = _product(L, case["model"])
        b, f = 10 * case["steps"] * b, 10 * case["steps"] * f
    elif kind == "liouville":
        b, f = _product(L, "liouville")
        b, f = 12 * case["steps"] * b, 12 * case["steps"] * f
    elif kind == "trotter":  # 32 flops an amplitude and gate; the state read and written once a step
        layers = 11 if case["order"] == 4 else 3
        D = float(1 << L)
        b, f = 32 * D * case["steps"], 32 * D * layers * (L - 1) / 2 * case["steps"]
    elif kind == "entropy":
        n, K = float(1 << case["cut"]), float(1 << (L - case["cut"]))
        z = 1 if case["real"] else 4
        b, f = 16 * n * K, z * (n * n * K + 4 / 3 * n ** 3)
    elif kind == "rdm":  # one complex multiply-add per site, or two per pair, on each pair or quad of amplitudes
        D = float(1 << L)
        b = 16 * D
        f = D * (4 * L + (4 * L * (L - 1) / 2 if case["two_site"] else 0))
    elif kind == "traj":
        b = f = 0.0
        for i, l in enumerate(_lengths(case)):
            n = len(range(i, case["n_traj"], len(_lengths(case))))
            pb, pf = _product(l, "xxz")
            b += n * case["steps"] * 8 * pb
            f += n * case["steps"] * 8 * pf
    else:  # forward and backward, two sub-steps of twenty products a slice
        pb, pf = _product(L, "xxz")
        n = case["slices"] * 2 * 20 * 3
        b, f = n * pb, n * pf
    return {"bytes": b, "flops": f}


# ---- the same in plain torch and numpy ------------------------------------------------------

class _Plain:
    """H on a torch state, term by term: a real diagonal, and flips on one or two bits."""

    def __init__(self, desc, J=None):
        L = self.L = desc.L
        self.site = np.zeros((L, 2, 2), np.complex128)
        self.bond = np.zeros((L - 1, 4, 4), np.complex128)
        for op, co in zip(desc.site_ops, desc.site_coef):
            self.site += co[:, None, None] * op
        for op, co in zip(desc.bond_ops, desc.bond_coef):
            self.bond += co[:, None, None] * op
        if J is not None:
            self.bond *= J[:, None, None]
        self.pairs = {}
        if getattr(desc, "inf_f", None) is not None:
            for k in range(L):
                for j in range(k + 1, L):
                    self.pairs[k, j] = desc.inf_coef[0, k] * desc.inf_f[0, j - k - 1]
        self.bound = sum(np.linalg.norm(a, 2) for a in self.site) + sum(np.linalg.norm(a, 2) for a in self.bond) + \
            sum(abs(v) for v in self.pairs.values())
        self._diag = None

    def z(self, k):
        return torch.tensor([1.0, -1.0], dtype=torch.float64, device=DEV).repeat_interleave(1 << (self.L - 1 - k)).repeat(1 << k)

    def diag(self):
        if self._diag is None:
            d = torch.zeros(1 << self.L, dtype=torch.float64, device=DEV)
            for k in range(self.L):
                v = d.view(1 << k, 2, -1)
                for a in range(2):
                    v[:, a] += float(self.site[k, a, a].real)
            for k in range(self.L - 1):
                v = d.view(1 << k, 4, -1)
                for a in range(4):
                    v[:, a] += float(self.bond[k, a, a].real)
            for (k, j), c in self.pairs.items():
                v = d.view(1 << k, 2, 1 << (j - k - 1), 2, -1)
                for a in range(2):
                    for b in range(2):
                        v[:, a, :, b] += float(c) * (1 - 2 * a) * (1 - 2 * b)
            self._diag = d
        return self._diag

    def bond_into(self, out, psi, k, op):
        o, p = out.view(1 << k, 4, -1), psi.view(1 << k, 4, -1)
        for a in range(4):
            for b in range(4):
                if op[a, b] != 0:
                    o[:, a].add_(p[:, b], alpha=complex(op[a, b]))

    def __call__(self, psi):
        out = psi * self.diag()
        for k in range(self.L):
            o, p = out.view(1 << k, 2, -1), psi.view(1 << k, 2, -1)
            for a in range(2):
                if self.site[k, a, 1 - a] != 0:
                    o[:, a].add_(p[:, 1 - a], alpha=complex(self.site[k, a, 1 - a]))
        for k in range(self.L - 1):
            self.bond_into(out, psi, k, self.bond[k] * (1 - np.eye(4)))
        return out


class _PlainLiouville:
    """i Lcal on the superket of a density matrix: the Hamiltonian on both sides and the jumps."""

    def __init__(self, desc):
        self.H, L = _Plain(desc), desc.L
        self.L, self.D = L, 1 << L
        n_up = torch.zeros(self.D, dtype=torch.float64, device=DEV)
        for k in range(L):
            n_up += 0.5 * (1 + self.H.z(k))
        self.decay = 0.5 * GAMMA * n_up
        self.bound = 2 * self.H.bound + 2 * GAMMA * L

    def __call__(self, x):
        D, L = self.D, self.L
        big = _Plain.__new__(_Plain)
        big.L = 2 * L
        rho = x.view(D, D)
        h = self.H
        out = (h.diag()[:, None] - h.diag()[None, :] - 1j * (self.decay[:, None] + self.decay[None, :])) * rho
        out = out.reshape(-1)
        for k in range(L - 1):
            flips = h.bond[k] * (1 - np.eye(4))
            big.bond_into(out, x, k, flips)
            big.bond_into(out, x, L + k, -flips.conj())
        o = out
        for k in range(L):
            ov = o.view(1 << k, 2, 1 << (L - 1), 2, -1)
            xv = x.view(1 << k, 2, 1 << (L - 1), 2, -1)
            ov[:, 1, :, 1].add_(xv[:, 0, :, 0], alpha=1j * GAMMA)
        return out


def _expm_apply(H, psi, t):
    """exp(-i t H) psi by a Taylor series on pieces with |H| t <= 3."""
    n = max(1, math.ceil(H.bound * abs(t) / 3))
    for _ in range(n):
        term, psi = psi, psi.clone()
        for k in range(1, 80):
            term = H(term).mul_(-1j * (t / n) / k)
            psi.add_(term)
            if float(torch.linalg.vector_norm(term)) < 1e-18 * float(torch.linalg.vector_norm(psi)):
                break
    return psi


def _sz(p, L):
    """<sigma^z_k> of a weight per basis state, and the weights' sum."""
    tot = float(p.sum())
    return np.array([float((p.view(1 << k, 2, -1)[:, 0].sum() - p.view(1 << k, 2, -1)[:, 1].sum()) / tot) for k in range(L)]), tot


def exact(case, seed):
    kind, L = case["kind"], case.get("L", 0)
    if kind == "traj":
        return None
    if kind == "apply":
        psi = prepare(case, seed).psi
        desc = _desc(case, seed)
        return (_PlainLiouville(desc) if case["model"] == "liouville" else _Plain(desc))(psi)
    if kind == "lanczos":
        H, v, prev, b = _Plain(_desc(case, seed)), prepare(case, seed).psi, None, 0.0
        al, be, e = [], [], None
        for m in range(600):  # the three-term recurrence: its lowest Ritz value needs no reorthogonalisation
            w = H(v)
            if prev is not None:
                w.sub_(prev, alpha=b)
            al.append(float(torch.vdot(v, w).real))
            w.sub_(v, alpha=al[-1])
            b = float(torch.linalg.vector_norm(w))
            be.append(b)
            prev, v = v, w.div_(b)
            if m % 10 == 9:
                new = float(np.linalg.eigvalsh(np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1))[0])
                if e is not None and abs(new - e) < 1e-15 * abs(new):
                    break
                e = new
        return [new, None]
    if kind == "krylov":
        H, psi = _Plain(_desc(case, seed)), prepare(case, seed).psi
        rec = {"sz": [], "energy": [], "norm": []}
        for n in range(case["steps"] + 1):
            if n:
                psi = _expm_apply(H, psi, 0.05)
            sz, tot = _sz((psi.real ** 2).add_(psi.imag ** 2), L)
            rec["sz"].append(sz)
            rec["norm"].append(math.sqrt(tot))
            rec["energy"].append(float(torch.vdot(psi, H(psi)).real) / tot)
        return [psi, {k: np.array(v) for k, v in rec.items()}]
    if kind == "liouville":
        H, x = _PlainLiouville(_desc(case, seed)), prepare(case, seed).psi
        rec = {"sz": [], "norm": []}
        for n in range(case["steps"] + 1):
            if n:
                x = _expm_apply(H, x, 0.05)
            sz, tot = _sz(x.view(1 << L, 1 << L).diagonal().real.contiguous(), L)
            rec["sz"].append(sz)
            rec["norm"].append(tot)
        return [x, {k: np.array(v) for k, v in rec.items()}]
    if kind == "trotter":
        H, psi = _Plain(_desc(case, seed)), prepare(case, seed).psi
        t3 = 1.0 / (2.0 * (4.0 - 4.0 ** (1.0 / 3.0)))
        t1, t2, t4 = 1.0 - 8.0 * t3, 0.5 * (1.0 - 6.0 * t3), 2.0 * t3
        seq = [(0, 0.5), (1, 1.0), (0, 0.5)] if case["order"] == 2 else \
            [(0, t3), (1, t4), (0, t4), (1, t4), (0, t2), (1, t1), (0, t2), (1, t4), (0, t4), (1, t4), (0, t3)]
        rec = {"sz": [], "norm": []}
        for n in range(case["steps"] + 1):
            for part, frac in seq if n else ():
                for k in range(L - 1):  # the bond of sites k+1, k+2; part 1: odd k+1
                    if (k + 1) % 2 != part:
                        continue
                    wl, wr = (1.0 if k == 0 else 0.5), (1.0 if k + 1 == L - 1 else 0.5)
                    h = H.bond[k] + wl * np.kron(H.site[k], np.eye(2)) + wr * np.kron(np.eye(2), H.site[k + 1])
                    e, Q = np.linalg.eigh(h)
                    U = (Q * np.exp(-1j * frac * 0.05 * e)) @ Q.conj().T
                    out = torch.zeros_like(psi)
                    H.bond_into(out, psi, k, U)
                    psi = out
            sz, tot = _sz((psi.real ** 2).add_(psi.imag ** 2), L)
            rec["sz"].append(sz)
            rec["norm"].append(math.sqrt(tot))
        return [psi, {k: np.array(v) for k, v in rec.items()}]
    if kind == "entropy":
        if case["cut"] > 11:
            return None
        M = prepare(case, seed).psi.view(1 << case["cut"], -1)
        G = (M @ M.conj().T.contiguous()).cpu().numpy()
        lam = np.clip(np.linalg.eigvalsh(G / np.trace(G).real)[::-1], 0.0, None)
        return [float(-sum(x * math.log(x) for x in lam if x > 0)), lam.copy()]
    if kind == "rdm":
        psi = prepare(case, seed).psi

        def block(v):
            n = len(v)
            r = np.zeros((n, n), np.complex128)
            for a in range(n):
                for b in range(a, n):
                    r[a, b] = complex(torch.vdot(v[b], v[a]))
                    r[b, a] = r[a, b].conjugate()
            return r
        r1 = np.stack([block([psi.view(1 << k, 2, -1)[:, a].reshape(-1) for a in range(2)]) for k in range(L)])
        if not case["two_site"]:
            return [torch.from_numpy(r1)]
        r2 = []
        for k in range(L):
            for j in range(k + 1, L):
                v = psi.view(1 << k, 2, 1 << (j - k - 1), 2, -1)
                r2.append(block([v[:, a, :, b].reshape(-1) for a in range(2) for b in range(2)]))
        return [torch.from_numpy(r1), torch.from_numpy(np.stack(r2))]
    # adjoint: the Taylor series of every piece, differentiated term by term
    J, w = _adjoint_args(case, seed)
    desc, psi = _desc(case, seed), _neel(L)
    unit = _Plain(desc)
    O = sum(float(w[k]) * unit.z(k) for k in range(L))
    hs = [_Plain(desc, Js) for Js in J]
    n = max(1, math.ceil(max(h.bound for h in hs) * 0.1 / 3))
    K, tau, starts = 45, 0.1 / n, []
    for h in hs:
        for _ in range(n):
            starts.append(psi)
            psi = _taylor(h, psi, tau, K)[1]
    loss = float(torch.vdot(psi, O * psi).real)
    lam, grad = 2 * O * psi, np.zeros_like(J)
    for s in range(len(hs) - 1, -1, -1):
        for p in range(n - 1, -1, -1):
            terms, _ = _taylor(hs[s], starts[s * n + p], tau, K)
            a = lam
            for k in range(K, 0, -1):
                c = -1j * tau / k
                if float(torch.linalg.vector_norm(terms[k - 1])) > 1e-19:
                    for b in range(L - 1):
                        hb = torch.zeros_like(psi)
                        unit.bond_into(hb, terms[k - 1], b, unit.bond[b])
                        grad[s, b] += (c * complex(torch.vdot(a, hb))).real
                a = lam + np.conj(c) * hs[s](a)
            lam = a
    return [loss, grad]


def _taylor(H, psi, tau, K):
    terms, out = [psi], psi.clone()
    for k in range(1, K + 1):
        terms.append(H(terms[-1]).mul_(-1j * tau / k))
        out.add_(terms[-1])
    return terms, out
