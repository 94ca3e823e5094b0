"""The workloads this framework is timed on: J/K builds of water clusters
through the package's public entry points, from one molecule (where launches
and latency count) to 128, in the precisions and routes that SCF programs use.

A case names its kind of call and its sizes.  The molecules are clusters of
rigid waters at the density of 32 waters in a 10 A box with the 30-AO /
87-aux basis per water of the benchmark, placed from the seed; the orbitals are
random and orthonormal in the AO overlap, also from the seed.

`exact` evaluates the same quantities in 64-bit torch from the integral
definitions (McMurchie-Davidson on whole shell classes), without the package.
"""
import math

import numpy as np
import torch

from paper_2404_09452_amd.dfjk import Batch, Plan, setup_batch

BOHR = 1.0 / 0.529177210903
WATER = np.array([[0.0, 0.0, 0.0], [0.757, 0.587, 0.0], [-0.757, 0.587, 0.0]])   # O, H, H in Angstrom
AO_SHELLS = {"O": [(0, 5000.0 * 0.2 ** k) for k in range(4)] + [(1, 20.0 * 0.3 ** k) for k in range(3)] + [(2, 0.8)],
             "H": [(0, 20.0 * 0.2 ** k) for k in range(3)] + [(1, 0.7)]}
AUX_SHELLS = {"O": [(l, 10000.0 * 0.25 ** k) for l, n in enumerate((8, 5, 4, 2)) for k in range(n)],
              "H": [(l, 50.0 * 0.3 ** k) for l, n in enumerate((4, 2, 1)) for k in range(n)]}
NAO, NAUX, NOCC = 30, 87, 5     # per water


def listed():
    return [
        # one SCF iteration of the smallest molecule: launch latency
        {"name": "build w1 fp64", "kind": "build", "n": 1, "precision": "fp64", "tau": 1e-14},
        # the same from a density (no orbitals at hand), a small ragged molecule
        {"name": "density w7 fp64", "kind": "density", "n": 7, "tau": 1e-14},
        # open shell (two electrons more alpha than beta), odd sizes
        {"name": "uks w13 fp64", "kind": "uks", "n": 13, "precision": "fp64", "tau": 1e-14},
        # FP32 exchange, as proposed for later SCF iterations
        {"name": "build w24 fp32", "kind": "build", "n": 24, "precision": "fp32", "tau": 1e-14},
        # the benchmark's SCF iteration, in FP64 and in the fastest precision within 1e-6 Eh
        {"name": "build w32 fp64", "kind": "build", "n": 32, "precision": "fp64", "tau": 1e-14},
        {"name": "build w32 int8_fast", "kind": "build", "n": 32, "precision": "int8_fast", "tau": 1e-14},
        # the large cluster: several aux slabs
        {"name": "build w128 int8_fast", "kind": "build", "n": 128, "precision": "int8_fast", "tau": 1e-10},
        # one step of a server's batch: many small molecules of uneven sizes
        {"name": "batch 16 fp64", "kind": "batch", "sizes": "12 8 9 11 7 10 11 3 1 4 4 11 11 1 6 10",
         "precision": "fp64", "tau": 1e-14},
        # a new molecule from its coordinates to its first J and K: host preparation, screening, setup, build
        {"name": "job w4 fp64", "kind": "job", "n": 4, "precision": "fp64", "tau": 1e-14},
        {"name": "job w32 fp64", "kind": "job", "n": 32, "precision": "fp64", "tau": 1e-14},
        # exact (unfitted) J and K of direct SCF, and the increment of a later iteration
        {"name": "direct w32", "kind": "direct", "n": 32, "tau": 1e-10},
        {"name": "direct delta w8", "kind": "direct_delta", "n": 8, "tau": 1e-10, "eps": 1e-2},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))

    kind = rng.choice(["build", "build", "build", "density", "uks", "batch", "job", "direct", "direct_delta"])
    case = {"kind": kind, "tau": rng.choice([1e-14, 1e-12, 1e-10])}
    if kind == "build":
        case["precision"] = rng.choice(["fp64", "int8", "int8_fast", "fp32", "bf16x3"])
        case["n"] = size(1, 64)
    elif kind == "density":
        case["n"] = size(1, 16)
    elif kind == "uks":
        case["precision"] = rng.choice(["fp64", "int8_fast"])
        case["n"] = size(1, 32)
    elif kind == "batch":
        case["precision"] = rng.choice(["fp64", "int8", "int8_fast"])
        case["sizes"] = " ".join(str(rng.randint(1, 12)) for _ in range(rng.randint(2, 20)))
    elif kind == "job":
        case["precision"] = "fp64"
        case["n"] = size(1, 48)
    else:
        case["n"] = size(1, 32 if kind == "direct" else 16)
        case["tau"] = rng.choice([1e-12, 1e-10])
        if kind == "direct_delta":
            case["eps"] = rng.choice([1e-2, 1e-3, 1e-4])
    return case


# --------------------------------------------------------------------------
# Inputs

class Mol:
    """Coordinates (Bohr) and the shells of both bases: atom, l, exponent."""

    def __init__(self, coords, symbols):
        self.coords = coords
        self.ao = self._shells(symbols, AO_SHELLS)
        self.aux = self._shells(symbols, AUX_SHELLS)

    @staticmethod
    def _shells(symbols, table):
        rows = [(i, l, e) for i, s in enumerate(symbols) for l, e in table[s]]
        return (np.array([r[0] for r in rows], dtype=np.int32), np.array([r[1] for r in rows], dtype=np.int32),
                np.array([r[2] for r in rows], dtype=np.float64))

    def plan(self, tau):
        return Plan(self.coords, *self.ao, *self.aux, schwarz_thresh=tau)


def cluster(n, seed):
    """n waters with O-O >= 2.6 A and random rotations in a box of the benchmark's density."""
    rng = np.random.default_rng([n, seed])
    box = 10.0 * (n / 32.0) ** (1.0 / 3.0)
    oxygen = np.empty((0, 3))
    while len(oxygen) < n:
        for tries in range(20000):
            cand = rng.uniform(0.0, box, size=3)
            if len(oxygen) == 0 or np.min(np.sum((oxygen - cand) ** 2, axis=1)) >= 2.6 ** 2:
                oxygen = np.vstack([oxygen, cand])
                break
        else:
            oxygen = oxygen[: len(oxygen) // 2]      # packed itself in: take some out again
    coords = []
    for o in oxygen:
        w, x, y, z = (q := rng.standard_normal(4)) / np.linalg.norm(q)
        rot = np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)],
                        [2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)],
                        [2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]])
        coords += [o + rot @ r for r in WATER]
    return Mol(np.array(coords) * BOHR, ["O", "H", "H"] * n)


def orthonormal(X, S):
    """X R^-1 with X^T S X = R^T R."""
    L = torch.linalg.cholesky(X.T @ S @ X)
    return torch.linalg.solve_triangular(L, X.T.contiguous(), upper=False).T.contiguous()


def orbitals(mol, ncol, seed):
    g = torch.Generator().manual_seed(seed * 7919 + 13)
    X = torch.randn(len_ao(mol), ncol, generator=g, dtype=torch.float64).cuda()
    return orthonormal(X, overlap(mol))


def len_ao(mol):
    return int(np.sum(2 * mol.ao[1] + 1))


def stepped(mol, C, eps, seed):
    """Orbitals of a later SCF iteration: a random step of eps, orthonormalised."""
    g = torch.Generator().manual_seed(seed * 7919 + 14)
    R = torch.randn(*C.shape, generator=g, dtype=torch.float64).cuda()
    return orthonormal(C + eps * R, overlap(mol))


def sizes_of(case):
    return [int(x) for x in case["sizes"].split()] if case["kind"] == "batch" else [case["n"]]


def spins(n):
    return NOCC * n + 1, NOCC * n - 1


def inputs(case, seed):
    """The molecules and, per molecule, the orbital or density matrices of the call."""
    mols = [cluster(n, 1000 * seed + i) for i, n in enumerate(sizes_of(case))]
    out = []
    for i, (mol, n) in enumerate(zip(mols, sizes_of(case))):
        if case["kind"] == "uks":
            a, b = spins(n)
            C = orbitals(mol, a, seed)
            out.append((C, stepped(mol, C, 0.05, seed)[:, :b].contiguous()))
        else:
            out.append((orbitals(mol, NOCC * n, seed + 31 * i),))
    if case["kind"] == "density":
        out = [(2.0 * C @ C.T,) for (C,) in out]
    elif case["kind"] == "direct_delta":
        out = [(2.0 * (C1 := stepped(mols[0], C, case["eps"], seed)) @ C1.T, 2.0 * C @ C.T) for (C,) in out]
    return mols, out


def prepare(case, seed):
    mols, mats = inputs(case, seed)
    state = {"case": case, "mols": mols, "mats": mats}
    if case["kind"] == "job":
        return state
    plans = [mol.plan(case["tau"]).screen() for mol in mols]
    if case["kind"] == "batch":
        setup_batch(plans)
        state["batch"] = Batch(plans, [C.shape[1] for (C,) in mats], case["precision"])
    elif case["kind"].startswith("direct"):
        plans[0].direct_setup()
        if case["kind"] == "direct_delta":
            state["ref"] = plans[0].direct_build(D=mats[0][1])[:2]
    else:
        plans[0].setup()
    state["plans"] = plans
    return state


def run(state):
    case = state["case"]
    kind, m = case["kind"], state["mats"][0]
    if kind == "batch":
        return state["batch"].build([C for (C,) in state["mats"]])
    if kind == "job":
        plan = state["mols"][0].plan(case["tau"]).screen().setup()
        out = plan.build(C=m[0], precision=case["precision"])
        state["plans"] = [plan]      # the program keeps it for its next iterations
        return out
    plan = state["plans"][0]
    if kind == "build":
        return plan.build(C=m[0], precision=case["precision"])
    if kind == "density":
        return plan.build(D=m[0])
    if kind == "uks":
        return plan.build_uks(m[0], m[1], precision=case["precision"])
    if kind == "direct":
        return plan.direct_build(C=m[0])
    return plan.direct_build_delta(m[0], m[1], *state["ref"])


# --------------------------------------------------------------------------
# What a pass cannot do without

def shell_pairs(n):
    """Classes and Schwarz factors of the shell pairs (those of s Gaussians with the
    shells' exponents), on one geometry of the size."""
    mol = cluster(n, 0)
    atom, l, e = mol.ao
    a, b = np.tril_indices(len(l))
    la, lb = np.maximum(l[a], l[b]), np.minimum(l[a], l[b])
    p = e[a] + e[b]
    r2 = np.sum((mol.coords[atom[a]] - mol.coords[atom[b]]) ** 2, axis=1)
    norm = (2 * e / math.pi) ** 0.75
    q = norm[a] * norm[b] * np.exp(-e[a] * e[b] / p * r2) * np.sqrt(2 * math.pi ** 2.5 / (p * p * np.sqrt(2 * p)))
    return la, lb, q


def work(case):
    total = {"bytes": 0.0, "flops": 0.0}
    cache = {}
    for n in sizes_of(case):
        if n not in cache:
            cache[n] = work_of_one(case, n)
        for k, v in cache[n].items():
            total[k] += v
    return total


def work_of_one(case, n):
    kind, tau = case["kind"], case["tau"]
    nao, naux, nocc = NAO * n, NAUX * n, NOCC * n
    la, lb, q = shell_pairs(n)
    la, lb, q = la[q > 1e-30], lb[q > 1e-30], q[q > 1e-30]
    if kind.startswith("direct"):
        # every unique quartet once: its Hermite integrals, the transformation to functions, six contractions
        nh = lambda l: (l + 1) * (l + 2) * (l + 3) // 6      # noqa: E731
        cls = {}
        for key in {(int(x), int(y)) for x, y in zip(la, lb)}:
            cls[key] = np.sort(q[(la == key[0]) & (lb == key[1])])
        flops = 0.0
        for (a, b), qb in cls.items():
            for (c, d), qk in cls.items():
                pairs = float(np.sum(len(qk) - np.searchsorted(qk, tau / qb)))
                fb, fk = (2 * a + 1) * (2 * b + 1), (2 * c + 1) * (2 * d + 1)
                flops += 0.5 * pairs * (60 + 4 * nh(a + b + c + d) + 2 * fb * nh(a + b) * nh(c + d) +
                                        2 * fb * fk * nh(c + d) + 12 * fb * fk)
        mats = 6 if kind == "direct_delta" else 3
        return {"bytes": 8.0 * mats * nao * nao, "flops": flops}
    qaux = max(((2 * e / math.pi) ** 1.5 * 2 * math.pi ** 2.5 / (e * e * math.sqrt(2 * e))) ** 0.5
               for t in AUX_SHELLS.values() for l, e in t)
    keep = q * qaux >= tau
    nf = float(np.sum(((2 * la + 1) * (2 * lb + 1))[keep]))
    cols = nao if kind == "density" else sum(spins(n)) if kind == "uks" else nocc
    # J: two products with B; K: the half transform of both orientations and the triangle of its square
    flops = 4.0 * nf * naux + 4.0 * nf * naux * cols + float(nao) * (nao + 1) * naux * cols
    nbytes = 8.0 * (nf * naux + nao * cols + (3 if kind == "uks" else 2) * nao * nao)
    if kind == "job":
        # integrals (about 100 operations a triplet function), the metric's factor, its inverse, whitening
        flops += 100.0 * nf * naux + 2.0 * naux ** 3 / 3.0 + nf * naux * naux
    return {"bytes": nbytes, "flops": flops}


# --------------------------------------------------------------------------
# The same quantities from their definitions, in 64 bits

HARMONIC = {    # real solid harmonics as {(i, j, k): coefficient of x^i y^j z^k}, up to a factor per function
    0: [{(0, 0, 0): 1.0}],
    1: [{(1, 0, 0): 1.0}, {(0, 1, 0): 1.0}, {(0, 0, 1): 1.0}],
    2: [{(1, 1, 0): 1.0}, {(0, 1, 1): 1.0}, {(0, 0, 2): 2.0, (2, 0, 0): -1.0, (0, 2, 0): -1.0}, {(1, 0, 1): 1.0},
        {(2, 0, 0): 1.0, (0, 2, 0): -1.0}],
    3: [{(2, 1, 0): 3.0, (0, 3, 0): -1.0}, {(1, 1, 1): 1.0}, {(0, 1, 2): 4.0, (2, 1, 0): -1.0, (0, 3, 0): -1.0},
        {(0, 0, 3): 2.0, (2, 0, 1): -3.0, (0, 2, 1): -3.0}, {(1, 0, 2): 4.0, (3, 0, 0): -1.0, (1, 2, 0): -1.0},
        {(2, 0, 1): 1.0, (0, 2, 1): -1.0}, {(3, 0, 0): 1.0, (1, 2, 0): -3.0}],
}


def orders(L):
    return [(t, u, v) for t in range(L + 1) for u in range(L + 1 - t) for v in range(L + 1 - t - u)]


def dev(x, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=dtype, device="cuda")


def expansion(la, lb, ea, eb, A, B):
    """Hermite expansion [pair][function pair][tuv] of every product of two shells, its exponent and centre."""
    p = ea + eb
    P = (ea[:, None] * A + eb[:, None] * B) / p[:, None]
    E = []
    for x in range(3):
        pa, pb = P[:, x] - A[:, x], P[:, x] - B[:, x]
        e = {(0, 0, 0): torch.exp(-ea * eb / p * (A[:, x] - B[:, x]) ** 2)}
        at = lambda i, j, t: e.get((i, j, t), 0.0)      # noqa: E731
        for i in range(la + 1):
            for j in range(lb + 1):
                for t in range(i + j + 1):
                    if (i, j) == (0, 0):
                        continue
                    r, c = ((i - 1, j), pa) if i else ((i, j - 1), pb)
                    e[i, j, t] = at(*r, t - 1) * (0.5 / p) + at(*r, t) * c + at(*r, t + 1) * (t + 1)
        E.append(e)
    herm = orders(la + lb)
    out = torch.zeros(len(p), len(HARMONIC[la]) * len(HARMONIC[lb]), len(herm), dtype=torch.float64, device="cuda")
    for ma, fa in enumerate(HARMONIC[la]):
        for mb, fb in enumerate(HARMONIC[lb]):
            for (ax, ay, az), ca in fa.items():
                for (bx, by, bz), cb in fb.items():
                    for h, (t, u, v) in enumerate(herm):
                        if t <= ax + bx and u <= ay + by and v <= az + bz:
                            out[:, ma * len(HARMONIC[lb]) + mb, h] += (
                                ca * cb * E[0][ax, bx, t] * E[1][ay, by, u] * E[2][az, bz, v])
    return out, p, P


def unit(l, e):
    """Factors that make the functions of one-centre shells unit-normalised, [shell][function]."""
    O = torch.zeros(len(e), 3, dtype=torch.float64, device="cuda")
    E, p, _ = expansion(l, l, e, e, O, O)
    k = 2 * l + 1
    return (E[:, [m * k + m for m in range(k)], 0] * (math.pi / p[:, None]) ** 1.5).rsqrt()


class Side:
    """One class of charge distributions: Hermite expansions, exponents, centres and function indices."""

    def __init__(self, E, p, P, L, index):
        self.E, self.p, self.P, self.L, self.index = E, p, P, L, index


def offsets(l):
    return np.concatenate([[0], np.cumsum(2 * l + 1)])


def pair_sides(mol):
    """Every ordered pair of AO shells, by class; index holds mu and nu of each function pair."""
    atom, l, e = mol.ao
    off = offsets(l)
    for la in range(3):
        for lb in range(3):
            ia, ib = np.nonzero(l == la)[0], np.nonzero(l == lb)[0]
            a, b = np.repeat(ia, len(ib)), np.tile(ib, len(ia))
            if len(a) == 0:
                continue
            ea, eb = dev(e[a]), dev(e[b])
            E, p, P = expansion(la, lb, ea, eb, dev(mol.coords[atom[a]]), dev(mol.coords[atom[b]]))
            E *= (unit(la, ea)[:, :, None] * unit(lb, eb)[:, None, :]).reshape(len(a), -1, 1)
            mu = off[a][:, None] + np.repeat(np.arange(2 * la + 1), 2 * lb + 1)[None, :]
            nu = off[b][:, None] + np.tile(np.arange(2 * lb + 1), 2 * la + 1)[None, :]
            yield Side(E, p, P, la + lb, (dev(mu, torch.int64), dev(nu, torch.int64)))


def aux_sides(mol):
    atom, l, e = mol.aux
    off = offsets(l)
    for lc in range(4):
        c = np.nonzero(l == lc)[0]
        if len(c) == 0:
            continue
        ec, R = dev(e[c]), dev(mol.coords[atom[c]])
        E, p, P = expansion(lc, 0, ec, torch.zeros_like(ec), R, R)
        yield Side(E * unit(lc, ec)[:, :, None], p, P, lc, dev(off[c][:, None] + np.arange(2 * lc + 1), torch.int64))


def overlap(mol):
    nao = len_ao(mol)
    S = torch.zeros(nao, nao, dtype=torch.float64, device="cuda")
    for s in pair_sides(mol):
        S[s.index[0], s.index[1]] = s.E[:, :, 0] * (math.pi / s.p[:, None]) ** 1.5
    return S


def boys(M, T):
    F = [None] * (M + 1)
    a = M + 0.5
    big = torch.clamp(T, min=1e-7)
    F[M] = torch.where(T < 1e-7, 1.0 / (2 * M + 1) - T / (2 * M + 3),
                       torch.special.gammainc(torch.full_like(T, a), big) * math.gamma(a) / (2.0 * big ** a))
    e = torch.exp(-T)
    for m in range(M - 1, -1, -1):
        F[m] = (2.0 * T * F[m + 1] + e) / (2 * m + 1)
    return F


def coulomb(x, y, most=1 << 27):
    """(f|g) of the distributions of two sides, in blocks over x: yields (slice of x, [x][f][y][g])."""
    hx, hy, L = orders(x.L), orders(y.L), x.L + y.L
    where = {h: i for i, h in enumerate(orders(L))}
    gather = torch.tensor([where[tuple(i + j for i, j in zip(a, b))] for a in hx for b in hy], device="cuda")
    sign = torch.tensor([(-1.0) ** sum(b) for b in hy], dtype=torch.float64, device="cuda")
    Ey = (y.E * sign).permute(0, 2, 1).contiguous()
    step = max(1, most // (len(gather) * len(y.p)))
    for i in range(0, len(x.p), step):
        p, P = x.p[i:i + step], x.P[i:i + step]
        s = p[:, None] + y.p[None, :]
        alpha = p[:, None] * y.p[None, :] / s
        X = [P[:, None, d] - y.P[None, :, d] for d in range(3)]
        F = boys(L, alpha * sum(v * v for v in X))
        R = {(0, 0, 0): (-2.0 * alpha) ** L * F[L]}
        for n in range(L - 1, -1, -1):
            up, R = R, {(0, 0, 0): (-2.0 * alpha) ** n * F[n]}
            for h in orders(L - n)[1:]:
                d = next(k for k in range(3) if h[k])
                low = tuple(v - (k == d) for k, v in enumerate(h))
                R[h] = X[d] * up[low]
                if h[d] > 1:
                    R[h] = R[h] + (h[d] - 1) * up[tuple(v - 2 * (k == d) for k, v in enumerate(h))]
        pref = 2.0 * math.pi ** 2.5 / (p[:, None] * y.p[None, :] * s.sqrt())
        R = torch.stack([R[h] * pref for h in orders(L)])
        n = len(p)
        R = R[gather].reshape(len(hx), len(hy), n, len(y.p)).permute(3, 2, 0, 1).reshape(len(y.p), n * len(hx), -1)
        W = torch.bmm(R, Ey).reshape(len(y.p), n, len(hx), -1).permute(1, 2, 0, 3).reshape(n, len(hx), -1)
        yield slice(i, i + n), torch.bmm(x.E[i:i + n], W.contiguous()).reshape(n, x.E.shape[1], len(y.p), -1)


def fitted(mol):
    """B [aux][nao][nao] of the fit, whitened by the metric's Cholesky factor."""
    nao, naux = len_ao(mol), int(np.sum(2 * mol.aux[1] + 1))
    aux = list(aux_sides(mol))
    V = torch.empty(naux, naux, dtype=torch.float64, device="cuda")
    for c in aux:
        for d in aux:
            for s, I in coulomb(c, d):
                V[c.index[s][:, :, None, None], d.index[None, None]] = I
    U = torch.empty(nao, nao, naux, dtype=torch.float64, device="cuda")
    for x in pair_sides(mol):
        for c in aux:
            for s, I in coulomb(x, c):
                U[x.index[0][s][:, :, None, None], x.index[1][s][:, :, None, None], c.index[None, None]] = I
    L = torch.linalg.cholesky(V)
    Linv = torch.linalg.solve_triangular(L.cpu(), torch.eye(naux, dtype=torch.float64), upper=False).cuda()
    B = torch.empty(naux, nao, nao, dtype=torch.float64, device="cuda")
    for i in range(nao):
        B[:, i] = Linv @ U[i].T
    return B


def exchange(B, C):
    """sum_P B_P C C^T B_P, in blocks of aux functions."""
    K = torch.zeros(B.shape[1], B.shape[1], dtype=torch.float64, device="cuda")
    step = max(1, (1 << 27) // (B.shape[1] * C.shape[1]))
    for i in range(0, len(B), step):
        X = torch.matmul(B[i:i + step].reshape(-1, B.shape[1]), C).reshape(-1, B.shape[1], C.shape[1])
        X = X.permute(1, 0, 2).reshape(B.shape[1], -1)
        K += X @ X.T
    return K


def fitted_jk(mol, D, Cs):
    """J of D, then sum_P B_P C C^T B_P of each C."""
    B = fitted(mol)
    flat = B.reshape(len(B), -1)
    J = (flat.T @ (flat @ D.reshape(-1))).reshape(D.shape)
    return J, [exchange(B, C) for C in Cs]


def four_centre_jk(mol, D):
    nao = len_ao(mol)
    J = torch.zeros(nao, nao, dtype=torch.float64, device="cuda")
    K = torch.zeros_like(J)
    sides = list(pair_sides(mol))
    for x in sides:
        mu, nu = x.index
        for y in sides:
            la, si = y.index[0].reshape(-1), y.index[1].reshape(-1)
            for s, I in coulomb(x, y, 1 << 26):
                I = I.reshape(I.shape[0] * I.shape[1], -1)       # rows: (mu nu|, columns: |la si)
                m, v = mu[s].reshape(-1), nu[s].reshape(-1)
                J.index_put_((m, v), I @ D[la, si], accumulate=True)
                # K[mu][la] += (mu nu|la si) D[nu][si]
                T = I * D[v[:, None], si[None, :]]
                row = torch.zeros(len(m), nao, dtype=torch.float64, device="cuda").index_add_(1, la, T)
                K.index_add_(0, m, row)
    return J, K


def exact(case, seed):
    kind = case["kind"]
    if max(sizes_of(case)) > (8 if kind.startswith("direct") else 32):
        return None
    mols, mats = inputs(case, seed)
    out = []
    for mol, m in zip(mols, mats):
        if kind == "uks":
            D = [C @ C.T for C in m]
            J, (Ka, Kb) = fitted_jk(mol, D[0] + D[1], m)
            E = torch.stack([0.5 * ((D[0] + D[1]) * J).sum(), -0.5 * ((D[0] * Ka).sum() + (D[1] * Kb).sum())])
            return J, Ka, Kb, E
        D = m[0] if kind in ("density", "direct_delta") else 2.0 * m[0] @ m[0].T
        if kind.startswith("direct"):
            J, K = four_centre_jk(mol, D)
        elif kind == "density":
            w, v = torch.linalg.eigh(D)
            keep = w > 1e-12 * w.max()
            J, (K,) = fitted_jk(mol, D, [(v[:, keep] * w[keep].sqrt()).contiguous()])
        else:
            J, (K,) = fitted_jk(mol, D, [math.sqrt(2.0) * m[0]])
        out.append((J, K, torch.stack([0.5 * (D * J).sum(), -0.25 * (D * K).sum()])))
    return out if kind == "batch" else out[0]
