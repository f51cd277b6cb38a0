"""Timed cases of the Fock-build library, through the calls of its ctypes binding.

Each case is one thing that a program does with the library: a direct Fock
build of a molecule at one of the sizes of the tests and the benchmark (one
molecule or a batch, FP64 or mixed precision, one density or several, eager
or replayed from a captured graph), the load of a new geometry, a whole SCF,
and one gradient of the learned-guess network.  A case is a dict of plain
values; ``prepare`` makes its inputs on the GPU and the handle that a program
keeps, ``run`` is one pass, ``work`` its minimal bytes and flops and ``exact``
the same result in plain numpy FP64 where that is affordable.

Launch settings are the library's defaults, or (``"persistent": 1``) the
resident-grid form with 32768-quartet tasks that the benchmark sets for
systems of about a thousand basis functions and more.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import workloads as W

TAU = 1e-10


# ---- the cases ----------------------------------------------------------------------

def listed():
    return [
        # the smallest build: (H2O)2 without d shells, 26 basis functions; launch latency
        {"name": "fock_dimer", "kind": "fock", "mol": "dimer", "n": 2, "precision": 0, "persistent": 0},
        # a small molecule replayed from a captured HIP graph (all 21 classes, odd size)
        {"name": "graph_5_waters", "kind": "graph", "mol": "water", "n": 5, "precision": 0, "persistent": 0},
        # an ordinary mid-size molecule with the default settings: 247 basis functions
        {"name": "fock_13_waters", "kind": "fock", "mol": "water", "n": 13, "precision": 0, "persistent": 0},
        # the benchmark's headline build: 1216 basis functions
        {"name": "fock_64_waters", "kind": "fock", "mol": "water", "n": 64, "precision": 0, "persistent": 1},
        # mixed FP32/FP64 evaluation, default settings
        {"name": "mixed_33_waters", "kind": "fock", "mol": "water", "n": 33, "precision": 1, "persistent": 0},
        # the largest: 2128 basis functions, where the staged rows are column-windowed
        {"name": "fock_112_waters", "kind": "fock", "mol": "water", "n": 112, "precision": 0, "persistent": 1},
        # the 0.5 nm graphene bilayer: contracted SP shells, primitive-heavy p and d classes
        {"name": "fock_graphene_44", "kind": "fock", "mol": "graphene", "n": 22, "precision": 0, "persistent": 1},
        # J and K of an alpha and a beta density in one pass (unrestricted builds)
        {"name": "jk_2_densities_27", "kind": "multi", "mol": "water", "n": 27, "ndens": 2},
        # a batch of small clusters of 1-16 waters: short tasks
        {"name": "batch_48_clusters", "kind": "batch", "nmol": 48, "lo": 1, "hi": 16, "precision": 0},
        # a new geometry: shell pairs, Schwarz bounds, plans, one-electron integrals; S and H out
        {"name": "load_29_waters", "kind": "load", "mol": "water", "n": 29},
        # a whole SCF of a small molecule, from SAD to convergence
        {"name": "scf_4_waters", "kind": "scf", "mol": "water", "n": 4},
        # one training gradient of the learned-guess network on a minibatch of pairs
        {"name": "guess_grad_8192", "kind": "guess", "rows": 8192},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fock", "fock", "fock", "graphene", "mixed", "graph", "multi", "batch", "load", "scf", "guess"])
    if kind in ("fock", "mixed"):
        n = _log_int(rng, 1, 80)
        return {"kind": "fock", "mol": "water", "n": n, "precision": int(kind == "mixed"),
                "persistent": rng.randint(0, 1)}
    if kind == "graphene":
        return {"kind": "fock", "mol": "graphene", "n": _log_int(rng, 2, 26), "precision": 0,
                "persistent": rng.randint(0, 1)}
    if kind == "graph":
        return {"kind": "graph", "mol": "water", "n": _log_int(rng, 1, 24), "precision": rng.randint(0, 1),
                "persistent": rng.randint(0, 1)}
    if kind == "multi":
        return {"kind": "multi", "mol": "water", "n": _log_int(rng, 1, 30), "ndens": rng.randint(1, 4)}
    if kind == "batch":
        lo = rng.randint(1, 4)
        return {"kind": "batch", "nmol": _log_int(rng, 2, 80), "lo": lo, "hi": lo + rng.randint(0, 12),
                "precision": rng.randint(0, 1)}
    if kind == "load":
        return {"kind": "load", "mol": rng.choice(["water", "graphene"]), "n": _log_int(rng, 1, 40)}
    if kind == "scf":
        return {"kind": "scf", "mol": "water", "n": _log_int(rng, 1, 12)}
    return {"kind": "guess", "rows": _log_int(rng, 100, 16384)}


# ---- inputs ---------------------------------------------------------------------------

def _molecule(case, seed):
    """The case's molecule: waters are placed from the seed; the graphene
    bilayer's sites are displaced by up to 0.02 bohr (a step of an optimisation)."""
    if case["mol"] == "dimer":
        return W.water_dimer(seed, W.BASIS_SP)
    if case["mol"] == "graphene":
        m = W.graphene_bilayer(case["n"])
        m.xyz = m.xyz + np.random.default_rng(seed).uniform(-0.02, 0.02, size=m.xyz.shape)
        return m
    return W.water_cluster(case["n"], seed)


def _batch(case, seed):
    """The batch's clusters: sizes uniform in lo..hi (the same for every seed), placed from the seed."""
    sizes = W.batch_sizes(case["nmol"], 2, case["lo"], case["hi"])
    return [W.water_cluster(int(n), seed * 1000 + i) for i, n in enumerate(sizes)]


def _density(n, nocc, seed):
    """A density of the right rank and size of entries: C C^T with n x nocc
    columns of variance 1/n (near-orthonormal, entries like a converged D)."""
    c = np.random.default_rng(seed).standard_normal((n, nocc)) / math.sqrt(n)
    ct = torch.tensor(c, device="cuda") if torch.cuda.is_available() else torch.tensor(c)
    return ct @ ct.T


def _guess_inputs(rows, seed):
    """A minibatch as the trainer packs it: rows by pair type (O-O, O-H, H-H
    about 1:4:4), features with one-hot elements, radial values in [0, 1] and
    log environments, targets of unit size, a seeded start of the network."""
    rng = np.random.default_rng(seed)
    counts = [rows // 9, rows * 4 // 9, rows - rows // 9 - rows * 4 // 9]
    X = np.zeros((rows, 164), np.float32)
    t = np.repeat(np.arange(3), counts)
    X[np.arange(rows), (t == 2).astype(int)] = 1.0
    X[np.arange(rows), 2 + (t > 0).astype(int)] = 1.0
    mu = np.linspace(0.5, 6.0, 32)
    r = rng.uniform(0.9, 6.0, rows)
    X[:, 4:36] = np.exp(-0.5 * ((r[:, None] - mu) / (mu[1] - mu[0])) ** 2) * (0.5 * np.cos(np.pi * r / 6.0) + 0.5)[:, None]
    X[:, 36:] = np.log1p(rng.gamma(1.0, 0.7, size=(rows, 128)))
    T = rng.standard_normal(counts[0] * 225 + counts[1] * 30 + counts[2] * 4).astype(np.float32) * 0.05
    return X, T, counts, X.mean(0), X.std(0) + 0.05, np.full(3, 0.05)


def prepare(case, seed):
    from paper_1708_00033_amd import hfx
    sp = torch.cuda.current_stream().cuda_stream
    kind = case["kind"]
    if kind == "guess":
        X, T, counts, mean, scale, ts = _guess_inputs(case["rows"], seed)
        net = hfx.GuessNet(0, hfx.GuessNet.init_params(seed, mean, scale, ts))
        return {"net": net, "X": torch.tensor(X, device="cuda"), "T": torch.tensor(T, device="cuda"),
                "counts": counts, "case": case, "stream": sp}
    prec = hfx.HFX_PREC_MIXED if case.get("precision") else hfx.HFX_PREC_FP64
    ctx = hfx.Context(device=0, schwarz_tau=TAU, precision=prec)
    s = {"ctx": ctx, "case": case, "stream": sp}
    if case.get("persistent"):
        ctx.set_class_tuning(-1, 32768, 0, 1, -1)
    if kind == "load":
        s["mol"] = _molecule(case, seed)
        return s
    if kind == "batch":
        ctx.load_batch(_batch(case, seed))
        nbf, nocc, _, tot = ctx.layout
        s["D"] = torch.cat([_density(int(n), int(o), seed * 1000 + i).reshape(-1)
                            for i, (n, o) in enumerate(zip(nbf, nocc))])
        assert s["D"].numel() == tot
        s["F"] = torch.empty_like(s["D"])
        return s
    ctx.load(_molecule(case, seed))
    if kind == "scf":
        return s
    if kind == "multi":
        s["D"] = torch.stack([_density(ctx.nbf, ctx.nocc, seed * 100 + d) for d in range(case["ndens"])]).contiguous()
        s["J"], s["K"] = torch.empty_like(s["D"]), torch.empty_like(s["D"])
        return s
    s["D"] = _density(ctx.nbf, ctx.nocc, seed).contiguous()
    s["F"] = torch.empty_like(s["D"])
    if kind == "graph":
        s["gstream"] = torch.cuda.Stream()
        torch.cuda.synchronize()
        ctx.graph_capture(s["D"].data_ptr(), s["F"].data_ptr(), s["gstream"].cuda_stream)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("fock", "batch"):
        s["ctx"].build_fock_dev(s["D"].data_ptr(), s["F"].data_ptr(), s["stream"])
        return s["F"]
    if kind == "graph":
        s["ctx"].graph_launch(s["stream"])
        return s["F"]
    if kind == "multi":
        s["ctx"].build_jk_multi_dev(case["ndens"], s["D"].data_ptr(), s["J"].data_ptr(), s["K"].data_ptr(), s["stream"])
        return {"J": s["J"], "K": s["K"]}
    if kind == "load":
        ctx = s["ctx"].load(s["mol"])
        S, H, e = ctx.core()
        return {"S": S, "H": H, "e_nuc": float(e)}
    if kind == "scf":
        r = s["ctx"].scf()
        return {"energy": float(r["energy"]), "D": r["D"], "eps": r["eps"]}
    net = s["net"]
    loss = net.grad_dev(s["X"].data_ptr(), s["counts"], s["T"].data_ptr(), s["stream"])
    return {"loss": float(loss), "grad": net.get_grads()}


# ---- minimal work ------------------------------------------------------------------------

_L = [(0, 0), (1, 0), (1, 1), (2, 0), (2, 1), (2, 2)]


def _nc(l):
    return (l + 1) * (l + 2) // 2


def _ntarget(la, lb):
    return sum(_nc(k) for k in range(la, la + lb + 1))


def _class_flops(counts):
    """Per primitive quartet: 20 for the Gaussian products, 25 + 4 L for the
    Boys functions, 2 per contracted intermediate; per integral 12 for the six
    Fock updates."""
    total, k = 0.0, 0
    for B in range(6):
        for K in range(B + 1):
            (la, lb), (lc, ld) = _L[B], _L[K]
            per_prim = 45 + 4 * (la + lb + lc + ld) + 2 * _ntarget(la, lb) * _ntarget(lc, ld)
            total += counts[k, 2] * per_prim + 12.0 * counts[k, 1]
            k += 1
    return float(total)


def work(case):
    """The screened quartets are counted by the library's planner on the
    molecule of seed 0; matrices are read and written once."""
    kind = case["kind"]
    if kind == "guess":
        rows = case["rows"]
        c = [rows // 9, rows * 4 // 9, rows - rows // 9 - rows * 4 // 9]
        mac = rows * (164 + 2 * 256) * 256 + sum(n * w * 256 for n, w in zip(c, (225, 30, 4)))
        npar = 256 * (164 + 1) + 2 * 256 * 257 + sum(w * 257 for w in (225, 30, 4)) + 164 * 2 + 3
        return {"bytes": 4.0 * (rows * 164 + sum(n * w for n, w in zip(c, (225, 30, 4))) + 2 * npar),
                "flops": 6.0 * mac - 2.0 * rows * 164 * 256}
    from paper_1708_00033_amd import hfx
    ctx = hfx.Context(device=0, schwarz_tau=TAU)
    if kind == "batch":
        ctx.load_batch(_batch(case, 0))
        nn = int(ctx.layout[3])
    else:
        mol = _molecule(case, 0)
        ctx.load(mol)
        nn = ctx.nbf * ctx.nbf
    flops = _class_flops(ctx.class_counts())
    ctx.close()
    if kind == "multi":
        return {"bytes": 24.0 * nn * case["ndens"], "flops": flops}
    if kind == "load":
        return {"bytes": 16.0 * nn, "flops": 60.0 * nn / 2 * mol.natom}
    if kind == "scf":
        n = math.sqrt(nn)
        return {"bytes": 10 * 24.0 * nn, "flops": 10 * (flops + 10.0 * n ** 3)}
    return {"bytes": 24.0 * nn, "flops": flops}


# ---- plain FP64 ---------------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind == "guess":
        return _exact_guess(case["rows"], seed)
    if kind == "load":
        mol = _molecule(case, seed)
        if mol.nbf > 560:
            return None
        b = _Basis(mol)
        S, H = b.one_electron()
        d = np.linalg.norm(mol.xyz[:, None] - mol.xyz[None], axis=2)[np.triu_indices(mol.natom, 1)]
        zz = np.outer(mol.Z, mol.Z)[np.triu_indices(mol.natom, 1)]
        return {"S": S, "H": H, "e_nuc": float((zz / d).sum())}
    if kind not in ("fock", "graph", "multi") or case["mol"] == "graphene" or case["n"] > 5 or case.get("precision"):
        return None
    mol = _molecule(case, seed)
    b = _Basis(mol)
    G = b.eri(TAU)
    nocc = int(mol.Z.sum()) // 2
    dens = [_density(b.n, nocc, s).cpu().numpy() for s in
            ([seed * 100 + d for d in range(case["ndens"])] if kind == "multi" else [seed])]
    J = np.stack([np.tensordot(G, D, 2) for D in dens])
    K = np.stack([np.tensordot(G, D, ((1, 3), (0, 1))) for D in dens])
    if kind == "multi":
        return {"J": J, "K": K}
    return b.one_electron()[1] + 2.0 * J[0] - K[0]


def _exact_guess(rows, seed):
    from paper_1708_00033_amd import hfx
    X, T, counts, mean, scale, ts = _guess_inputs(rows, seed)
    flat = hfx.GuessNet.init_params(seed, mean, scale, ts).astype(np.float64)
    p, o = {}, 0
    for name, r, c in hfx.GuessNet.LAYOUT:
        p[name] = flat[o:o + r * c].reshape(r, c)
        o += r * c
    sig = lambda z: 1.0 / (1.0 + np.exp(-z))  # noqa: E731
    h = [np.clip((X - p["fmean"][:, 0]) / p["fscale"][:, 0], -4.0, 4.0)]
    z = []
    for k in (1, 2, 3):
        z.append(h[-1] @ p["W%d" % k].T + p["b%d" % k][:, 0])
        h.append(z[-1] * sig(z[-1]))
    ny = sum(c * w for c, w in zip(counts, (225, 30, 4)))
    g, loss, dh, r0, t0 = {}, 0.0, np.zeros_like(h[-1]), 0, 0
    for t, w in enumerate((225, 30, 4)):
        c = counts[t]
        hb = h[-1][r0:r0 + c]
        d = hb @ p["H%d" % t].T + p["c%d" % t][:, 0] - T[t0:t0 + c * w].reshape(c, w) / p["tscale"][t, 0]
        loss += float((d * d).sum())
        d *= 2.0 / ny
        g["H%d" % t], g["c%d" % t] = d.T @ hb, d.sum(0)
        dh[r0:r0 + c] = d @ p["H%d" % t]
        r0, t0 = r0 + c, t0 + c * w
    for k in (3, 2, 1):
        s = sig(z[k - 1])
        dz = dh * s * (1.0 + z[k - 1] * (1.0 - s))
        g["W%d" % k], g["b%d" % k] = dz.T @ h[k - 1], dz.sum(0)
        dh = dz @ p["W%d" % k]
    out = [g[n].ravel() if n in g else np.zeros(r * c) for n, r, c in hfx.GuessNet.LAYOUT]
    return {"loss": loss / ny, "grad": np.concatenate(out)}


def _cart(l):
    return [(x, y, l - x - y) for x in range(l, -1, -1) for y in range(l - x, -1, -1)]


def _boys(m_max, T):
    """F_0..F_m_max: ascending series and downward recursion below T = 45, the
    asymptotic value and upward recursion above."""
    T = np.asarray(T, float)
    F = np.empty((m_max + 1,) + T.shape)
    lo = T < 45.0
    t = T[lo]
    e = np.exp(-t)
    term = np.full_like(t, 1.0 / (2 * m_max + 1))
    acc = term.copy()
    for i in range(1, 190):
        term = term * (2.0 * t) / (2 * m_max + 2 * i + 1)
        acc += term
        if not t.size or term.max() < 1e-18 * acc.min():
            break
    f = e * acc
    F[m_max][lo] = f
    for m in range(m_max - 1, -1, -1):
        f = (2.0 * t * f + e) / (2 * m + 1)
        F[m][lo] = f
    t = T[~lo]
    e = np.exp(-t)
    f = 0.5 * np.sqrt(np.pi / t)
    F[0][~lo] = f
    for m in range(m_max):
        f = ((2 * m + 1) * f - e) / (2.0 * t)
        F[m + 1][~lo] = f
    return F


def _hermite_r(L, alpha, pq):
    """R_tuv(alpha, PQ) for t + u + v <= L (McMurchie and Davidson)."""
    F = _boys(L, alpha * (pq ** 2).sum(0))
    lev = {(0, 0, 0): (-2.0 * alpha) ** L * F[L]}
    for n in range(L - 1, -1, -1):
        new = {(0, 0, 0): (-2.0 * alpha) ** n * F[n]}
        for k in range(1, L - n + 1):
            for t in _cart(k):
                i = max(range(3), key=lambda q: t[q])
                d = list(t)
                d[i] -= 1
                v = pq[i] * lev[tuple(d)]
                if d[i] > 0:
                    c = d[i]
                    d[i] -= 1
                    v = v + c * lev[tuple(d)]
                new[t] = v
        lev = new
    return lev


def _hermite_e(la, lb, p, pa, pb):
    """E^{ij}_t along one axis without the Gaussian prefactor (arrays over pairs)."""
    z = np.zeros_like(pa)
    E = {(0, 0, 0): np.ones_like(pa)}
    get = lambda i, j, t: E.get((i, j, t), z)  # noqa: E731
    for i in range(la + 1):
        for j in range(lb + 1):
            if i == j == 0:
                continue
            for t in range(i + j + 1):
                if i > 0:
                    E[i, j, t] = get(i - 1, j, t - 1) / (2 * p) + pa * get(i - 1, j, t) + (t + 1) * get(i - 1, j, t + 1)
                else:
                    E[i, j, t] = get(i, j - 1, t - 1) / (2 * p) + pb * get(i, j - 1, t) + (t + 1) * get(i, j - 1, t + 1)
    return E


class _Basis:
    """Shells (SP written out as s and p) and their shell pairs by class, each
    with its primitive pairs and Hermite expansion coefficients."""

    def __init__(self, mol):
        sh, n = [], 0
        for s in mol.shells:
            for l, co in (((0, s.coefs), (1, s.coefs_p)) if s.l == W.SP else ((s.l, s.coefs),)):
                a = np.asarray(s.exps, float)
                c = np.asarray(co, float) * (2 * a / np.pi) ** 0.75 * (4 * a) ** (0.5 * l)
                pp = a[:, None] + a[None]
                c = c / math.sqrt((np.outer(c, c) * (np.pi / pp) ** 1.5 / (2 * pp) ** l).sum())
                sh.append((l, mol.xyz[s.atom], a, c, n))
                n += _nc(l)
        self.n, self.mol = n, mol
        self.scale = np.concatenate([[1.0 / math.sqrt(np.prod([_odd(x) for x in e])) for e in _cart(l)]
                                     for l, *_ in sh])
        groups = {}
        for i in range(len(sh)):
            for j in range(i + 1):
                a, b = (sh[i], sh[j]) if sh[i][0] >= sh[j][0] else (sh[j], sh[i])
                groups.setdefault((a[0], b[0]), []).append((a, b))
        self.cls = {k: self._pairs(k, v) for k, v in groups.items()}

    def _pairs(self, key, pairs):
        la, lb = key
        al, be, cc, A, B, start = [], [], [], [], [], []
        for a, b in pairs:
            start.append(sum(map(len, al)))
            al.append(np.repeat(a[2], len(b[2])))
            be.append(np.tile(b[2], len(a[2])))
            cc.append(np.outer(a[3], b[3]).ravel())
            A.append(np.tile(a[1], (len(al[-1]), 1)))
            B.append(np.tile(b[1], (len(al[-1]), 1)))
        al, be, cc, A, B = map(np.concatenate, (al, be, cc, A, B))
        p = al + be
        P = (al[:, None] * A + be[:, None] * B) / p[:, None]
        k = cc * np.exp(-al * be / p * ((A - B) ** 2).sum(1))
        E = [_hermite_e(la, lb + 2, p, P[:, x] - A[:, x], P[:, x] - B[:, x]) for x in range(3)]
        herm = [t for q in range(la + lb + 1) for t in _cart(q)]
        ab = [(a, b) for a in _cart(la) for b in _cart(lb)]
        Eab = np.zeros((len(p), len(ab), len(herm)))
        for m, (a, b) in enumerate(ab):
            for h, t in enumerate(herm):
                if all(t[x] <= a[x] + b[x] for x in range(3)):
                    Eab[:, m, h] = k * np.prod([E[x][a[x], b[x], t[x]] for x in range(3)], axis=0)
        rows = np.array([[a[4] + i for i in range(_nc(la)) for _ in range(_nc(lb))] for a, b in pairs])
        cols = np.array([[b[4] + j for _ in range(_nc(la)) for j in range(_nc(lb))] for a, b in pairs])
        return dict(p=p, P=P, be=be, k=k, E=E, Eab=Eab, herm=herm, ab=ab, start=np.array(start), rows=rows,
                    cols=cols, key=key)

    def one_electron(self):
        S, H = np.zeros((self.n, self.n)), np.zeros((self.n, self.n))
        for c in self.cls.values():
            p, be, E, k = c["p"], c["be"], c["E"], c["k"]
            s, h = [], []
            for a, b in c["ab"]:
                f = np.sqrt(np.pi / p)
                ov = [f * E[x][a[x], b[x], 0] for x in range(3)]
                kin = [f * (-2.0 * be ** 2 * E[x][a[x], b[x] + 2, 0] + be * (2 * b[x] + 1) * E[x][a[x], b[x], 0]
                            - (0.5 * b[x] * (b[x] - 1) * E[x][a[x], b[x] - 2, 0] if b[x] > 1 else 0.0))
                       for x in range(3)]
                s.append(k * ov[0] * ov[1] * ov[2])
                h.append(k * (kin[0] * ov[1] * ov[2] + ov[0] * kin[1] * ov[2] + ov[0] * ov[1] * kin[2]))
            s, h = np.array(s).T, np.array(h).T
            for z, xyz in zip(self.mol.Z, self.mol.xyz):
                R = _hermite_r(sum(c["key"]), p, (c["P"] - xyz).T)
                h -= z * (2 * np.pi / p)[:, None] * np.einsum("pmh,hp->pm", c["Eab"], np.stack([R[t] for t in c["herm"]]))
            for M, v in ((S, s), (H, h)):
                v = np.add.reduceat(v, c["start"], axis=0) * self.scale[c["rows"]] * self.scale[c["cols"]]
                M[c["rows"], c["cols"]] = v
                M[c["cols"], c["rows"]] = v
        return S, H

    def eri(self, tau):
        """(mn|ls) of the quartets that Schwarz screening keeps, all n^4."""
        G = np.zeros((self.n,) * 4)
        Q = {key: self._schwarz(c) for key, c in self.cls.items()}
        keys = list(self.cls)
        for i, kb in enumerate(keys):
            for kk in keys[:i + 1]:
                b, c = self.cls[kb], self.cls[kk]
                v = self._block(b, c) * (Q[kb][:, None] * Q[kk][None] >= tau)[:, :, None, None]
                r, s = b["rows"][:, None, :, None], b["cols"][:, None, :, None]
                t, u = c["rows"][None, :, None, :], c["cols"][None, :, None, :]
                v = v * self.scale[r] * self.scale[s] * self.scale[t] * self.scale[u]
                for x, y in ((r, s), (s, r)):
                    for z, w in ((t, u), (u, t)):
                        G[x, y, z, w] = v
                        G[z, w, x, y] = v
        return G

    def _schwarz(self, c):
        v = self._block(c, c, diagonal=True)
        d = np.einsum("pmm->pm", v) * (self.scale[c["rows"]] * self.scale[c["cols"]]) ** 2
        return np.sqrt(d.max(1))

    def _block(self, b, c, diagonal=False):
        """Contracted blocks (bra pair, ket pair, ab, cd); with diagonal, of every pair with itself."""
        nb, ne = len(b["start"]), np.append(b["start"], len(b["p"]))
        ns = np.append(c["start"], len(c["p"]))
        out = np.zeros((nb,) + (() if diagonal else (len(c["start"]),)) + (len(b["ab"]), len(c["ab"])))
        sign = np.array([(-1.0) ** sum(t) for t in c["herm"]])
        step = 1 if diagonal else max(1, int(4e6 // (len(c["p"]) * len(b["herm"]) * len(c["herm"]) * 9)))
        for i in range(0, nb, step):
            pi = slice(ne[i], ne[min(nb, i + step)])
            ci = slice(ns[i], ns[i + 1]) if diagonal else slice(None)
            p, q = b["p"][pi, None], c["p"][None, ci]
            pq = (b["P"][pi, None] - c["P"][None, ci]).transpose(2, 0, 1)
            pre = 2 * np.pi ** 2.5 / (p * q * np.sqrt(p + q))
            R = _hermite_r(sum(b["key"]) + sum(c["key"]), p * q / (p + q), pq)
            M = np.stack([np.stack([R[tuple(x + y for x, y in zip(s, t))] for t in c["herm"]], -1)
                          for s in b["herm"]], -2) * pre[..., None, None] * sign
            v = b["Eab"][pi, None] @ M @ c["Eab"][None, ci].transpose(0, 1, 3, 2)
            if diagonal:
                out[i] = v.sum((0, 1))
            else:
                v = np.add.reduceat(v, c["start"], axis=1)
                out[i:i + step] = np.add.reduceat(v, b["start"][i:i + step] - ne[i], axis=0)
        return out


def _odd(l):
    """(2 l - 1)!!"""
    return float(np.prod(np.arange(2 * l - 1, 1, -2))) if l > 1 else 1.0
