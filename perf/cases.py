"""The work that a user of this eigensolver has it do, as timed cases.

A case is one call (or, for the fit, one forward and backward pass) through the
package's public entry points:

  apply   one block product W = H V, the step that an outside eigensolver, a
          strength-function code or the library's own solver repeats
  solve   the lowest levels of one space, start to end
  grad    the Hellmann-Feynman gradient of a weighted eigenvalue sum for
          eigenvectors that the program already holds
  fit     one step of an interaction fit: new matrix elements, the lowest levels
          and their gradient (torch autograd)

Spaces are the shells and nucleon numbers of the workloads, tests and benchmark
of this repository (sd, pf, and the 50-82 neutron shell) and their odd
neighbours. Interactions and vectors are drawn from the seed: i.i.d. normal
J-coupled elements and normal columns of about unit norm.

`exact` holds a plain torch statement of the same quantities in 64 bits: every
m-scheme term is applied one at a time.
"""
from __future__ import annotations

import itertools
import math
from functools import lru_cache

import numpy as np
import torch

import paper_1902_02064_amd as trbl

# shells: orbits (n, l, 2j) and their single-particle energies
SHELLS = {
    "sd": (((0, 2, 5), (1, 0, 1), (0, 2, 3)), (-3.9, -3.2, 2.1)),
    "pf": (((0, 3, 7), (1, 1, 3), (0, 3, 5), (1, 1, 1)), (0.0, 2.0, 4.0, 6.0)),
    "sn": (((0, 4, 7), (1, 2, 5), (1, 2, 3), (2, 0, 1), (0, 5, 11)), (0.0, 0.2, 1.5, 1.8, 2.4)),
}


def _space(shell, n_prot, n_neut):
    return {"shell": shell, "n_prot": n_prot, "n_neut": n_neut, "twoM": (n_prot + n_neut) % 2,
            "parity": 1 if shell == "sn" else 0}


def listed():
    return [
        # the smallest product: 20Ne in the sd shell (D = 640), where the launches count
        {"name": "apply sd 2+2 nb4 f64", "do": "apply", **_space("sd", 2, 2), "nb": 4, "dtype": "f64"},
        # the largest sd space, 28Si (D = 93,710)
        {"name": "apply sd 6+6 nb8 f64", "do": "apply", **_space("sd", 6, 6), "nb": 8, "dtype": "f64"},
        # an odd-mass pf nucleus (47V shape) with a block width that fills no tile
        {"name": "apply pf 3+4 nb12 f64", "do": "apply", **_space("pf", 3, 4), "nb": 12, "dtype": "f64"},
        # 48Cr shape (D = 1,963,461): the ordinary product of the block solver, in both precisions
        {"name": "apply pf 4+4 nb16 f64", "do": "apply", **_space("pf", 4, 4), "nb": 16, "dtype": "f64"},
        {"name": "apply pf 4+4 nb16 f32", "do": "apply", **_space("pf", 4, 4), "nb": 16, "dtype": "f32"},
        # the same space one vector at a time: plain Lanczos, strength functions
        {"name": "apply pf 4+4 nb1 f64", "do": "apply", **_space("pf", 4, 4), "nb": 1, "dtype": "f64"},
        # the largest space one GPU solves (D = 109,954,620), in the precision it is solved in
        {"name": "apply pf 6+6 nb32 f32", "do": "apply", **_space("pf", 6, 6), "nb": 32, "dtype": "f32"},
        # 112Sn shape (D = 6,210,638): one species only
        {"name": "apply sn 0+12 nb8 f64", "do": "apply", **_space("sn", 0, 12), "nb": 8, "dtype": "f64"},
        # level schemes: 28Si, 20 lowest, and 48Cr, 10 lowest
        {"name": "solve sd 6+6 n20", "do": "solve", **_space("sd", 6, 6), "nb": 8, "n_eig": 20, "l_s": 40,
         "l_m": 120, "tol": 1e-10},
        {"name": "solve pf 4+4 n10", "do": "solve", **_space("pf", 4, 4), "nb": 16, "n_eig": 10, "l_s": 40,
         "l_m": 200, "tol": 1e-8},
        # the gradient of 20 levels of 28Si with eigenvectors at hand
        {"name": "grad sd 6+6 n20", "do": "grad", **_space("sd", 6, 6), "n_eig": 20},
        # one step of an interaction fit to the 10 lowest levels of 20Ne (the tolerance that the gradient's
        # own solve takes by default)
        {"name": "fit sd 2+2 n10", "do": "fit", **_space("sd", 2, 2), "nb": 4, "n_eig": 10, "l_s": 20, "l_m": 60,
         "tol": 1e-10},
    ]


def draw(rng):
    """One more case: the same calls on spaces, widths and precisions between the listed ones."""
    what = rng.choice(("apply",) * 7 + ("solve", "grad", "fit"))
    if what == "apply":
        shell = rng.choice(("sd", "pf", "pf", "sn"))
        while True:
            if shell == "sn":
                case = _space("sn", 0, rng.choice((4, 6, 8, 10, 12)))
            else:
                hi = 6 if shell == "sd" else 5
                case = _space(shell, rng.randint(1, hi), rng.randint(1, hi))
            nb = int(round(math.exp(rng.uniform(0.0, math.log(40.0)))))
            # memory and time stay below the largest listed product
            if 300 <= _dimension(case) and _dimension(case) * nb <= 4e8:
                break
        return {"do": "apply", **case, "nb": nb, "dtype": rng.choice(("f64", "f32"))}
    if what == "solve":
        shell, a, b = rng.choice((("sd", 3, 4), ("sd", 4, 4), ("sd", 5, 5), ("sd", 6, 5), ("pf", 2, 3), ("pf", 3, 3)))
        n, nb = rng.randint(1, 24), rng.choice((2, 4, 6, 8, 12, 16))
        l_s = max(2 * n, 16)
        return {"do": "solve", **_space(shell, a, b), "nb": nb, "n_eig": n, "l_s": l_s,
                "l_m": l_s + 10 * nb + rng.randint(0, 3), "tol": 1e-9}
    if what == "grad":
        shell, a, b = rng.choice((("sd", 3, 4), ("sd", 4, 4), ("sd", 5, 6), ("pf", 2, 2), ("pf", 3, 3)))
        return {"do": "grad", **_space(shell, a, b), "n_eig": rng.randint(1, 32)}
    a, b = rng.choice(((2, 2), (2, 3), (3, 2), (1, 4)))
    n, nb = rng.randint(2, 12), rng.choice((2, 3, 4, 6))
    return {"do": "fit", **_space("sd", a, b), "nb": nb, "n_eig": n, "l_s": 2 * n + 4, "l_m": 2 * n + 4 + 8 * nb,
            "tol": 1e-10}


# ------------------------------------------------------------------ inputs
def _pairs(orbits, channel, twoJ, parity):
    """Orbit pairs of one channel (0 pp, 1 nn, 2 pn) that couple to J and the parity."""
    out = []
    for a, b in itertools.product(range(len(orbits)), repeat=2):
        (_, la, ja), (_, lb, jb) = orbits[a], orbits[b]
        if (la + lb) % 2 != parity or not abs(ja - jb) <= twoJ <= ja + jb:
            continue
        if channel != 2 and (a > b or (a == b and twoJ % 4 == 2)):
            continue
        out.append((a, b))
    return out


@lru_cache(maxsize=None)
def _elements(shell):
    """(channel, a, b, c, d, 2J) of every independent J-coupled element of a shell."""
    orbits = SHELLS[shell][0]
    out = []
    for ch in range(3):
        for twoJ in range(0, 2 * max(o[2] for o in orbits) + 1, 2):
            for parity in (0, 1):
                p = _pairs(orbits, ch, twoJ, parity)
                out += [(ch, *p[i], *p[j], twoJ) for i in range(len(p)) for j in range(i, len(p))]
    return tuple(out)


def _interaction(case, seed):
    v = np.random.default_rng(seed).standard_normal(len(_elements(case["shell"])))
    return [(*e, float(x)) for e, x in zip(_elements(case["shell"]), v)]


def _vectors(case, D, cols, seed, device="cuda"):
    dtype = torch.float32 if case.get("dtype") == "f32" else torch.float64
    g = torch.Generator(device=device).manual_seed(seed)
    return torch.randn(D, cols, generator=g, dtype=dtype, device=device).div_(math.sqrt(D))


def prepare(case, seed):
    orbits, spe = SHELLS[case["shell"]]
    model = trbl.Model(orbits, case["n_prot"], case["n_neut"], case["twoM"], case["parity"])
    s = {"case": case, "model": model}
    tbme = _interaction(case, seed)
    if case["do"] == "fit":
        s["structure"] = [t[:6] for t in tbme]
        s["v"] = torch.tensor([t[6] for t in tbme], dtype=torch.float64)
        s["spe"] = torch.tensor(spe, dtype=torch.float64)
        return s
    model.set_hamiltonian(spe, spe, tbme)
    if case["do"] == "apply":
        s["V"] = _vectors(case, model.dim, case["nb"], seed)
        s["W"] = torch.empty_like(s["V"])
    elif case["do"] == "grad":
        s["X"] = _vectors(case, model.dim, case["n_eig"], seed)
        s["w"] = _weights(case, seed)
    return s


def _weights(case, seed):
    return np.random.default_rng(seed + 1).uniform(0.1, 1.0, case["n_eig"])


def run(s):
    c, m = s["case"], s["model"]
    if c["do"] == "apply":
        return m.apply(s["V"], s["W"])
    if c["do"] == "solve":
        ev, _, info = m.solve(c["nb"], c["n_eig"], c["l_s"], c["l_m"], c["tol"], check_every=-1)
        return {"levels": ev, "converged": info.converged}
    if c["do"] == "grad":
        gv, gs = m.tbme_grad(s["w"], evecs=s["X"])
        return {"tbme": gv, "spe": gs}
    v, ep, en = s["v"].clone().requires_grad_(), s["spe"].clone().requires_grad_(), s["spe"].clone().requires_grad_()
    e = trbl.eigenvalues(m, s["structure"], v, ep, en, c["nb"], c["n_eig"], c["l_s"], c["l_m"], c["tol"])
    e.sum().backward()
    return {"levels": e.detach(), "tbme": v.grad, "spe_p": ep.grad, "spe_n": en.grad}


# ------------------------------------------------------------------ sizes
@lru_cache(maxsize=None)
def _states(shell):
    """(orbit, 2m, odd l) of the m-states of a shell: orbits in order, 2m ascending."""
    return tuple((o, tm, l % 2) for o, (_, l, tj) in enumerate(SHELLS[shell][0]) for tm in range(-tj, tj + 1, 2))


@lru_cache(maxsize=None)
def _counts(shell, n):
    """Number of n-particle determinants by (2M, odd parity)."""
    have = {(0, 0, 0): 1}
    for _, tm, par in _states(shell):
        for (k, M, p), cnt in list(have.items()):
            if k < n:
                key = (k + 1, M + tm, p ^ par)
                have[key] = have.get(key, 0) + cnt
    return {key[1:]: cnt for key, cnt in have.items() if key[0] == n}


def _dimension(case):
    neut = _counts(case["shell"], case["n_neut"])
    return sum(cnt * neut.get((case["twoM"] - M, q), 0)
               for (M, p), cnt in _counts(case["shell"], case["n_prot"]).items()
               for q in (0, 1) if case["parity"] == 0 or (p ^ q) == (case["parity"] < 0))


def _elements_per_row(case):
    """Matrix elements of H that one basis state links to, estimated: for each pair of its nucleons,
    the pair states of the same 2M and parity that the other nucleons leave free, on average."""
    st = _states(case["shell"])
    ns, a, b = len(st), case["n_prot"], case["n_neut"]

    def mean_group(same):
        size = {}
        for i, j in itertools.product(range(ns), repeat=2):
            if not same or i < j:
                key = (st[i][1] + st[j][1], st[i][2] ^ st[j][2])
                size[key] = size.get(key, 0) + 1
        return sum(x * x for x in size.values()) / sum(size.values())

    def free(n):
        return max(0.0, (ns - n) / ns)

    return (1 + a * b * mean_group(False) * free(a - 1) * free(b - 1)
            + a * (a - 1) / 2 * mean_group(True) * free(a - 2) ** 2
            + b * (b - 1) / 2 * mean_group(True) * free(b - 2) ** 2)


def work(case):
    """apply: V once, W once, two operations per element and column. grad: the vectors once, two
    operations per element and vector. solve and fit: at least one basis of l_s vectors built with
    one product and one orthogonalisation against the earlier ones for each."""
    D, G = _dimension(case), _elements_per_row(case)
    if case["do"] == "apply":
        size = 4 if case["dtype"] == "f32" else 8
        return {"bytes": 2.0 * D * case["nb"] * size, "flops": 2.0 * D * case["nb"] * G}
    if case["do"] == "grad":
        n = case["n_eig"]
        return {"bytes": 8.0 * D * n, "flops": 2.0 * D * n * G}
    n = case["l_s"]
    return {"bytes": 8.0 * D * n * (2 + n / (2.0 * case["nb"])), "flops": 2.0 * D * n * (G + 2.0 * n)}


# ------------------------------------------------------------------ the same in plain torch, 64 bits
@lru_cache(maxsize=None)
def _cg(j1, m1, j2, m2, J, M):
    """<j1 m1 j2 m2 | J M> (Racah's sum), all arguments doubled."""
    if m1 + m2 != M or not abs(j1 - j2) <= J <= j1 + j2 or abs(M) > J:
        return 0.0
    f = lambda x: math.factorial(x // 2)  # noqa: E731
    pre = (J + 1) * f(j1 + j2 - J) * f(j1 - j2 + J) * f(j2 - j1 + J) / f(j1 + j2 + J + 2)
    pre *= f(j1 + m1) * f(j1 - m1) * f(j2 + m2) * f(j2 - m2) * f(J + M) * f(J - M)
    total = 0.0
    for k in range(0, j1 + j2 + 2, 2):
        args = (k, j1 + j2 - J - k, j1 - m1 - k, j2 + m2 - k, J - j2 + m1 + k, J - j1 - m2 + k)
        if min(args) >= 0:
            total += (-1) ** (k // 2) / math.prod(f(x) for x in args)
    return math.sqrt(pre) * total


def _terms(shell, channel):
    """{(alpha, beta, gamma, delta): [(element, coefficient)]} of c+_alpha c+_beta c_delta c_gamma
    (alpha < beta and gamma < delta for identical particles; alpha, gamma protons for pn)."""
    orbits, st, out = SHELLS[shell][0], _states(shell), {}

    def coupled(a, b, twoJ):
        for i, (oi, mi, _) in enumerate(st):
            for j, (oj, mj, _) in enumerate(st):
                if (oi, oj) == (a, b) and (channel == 2 or i < j):
                    c = _cg(orbits[a][2], mi, orbits[b][2], mj, twoJ, mi + mj)
                    c *= math.sqrt(2.0) if channel != 2 and a == b else 1.0
                    if c:
                        yield i, j, mi + mj, c

    for n, (ch, a, b, c, d, twoJ) in enumerate(_elements(shell)):
        if ch != channel:
            continue
        for left, right in {((a, b), (c, d)), ((c, d), (a, b))}:
            r = list(coupled(*right, twoJ))
            for i, j, M, x in coupled(*left, twoJ):
                for k, l, N, y in r:
                    if M == N:
                        out.setdefault((i, j, k, l), []).append((n, x * y))
    return out


class _Plain:
    """Determinants of one species in the library's order, as tensors: words, sectors, occupations."""

    def __init__(self, shell, n, keep=None, device="cpu"):
        st = _states(shell)
        comb = np.array(list(itertools.combinations(range(len(st)), n)), dtype=np.int64)
        comb = comb.reshape(math.comb(len(st), n), n)
        tm = np.array([s[1] for s in st])[comb].sum(1)
        par = np.array([s[2] for s in st])[comb].sum(1) % 2
        if keep is not None:
            ok = np.array([(int(M), int(p)) in keep for M, p in zip(tm, par)], dtype=bool)
            comb, tm, par = comb[ok], tm[ok], par[ok]
        orb = np.array([s[0] for s in st])[comb]
        occ = [-(orb == o).sum(1) for o in range(len(SHELLS[shell][0]))]
        order = np.lexsort([*reversed(occ), par, tm])  # stable: tuples stay ascending inside a partition
        comb, self.tm, self.par = comb[order], tm[order], par[order]
        words = (np.int64(1) << comb).sum(1)
        self.ns, self.n, self.words = len(st), n, torch.from_numpy(words).to(device)
        self.sorted, self.place = torch.sort(self.words)
        bits = (words[:, None] >> np.arange(len(st))) & 1
        self.occ = torch.from_numpy(bits.astype(bool)).to(device)
        self.below = torch.from_numpy(np.cumsum(bits, 1) - bits).to(device)  # occupied states below s

    def at(self, words):
        return self.place[torch.searchsorted(self.sorted, words).clamp_(max=len(self.sorted) - 1)]

    def known(self, words):
        return self.words[self.at(words)] == words

    def move(self, new, old):
        """c+_new c_old: (targets, sources, signs); lists of one or two distinct states, ascending."""
        ok = torch.ones(len(self.words), dtype=torch.bool, device=self.words.device)
        for s in old:
            ok &= self.occ[:, s]
        for s in new:
            if s not in old:
                ok &= ~self.occ[:, s]
        src = torch.nonzero(ok)[:, 0]
        w = self.words[src]
        for s in old:
            w = w ^ (1 << s)
        swaps = torch.zeros_like(src)
        for s in (*old, *new):
            swaps += self.below[src, s] - sum(o < s for o in old)
        for s in new:
            w = w | (1 << s)
        hit = self.known(w)
        src, w, swaps = src[hit], w[hit], swaps[hit]
        return self.at(w), src, (1 - 2 * (swaps & 1)).to(torch.float64)


class _Reference:
    """One space: the products and densities of its Hamiltonian, one m-scheme term at a time."""

    def __init__(self, case):
        self.case = case
        dev = self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        shell, want = case["shell"], case["parity"]
        kp, kn = _counts(shell, case["n_prot"]), _counts(shell, case["n_neut"])
        fits = [((M, p), (N, q)) for M, p in sorted(kp) for N, q in sorted(kn)
                if M + N == case["twoM"] and (want == 0 or (p ^ q) == (want < 0))]
        self.sp = [_Plain(shell, case["n_prot"], {f[0] for f in fits}, dev),
                   _Plain(shell, case["n_neut"], {f[1] for f in fits}, dev)]
        rows = []
        for fp, fn in fits:
            r = [torch.from_numpy(np.flatnonzero((s.tm == f[0]) & (s.par == f[1]))).to(dev)
                 for s, f in zip(self.sp, (fp, fn))]
            rows.append((r[0][:, None] * len(self.sp[1].words) + r[1][None, :]).reshape(-1))
        self.cell = torch.cat(rows)  # basis state -> cell of the proton x neutron grid

    def grid(self, V):
        g = torch.zeros(len(self.sp[0].words) * len(self.sp[1].words), V.shape[1], dtype=torch.float64, device=self.dev)
        g[self.cell] = V.to(torch.float64)
        return g.view(len(self.sp[0].words), len(self.sp[1].words), V.shape[1])

    def energies(self, s):
        e = torch.tensor([SHELLS[self.case["shell"]][1][o] for o, _, _ in _states(self.case["shell"])],
                         dtype=torch.float64, device=self.dev)
        return self.sp[s].occ.to(torch.float64) @ e

    def identical(self, s):
        """(term, targets, sources, signs) of every two-body move of one species."""
        if self.sp[s].n >= 2:
            for t, elements in _terms(self.case["shell"], s).items():
                i, j, x = self.sp[s].move(t[:2], t[2:])
                if len(j):
                    yield elements, i, j, x

    def apply(self, V, v):
        A = self.grid(V)
        W = (self.energies(0)[:, None, None] + self.energies(1)[None, :, None]) * A
        h = lambda elements: sum(v[n] * c for n, c in elements)  # noqa: E731
        for elements, i, j, x in self.identical(0):
            W.index_add_(0, i, A[j] * (h(elements) * x)[:, None, None])
        for elements, i, j, x in self.identical(1):
            W.index_add_(1, i, A[:, j] * (h(elements) * x)[None, :, None])
        if self.sp[0].n and self.sp[1].n:
            moves = {}
            for (a, b, c, d), elements in _terms(self.case["shell"], 2).items():
                moves.setdefault((a, c), []).append((b, d, h(elements)))
            inner = {}
            for (a, c), lst in moves.items():
                i, j, x = self.sp[0].move((a,), (c,))
                if not len(j):
                    continue
                B, Y = A[j] * x[:, None, None], torch.zeros(len(j), *A.shape[1:], dtype=torch.float64, device=self.dev)
                for b, d, hv in lst:
                    if (b, d) not in inner:
                        inner[b, d] = self.sp[1].move((b,), (d,))
                    k, l, y = inner[b, d]
                    if len(l):
                        Y.index_add_(1, k, B[:, l] * (hv * y)[None, :, None])
                W.index_add_(0, i, Y)
        return W.reshape(-1, V.shape[1])[self.cell]

    def gradient(self, X, w):
        """d(sum_k w_k <x_k|H|x_k>) by element, and by proton then neutron orbit energy."""
        A = self.grid(X)
        Aw = A * torch.as_tensor(w, dtype=torch.float64, device=self.dev)
        out = [torch.zeros((), dtype=torch.float64, device=self.dev) for _ in _elements(self.case["shell"])]
        rho = [None, None]
        n = A.shape[0] * A.shape[1]
        rho[0] = A.reshape(A.shape[0], -1) @ Aw.reshape(A.shape[0], -1).T
        At, Awt = (t.transpose(0, 1).reshape(A.shape[1], -1) for t in (A, Aw))
        rho[1] = At @ Awt.T
        for s in (0, 1):
            for elements, i, j, x in self.identical(s):
                r = (rho[s][i, j] * x).sum()
                for e, c in elements:
                    out[e] = out[e] + c * r
        if self.sp[0].n and self.sp[1].n:
            pairs = {}
            for (a, b, c, d), elements in _terms(self.case["shell"], 2).items():
                pairs.setdefault((a, c), []).append((b, d, elements))
            inner = {}
            for (a, c), lst in pairs.items():
                i, j, x = self.sp[0].move((a,), (c,))
                if not len(j):
                    continue
                # density between neutron determinants for this proton move
                L = (A[i] * x[:, None, None]).transpose(0, 1).reshape(A.shape[1], -1)
                R = Aw[j].transpose(0, 1).reshape(A.shape[1], -1)
                Rho = L @ R.T
                for b, d, elements in lst:
                    if (b, d) not in inner:
                        inner[b, d] = self.sp[1].move((b,), (d,))
                    k, l, y = inner[b, d]
                    if len(l):
                        r = (Rho[k, l] * y).sum()
                        for e, cc in elements:
                            out[e] = out[e] + cc * r
        gs = []
        for s in (0, 1):
            occ = torch.diagonal(rho[s]) @ self.sp[s].occ.to(torch.float64)
            for o in range(len(SHELLS[self.case["shell"]][0])):
                gs.append(sum((occ[k] for k, st in enumerate(_states(self.case["shell"])) if st[0] == o),
                              torch.zeros((), dtype=torch.float64, device=self.dev)))
        return torch.stack(out).cpu().numpy(), torch.stack(gs).cpu().numpy()


def exact(case, seed):
    grid = math.comb(len(_states(case["shell"])), case["n_prot"]) * math.comb(len(_states(case["shell"])), case["n_neut"])
    v = [t[6] for t in _interaction(case, seed)]
    if case["do"] == "apply":
        if grid * case["nb"] * 8 > 6e9 or (case["shell"] == "sn" and _dimension(case) > 150_000):
            return None  # minutes of single terms
        V = _vectors(case, _dimension(case), case["nb"], seed)
        return _Reference(case).apply(V, v)
    if case["do"] == "grad":
        if grid > 1_500_000:
            return None
        gv, gs = _Reference(case).gradient(_vectors(case, _dimension(case), case["n_eig"], seed), _weights(case, seed))
        return {"tbme": gv, "spe": gs}
    if _dimension(case) > 2000:
        return None  # no dense matrix of that size in the time
    ref, n = _Reference(case), case["n_eig"]
    H = ref.apply(torch.eye(_dimension(case), dtype=torch.float64, device=ref.dev), v)
    e, U = np.linalg.eigh(H.cpu().numpy())
    if case["do"] == "solve":
        return {"levels": e[:n], "converged": None}
    gv, gs = ref.gradient(torch.from_numpy(np.ascontiguousarray(U[:, :n])).to(ref.dev), np.ones(n))
    half = len(gs) // 2
    return {"levels": e[:n], "tbme": gv, "spe_p": gs[:half], "spe_n": gs[half:]}
