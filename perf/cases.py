"""Timed work of the library through its public entry points.

A pass is one Newton step as an interior-point program takes it: the values of
the condensed system on the GPU are refactored and solved (Lifted-KKT, HyKKT,
the augmented system, a whole interior-point solve, a batch, a burst of served
requests, the stage-structured solver). The patterns are the generators'
(``kktgen``): NMPC stages with dense Hessian blocks, distillation-column-shaped
stages, band-limited unstructured systems. A pattern's symbolic analysis is kept
for its lifetime, as a program does that solves one pattern many times.

``sigma`` is the decimal exponent of the diagonals' range, Sigma ~
logU[10^-sigma, 10^sigma]: 2 early in an interior-point run, 6 late in it.
"""
import functools
import math

import kktgen
import numpy as np
import torch

from paper_2403_15913_amd import kkt

DEV = "cuda" if torch.cuda.is_available() else "cpu"


def listed():
    return [
        # the smallest call: one controller's step on a short horizon (latency and launches)
        dict(name="small", do="lifted", kind="nmpc", N=50, nx=8, nu=1, sigma=2),
        # an ordinary horizon of odd sizes late in the iterations; predictor and corrector share the factor
        dict(name="nmpc_two_solves", do="lifted", kind="nmpc", N=173, nx=37, nu=3, sigma=6, solves=2),
        # the paper's scale: 2,000 stages of a distillation column at the analysis options the autotuner keeps for it
        dict(name="paper", do="lifted", kind="dist", N=2000, sigma=6, ordering=2, nd_leaf=417),
        # no stages: a band-limited unstructured system (a one-dimensional mesh) with default options
        dict(name="banded", do="lifted", kind="band", n=20001, m=11987, band=40, sigma=4),
        # equality constraints kept: K_gamma and the Schur-complement CG at the paper's scale
        dict(name="hykkt", do="hykkt", kind="dist", N=2000, sigma=2, gamma=1e6, ordering=2, nd_leaf=417),
        # one interior-point step on the augmented system: inertia-checked refactor, slack and multiplier steps
        dict(name="augmented", do="augmented", kind="dist", N=301, sigma=4),
        # a whole convex QP by the interior-point loop
        dict(name="ipm", do="ipm", kind="dist", N=200, sigma=2),
        # many plants at once: 256 instances of mixed horizons and widths, eager refactor and solve
        dict(name="batch_mixed", do="batch", kind="nmpc", count=256, shapes=64, sigma=6, ordering=2, nd_leaf=512,
             max_super=48, small=48),
        # an ensemble of one small controller, replayed as a graph
        dict(name="batch_small", do="graph", kind="nmpc", N=50, nx=8, nu=1, count=256, sigma=2),
        # a burst of requests over resident patterns of different sizes
        dict(name="served", do="served", kind="nmpc", patterns=8, requests=24, n_lo=1000, n_hi=30000, sigma=6),
        # the block-tridiagonal solver at the paper's scale
        dict(name="stagewise", do="stagewise", kind="dist", N=2000, count=1, sigma=6),
        # stages hundreds of variables wide: fronts too tall for LDS
        dict(name="wide", do="lifted", kind="nmpc", N=4, nx=700, nu=4, sigma=6, ordering=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["nmpc", "nmpc", "dist", "dist", "band", "hykkt", "augmented", "ipm", "batch", "graph", "served",
                     "stagewise", "wide"])
    sigma = rng.randint(2, 6)
    nmpc = dict(kind="nmpc", nx=rng.randint(5, 64), nu=rng.randint(1, 4))
    if do == "nmpc":
        return dict(do="lifted", N=_log(rng, 20, 1500), sigma=sigma, solves=rng.randint(1, 2), **nmpc)
    if do == "dist":
        return dict(do="lifted", kind="dist", N=_log(rng, 20, 2000), sigma=sigma)
    if do == "band":
        n = _log(rng, 300, 40000)
        return dict(do="lifted", kind="band", n=n, m=int(n * rng.uniform(0.2, 1.0)), band=rng.randint(12, 48), sigma=4)
    if do == "hykkt":
        shape = dict(kind="dist") if rng.random() < 0.5 else nmpc
        return dict(do="hykkt", N=_log(rng, 30, 1500), sigma=2, gamma=rng.choice([1e4, 1e5, 1e6]), **shape)
    if do == "augmented":
        shape = dict(kind="dist") if rng.random() < 0.5 else nmpc
        return dict(do="augmented", N=_log(rng, 30, 1200), sigma=rng.randint(2, 4), **shape)
    if do == "ipm":
        return dict(do="ipm", N=_log(rng, 20, 200), sigma=2, **nmpc)
    if do == "batch":
        return dict(do="batch", kind="nmpc", count=_log(rng, 8, 200), shapes=rng.randint(3, 24), sigma=sigma,
                    ordering=2, nd_leaf=rng.choice([0, 256, 512]), max_super=48, small=rng.choice([0, 48]))
    if do == "graph":
        return dict(do="graph", kind="nmpc", N=_log(rng, 10, 60), nx=rng.randint(3, 20), nu=rng.randint(1, 3),
                    count=_log(rng, 1, 256), sigma=2)
    if do == "served":
        return dict(do="served", kind="nmpc", patterns=rng.randint(2, 6), requests=_log(rng, 4, 24), n_lo=1000,
                    n_hi=_log(rng, 4000, 30000), sigma=sigma)
    if do == "stagewise":
        shape = dict(kind="dist") if rng.random() < 0.5 else nmpc
        return dict(do="stagewise", N=_log(rng, 20, 1000), count=rng.choice([1, 1, 4]), sigma=sigma, **shape)
    return dict(do="lifted", kind="nmpc", N=rng.randint(3, 6), nx=rng.randint(160, 600), nu=rng.randint(1, 4),
                sigma=sigma, ordering=rng.choice([0, 2]))


# ---------------------------------------------------------------------------
# patterns, analyses and values
# ---------------------------------------------------------------------------

class Shape:
    """One pattern: its arrays, stage (or band) width, and the recipe of its J values."""

    def __init__(self, key):
        kind, a, b, c = key
        self.kind = kind
        if kind == "band":
            self.pat = kktgen.general_pattern(kktgen.rng_for(5, a, c), a, b, 0.12, band=c)
            self.s = c
            return
        self.pat = p = kktgen.nmpc_pattern(a, b, c) if kind == "nmpc" else kktgen.distillation_pattern(a)
        nx = p.meta["nx"]
        self.s = s = p.meta["stage"]
        row = np.repeat(np.arange(p.m), np.diff(p.j_rowptr))
        last = p.j_colind[p.j_rowptr[1:] - 1][row]
        stage, local = p.j_colind // s, p.j_colind % s
        base, uni, nor = np.zeros(p.nnz_j), np.zeros(p.nnz_j), np.zeros(p.nnz_j)
        first = row < nx
        one = first | ((p.j_colind == last) & (last % s < nx) & (np.diff(p.j_rowptr)[row] > 1))
        if kind == "nmpc":
            i = (row - nx) % nx
            state = ~one & (local < nx)
            uni[state] = 0.5
            base[state & (local == i)] = -0.9
            nor[~one & (local >= nx)] = 1.0
        else:
            na = p.meta["na"]
            uni[~one] = 1.0
            alg = ~one & (last % s >= nx)             # the stage's own algebraic rows: identity plus a small part
            k = (row - nx) - stage * (nx + na)
            eye = alg & (local - nx < na)
            uni[eye] = np.where(local[eye] - nx == k[eye], 0.0, 0.25)
            base[eye & (local - nx == k)] = 1.0
        base[one] = 1.0
        self.recipe = [torch.tensor(v, device=DEV) for v in (base, uni, nor)]
        if kind == "nmpc":
            self.tril = torch.tril_indices(s, s, device=DEV)
        else:
            self.keep = torch.tensor(np.arange(s)[:, None] + np.arange(-2, 1)[None] >= 0, device=DEV)


@functools.lru_cache(maxsize=96)
def shape(key):
    return Shape(key)


@functools.lru_cache(maxsize=96)
def analysis(key, ordering=0, nd_leaf=0, max_super=0):
    return kkt.Symbolic.from_pattern(shape(key).pat, ordering=ordering, nd_leaf=nd_leaf, max_super=max_super)


def keys(case):
    """The pattern of every instance of a case."""
    if case["do"] == "batch":
        mixed = [("nmpc", *sh) for sh in kktgen.batch_shapes(case["shapes"])]
        return [mixed[q % len(mixed)] for q in range(case["count"])]
    if case["do"] == "served":
        pats = [("nmpc", *sh) for sh in kktgen.serving_shapes(case["patterns"], n_lo=case["n_lo"], n_hi=case["n_hi"])]
        return [pats[q % len(pats)] for q in range(case["requests"])]
    if case["kind"] == "band":
        key = ("band", case["n"], case["m"], case["band"])
    elif case["kind"] == "dist":
        key = ("dist", case["N"], 0, 0)
    else:
        key = ("nmpc", case["N"], case["nx"], case["nu"])
    return [key] * case.get("count", 1)


def options(case):
    return tuple(case.get(k, 0) for k in ("ordering", "nd_leaf", "max_super"))


def values(key, sigma, gen, seed):
    """w, j, Sigma_x, Sigma_s of one instance."""
    sh = shape(key)
    p = sh.pat

    def uniform(*size):
        return torch.rand(*size, generator=gen, device=DEV, dtype=torch.float64)

    def normal(*size):
        return torch.randn(*size, generator=gen, device=DEV, dtype=torch.float64)

    if key[0] == "band":
        v = kktgen.general_values(p, np.random.default_rng(seed), 0.1, 1.0)
        w, j = (torch.tensor(a, device=DEV) for a in (v.w_vals, v.j_vals))
    else:
        N, s = p.meta["N"], sh.s
        if key[0] == "nmpc":
            M = normal(N, s, s)
            W = torch.bmm(M, M.transpose(1, 2).contiguous())
            W.diagonal(dim1=1, dim2=2).add_(0.1)
            w = W[:, sh.tril[0], sh.tril[1]].reshape(-1)
        else:
            # W_k = M M^T + 0.1 I with M lower banded (three diagonals m0, m1, m2)
            m = normal(3, N, s)
            m[1, :, :1] = 0.0
            m[2, :, :2] = 0.0
            band = torch.zeros(N, s, 3, dtype=torch.float64, device=DEV)
            band[:, :, 2] = (m * m).sum(0) + 0.1
            band[:, 1:, 1] = m[1, :, 1:] * m[0, :, :-1] + m[2, :, 1:] * m[1, :, :-1]
            band[:, 2:, 0] = m[2, :, 2:] * m[0, :, :-2]
            w = band[:, sh.keep].reshape(-1)
        base, uni, nor = sh.recipe
        j = base + uni * (2.0 * uniform(p.nnz_j) - 1.0) + nor * normal(p.nnz_j)
    span = sigma * math.log(10.0)
    sx, ss = (torch.exp(span * (2.0 * uniform(k) - 1.0)) for k in (p.n, p.m))
    return w, j, sx, ss


def inputs(case, seed):
    """One dict of tensors per instance."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    out = []
    for q, key in enumerate(keys(case)):
        p = shape(key).pat
        d = dict(zip(("w", "j", "sx", "ss"), values(key, case["sigma"], gen, seed * 1000 + q)))
        for name, k in (("b", p.n), ("b2", p.n), ("g", p.m), ("r4", p.m)):
            d[name] = torch.randn(k, generator=gen, device=DEV, dtype=torch.float64)
        if case["do"] == "ipm":
            d["u"] = 0.1 + d["g"].abs()
        out.append(d)
    return out


# ---------------------------------------------------------------------------
# the passes
# ---------------------------------------------------------------------------

def prepare(case, seed):
    ins = inputs(case, seed)
    ks = keys(case)
    do = case["do"]
    st = dict(case=case, **ins[0])
    zeros = [torch.zeros(d["b"].shape[0], dtype=torch.float64, device=DEV) for d in ins]
    if do in ("lifted", "hykkt", "augmented", "ipm"):
        st["factor"] = f = kkt.Factor(analysis(ks[0], *options(case)))
        f.keep_augmented(do == "augmented")
        st["x"] = [torch.zeros_like(ins[0]["b"]) for _ in range(case.get("solves", 1))]
        st["dual"] = [torch.zeros_like(ins[0]["g"]) for _ in range(2)]
    elif do in ("batch", "graph", "stagewise"):
        cat = {k: torch.cat([d[k] for d in ins]) for k in ("w", "j", "sx", "ss", "b")}
        st.update(cat, x=torch.cat(zeros))
        syms = [analysis(k, *options(case)) for k in ks]
        if do == "stagewise":
            ends = [np.arange(0, shape(k).pat.n + 1, shape(k).s, dtype=np.int32) for k in ks]
            st["solver"] = kkt.Stagewise(syms, ends)
        else:
            st["solver"] = B = kkt.Batch(syms)
            B.set_small_fronts(case.get("small", 0))
            if do == "graph":
                B.capture(st["w"], st["j"], st["sx"], st["ss"], st["b"], st["x"], rounds=1)
    else:
        st["server"] = S = kkt.Server(hbm_budget=4 << 30)
        pid = {}
        for k in ks:
            if k not in pid:
                pid[k] = S.register(analysis(k, *options(case)))
        st["requests"] = [(pid[k], d["w"], d["j"], d["sx"], d["ss"], d["b"], x) for k, d, x in zip(ks, ins, zeros)]
    return st


def run(st):
    case = st["case"]
    do = case["do"]
    if do == "lifted":
        f = st["factor"]
        f.refactor(st["w"], st["j"], st["sx"], st["ss"])
        for x, b in zip(st["x"], (st["b"], st["b2"])):
            f.solve(b, x)
        return st["x"]
    if do == "hykkt":
        f, (x,), (dy, _) = st["factor"], st["x"], st["dual"]
        f.refactor(st["w"], st["j"], st["sx"], None, case["gamma"])
        f.cg_schur(st["b"], st["g"], x, dy, tol=1e-10)
        return [x, dy]
    if do == "augmented":
        f, (x,), (ds, dz) = st["factor"], st["x"], st["dual"]
        f.refactor_inertia(st["w"], st["j"], st["sx"], st["ss"])
        f.solve_augmented(st["b"], st["g"], st["r4"], x, ds, dz)
        return [x, ds, dz]
    if do == "ipm":
        f, (x,), (s, z) = st["factor"], st["x"], st["dual"]
        x.zero_()
        s.copy_(st["u"])
        z.fill_(1.0)
        f.ipm_qp(st["w"], st["j"], st["b"], st["u"], x, s, z, tol=1e-8)
        return [x, s, z]
    if do in ("batch", "stagewise"):
        B = st["solver"]
        B.refactor(st["w"], st["j"], st["sx"], st["ss"])
        B.solve(st["b"], st["x"])
        return st["x"]
    if do == "graph":
        st["solver"].replay()
        return st["x"]
    S = st["server"]
    tickets = [S.submit(*r) for r in st["requests"]]
    for t in tickets:
        S.wait(t)
    return [r[-1] for r in st["requests"]]


def work(case):
    """Every input read once and every solution written once; the flops of the exact Cholesky factor in stage order
    (the fewest of the orders in use) and one forward and backward sweep per solve with it."""
    size = flops = 0.0
    counted = {}
    for key in keys(case):
        if key not in counted:
            p, st = shape(key).pat, analysis(key, kkt.ORDER_NATURAL).stats()
            counted[key] = (8.0 * (p.nnz_w + p.nnz_j + 3 * p.n + p.m), st["flops_exact"], 4.0 * st["nnz_l_exact"], p)
        b, fl, sweep, p = counted[key]
        size += b
        if case["do"] == "ipm":
            flops += 10 * (fl + sweep)  # an interior-point run of ten steps at the least
        else:
            flops += fl + sweep * case.get("solves", 1)
        if case["do"] in ("hykkt", "augmented", "ipm"):
            size += 16.0 * p.m + 8.0 * p.n
        size += 16.0 * p.n * (case.get("solves", 1) - 1)
    return dict(bytes=size, flops=flops)


# ---------------------------------------------------------------------------
# the same results in plain numpy
# ---------------------------------------------------------------------------

def block_solve(nb, w, entries, rhs):
    """x of A x = rhs for instances of one block-tridiagonal pattern: `entries` holds the lower triangle as
    (row, column, values (instances, entries)), rhs (instances, vectors, nb * w)."""
    D, E = np.zeros((rhs.shape[0], nb * w * w)), np.zeros((rhs.shape[0], nb * w * w))
    for i, j, v in entries:
        bi, bj, li, lj = i // w, j // w, i % w, j % w
        for A, at, pos in ((D, bi == bj, (bi * w + li) * w + lj), (D, (bi == bj) & (li != lj), (bi * w + lj) * w + li),
                           (E, bi == bj + 1, (bj * w + li) * w + lj)):
            for q in range(len(A)):
                A[q] += np.bincount(pos[at], weights=v[q][at], minlength=nb * w * w)
    D, E = (A.reshape(-1, nb, w, w) for A in (D, E))
    inv, G = [], []
    S = D[:, 0]
    for k in range(nb):
        inv.append(np.linalg.inv(S))
        if k + 1 < nb:
            G.append(E[:, k] @ inv[k])
            S = D[:, k + 1] - G[k] @ E[:, k].transpose(0, 2, 1)

    def once(r):
        y = [r[:, 0]]
        for k in range(1, nb):
            y.append(r[:, k] - G[k - 1] @ y[k - 1])
        x = [inv[nb - 1] @ y[nb - 1]]
        for k in range(nb - 2, -1, -1):
            x.append(inv[k] @ y[k] - G[k].transpose(0, 2, 1) @ x[-1])
        return np.stack(x[::-1], 1)

    r = rhs.reshape(rhs.shape[0], -1, nb, w).transpose(0, 2, 3, 1)  # instance, block, row, vector
    x = once(r)
    for _ in range(2):
        res = r - D @ x
        res[:, 1:] -= E[:, :nb - 1] @ x[:, :-1]
        res[:, :-1] -= E[:, :nb - 1].transpose(0, 1, 3, 2) @ x[:, 1:]
        x = x + once(res)
    return x.transpose(0, 3, 1, 2).reshape(rhs.shape)


def j_products(p, jv, d):
    """Lower entries of J^T diag(d) J: rows, columns, products (instances, products)."""
    start, length = p.j_rowptr[:-1].astype(np.int64), np.diff(p.j_rowptr)
    for ln in np.unique(length[length > 0]):
        rows = np.flatnonzero(length == ln)
        e = start[rows][:, None] + np.arange(ln)[None]
        a, b = np.tril_indices(ln)
        i, j = e[:, a].ravel(), e[:, b].ravel()
        yield p.j_colind[i].astype(np.int64), p.j_colind[j].astype(np.int64), \
            jv[:, i] * jv[:, j] * np.repeat(d[:, rows], len(a), axis=1)


def lifted_exact(key, ins, rhs):
    """K x = rhs of instances of one pattern; rhs (instances, vectors, n)."""
    sh = shape(key)
    p, w = sh.pat, sh.s
    nb = -(-p.n // w)
    wv, jv, sx, ss = (np.stack([d[k].cpu().numpy() for d in ins]) for k in ("w", "j", "sx", "ss"))
    row = np.repeat(np.arange(p.n), np.diff(p.w_rowptr))
    pad = np.arange(p.n, nb * w)
    eye = np.arange(p.n)
    entries = [(row, p.w_colind.astype(np.int64), wv), (eye, eye, sx), (pad, pad, np.ones((len(ins), len(pad))))]
    entries += list(j_products(p, jv, ss))
    full = np.concatenate([rhs, np.zeros(rhs.shape[:2] + (len(pad),))], 2)
    return block_solve(nb, w, entries, full)[:, :, :p.n]


def hykkt_exact(key, d):
    """[[W + Sx, J^T], [J, 0]] [dx; dy] = [b; g] with every row of J placed in the stage of its last variable."""
    sh = shape(key)
    p, s = sh.pat, sh.s
    nb = p.meta["N"]
    w = s + p.m // nb
    stage_of = p.j_colind[p.j_rowptr[1:] - 1] // s
    order = np.argsort(stage_of, kind="stable")
    at_row = np.empty(p.m, np.int64)
    at_row[order] = stage_of[order] * w + s + np.arange(p.m) % (p.m // nb)
    at_col = np.arange(p.n) // s * w + np.arange(p.n) % s
    wv, jv, sx, b, g = (d[k].cpu().numpy() for k in ("w", "j", "sx", "b", "g"))
    row = np.repeat(np.arange(p.n), np.diff(p.w_rowptr))
    jr, jc = at_row[np.repeat(np.arange(p.m), np.diff(p.j_rowptr))], at_col[p.j_colind]
    low = jr // w >= jc // w
    assert low.all()
    rhs = np.zeros(nb * w)
    rhs[at_col], rhs[at_row] = b, g
    x = block_solve(nb, w, [(at_col[row], at_col[p.w_colind], wv[None]), (at_col, at_col, sx[None]),
                            (jr, jc, jv[None])], rhs[None, None])[0, 0]
    return x[at_col], x[at_row]


def exact(case, seed):
    do = case["do"]
    if do == "ipm":
        return None  # the loop's iterates, not the optimum, are what it returns
    ins, ks = inputs(case, seed), keys(case)
    if do == "hykkt":
        return list(hykkt_exact(ks[0], ins[0]))
    if do == "augmented":
        d = {k: v.cpu().numpy() for k, v in ins[0].items()}
        p = shape(ks[0]).pat
        row = np.repeat(np.arange(p.m), np.diff(p.j_rowptr))
        t = d["ss"] * d["r4"] - d["g"]
        rhs = -(d["b"] + np.bincount(p.j_colind, weights=d["j"] * t[row], minlength=p.n))
        x = lifted_exact(ks[0], ins, rhs[None, None])[0, 0]
        ds = -d["r4"] - np.bincount(row, weights=d["j"] * x[p.j_colind], minlength=p.m)
        return [x, ds, -d["g"] - d["ss"] * ds]
    if do == "lifted":
        rhs = np.stack([ins[0][k].cpu().numpy() for k in ("b", "b2")[:case.get("solves", 1)]])
        return list(lifted_exact(ks[0], ins, rhs[None])[0])
    x = [None] * len(ks)
    for key in dict.fromkeys(ks):
        at = [q for q, k in enumerate(ks) if k == key]
        sol = lifted_exact(key, [ins[q] for q in at], np.stack([ins[q]["b"].cpu().numpy()[None] for q in at]))
        for q, v in zip(at, sol):
            x[q] = v[0]
    return x if do == "served" else np.concatenate(x)
