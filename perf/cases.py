"""Performance cases of mbrank: the calls a user's program makes, over the sizes it makes them.

listed() names the cases that stand for the uses of the library, draw() gives
further ones of the same ranges.  prepare() makes what a program holds before
the call (inputs on the device, sector, ranker, Hamiltonian or Lanczos
handle), run() is one pass through the public entry points, work() the bytes
and operations that pass cannot do without, and exact() the same outputs from
plain torch in 64 bits, with none of the library's code.

A case's "use" field names the path:
  rank      patterns to ranks, one batch through a ranker
  setup     a momentum sector listed, its trie built and a first batch ranked
  hx        one product with a Hubbard-type Hamiltonian
  lanczos   a whole ground-state search: start, steps, energies, coefficients
  operator  one product with a general operator from Eq. H
  gradient  one loss and gradient of the learned index's network
"""
import math

import numpy as np
import torch

import paper_2203_04158_amd as mbr

DEV = "cuda"


def listed():
    return [
        # A lookup inside an interactive or per-term loop: a thousand patterns, where the call itself is the cost.
        {"name": "rank_small", "use": "rank", "method": "staggered", "M": 16, "N": 8, "ras": 0, "k": 8, "width": 32, "n": 1003},
        # The staggered lookup at the size the ranking microbenchmark uses (half filling, 2^22 unsorted queries).
        {"name": "rank_staggered", "use": "rank", "method": "staggered", "M": 24, "N": 12, "ras": 0, "k": 8, "width": 32, "n": 4194304},
        # An irregular (RAS-like) sector of 64-bit patterns, where only a trie ranks; a tenth of the queries are no members.
        {"name": "rank_bitmap", "use": "rank", "method": "bitmap", "M": 36, "N": 8, "ras": 3, "k": 8, "width": 64, "n": 8000003},
        # Moving to the next total-momentum sector of the ring: list it, build its trie, rank a batch.
        {"name": "setup_ring", "use": "setup", "L": 14, "n_up": 7, "n_dn": 7, "K": 3, "k": 8, "n": 1000001},
        # One product on a small chain, as in a time-evolution or Davidson loop over small sectors: latency.
        {"name": "hx_small", "use": "hx", "model": "chain", "L": 8, "n_up": 3, "n_dn": 5, "precision": "f64"},
        # The headline product: half-filled 14-site chain, fp64, launch shape tuned once as the benchmark does.
        {"name": "hx_chain", "use": "hx", "model": "chain", "L": 14, "n_up": 7, "n_dn": 7, "precision": "f64"},
        # Every sector of the 12-site impurity model in one product, fp32 vectors (the mixed form).
        {"name": "hx_impurity", "use": "hx", "model": "impurity", "L": 12, "n_up": -1, "n_dn": -1, "precision": "f32"},
        # A ground-state search on an ordinary chain, three-term recurrence, graph-replayed steps.
        {"name": "lanczos_chain", "use": "lanczos", "model": "chain", "L": 12, "n_up": 6, "n_dn": 6, "precision": "f64", "reorth": False, "steps": 40},
        # The impurity solver's search: all 121 sectors of a 10-site model in one batch, full Gram-Schmidt.
        {"name": "lanczos_impurity", "use": "lanczos", "model": "impurity", "L": 10, "n_up": -1, "n_dn": -1, "precision": "f64", "reorth": True, "steps": 40},
        # The momentum-space ring: an irregular sector, a trie for its ranks, L^3 interaction terms.
        {"name": "operator_ring", "use": "operator", "model": "ring", "L": 14, "N": 7, "K": 0, "k": 14},
        # A general two-body Hamiltonian on 15 orbitals, every integral non-zero, staggered ranks.
        {"name": "operator_general", "use": "operator", "model": "general", "L": 15, "N": 7, "K": 0, "k": 8},
        # One optimiser step's loss and gradient at the batch the learned index trains with.
        {"name": "learned_gradient", "use": "gradient", "batch": 4096},
    ]


def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    use = rng.choice(["rank", "rank", "rank", "setup", "hx", "hx", "hx", "lanczos", "lanczos", "operator", "operator", "gradient"])
    if use == "rank":
        method = rng.choice(["staggered", "spin", "trie", "bitmap"])
        n = _log(rng, 300, 8000003)
        if method == "spin":
            L = rng.randint(4, 14)
            return {"use": use, "method": method, "M": L, "N": rng.randint(1, L - 1), "ras": rng.randint(1, L - 1), "k": rng.randint(4, 8), "width": 32, "n": n}
        if method == "staggered":
            width = rng.choice([32, 32, 64])
            M = rng.randint(8, 32) if width == 32 else rng.randint(33, 40)
            return {"use": use, "method": method, "M": M, "N": rng.randint(1, M - 1) if width == 32 else rng.randint(1, 8), "ras": 0, "k": rng.randint(4, 10), "width": width, "n": n}
        width = rng.choice([32, 64])
        M = rng.randint(16, 24) if width == 32 else rng.randint(33, 36)
        return {"use": use, "method": method, "M": M, "N": rng.randint(4, 12) if width == 32 else rng.randint(4, 6), "ras": rng.randint(0, 3), "k": rng.randint(4, 8), "width": width, "n": n}
    if use == "setup":
        L = rng.randint(5, 13)
        return {"use": use, "L": L, "n_up": rng.randint(2, L - 2), "n_dn": rng.randint(2, L - 2), "K": rng.randrange(L), "k": rng.randint(4, 12), "n": _log(rng, 1000, 1000001)}
    if use == "hx":
        if rng.random() < 0.4:
            return {"use": use, "model": "impurity", "L": rng.randint(4, 12), "n_up": -1, "n_dn": -1, "precision": rng.choice(["f64", "f32"])}
        L = rng.randint(5, 14)
        return {"use": use, "model": "chain", "L": L, "n_up": rng.randint(1, L - 1), "n_dn": rng.randint(1, L - 1), "precision": rng.choice(["f64", "f64", "f32"])}
    if use == "lanczos":
        if rng.random() < 0.5:
            return {"use": use, "model": "impurity", "L": rng.randint(6, 9), "n_up": -1, "n_dn": -1, "precision": "f64", "reorth": True, "steps": rng.randint(8, 40)}
        L = rng.randint(8, 12)
        return {"use": use, "model": "chain", "L": L, "n_up": rng.randint(3, L - 3), "n_dn": rng.randint(3, L - 3), "precision": "f64", "reorth": rng.random() < 0.3, "steps": rng.randint(8, 24)}
    if use == "operator":
        if rng.random() < 0.6:
            L = rng.randint(5, 13)
            return {"use": use, "model": "ring", "L": L, "N": rng.randint(2, L - 2), "K": rng.randrange(L), "k": rng.randint(5, 14)}
        L = rng.randint(8, 15)
        return {"use": use, "model": "general", "L": L, "N": rng.randint(2, L - 2), "K": 0, "k": rng.randint(4, 8)}
    return {"use": "gradient", "batch": 64 * _log(rng, 1, 128)}


# ---------------------------------------------------------------- inputs
def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + salt)
    return g


def _uniform(n, seed, salt=0):
    """Vector entries uniform in [-1, 1), fp64."""
    return torch.rand(n, generator=_gen(seed, salt), device=DEV, dtype=torch.float64) * 2 - 1


def _subsets(n, M, N, seed, salt=0):
    """n uniform patterns with N of M bits set (int64)."""
    out = torch.empty(n, dtype=torch.int64, device=DEV)
    g = _gen(seed, salt)
    for a in range(0, n, 1 << 20):
        b = min(n, a + (1 << 20))
        pos = torch.rand(b - a, M, generator=g, device=DEV).argsort(dim=1)[:, :N]
        out[a:b] = (torch.ones_like(pos) << pos).sum(dim=1)
    return out


def _patterns(v, width):
    return v if width == 64 else v.to(torch.int32)


def _ras_windows(c):
    """The particle number of a trie sector, and at least `ras` particles among orbitals 0-7."""
    full = (1 << c["M"]) - 1
    return [(full, c["N"], c["N"])] + ([(0xFF, min(c["ras"], c["N"]), 8)] if c["ras"] else [])


def _ring_windows(L, n_up, n_dn):
    low = (1 << L) - 1
    return [(low, n_dn, n_dn), (low << L, n_up, n_up)]


def _ring_terms(L):
    """The momentum-space Hubbard ring at U = 4: one-body matrix and Coulomb list."""
    t = np.zeros((2 * L, 2 * L))
    for k in range(L):
        t[k, k] = t[L + k, L + k] = 2.0 * math.cos(2 * math.pi * k / L)
    u = [(L + a, b, L + (a + b - c) % L, c, 4.0 * 4.0 / L) for a in range(L) for b in range(L) for c in range(L)]
    return t, u


def _general_terms(M):
    """A Hermitian two-body Hamiltonian on M orbitals with every integral non-zero."""
    r = np.random.RandomState(1234 + M)
    t = r.standard_normal((M, M))
    t = 0.5 * (t + t.T)
    pairs = [(i, j) for i in range(M) for j in range(i + 1, M)]
    w = r.standard_normal((len(pairs), len(pairs)))
    w = 0.3 * (w + w.T)
    return t, [(i, j, k, l, w[a, b]) for a, (i, j) in enumerate(pairs) for b, (k, l) in enumerate(pairs)]


def _model(c):
    """(bonds, U, eps, sectors) of a Hubbard-type model."""
    L = c["L"]
    if c["model"] == "chain":
        bonds = [(i, (i + 1) % L, 1.0) for i in range(L)]
        return bonds, [4.0] * L, [0.0] * L, [(c["n_up"], c["n_dn"])]
    r = np.random.RandomState(5 + L)
    eps = [-4.0] + list(r.uniform(-2.0, 2.0, L - 1))
    bonds = [(0, i + 1, -float(v)) for i, v in enumerate(r.uniform(0.2, 0.8, L - 1))]
    return bonds, [8.0] + [0.0] * (L - 1), eps, [(a, b) for a in range(L + 1) for b in range(L + 1)]


def _hubbard(c):
    bonds, U, eps, sectors = _model(c)
    prec = mbr.F64 if c["precision"] == "f64" else mbr.F32
    h = mbr.hubbard_create(c["L"], bonds, sectors, U=U, eps=eps, precision=prec)
    # a program that will take many products of a large system tunes once; a small one takes the default shape
    if h.dim >= 1 << 20:
        mbr.hubbard_autotune(h, reps=3)
    return h


def _dim(c):
    _, _, _, sectors = _model(c)
    return sum(math.comb(c["L"], a) * math.comb(c["L"], b) for a, b in sectors)


def _params(seed):
    """He-uniform network parameters in the library's order (6337 fp32 values)."""
    u = torch.rand(6337, generator=_gen(seed, 1), device=DEV) * 2 - 1
    scale = torch.zeros(6337, device=DEV)
    scale[:2048], scale[2112:6208], scale[6272:6336] = math.sqrt(6 / 32), math.sqrt(6 / 64), math.sqrt(3 / 64)
    scale[2048:2112] = scale[6208:6272] = 0.05
    p = u * scale
    p[6336] = 0.5
    return p


def _samples(c, seed):
    """A training batch: members of the half-filled 14-site spin sector and their rank / size."""
    n = c["batch"]
    half = _half(14, 7)
    idx = torch.randint(half.numel() ** 2, (n,), generator=_gen(seed, 2), device=DEV)
    q = (half[idx // half.numel()] << 14) | half[idx % half.numel()]
    return q.to(torch.int32), (idx.double() / half.numel() ** 2).float()


# ---------------------------------------------------------------- the calls
def prepare(case, seed):
    c = case
    if c["use"] == "rank":
        if c["method"] == "spin":
            ranker = mbr.build_spin_ranker(c["M"], c["N"], c["ras"], c["k"])
            q = (_subsets(c["n"], c["M"], c["N"], seed, 3) << c["M"]) | _subsets(c["n"], c["M"], c["ras"], seed, 4)
            q = _patterns(q, ranker.info().width_bits)
        elif c["method"] == "staggered":
            ranker = mbr.build_staggered_tables(c["M"], c["N"], c["k"], c["width"])
            q = _patterns(_subsets(c["n"], c["M"], c["N"], seed, 3), c["width"])
        else:
            sector = mbr.sector_build(c["M"], _ras_windows(c), c["width"])
            ranker = (mbr.build_trie if c["method"] == "trie" else mbr.build_bitmap_trie)(sector, c["k"])
            idx = torch.randint(sector.size, (c["n"],), generator=_gen(seed, 3), device=DEV, dtype=torch.int32)
            q = mbr.unrank_batch(sector, idx)
            q[::10] = _patterns(_subsets((c["n"] + 9) // 10, c["M"], c["N"], seed, 4), c["width"])
        return {"use": "rank", "ranker": ranker, "q": q, "out": torch.empty(c["n"], dtype=torch.int32, device=DEV)}
    if c["use"] == "setup":
        L = c["L"]
        q = (_subsets(c["n"], L, c["n_up"], seed, 3) << L) | _subsets(c["n"], L, c["n_dn"], seed, 4)
        return {"use": "setup", "case": c, "windows": _ring_windows(L, c["n_up"], c["n_dn"]), "weights": list(range(L)) * 2, "q": q.to(torch.int32)}
    if c["use"] == "hx":
        h = _hubbard(c)
        x = _uniform(h.dim, seed).to(torch.float64 if c["precision"] == "f64" else torch.float32)
        return {"use": "hx", "h": h, "x": x, "y": torch.empty_like(x)}
    if c["use"] == "lanczos":
        lz = mbr.lanczos_create(_hubbard(c), c["steps"], reorth=c["reorth"])
        return {"use": "lanczos", "lz": lz, "v0": _uniform(_dim(c), seed), "steps": c["steps"]}
    if c["use"] == "operator":
        L = c["L"]
        if c["model"] == "ring":
            sector = mbr.sector_build_mod(2 * L, _ring_windows(L, c["N"], c["N"]), list(range(L)) * 2, L, c["K"])
            ranker = mbr.build_trie(sector, c["k"])
            terms = mbr.terms_from_hamiltonian(2 * L, *_ring_terms(L))
        else:
            sector = mbr.sector_build(L, [((1 << L) - 1, c["N"], c["N"])])
            ranker = mbr.build_staggered_tables(L, c["N"], c["k"])
            terms = mbr.terms_from_hamiltonian(L, *_general_terms(L))
        op = mbr.operator_create(sector, ranker, terms)
        x = _uniform(op.dim, seed)
        return {"use": "operator", "op": op, "x": x, "y": torch.empty_like(x)}
    q, tgt = _samples(c, seed)
    return {"use": "gradient", "params": _params(seed), "q": q, "tgt": tgt}


def run(state):
    s = state
    if s["use"] == "rank":
        return mbr.rank_batch(s["ranker"], s["q"], out=s["out"])
    if s["use"] == "setup":
        c = s["case"]
        sector = mbr.sector_build_mod(2 * c["L"], s["windows"], s["weights"], c["L"], c["K"])
        trie = mbr.build_trie(sector, c["k"])
        return {"states": sector.states(), "ranks": mbr.rank_batch(trie, s["q"])}
    if s["use"] == "hx":
        return mbr.hubbard_apply(s["h"], s["x"], s["y"])
    if s["use"] == "lanczos":
        mbr.lanczos_start(s["lz"], s["v0"])
        mbr.lanczos_step(s["lz"], s["steps"])
        e0, done = mbr.lanczos_result(s["lz"])
        alpha, beta = mbr.lanczos_coeffs(s["lz"])
        return {"e0": e0, "steps": done, "alpha": alpha, "beta": beta}
    if s["use"] == "operator":
        return mbr.operator_apply(s["op"], s["x"], s["y"])
    grad, loss = mbr.mlp_gradients(s["params"], s["q"], s["tgt"])
    return {"grad": grad, "loss": loss}


def _ring_dim(L, n_up, n_dn):
    return math.comb(L, n_up) * math.comb(L, n_dn) // L


def work(case):
    c = case
    if c["use"] == "rank":
        width = 64 if c["method"] == "spin" and c["M"] > 16 else c["width"]
        return {"bytes": c["n"] * (width // 8 + 4), "flops": 0}
    if c["use"] == "setup":
        # the list and the ranks are written, the queries read
        return {"bytes": 4 * _ring_dim(c["L"], c["n_up"], c["n_dn"]) + 8 * c["n"], "flops": 0}
    if c["use"] in ("hx", "lanczos"):
        dim, size = _dim(c), 8 if c["precision"] == "f64" else 4
        bonds, _, _, sectors = _model(c)
        L = c["L"]
        hops = 0
        for a, b in sectors:  # a bond hops in a spin half when one of its two sites is occupied
            rows = math.comb(L, a) * math.comb(L, b)
            hops += rows * len(bonds) * 2 * (a * (L - a) + b * (L - b)) // (L * (L - 1))
        if c["use"] == "hx":
            return {"bytes": 2 * size * dim, "flops": 2 * hops + 3 * dim}
        # a step reads the last two vectors and writes one, then reads two and writes one; Gram-Schmidt reads the basis twice
        m = c["steps"]
        basis = m * (m + 1) if c["reorth"] else 0
        return {"bytes": (6 * m + basis) * size * dim, "flops": m * (2 * hops + 10 * dim) + 2 * basis * dim}
    if c["use"] == "operator":
        L, N = c["L"], c["N"]
        if c["model"] == "ring":
            dim = _ring_dim(L, N, N)
            live = N * N * (L - N + 1)  # a pair of particles, and the momentum one of them takes up
        else:
            dim = math.comb(L, N)
            live = (N * (N - 1) // 2) * ((L - N + 2) * (L - N + 1) // 2)
        return {"bytes": 20 * dim, "flops": 2 * live * dim}
    # forward, and twice as much backward; parameters and samples read, gradients written
    return {"bytes": 8 * 6337 + 8 * c["batch"], "flops": 3 * 12416 * c["batch"]}


# ---------------------------------------------------------------- the same in 64 bits
def _popcount(v):
    n = torch.zeros_like(v)
    for b in range(40):
        n += (v >> b) & 1
    return n


def _half(L, n):
    """Ascending L-bit patterns with n bits set."""
    p = torch.arange(1 << L, device=DEV)
    return p[_popcount(p) == n]


def _half_rank(L, n):
    h = _half(L, n)
    r = torch.zeros(1 << L, dtype=torch.int64, device=DEV)
    r[h] = torch.arange(h.numel(), device=DEV)
    return h, r


def _hubbard_terms(c, n_up, n_dn):
    """[(coefficients, source rows)] of one (N_up, N_dn) sector: y = sum coefficient * x[source]."""
    L = c["L"]
    bonds, U, eps, _ = _model(c)
    up, r_up = _half_rank(L, n_up)
    dn, r_dn = _half_rank(L, n_dn)
    a_up, a_dn = up.repeat_interleave(dn.numel()), dn.repeat(up.numel())
    row = torch.arange(a_up.numel(), device=DEV)
    diag = torch.zeros(a_up.numel(), dtype=torch.float64, device=DEV)
    for i in range(L):
        bu, bd = ((a_up >> i) & 1).double(), ((a_dn >> i) & 1).double()
        diag += eps[i] * (bu + bd) + U[i] * bu * bd
    yield diag, row
    for i, j, t in bonds:
        lo, hi = min(i, j), max(i, j)
        flip, between = (1 << i) | (1 << j), ((1 << hi) - 1) & ~((1 << (lo + 1)) - 1)
        for a, other, spin in ((a_up, a_dn, "up"), (a_dn, a_up, "dn")):
            on = (((a >> i) ^ (a >> j)) & 1) == 1
            sign = 1.0 - 2.0 * (_popcount(a & between) & 1).double()
            to = torch.where(on, a ^ flip, a)
            src = r_up[to] * dn.numel() + r_dn[other] if spin == "up" else r_up[other] * dn.numel() + r_dn[to]
            yield torch.where(on, -t * sign, torch.zeros_like(sign)), src


def _exact_hx(c, seed):
    _, _, _, sectors = _model(c)
    x = _uniform(_dim(c), seed)
    if c["precision"] == "f32":
        x = x.float().double()
    y, off = torch.zeros_like(x), 0
    for a, b in sectors:
        n = math.comb(c["L"], a) * math.comb(c["L"], b)
        for coef, src in _hubbard_terms(c, a, b):
            y[off:off + n] += coef * x[off:off + n][src]
        off += n
    return y


def _exact_lanczos(c, seed):
    _, _, _, sectors = _model(c)
    v0, m = _uniform(_dim(c), seed), c["steps"]
    ns = len(sectors)
    alpha, beta, e0, done, off = np.zeros((ns, m)), np.zeros((ns, m)), np.zeros(ns), np.zeros(ns, dtype=np.int32), 0
    for s, (a, b) in enumerate(sectors):
        n = math.comb(c["L"], a) * math.comb(c["L"], b)
        terms = list(_hubbard_terms(c, a, b))
        v = v0[off:off + n]
        off += n
        v = v / v.norm()
        basis, al, be = [v], [], []
        for j in range(min(m, n)):
            w = torch.zeros_like(v)
            for coef, src in terms:
                w += coef * basis[j][src]
            if j:
                w -= be[j - 1] * basis[j - 1]
            al.append(float(torch.dot(basis[j], w)))
            w = w - al[j] * basis[j]
            if c["reorth"]:
                V = torch.stack(basis)
                for _ in range(2):
                    w = w - V.T @ (V @ w)
            be.append(float(w.norm()))
            if be[j] <= 1e-12 * (abs(al[j]) + (be[j - 1] if j else 0.0)):
                break
            basis.append(w / be[j])
        d = len(al)
        be[-1] = 0.0
        alpha[s, :d], beta[s, :d], done[s] = al, be, d
        tri = np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1)
        e0[s] = np.linalg.eigvalsh(tri)[0]
    return {"e0": e0, "steps": None, "alpha": alpha, "beta": beta}


def _exact_operator(c, seed):
    """Eq. H applied operator by operator, each term scattering x to the states it reaches."""
    L = c["L"]
    if c["model"] == "ring":
        n_bits = 2 * L
        h = _half(L, c["N"])
        st = ((h.repeat_interleave(h.numel()) << L) | h.repeat(h.numel()))
        mom = sum(((st >> b) & 1) * (b % L) for b in range(n_bits)) % L
        st = st[mom == c["K"]]
        t, u = _ring_terms(L)
    else:
        n_bits = L
        st = _half(L, c["N"])
        t, u = _general_terms(L)
    x = _uniform(st.numel(), seed)
    y = torch.zeros_like(x)

    def add(coef, ops):
        """y += coef * (product of ops, the last acting first) x."""
        a, sign, idx = st, torch.ones_like(x), None
        for create, i in reversed(ops):
            ok = ((a >> i) & 1) == (0 if create else 1)
            keep = ok.nonzero()[:, 0]
            idx = keep if idx is None else idx[keep]
            a, sign = a[keep], sign[keep]
            par = a & ((1 << i) - 1)
            for s in (32, 16, 8, 4, 2, 1):
                par = par ^ (par >> s)
            sign = sign * (1.0 - 2.0 * (par & 1).double())
            a = a ^ (1 << i)
        if idx.numel():
            y.index_add_(0, torch.searchsorted(st, a), coef * sign * x[idx])

    for i in range(n_bits):
        for j in range(n_bits):
            if t[i, j] != 0:
                add(-t[i, j], [(True, i), (False, j)])
    for i, j, k, l, U in u:
        if i != j and k != l:
            add(0.25 * U, [(True, i), (True, j), (False, l), (False, k)])
    return y


def _exact_gradient(c, seed):
    p = _params(seed).bfloat16().double()
    q, tgt = _samples(c, seed)
    bits = ((q.long()[:, None] >> torch.arange(32, device=DEV)) & 1).double()
    w1, b1, w2, b2, w3, b3 = p[:2048].view(64, 32), p[2048:2112], p[2112:6208].view(64, 64), p[6208:6272], p[6272:6336], p[6336]
    z1 = bits @ w1.T + b1
    h1 = z1.clamp(min=0)
    z2 = h1 @ w2.T + b2
    h2 = z2.clamp(min=0)
    d = h2 @ w3 + b3 - tgt.double()
    dy = 2 * d / c["batch"]
    dz2 = dy[:, None] * w3 * (z2 > 0)
    dz1 = (dz2 @ w2) * (z1 > 0)
    g = torch.cat([(dz1.T @ bits).reshape(-1), dz1.sum(0), (dz2.T @ h1).reshape(-1), dz2.sum(0), h2.T @ dy, dy.sum()[None]])
    return {"grad": g, "loss": (d * d).mean()[None]}


def exact(case, seed):
    if case["use"] == "hx":
        return _exact_hx(case, seed)
    if case["use"] == "lanczos":
        return _exact_lanczos(case, seed)
    if case["use"] == "operator":
        return _exact_operator(case, seed)
    if case["use"] == "gradient":
        return _exact_gradient(case, seed)
    return None  # ranks and state lists are whole numbers
