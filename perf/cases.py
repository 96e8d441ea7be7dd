"""The work that users of this package have it do, as timed cases, each through a public entry point.

listed() names the standing cases: one call of every route (potential family) of the library, from a
16-slice estimate of 1e5 paths, where launches and latency count, to runs that fill the GPU for tens of
milliseconds. draw(rng) gives more of the same routes over the ranges of levels, slice numbers, sample
counts, potentials and options that the tests and the benchmark span. exact(case, seed) restates a
case in FP64 with plain torch (the estimator of Balaz et al. on the same Philox streams).
"""
import functools
import math
import random

import numpy as np
import torch

import paper_1105_0542_amd as P

# Monomials of the derivative-symbol mode's level-p slice polynomial (counted from its recursion).
GENERAL_MONOMIALS = {1: 1, 2: 3, 3: 7, 4: 15, 5: 30, 6: 58, 7: 107, 8: 193, 9: 341, 10: 585, 11: 983, 12: 1629,
                     13: 2641, 14: 4223, 15: 6664, 16: 10360, 17: 15916, 18: 24196}
# Two particles on a line with a quartic pair interaction in a trap with a field; an anisotropic 3D
# trap with cubic and quartic couplings; two particles in two dimensions with a harmonic pair
# interaction; an anharmonic oscillator with odd terms: (coefficient, exponents per coordinate).
POLY_TERMS = {
    1: [(0.5, (2,)), (0.3, (1,)), (0.05, (3,)), (0.2, (4,))],
    2: [(0.5, (2, 0)), (0.7, (0, 2)), (0.1, (4, 0)), (-0.4, (3, 1)), (0.6, (2, 2)), (-0.4, (1, 3)), (0.1, (0, 4)),
        (0.3, (1, 0)), (0.2, (1, 1))],
    3: [(0.5, (2, 0, 0)), (0.4, (0, 2, 0)), (0.3, (0, 0, 2)), (0.2, (0, 2, 1)), (0.05, (1, 1, 2)), (0.05, (0, 0, 4)),
        (0.1, (2, 2, 0)), (0.1, (0, 0, 1))],
    4: [(0.5, (2, 0, 0, 0)), (0.5, (0, 2, 0, 0)), (0.5, (0, 0, 2, 0)), (0.5, (0, 0, 0, 2)), (-0.3, (1, 0, 1, 0)),
        (-0.3, (0, 1, 0, 1)), (0.05, (4, 0, 0, 0)), (0.05, (0, 0, 4, 0))],
}
FIELDS = ("amp", "err", "log_amp", "relvar", "ess", "n", "n_nonfinite")


def listed():
    return [
        # a first estimate of the anharmonic oscillator: every level of N = 16, 1e5 paths (latency)
        dict(name="quartic_p4_n16", kind="quartic", g=1.0, T=1.0, m=1.0, p=4, s=4, n=100_000, hier=True, fp32=False),
        # one point of the convergence sweep at the highest level: N = 1024, every coarser N with it
        dict(name="quartic_p18_n1024", kind="quartic", g=10.0, T=1.0, m=1.0, p=18, s=10, n=20_000_000, hier=True,
             fp32=False),
        # the finest N alone with FP32 slice polynomials, a million paths and a few
        dict(name="quartic_fp32_n512", kind="quartic", g=10.0, T=1.0, m=1.0, p=18, s=9, n=1_000_003, hier=False,
             fp32=True),
        # a polynomial potential outside the quartic family (odd terms, sixth power)
        dict(name="odd_sextic_p6_n64", kind="polynomial", degree=6, T=0.5, m=1.0, p=6, s=6, n=300_001, hier=True),
        # the Poeschl-Teller potential at the level and slice numbers of its convergence study
        dict(name="mpt_p10_n1024", kind="mpt", T=1.0, m=1.0, p=10, s=10, n=1_000_000, hier=True),
        # a potential with no table of its own: a Gaussian barrier in a trap, by the derivatives of V
        dict(name="barrier_p8_n256", kind="general", sech=False, T=1.0, m=1.0, p=8, s=8, n=1_000_000, hier=True),
        # the same at the highest level (24,196 monomials a slice)
        dict(name="barrier_p18_n64", kind="general", sech=False, T=1.0, m=1.0, p=18, s=6, n=50_000, hier=True),
        # three coordinates, rotation-invariant: every level of N = 1024
        dict(name="radial_d3_p18_n1024", kind="radial", d=3, g=10.0, T=1.0, m=1.0, p=18, s=10, n=1_000_000, hier=True),
        # two interacting particles on a line
        dict(name="pair_d2_p10_n256", kind="poly", d=2, T=1.0, m=1.0, p=10, s=8, n=500_000, hier=True),
        # a grid of endpoints with mixed N, p and T, planned once and run
        dict(name="batch_16x16", kind="batch", grid=16, n=20_000, hier=False),
        # the ten lowest levels of the anharmonic oscillator from the evolution operator on a fine grid
        dict(name="spectrum_n16384", kind="spectrum", A=1.0, g=48.0, t=0.02, L=8.0, p=21, n=16384, k=10),
        # a learned proposal: training steps from the identity map, then an estimate with it
        dict(name="proposal_n128", kind="proposal", g=10.0, T=2.0, p=12, s=7, batch=4096, steps=48, n=1 << 20),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


# Seconds of a slice evaluation per counted FP64 operation (vector rate, less for the wide codes), so
# that a drawn case is given as many paths as cost no more than the largest listed one.
_SECONDS_PER_OP = {"quartic": 1 / 3.5e13, "polynomial": 1 / 2e13, "mpt": 1 / 3e13, "general": 1 / 2e13,
                   "radial": 1 / 2.5e13, "poly": 1 / 1.2e13}


def draw(rng):
    kind = rng.choice(["quartic", "quartic", "polynomial", "mpt", "general", "radial", "poly", "batch", "spectrum",
                       "proposal"])
    if kind == "batch":
        return dict(kind=kind, grid=rng.randint(3, 16), n=int(_log_uniform(rng, 2_000, 40_000)),
                    hier=rng.random() < 0.3)
    if kind == "spectrum":
        n = int(_log_uniform(rng, 300, 9_000))
        return dict(kind=kind, A=1.0, g=rng.uniform(1.0, 48.0), t=rng.uniform(0.02, 0.1), L=rng.uniform(7.0, 10.0),
                    p=rng.randint(8, 21), n=n, k=rng.randint(2, 12))
    if kind == "proposal":
        return dict(kind=kind, g=rng.uniform(1.0, 10.0), T=rng.uniform(0.5, 2.0), p=rng.randint(4, 12),
                    s=rng.randint(3, 7), batch=int(_log_uniform(rng, 500, 16_384)), steps=rng.randint(4, 40),
                    n=int(_log_uniform(rng, 10_000, 1 << 20)))
    c = dict(kind=kind, T=rng.uniform(0.3, 1.2), m=rng.choice([1.0, 1.0, 2.0]), hier=rng.random() < 0.7)
    if kind == "quartic":
        c.update(g=rng.uniform(0.5, 10.0), p=rng.choice([1, 2, 4, 5, 8, 9, 12, 14, 18]), s=rng.randint(4, 10))
        c["fp32"] = rng.random() < 0.2
    elif kind == "polynomial":
        c.update(degree=rng.choice([4, 6, 8]), p=rng.randint(2, 7), s=rng.randint(2, 9))
        c["T"] *= 0.5
    elif kind == "mpt":
        c.update(p=rng.choice([1, 2, 4, 6, 10, 12]), s=rng.randint(2, 10))
    elif kind == "general":
        c.update(sech=rng.random() < 0.5, p=rng.choice([2, 4, 6, 8, 8, 10, 13, 18]), s=rng.randint(3, 8))
    elif kind == "radial":
        c.update(d=rng.randint(1, 4), g=rng.uniform(0.5, 10.0), p=rng.choice([2, 4, 6, 10, 18]), s=rng.randint(2, 10))
    else:
        d = rng.randint(1, 4)
        c.update(d=d, p=rng.randint(2, {1: 10, 2: 8, 3: 5, 4: 4}[d]), s=rng.randint(3, 9))
    spent = _slice_count(c) * _ops_per_slice(c) * _SECONDS_PER_OP[kind]
    if kind == "general" and c["p"] > 10:
        spent *= 8                      # code far beyond the instruction cache
    c["n"] = int(_log_uniform(rng, 1_000, max(2_000, min(4_000_000, 0.04 / spent)))) | 1
    return c


# ------------------------------------------------------------------------------ what a pass costs
def _slice_count(c):
    return (2 << c["s"]) - 1 if c["hier"] else 1 << c["s"]


@functools.lru_cache(maxsize=None)
def _monomials(kind, p, d, degree):
    """Terms of the level-p slice polynomial in its own variables."""
    if kind == "general":
        return GENERAL_MONOMIALS[p]
    if kind == "mpt":
        return p * (p + 1)
    if kind == "radial" and d > 1:       # u^i z^l (w^2)^j of V = r^2/2 + g r^4/24: 102 at p = 18
        return max(1, round(102 * (p / 18.0) ** 2))
    if kind == "quartic" or kind == "radial":
        return len(_slice_terms(_quartic_symbols(1.0, 1.0), 1, p, 1.0))
    if kind == "polynomial":
        return len(_slice_terms(_poly_symbols(_odd_terms(degree, 0.1), 1), 1, p, 1.0))
    return len(_slice_terms(_poly_symbols(POLY_TERMS[d], d), d, p, 1.0))


def _ops_per_slice(c):
    """FP64 operations: two per term, the slice's variables, and half a normal (about 60 operations
    a pair with its logarithm, square root, sine and cosine) per coordinate."""
    kind, d = c["kind"], c.get("d", 1)
    terms = _monomials(kind, c["p"], d, c.get("degree", 0))
    extra = {"mpt": 40, "general": 4 * c["p"] + 60}.get(kind, 0)
    normals = 32 * d * ((1 << c["s"]) - 1) / _slice_count(c)
    return 2 * terms + 6 * d + extra + normals


def work(case):
    kind = case["kind"]
    if kind == "batch":
        flops = out = 0
        for (_, _, _, _, _, N, p, n, _) in _batch_rows(case, 0)[1]:
            t = dict(kind="quartic", p=p, s=N.bit_length() - 1, hier=case["hier"])
            flops += n * _slice_count(t) * _ops_per_slice(t)
            out += 56 * N.bit_length()
        return {"bytes": out, "flops": flops}
    if kind == "spectrum":
        # the matrix's distinct elements once, and read once a Lanczos step (at least 4 k of them)
        el = case["n"] * (case["n"] + 1) / 2
        terms = _monomials("quartic", case["p"], 1, 0)
        return {"bytes": 8 * el * 4 * case["k"], "flops": el * (2 * terms + 40 + 4 * 4 * case["k"])}
    if kind == "proposal":
        N = 1 << case["s"]
        net = 2 * (64 * 128 + 128 * 128) * 8              # multiply-adds of eight couplings, both products
        flops = case["n"] * (2 * net / 2 + 64 * N) + case["steps"] * case["batch"] * (3 * net + 128 * N)
        return {"bytes": 8 * 24832 * 4 * 3 * case["steps"], "flops": flops}
    return {"bytes": 56 * (case["s"] + 1) + 64, "flops": case["n"] * _slice_count(case) * _ops_per_slice(case)}


# ------------------------------------------------------------------------------ inputs and the call
def _odd_terms(degree, c):
    t = [(0.3, (1,)), (0.5, (2,)), (c, (3,)), (0.2, (4,))]
    return t + [(0.02, (j,)) for j in range(6, degree + 1, 2)]


def _inputs(case, seed):
    """Potential strength, endpoints and sample stream of a problem, from the seed alone."""
    r = random.Random(1_000_003 * seed + 7)
    d = case.get("d", 1)
    return dict(scale=1.0 + 0.2 * r.random(), a=[0.2 * (r.random() - 0.5) for _ in range(d)],
                b=[(1.0, 0.4, -0.2, 0.3)[c] + 0.2 * (r.random() - 0.5) for c in range(d)], seed=r.getrandbits(62),
                stream=r.getrandbits(20))


def _batch_rows(case, seed):
    r = random.Random(1_000_003 * seed + 11)
    xs = [-2.0 + 4.0 * i / (case["grid"] - 1) + 0.05 * r.random() for i in range(case["grid"])]
    rows = []
    base = r.getrandbits(16) << 10
    for i, a in enumerate(xs):
        for j, b in enumerate(xs):
            k = i * len(xs) + j
            rows.append((k % 2, 1.0, a, b, (0.5, 1.0)[(i + j) % 2], 16 << ((7 * i + 3 * j) % 6), (8, 12, 18)[(i * 5 + j) % 3],
                         case["n"], base + k))
    return [[0.0, 0.0, 0.5, 0.0, 1.0 / 24.0], [0.0, 0.0, -0.5, 0.0, 4.0 / 24.0]], rows


def prepare(case, seed):
    ctx = P.Context()
    st = dict(case=case, ctx=ctx)
    kind = case["kind"]
    if kind == "batch":
        systems, rows = _batch_rows(case, seed)
        st["batch"] = P.Batch(ctx, systems, rows, 1 + seed, P.FLAG_HIERARCHY if case["hier"] else 0)
        return st
    x = st["x"] = _inputs(case, seed)
    if kind == "proposal":
        st["flow"] = P.Flow(ctx, P.quartic(1.0, case["g"] * x["scale"]), 1.0, x["a"][0], x["b"][0], case["T"],
                            1 << case["s"], case["p"], layers=8, batch=case["batch"], lr=1e-3, beta=0.9,
                            init_seed=seed)
        st["theta"] = st["flow"].get_params()
        return st
    if kind == "spectrum":
        return st
    st["flags"] = (P.FLAG_HIERARCHY if case["hier"] else 0) | (P.FLAG_FP32_POLY if case.get("fp32") else 0)
    if kind == "quartic":
        st["coefs"] = P.quartic(1.0, case["g"] * x["scale"])
    elif kind == "polynomial":
        st["coefs"] = [0.0] * (case["degree"] + 1)
        for c, (e,) in _odd_terms(case["degree"], 0.1 * x["scale"]):
            st["coefs"][e] = c
    elif kind == "radial":
        st["coefs"] = [0.0, 0.5, case["g"] * x["scale"] / 24.0]
    elif kind == "poly":
        st["terms"] = [(c * x["scale"], e) for c, e in POLY_TERMS[case["d"]]]
    return st


def run(st):
    case, ctx, kind = st["case"], st["ctx"], st["case"]["kind"]
    if kind == "batch":
        res, _, _ = st["batch"].run()
        return {f: res[f] for f in FIELDS}
    x = st["x"]
    if kind == "spectrum":
        E, _, _, _ = ctx.spectrum(P.quartic(case["A"], case["g"] * x["scale"]), 1.0, case["t"], case["p"], case["L"],
                                  case["n"], case["k"])
        return E
    if kind == "proposal":
        st["flow"].set_params(st["theta"])
        losses, _ = st["flow"].train(x["seed"], 1 << 31, case["steps"])
        r, _, _ = st["flow"].amplitude(case["n"], x["seed"], 1 << 30)
        return {"losses": losses, "theta": st["flow"].get_params(), **{f: getattr(r, f) for f in FIELDS}}
    N, T, p, n = 1 << case["s"], case["T"], case["p"], case["n"]
    tail = (T, N, p, n, x["seed"], x["stream"], st["flags"])
    a, b, m = x["a"], x["b"], case["m"]
    if kind in ("quartic", "polynomial"):
        res, _ = ctx.amplitude(st["coefs"], m, a[0], b[0], *tail)
    elif kind == "mpt":
        res, _ = ctx.amplitude_mpt(x["scale"], 1.0, m, a[0] - 0.5, b[0] - 0.5, *tail)
    elif kind == "general":
        res, _ = ctx.amplitude_general(m, a[0] - 0.3, b[0] - 0.6, *tail, poly=(0.0, 0.0, 0.5),
                                       sech2=((0.5, 0.8),) if case["sech"] else (), gauss=((2.0 * x["scale"], 1.0),))
    elif kind == "radial":
        res, _ = ctx.amplitude_radial(st["coefs"], case["d"], m, a, b, *tail)
    else:
        res, _ = ctx.amplitude_poly(st["terms"], case["d"], m, a, b, *tail)
    return {f: np.array([getattr(r, f) for r in res]) for f in FIELDS}


# ------------------------------------------------------------------------------ the same in plain FP64
# Polynomials are dicts {exponents: coefficient}; the last d exponents are those of the half-deviation
# xbar, the ones before belong to a ring in which x-derivatives are known: the components of x, tanh,
# or symbols V', V'', ...
def _add(a, b, s=1.0):
    for k, v in b.items():
        a[k] = a.get(k, 0.0) + s * v
    return a


def _mul(a, b, out, s):
    for ka, va in a.items():
        for kb, vb in b.items():
            k = tuple([x + y for x, y in zip(ka, kb)])
            out[k] = out.get(k, 0.0) + s * va * vb


def _partial(a, i):
    out = {}
    for k, v in a.items():
        if k[i]:
            e = k[:i] + (k[i] - 1,) + k[i + 1:]
            out[e] = out.get(e, 0.0) + v * k[i]
    return out


def _coefficients(V, dx, d, p):
    """W_{m,k} of W = sum eps^(m-k) W_{m,k}(x, xbar), m < p: eq.(DIA) on the diagonal, eq.(MBrec) below
    it (in one coordinate eq.(diagonal) and eq.(1Drec)). dx: the d derivatives in x."""
    nv = len(next(iter(V)))
    db = [functools.partial(_partial, i=nv - d + c) for c in range(d)]
    W, gx, gb = {(0, 0): dict(V)}, {}, {}

    def grad(store, ops, key):
        if key not in store:
            store[key] = [f(W[key]) for f in ops]
        return store[key]

    power = dict(V)
    for m in range(1, p):
        for _ in range(2):                                      # (xbar . d/dx) twice
            new = {}
            for c in range(d):
                for k, v in dx[c](power).items():
                    e = list(k)
                    e[nv - d + c] += 1
                    new[tuple(e)] = new.get(tuple(e), 0.0) + v
            power = new
        W[m, m] = {k: v / math.factorial(2 * m + 1) for k, v in power.items()}
        for k in range(m - 1, -1, -1):
            rhs = {}
            for c in range(d):
                _add(rhs, dx[c](dx[c](W[m - 1, k])))
                _add(rhs, db[c](db[c](W[m, k + 1])))
            for l in range(m - 1):
                for r in range(max(0, k - m + l + 2), min(k, l) + 1):
                    for f, g in zip(grad(gx, dx, (l, r)), grad(gx, dx, (m - l - 2, k - r))):
                        _mul(f, g, rhs, -1.0)
                    if l:
                        for f, g in zip(grad(gb, db, (l, r)), grad(gb, db, (m - l - 1, k - r + 1))):
                            _mul(f, g, rhs, -1.0)
            W[m, k] = {e: v / (8.0 * (m + k + 1)) for e, v in rhs.items() if v}
    return W


def _fold(W, eps):
    out = {}
    for (m, k), w in W.items():
        _add(out, w, eps ** (m - k + 1))
    return out


def _slice_terms(symbols, d, p, eps):
    V, dx = symbols
    return _fold(_coefficients(V, dx, d, p), eps)


def _poly_symbols(terms, d):
    return {tuple(e) + (0,) * d: float(c) for c, e in terms}, [functools.partial(_partial, i=c) for c in range(d)]


def _quartic_symbols(A, g):
    return _poly_symbols([(A / 2.0, (2,)), (g / 24.0, (4,))], 1)


def _tanh_symbols(lam, alpha):
    def dx(a):                                                  # d/dx = alpha (1 - y^2) d/dy
        out = {}
        for (e, x), v in a.items():
            if e:
                out[e - 1, x] = out.get((e - 1, x), 0.0) + alpha * e * v
                out[e + 1, x] = out.get((e + 1, x), 0.0) - alpha * e * v
        return out
    return {(0, 0): -lam, (2, 0): lam}, [dx]


def _derivative_symbols(p):
    J = 2 * p - 1                                               # V, V', ..., V^(2p-2)

    def dx(a):
        out = {}
        for k, v in a.items():
            for j in range(J - 1):
                if k[j]:
                    e = list(k)
                    e[j] -= 1
                    e[j + 1] += 1
                    out[tuple(e)] = out.get(tuple(e), 0.0) + v * k[j]
        return out
    return {(1,) + (0,) * J: 1.0}, [dx]


def _general_derivatives(x, J, poly, sech, gauss):
    """V^(j)(x), j = 0..J-1, of poly + sum A/cosh^2(a x) + sum B exp(-b x^2)."""
    out = [torch.zeros_like(x) for _ in range(J)]
    c = list(poly)
    for j in range(J):
        acc = torch.zeros_like(x)
        for v in reversed(c):
            acc = acc * x + v
        out[j] = out[j] + acc
        c = [i * c[i] for i in range(1, len(c))]
    for A, a in sech:
        t = torch.tanh(a * x)
        q = [A, 0.0, -A]                                        # A (1 - t^2); d/dx = a (1 - t^2) d/dt
        for j in range(J):
            acc = torch.zeros_like(x)
            for v in reversed(q):
                acc = acc * t + v
            out[j] = out[j] + acc
            dq = [i * q[i] for i in range(1, len(q))] + [0.0, 0.0, 0.0]
            q = [a * (dq[i] - (dq[i - 2] if i > 1 else 0.0)) for i in range(len(q) + 1)]
    for B, b in gauss:
        g = B * torch.exp(-b * x * x)
        h0, h1 = torch.ones_like(x), -2.0 * b * x               # exp(b x^2) (d/dx)^j exp(-b x^2)
        for j in range(J):
            out[j] = out[j] + g * h0
            h0, h1 = h1, -2.0 * b * (x * h1 + (j + 1) * h0)
    return out


def _normals(seed, stream, paths, pairs):
    """Standard normals of heap nodes (2 j, 2 j + 1), j in pairs: Philox4x32-10 and Box-Muller."""
    M = 0xFFFFFFFF
    c0, c1, c2, c3 = torch.broadcast_tensors(pairs[None, :], (paths & M)[:, None], (paths >> 32)[:, None],
                                             torch.full((1, 1), stream & M, device=paths.device))
    k0, k1 = seed & M, (seed >> 32) & M
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57               # modulo 2^64: the words are exact
        c0, c1, c2, c3 = ((p1 >> 32) & M) ^ c1 ^ k0, p1 & M, ((p0 >> 32) & M) ^ c3 ^ k1, p0 & M
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    u = [(((hi << 21) | (lo >> 11)) | 1).double() * 2.0 ** -53 for lo, hi in ((c0, c1), (c2, c3))]
    r, th = torch.sqrt(-2.0 * torch.log(u[0])), 2.0 * math.pi * u[1]
    return r * torch.cos(th), r * torch.sin(th)


def _paths(seed, stream, first, count, a, b, T, s, device):
    """Bridges of len(a) coordinates: [coordinate][path, 2^s + 1]."""
    N = 1 << s
    paths = torch.arange(first, first + count, device=device)
    out = []
    for c in range(len(a)):
        q = torch.empty(count, N + 1, dtype=torch.float64, device=device)
        q[:, 0], q[:, N] = a[c], b[c]
        for n in range(1, s + 1):
            st = N >> n
            off = c << 20
            if n == 1:
                z = _normals(seed, stream, paths, torch.tensor([off], device=device))[1]
            else:
                j = torch.arange(1 << (n - 2), 1 << (n - 1), device=device) + off
                z = torch.stack(_normals(seed, stream, paths, j), dim=2).reshape(count, -1)
            q[:, st::2 * st] = math.sqrt(T / 2.0 ** (n + 1)) * z + 0.5 * (q[:, 0:N:2 * st] + q[:, 2 * st::2 * st])
        out.append(q)
    return out


def _slice_sum(terms, values):
    """sum over terms of coefficient times the product of powers of the values, summed over slices."""
    powers = [[None, v] for v in values]
    for t in range(len(values)):
        for _ in range(max(e[t] for e in terms) - 1):
            powers[t].append(powers[t][-1] * values[t])
    total = torch.zeros_like(values[0])
    for e, c in terms.items():
        v = None
        for t, x in enumerate(e):
            if x:
                v = powers[t][x] if v is None else v * powers[t][x]
        total = total + c * (1.0 if v is None else v)
    return total.sum(dim=1)


def _estimate(problem, T, s, levels, n, seed, stream):
    """Amplitude, error, ... per level from paths 0..n-1, as the library's records."""
    W, variables, a, b, pref = problem["W"], problem["variables"], problem["a"], problem["b"], problem["pref"]
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    d = len(a)
    terms = [_fold(W, T / 2.0 ** k) for k in range(s + 1)]

    def actions(q, k):
        st = (q[0].shape[1] - 1) >> k
        qa, qb = [x[:, :-1:st] for x in q], [x[:, st::st] for x in q]
        return _slice_sum(terms[k], variables([0.5 * (u + v) for u, v in zip(qa, qb)])
                          + [0.5 * (v - u) for u, v in zip(qa, qb)])

    line = [torch.linspace(0.0, 1.0, (1 << s) + 1, dtype=torch.float64, device=dev)[None, :] * (b[c] - a[c]) + a[c]
            for c in range(d)]
    ref = [float(actions(line, k)) for k in range(s + 1)]
    sums = [[0.0, 0.0] for _ in range(s + 1)]
    step = max(1, min(n, (1 << 22) // ((1 << s) * d)))
    for first in range(0, n, step):
        q = _paths(seed, stream, first, min(step, n - first), a, b, T, s, dev)
        for k in levels:
            e = torch.expm1(ref[k] - actions(q, k))
            sums[k][0] += e.sum()
            sums[k][1] += (e * e).sum()
    dist2 = sum((v - u) ** 2 for u, v in zip(a, b))
    log_k0 = math.log(pref) - dist2 / (2.0 * T) - 0.5 * d * math.log(2.0 * math.pi * T)
    out = {f: np.zeros(s + 1) for f in FIELDS[:5]}
    base = log_k0 - ref[0]
    for f, v in zip(FIELDS[:5], (math.exp(base), 0.0, base, 0.0, float(n))):
        out[f][0] = v
    for k in levels:
        sd, sd2 = float(sums[k][0]), float(sums[k][1])
        mean = sd / n
        var = max(0.0, (sd2 - sd * mean) / (n - 1))
        base = log_k0 - ref[k]
        w2 = n + 2.0 * sd + sd2
        for f, v in zip(FIELDS[:5], (math.exp(base) * (1.0 + mean), math.exp(base) * math.sqrt(var / n),
                                     base + math.log1p(mean), var / (1.0 + mean) ** 2, (n + sd) ** 2 / w2)):
            out[f][k] = v
    return {**out, "n": None, "n_nonfinite": None}


def _problem(case, x):
    """Coefficients, variables and endpoints of a case after the mass rescaling q -> sqrt(m) q."""
    kind, m, p = case["kind"], case["m"], case["p"]
    sm, d, same = math.sqrt(m), case.get("d", 1), lambda mid: mid
    a, b = x["a"], x["b"]
    if kind == "mpt":
        alpha = 1.0 / sm
        W, var = _coefficients(*_tanh_symbols(x["scale"], alpha), 1, p), lambda mid: [torch.tanh(alpha * mid[0])]
        a, b = [a[0] - 0.5], [b[0] - 0.5]
    elif kind == "general":
        J = 2 * p - 1
        args = ((0.0, 0.0, 0.5 / m), ((0.5, 0.8 / sm),) if case["sech"] else (), ((2.0 * x["scale"], 1.0 / m),))
        W, var = _coefficients(*_derivative_symbols(p), 1, p), lambda mid: _general_derivatives(mid[0], J, *args)
        a, b = [a[0] - 0.3], [b[0] - 0.6]
    else:
        if kind == "quartic":
            terms = [(0.5, (2,)), (case["g"] * x["scale"] / 24.0, (4,))]
        elif kind == "polynomial":
            terms = _odd_terms(case["degree"], 0.1 * x["scale"])
        elif kind == "radial":
            c4, terms = case["g"] * x["scale"] / 24.0, []
            for i in range(d):
                e = [2 * (j == i) for j in range(d)]
                terms.append((0.5, e))
                terms += [(c4, [e[j] + 2 * (j == k) for j in range(d)]) for k in range(d)]
            merged = {}
            for c, e in terms:
                merged[tuple(e)] = merged.get(tuple(e), 0.0) + c
            terms = [(c, e) for e, c in merged.items()]
        else:
            terms = [(c * x["scale"], e) for c, e in POLY_TERMS[d]]
        W, var = _coefficients(*_poly_symbols([(c * sm ** -sum(e), e) for c, e in terms], d), d, p), same
    return dict(W=W, variables=var, a=[sm * v for v in a], b=[sm * v for v in b], pref=sm ** d)


def _exact_is_quick(case):
    """Whether the recursion and the paths take a few seconds in plain Python and torch."""
    kind, p, d = case["kind"], case["p"], case.get("d", 1)
    if p > {"general": 8, "radial": (18, 6, 4, 3)[d - 1], "poly": (10, 10, 4, 3)[d - 1]}.get(kind, 18):
        return False
    terms = _monomials("poly" if kind == "radial" and d > 1 else kind, p, d, case.get("degree", 0))
    return case["n"] * (_slice_count(case) * (2 * terms + 10) + 300 * d * (1 << case["s"])) < 1.5e12


def exact(case, seed):
    kind = case["kind"]
    if kind == "proposal":
        return None                     # trained weights have no value apart from the 16-bit products
    if kind == "spectrum":
        n, k, t = case["n"], case["k"], case["t"]
        if n > 2000:
            return None
        x = _inputs(case, seed)
        h = 2.0 * case["L"] / n
        grid = torch.arange(n, dtype=torch.float64) * h + (0.5 * h - case["L"])
        mid, dev = 0.5 * (grid[:, None] + grid[None, :]), 0.5 * (grid[None, :] - grid[:, None])
        terms = _slice_terms(_quartic_symbols(case["A"], case["g"] * x["scale"]), 1, case["p"], t)
        S = _slice_sum(terms, [mid.reshape(-1, 1), dev.reshape(-1, 1)]).reshape(n, n)
        free = 2.0 * dev * dev / t
        M = torch.where(free > 40.0, torch.zeros_like(S), h / math.sqrt(2.0 * math.pi * t) * torch.exp(-free - S))
        lam = np.linalg.eigvalsh(M.numpy())
        return -np.log(lam[::-1][:k]) / t
    if kind == "batch":
        systems, rows = _batch_rows(case, seed)
        if sum(r[7] * r[5] for r in rows) > 4e9:
            return None
        smax = max(r[5] for r in rows).bit_length() - 1
        out, coefficients = [], {}
        for system, m, a, b, T, N, p, n, stream in rows:
            if (system, p) not in coefficients:
                c = systems[system]
                coefficients[system, p] = _coefficients(*_quartic_symbols(2.0 * c[2], 24.0 * c[4]), 1, p)
            s = N.bit_length() - 1
            prob = dict(W=coefficients[system, p], variables=lambda mid: mid, a=[a], b=[b], pref=1.0)
            r = _estimate(prob, T, s, range(1, s + 1) if case["hier"] else [s], n, 1 + seed, stream)
            out.append({f: np.concatenate([r[f], np.zeros(smax - s)]) for f in FIELDS[:5]})
        return {**{f: np.stack([r[f] for r in out]) for f in FIELDS[:5]}, "n": None, "n_nonfinite": None}
    if not _exact_is_quick(case):
        return None
    x = _inputs(case, seed)
    s = case["s"]
    return _estimate(_problem(case, x), case["T"], s, range(1, s + 1) if case["hier"] else [s], case["n"], x["seed"],
                     x["stream"])
