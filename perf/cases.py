"""Timed cases of the solver's main paths.

Each case is one call (or the short run of calls) that an ADAPT-VQE or
classical pre-optimization program makes over and over:

  evaluate  one VQE evaluation: the ansatz applied from the reference, then
            the energy and all parameter gradients by the adjoint sweep
  pool      ADAPT's gradients of the whole operator pool on the current state
  screened  the gradients of the share of the pool a screener has selected
  sigma     the projected sigma vector of a large state, exported sorted
  screener  one screener iteration: features, scores and selection over the
            pool, then the network's gradient on the replay buffer

Orbital and electron counts, ansatz lengths, thresholds and the fixed ansatz
seeds are those of ``paper_2411_07920_amd.inputs.CONFIGS`` where a case says
``ops="config"``; elsewhere the ansatz is drawn from the excitations of the
reference (the operators ADAPT and UCCSD ansaetze are made of), which grows
states of the sizes that ADAPT reaches.  The integrals, the angles and the
random numbers of a case come from the seed; its operators do not, so a case
costs about the same for every seed.  States whose size shapes an output are
cut to a fixed count (N_CUT); the others are pruned by a threshold.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2411_07920_amd import spin, swcs
from paper_2411_07920_amd.inputs import CONFIGS, draw_ansatz, enumerate_pool, make_integrals

# ----------------------------------------------------------------- the cases


def _config(name, kind, config, **more):
    c = CONFIGS[config]
    case = {"name": name, "kind": kind, "n": c.n, "na": c.n_elec // 2, "nb": c.n_elec // 2, "ops": "config",
            "M": c.n_ops, "ops_seed": c.seed_ansatz, "theta": c.theta_hi, "eps": c.eps, "ncut": 0}
    case.update(more)
    return case


def _reference(name, kind, n, na, nb, M, theta, eps, ops="reference", ops_seed=7, ncut=0, **more):
    case = {"name": name, "kind": kind, "n": n, "na": na, "nb": nb, "ops": ops, "M": M, "ops_seed": ops_seed,
            "theta": theta, "eps": eps, "ncut": ncut}
    case.update(more)
    return case


def listed():
    return [
        # the smallest evaluation (12 spin-orbitals): launches and latency
        _config("evaluate_12so", "evaluate", "c1"),
        # an ordinary small one: 28 spin-orbitals, 100 gates, one workgroup's state
        _config("evaluate_28so", "evaluate", "c2"),
        # the paper's own truncation, N_CUT = 10,000, over spin-complemented generators
        _reference("evaluate_ncut_generators", "evaluate", 26, 4, 4, 100, 0.1, 0.0, ops="generators", ncut=10000),
        # the largest configured ansatz: 52 spin-orbitals, 300 gates
        _config("evaluate_52so", "evaluate", "c5"),
        # an ADAPT-sized state of about a million determinants
        _reference("evaluate_large", "evaluate", 26, 8, 8, 90, 0.1, 1e-8),
        # ADAPT's operator selection early on (hundreds of determinants) ...
        _config("pool_28so", "pool", "c2"),
        # ... on a large state of a small orbital space, odd electron count ...
        _reference("pool_30so_open_shell", "pool", 15, 6, 5, 90, 0.15, 1e-7),
        # ... and on a state of 10^5 determinants at 52 spin-orbitals
        _reference("pool_large_state", "pool", 26, 8, 8, 62, 0.1, 1e-8),
        # the screener's share (5 % + 1 %) of the pool at 52 spin-orbitals
        _config("screened_52so", "screened", "c5", share=0.06),
        # export of sigma_P: the energy path of a large state (N_CUT = 800,000)
        _reference("sigma_large", "sigma", 26, 8, 8, 84, 0.1, 0.0, ncut=800000),
        # screener over the 301,600 operators of 52 spin-orbitals, full replay buffer
        _config("screener_52so", "screener", "c5", M=40, rows=65536),
        # whole pool at 52 spin-orbitals on the configured ansatz
        _config("pool_52so", "pool", "c5"),
    ]


def draw(rng):
    kind = rng.choice(["evaluate", "evaluate", "pool", "pool", "screened", "sigma", "screener"])
    n = rng.randint(8, 26)
    na = rng.randint(3, max(3, min(8, n // 2)))
    nb = max(2, na - rng.randint(0, 2))

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    M = log_int(16, 80 if kind in ("evaluate", "sigma") else 56)
    eps = rng.choice([1e-6, 1e-7, 1e-8])
    theta = rng.choice([0.05, 0.1, 0.15])
    ops, ncut = rng.choice(["reference", "reference", "mixed"]), 0
    more = {}
    if kind == "evaluate":
        ops = rng.choice(["reference", "mixed", "generators"])
        if rng.random() < 0.35:
            ncut, eps = log_int(300, 12000), 0.0
    elif kind == "sigma":
        ncut, eps = log_int(200, 600000), 0.0
    elif kind == "screened":
        more["share"] = rng.uniform(0.01, 0.1)
    elif kind == "screener":
        more["rows"] = log_int(1000, 65536)
        M = log_int(5, 40)
    case = _reference("", kind, n, na, nb, M, theta, eps, ops=ops, ops_seed=rng.randrange(1 << 20), ncut=ncut, **more)
    del case["name"]
    return case


# ------------------------------------------------------- problem and ansatz


@functools.lru_cache(maxsize=8)
def _pool(n):
    return enumerate_pool(n)


@functools.lru_cache(maxsize=4)
def _generator_pool(n):
    return spin.spin_complemented(_pool(n))


def _reference_key(case):
    return sum(1 << (2 * p) for p in range(case["na"])) | sum(1 << (2 * p + 1) for p in range(case["nb"]))


def _masks(pool):
    p = pool.astype(np.int64)
    two = p[:, 2] >= 0
    one = np.int64(1)
    cre = np.where(two, (one << p[:, 0]) | (one << p[:, 1]), one << p[:, 0])
    ann = np.where(two, (one << np.maximum(p[:, 2], 0)) | (one << np.maximum(p[:, 3], 0)), one << p[:, 1])
    return ann, cre


@functools.lru_cache(maxsize=64)
def _ansatz(n, na, nb, ops, M, ops_seed):
    """Pool rows (int32 [M]), or generator rows (k, k', sign) [M, 3]."""
    pool = _pool(n)
    if ops == "config":
        return draw_ansatz(len(pool), M, -1.0, 1.0, ops_seed)[0]
    rng = np.random.default_rng(ops_seed)
    ref = _reference_key({"na": na, "nb": nb})
    ann, cre = _masks(pool)
    exc = np.flatnonzero((((ref & ann) == ann) & ((ref & cre) == 0)) | (((ref & cre) == cre) & ((ref & ann) == 0)))
    if ops == "generators":
        gp = _generator_pool(n)
        g = np.flatnonzero(np.isin(gp.first, exc))
        return spin.gen_rows(gp, rng.choice(g, min(M, len(g)), replace=False))
    take = rng.choice(exc, min(M, len(exc)), replace=False)
    if ops == "mixed":  # one operator in four from anywhere in the pool, once the state has grown
        late = np.arange(len(take)) % 4 == 3
        take[late] = rng.choice(np.setdiff1d(np.arange(len(pool)), take), int(late.sum()), replace=False)
    return take.astype(np.int32)


def _rows(case):
    return _ansatz(case["n"], case["na"], case["nb"], case["ops"], case["M"], case["ops_seed"])


def _draw(case, seed):
    """(h, eri, angles, generator for the rest) of a seed."""
    h, eri = make_integrals(case["n"], case["n"], 10_000 + seed)
    rng = np.random.default_rng([seed, 77])
    theta = rng.uniform(-case["theta"], case["theta"], len(_rows(case)))
    return h, eri, theta, rng


def _subset(case, rng):
    K = len(_pool(case["n"]))
    return np.sort(rng.choice(K, max(1, int(case["share"] * K)), replace=False)).astype(np.int32)


def _screener_inputs(case, rng):
    K, B = len(_pool(case["n"])), case["rows"]
    prev = np.exp(rng.uniform(np.log(1e-9), 0.0, K)).astype(np.float32)
    age = rng.integers(0, 11, K).astype(np.float32)
    count = (rng.random(K) < 0.002).astype(np.float32)
    rnd = rng.integers(0, 1 << 32, K, dtype=np.uint64).astype(np.uint32)
    P = 16 * 128 + 128 + 128 * 128 + 128 + 128 + 1
    W = np.zeros(P, dtype=np.float32)
    W[:2048] = rng.normal(0, math.sqrt(2 / 16), 2048)
    W[2176:2176 + 16384] = rng.normal(0, math.sqrt(2 / 128), 16384)
    W[2048:2176] = rng.normal(0, 0.05, 128)
    W[18688:18816] = rng.normal(0, 0.05, 128)
    bx = rng.normal(0, 1, (B, 16)).astype(np.float32)
    bx[:, 10] = rng.uniform(-9, 0, B)
    bt = rng.normal(0, 0.5, B).astype(np.float32)
    return prev, age, count, rnd, W, bx, bt


# ------------------------------------------------------------- the program


def _apply(ctx, case, rows, theta):
    if case["ops"] == "generators":
        return ctx.apply_generators(rows, theta, case["eps"], case["ncut"])
    return ctx.apply_ansatz(rows, theta, case["eps"], case["ncut"])


def prepare(case, seed):
    h, eri, theta, rng = _draw(case, seed)
    rows = _rows(case)
    ctx = swcs.make_context(case["n"], case["na"], case["nb"], h, eri, _pool(case["n"]), _reference_key(case))
    s = {"case": case, "kind": case["kind"], "ctx": ctx, "rows": rows, "theta": theta}
    if case["kind"] != "evaluate":
        _apply(ctx, case, rows, theta)
    if case["kind"] == "screened":
        sub = _subset(case, rng)
        s["subset"] = torch.from_numpy(sub).cuda()
        s["g"] = torch.zeros(len(sub), dtype=torch.float64, device="cuda")
    if case["kind"] == "screener":
        prev, age, count, rnd, W, bx, bt = _screener_inputs(case, rng)
        K, B = len(prev), len(bx)
        s["n_top"], s["n_rand"] = math.ceil(0.05 * K), math.ceil(0.01 * K)
        for name, a in (("prev", prev), ("age", age), ("count", count), ("rnd", rnd.view(np.int32)), ("W", W),
                        ("bx", bx), ("bt", bt)):
            s[name] = torch.from_numpy(a).cuda()
        for name, shape in (("feat", (K, 16)), ("score", (K,)), ("y", (B,)), ("act", (B, 256)), ("dy", (B,)),
                            ("loss", (1,)), ("dW", (len(W),))):
            s[name] = torch.zeros(shape, device="cuda")
        s["idx"] = torch.zeros(s["n_top"] + s["n_rand"], dtype=torch.int32, device="cuda")
    return s


def run(s):
    ctx, kind = s["ctx"], s["kind"]
    if kind == "evaluate":
        n_det = _apply(ctx, s["case"], s["rows"], s["theta"])
        dE, E = ctx.param_gradients(len(s["rows"]))
        return {"n_det": n_det, "E": E, "dE": dE}
    if kind == "pool":
        return {"g": ctx.pool_gradients()}
    if kind == "screened":
        ctx.pool_gradients_device(s["subset"], s["g"])
        return {"g": s["g"]}
    if kind == "sigma":
        keys, sigma = ctx.sigma_projected()
        return {"keys": keys.view(np.int64), "sigma": sigma}
    ctx.features(s["prev"], s["age"], s["count"], s["feat"])
    ctx.mlp_forward(s["W"], s["feat"], s["score"])
    ctx.add_feature(s["score"], s["feat"], 10, +1, 0.25)
    ctx.select(s["score"], s["rnd"], s["n_top"], s["n_rand"], s["idx"])
    ctx.mlp_forward(s["W"], s["bx"], s["y"], s["act"])
    ctx.mse(s["y"], s["bt"], s["dy"], s["loss"])
    ctx.mlp_backward(s["W"], s["bx"], s["act"], s["dy"], s["dW"])
    return {"feat": s["feat"], "score": s["score"], "idx": s["idx"], "y": s["y"], "loss": s["loss"], "dW": s["dW"]}


# ------------------------------------------- the same quantities, plainly


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _par(x):
    for sh in (32, 16, 8, 4, 2, 1):
        x = x ^ (x >> sh)
    return x & 1


def _sign_of(x):
    return 1.0 - 2.0 * _par(x).double()


class _Op:
    """T of a pool row (P, Q, R, S) as the ladder operators that act, in order."""

    def __init__(self, row):
        P, Q, R, S = (int(x) for x in row)
        self.order = (Q, P) if R < 0 else (R, S, Q, P)
        n_ann = len(self.order) // 2
        self.ann = sum(1 << x for x in self.order[:n_ann])
        self.cre = sum(1 << x for x in self.order[n_ann:])
        self.both = self.ann | self.cre

    def phase(self, D):
        """<T D|T|D> for determinants D that T acts on."""
        x = torch.zeros_like(D)
        for q in self.order:
            x = x ^ _par(D & ((1 << q) - 1))
            D = D ^ (1 << q)
        return 1.0 - 2.0 * x.double()


def _find(keys, q):
    at = torch.searchsorted(keys, q).clamp(max=len(keys) - 1)
    return at, keys[at] == q


def _value(keys, v, q):
    at, hit = _find(keys, q)
    return torch.where(hit, v[at], torch.zeros_like(v[at])), hit


def _pairs(keys, op):
    """The pairs (D, T D) with a member among keys, as sorted D, and the keys of none."""
    isT = ((keys & op.ann) == op.ann) & ((keys & op.cre) == 0)
    isTd = ((keys & op.cre) == op.cre) & ((keys & op.ann) == 0)
    return torch.unique(torch.cat([keys[isT], keys[isTd] ^ op.both])), ~(isT | isTd)


def _prune(keys, amps, eps, ncut):
    keys, at = torch.sort(keys)
    amps = amps[at]
    if ncut:
        if len(keys) > ncut:
            at = torch.sort(torch.sort(amps.abs(), descending=True, stable=True)[1][:ncut])[0]
            keys, amps = keys[at], amps[at]
    elif eps > 0:
        keep = ~(amps.abs() < eps)
        keys, amps = keys[keep], amps[keep]
    return keys, amps


class _Row:
    """exp(angle A) of one pool row: every pair rotates."""

    def __init__(self, row, c, sn):
        self.op, self.c, self.sn = _Op(row), c, sn

    def forward(self, keys, amps):
        D, free = _pairs(keys, self.op)
        X = D ^ self.op.both
        (a, _), (b, _) = _value(keys, amps, D), _value(keys, amps, X)
        s = self.op.phase(D)
        nd, nx = self.c * a - s * (self.sn * b), self.c * b + s * (self.sn * a)
        return torch.cat([keys[free], D, X]), torch.cat([amps[free], nd, nx])

    def backward(self, keys, amps, keys2, mu2):
        D, _ = _pairs(keys, self.op)
        X = D ^ self.op.both
        (a, hd), (b, hx) = _value(keys, amps, D), _value(keys, amps, X)
        s = self.op.phase(D)
        m, _ = _value(keys2, mu2, D)
        w, _ = _value(keys2, mu2, X)
        dE = (m * (-self.sn * a - s * self.c * b) + w * (-self.sn * b + s * self.c * a)).sum()
        mu, _ = _value(keys2, mu2, keys)
        mu[_find(keys, D[hd])[0]] = (self.c * m + s * self.sn * w)[hd]
        mu[_find(keys, X[hx])[0]] = (self.c * w - s * self.sn * m)[hx]
        return dE, mu


class _Star:
    """exp(theta (A1 + sg A2)) of two rows that share spin-orbitals, by its power series."""

    def __init__(self, row1, row2, sg, theta):
        self.terms = ((_Op(row1), 1.0), (_Op(row2), float(sg)))
        self.theta = theta

    def _space(self, keys):
        while True:
            more = [keys]
            for op, _ in self.terms:
                D, _free = _pairs(keys, op)
                more += [D, D ^ op.both]
            grown = torch.unique(torch.cat(more))
            if len(grown) == len(keys):
                return keys
            keys = grown

    def _maps(self, keys):
        maps = []
        for op, f in self.terms:
            D, _ = _pairs(keys, op)
            s = f * op.phase(D)
            maps.append((_find(keys, D)[0], _find(keys, D ^ op.both)[0], s))
        return maps

    @staticmethod
    def _g(maps, v):
        out = torch.zeros_like(v)
        for i, j, s in maps:
            out[j] += s * v[i]
            out[i] -= s * v[j]
        return out

    def _exp(self, maps, v, t):
        out, term = v.clone(), v
        for k in range(1, 30):
            term = self._g(maps, term) * (t / k)
            out = out + term
        return out

    def forward(self, keys, amps):
        space = self._space(keys)
        v, _ = _value(keys, amps, space)
        u = self._exp(self._maps(space), v, self.theta)
        keep = _find(keys, space)[1] | (u != 0)
        return space[keep], u[keep]

    def backward(self, keys, amps, keys2, mu2):
        space = self._space(keys)
        maps = self._maps(space)
        v, _ = _value(keys, amps, space)
        m, _ = _value(keys2, mu2, space)
        dE = (m * self._g(maps, self._exp(maps, v, self.theta))).sum()
        return dE, _value(space, self._exp(maps, m, -self.theta), keys)[0]


def _chain(case, theta):
    """The unitaries of a case with the parameter of each and d(angle)/d(parameter)."""
    pool, gates = _pool(case["n"]), []
    for i, r in enumerate(_rows(case)):
        c, s = math.cos(theta[i]), math.sin(theta[i])
        if case["ops"] != "generators" or r[1] < 0:
            gates.append((_Row(pool[int(r) if case["ops"] != "generators" else int(r[0])], c, s), i, 1.0))
            continue
        a, b, sg = int(r[0]), int(r[1]), float(r[2])
        if _Op(pool[a]).both & _Op(pool[b]).both:
            gates.append((_Star(pool[a], pool[b], sg, theta[i]), i, 1.0))
        else:
            gates.append((_Row(pool[a], c, s), i, 1.0))
            gates.append((_Row(pool[b], c, sg * s), i, sg))
    return gates


def _state(case, theta, keep=None):
    """The pruned state of the ansatz, keys ascending; keep collects the state before each unitary."""
    keys = torch.tensor([_reference_key(case)], dtype=torch.int64, device=_device())
    amps = torch.ones(1, dtype=torch.float64, device=_device())
    for gate, _, _ in _chain(case, theta):
        if keep is not None:
            keep.append((keys, amps))
        keys, amps = _prune(*gate.forward(keys, amps), case["eps"], case["ncut"])
    return keys, amps


class _Hamiltonian:
    def __init__(self, h, eri):
        dev = _device()
        self.n = len(h)
        self.h = torch.from_numpy(h).to(dev)
        self.eri = torch.from_numpy(eri).to(dev)
        self.flat = self.eri.reshape(-1)

    def two(self, p, q, r, s):
        """Spin-orbital (pq|rs) with the spin deltas."""
        v = self.flat[(((p >> 1) * self.n + (q >> 1)) * self.n + (r >> 1)) * self.n + (s >> 1)]
        return torch.where((((p ^ q) & 1) | ((r ^ s) & 1)) == 0, v, torch.zeros_like(v))

    def diagonal(self, keys):
        n = self.n
        bit = ((keys[:, None] >> torch.arange(2 * n, device=keys.device)) & 1).double()
        a, b = bit[:, 0::2], bit[:, 1::2]
        J = torch.einsum("ppqq->pq", self.eri).contiguous()
        K = torch.einsum("pqqp->pq", self.eri).contiguous()
        t = a + b
        return t @ torch.diagonal(self.h) + 0.5 * ((t @ J * t).sum(1) - (a @ K * a).sum(1) - (b @ K * b).sum(1))

    def single(self, D, i, a):
        """<X|H|D>, X = a+_a a_i D, without its sign."""
        v = self.h[a >> 1, i >> 1].clone()
        for Q in range(2 * self.n):
            q = torch.full_like(i, Q)
            occ = ((D >> Q) & 1).double()
            v += occ * (self.two(a, i, q, q) - self.two(a, q, q, i))
        return v


def _bit_position(x):
    return torch.log2(x.double()).round().long()


def _sigma(keys, amps, ham):
    """sigma_P over the stored determinants: pairs that share a subset of all but two electrons."""
    n = 2 * ham.n
    sigma = ham.diagonal(keys) * amps
    bits = (keys[:, None] >> torch.arange(n, device=keys.device)) & 1
    N = int(bits[0].sum())
    occ = torch.nonzero(bits)[:, 1].reshape(len(keys), N)
    del bits
    subs, who = [], []
    at = torch.arange(len(keys), device=keys.device, dtype=torch.int32)
    for i in range(N):
        for j in range(i):
            subs.append(keys ^ (torch.ones_like(keys) << occ[:, i]) ^ (torch.ones_like(keys) << occ[:, j]))
            who.append(at)
    subs, order = torch.sort(torch.cat(subs))
    who = torch.cat(who)[order].long()
    del order
    first = torch.arange(len(subs) - 1, device=keys.device)
    step = 1
    while True:
        first = first[first + step < len(subs)]
        first = first[subs[first] == subs[first + step]]
        if len(first) == 0:
            return sigma
        for lo in range(0, len(first), 1 << 25):
            f = first[lo:lo + (1 << 25)]
            i, j, S = who[f], who[f + step], subs[f]
            D, X = keys[i], keys[j]
            holes, parts = D & ~X, X & ~D
            h0, p0 = holes & -holes, parts & -parts
            h1, p1 = holes ^ h0, parts ^ p0
            two = h1 != 0
            v = torch.zeros(len(f), dtype=torch.float64, device=keys.device)
            A, B, I, J = (_bit_position(x[two]) for x in (p0, p1, h0, h1))
            d, s = D[two], None
            for q in (I, J, B, A):
                m = torch.ones_like(q) << q
                s = _par(d & (m - 1)) if s is None else s ^ _par(d & (m - 1))
                d = d ^ m
            v[two] = (1.0 - 2.0 * s.double()) * (ham.two(A, I, B, J) - ham.two(A, J, B, I))
            common = D & X
            one = ~two & (S == (common & (common - 1)))  # a single shares many subsets: one of them counts
            I, A, d = _bit_position(h0[one]), _bit_position(p0[one]), D[one]
            s = _par(d & (h0[one] - 1)) ^ _par((d ^ h0[one]) & (p0[one] - 1))
            v[one] = (1.0 - 2.0 * s.double()) * ham.single(d, I, A)
            sigma.index_add_(0, i, v * amps[j])
            sigma.index_add_(0, j, v * amps[i])
        step += 1


def _pool_gradients(case, keys, amps, ham):
    """g_k = 2 <H psi|A_k psi> / <psi|psi> with sigma = H psi on every determinant A_k psi reaches."""
    pool = _pool(case["n"])
    ann, cre = _masks(pool)
    dev = keys.device
    ann_t, cre_t = torch.from_numpy(ann).to(dev), torch.from_numpy(cre).to(dev)
    rows = torch.from_numpy(pool.astype(np.int64)).to(dev)
    P, Q, R, S = rows[:, 0], rows[:, 1], rows[:, 2].clamp(min=0), rows[:, 3].clamp(min=0)
    double = rows[:, 2] >= 0
    w_double = ham.two(P, R, Q, S) - ham.two(P, S, Q, R)
    Xs, vs, ks, ws = [], [], [], []
    step = max(1, (1 << 26) // len(keys))
    for lo in range(0, len(pool), step):
        an, cr = ann_t[lo:lo + step, None], cre_t[lo:lo + step, None]
        isT = ((keys & an) == an) & ((keys & cr) == 0)
        isTd = ((keys & cr) == cr) & ((keys & an) == 0)
        k, d = torch.nonzero(isT | isTd, as_tuple=True)
        T = isT[k, d]
        k = k + lo
        D = keys[d]
        X = D ^ ann_t[k] ^ cre_t[k]
        low = torch.where(T, D, X)
        s = torch.zeros_like(low)
        x = low
        dbl = double[k].long()
        for q, on in ((R[k], dbl), (S[k], dbl), (Q[k], None), (P[k], None)):
            m = torch.ones_like(q) << q
            b, flip = _par(x & (m - 1)), m
            if on is not None:
                b, flip = b * on, m * on
            s = s ^ b
            x = x ^ flip
        ph = 1.0 - 2.0 * s.double()
        v = w_double[k]
        one = dbl == 0
        if bool(one.any()):
            v[one] = ham.single(low[one], Q[k[one]], P[k[one]])
        psi = amps[d]
        Xs.append(X)
        vs.append(ph * v * psi)
        ks.append(k.int())
        ws.append(torch.where(T, ph, -ph) * psi)
    X, v, k, w = torch.cat(Xs), torch.cat(vs), torch.cat(ks), torch.cat(ws)
    del Xs, vs, ks, ws
    ext, order = torch.sort(X)
    new = torch.ones(len(ext), dtype=torch.bool, device=dev)
    new[1:] = ext[1:] != ext[:-1]
    group = torch.cumsum(new, 0) - 1
    ext = ext[new]
    sigma = torch.zeros(len(ext), dtype=torch.float64, device=dev)
    sigma.index_add_(0, group, v[order])
    at, hit = _find(ext, keys)
    sigma[at[hit]] += (ham.diagonal(keys) * amps)[hit]
    g = torch.zeros(len(pool), dtype=torch.float64, device=dev)
    g.index_add_(0, k[order].long(), w[order] * sigma[group])
    return 2.0 * g / (amps * amps).sum()


def _connections(case):
    n, a, b = case["n"], case["na"], case["nb"]
    va, vb, c2 = n - a, n - b, lambda m: m * (m - 1) // 2
    return a * va + b * vb + c2(a) * c2(va) + c2(b) * c2(vb) + a * b * va * vb


def _exact_screener(case, seed):
    h, eri, theta, rng = _draw(case, seed)
    prev, age, count, _, W, bx, bt = _screener_inputs(case, rng)
    keys, amps = _state(case, theta)
    dev = keys.device
    n, rows = case["n"], _pool(case["n"]).astype(np.int64)
    two = rows[:, 2] >= 0
    bit = ((keys[:, None] >> torch.arange(2 * n, device=dev)) & 1).double()
    occ = ((amps * amps)[:, None] * bit).sum(0).cpu().numpy() / float((amps * amps).sum())
    fock = h + sum(2.0 * eri[:, :, j, j] - eri[:, j, j, :] for j in range(case["na"]))
    f = np.zeros((len(rows), 16))
    for t in range(4):
        on = rows[:, t] >= 0
        p = rows[on, t]
        f[on, t] = fock[p >> 1, p >> 1]
        f[on, 5 + t] = occ[p]
    p, q, r, s = (rows[:, t] >> 1 for t in range(4))
    f[:, 4] = np.where(two, np.abs(eri[p, r, q, s]), np.abs(fock[p, q]))
    f[:, 9], f[:, 11], f[:, 15] = prev, age / 10.0, count
    f[:, 10] = np.log10(prev.astype(np.float64) + 1e-16)
    same = ((rows[:, 0] ^ rows[:, 1]) & 1) == 0
    f[:, 12], f[:, 13], f[:, 14] = ~two, two & same, two & ~same
    w = torch.from_numpy(W.astype(np.float64)).to(dev)
    parts = torch.split(w, [2048, 128, 16384, 128, 128, 1])
    w1, b1, w2, b2, w3, b3 = [p.clone().requires_grad_() for p in parts]

    def net(x):
        a1 = torch.relu(x @ w1.reshape(16, 128) + b1)
        return torch.relu(a1 @ w2.reshape(128, 128) + b2) @ w3 + b3

    ft = torch.from_numpy(f).to(dev)
    with torch.no_grad():
        score = 0.25 * net(ft) + ft[:, 10]
    x, t = torch.from_numpy(bx).to(dev).double(), torch.from_numpy(bt).to(dev).double()
    y = net(x)
    loss = ((y - t) ** 2).mean()
    dW = torch.cat(torch.autograd.grad(loss, [w1, b1, w2, b2, w3, b3]))
    return {"feat": ft, "score": score, "idx": None, "y": y.detach(), "loss": loss.detach().reshape(1), "dW": dW}


def exact(case, seed):
    if case["kind"] == "screener":
        return _exact_screener(case, seed)
    h, eri, theta, rng = _draw(case, seed)
    ham = _Hamiltonian(h, eri)
    if case["kind"] != "evaluate":
        keys, amps = _state(case, theta)
        if case["kind"] == "sigma":
            return {"keys": None, "sigma": _sigma(keys, amps, ham)}
        if len(keys) * _connections(case) > 2 ** 31 - 2:
            return None  # more pairs than one plain sort takes
        g = _pool_gradients(case, keys, amps, ham)
        if case["kind"] == "screened":
            g = g[torch.from_numpy(_subset(case, rng)).long().to(g.device)]
        return {"g": g}
    before = []
    keys, amps = _state(case, theta, before)
    sigma = _sigma(keys, amps, ham)
    norm = (amps * amps).sum()
    E = (amps * sigma).sum() / norm
    mu = (2.0 / norm) * (sigma - E * amps)
    dE = np.zeros(len(theta))
    after = keys
    for (gate, i, factor), (kb, ab) in zip(reversed(_chain(case, theta)), reversed(before)):
        d, mu = gate.backward(kb, ab, after, mu)
        dE[i] += factor * float(d)
        after = kb
    return {"n_det": None, "E": float(E), "dE": dE}


# ------------------------------------------------------------------- work


@functools.lru_cache(maxsize=256)
def _sizes(items):
    """(determinants entering each unitary, final determinants) at one seed."""
    case = dict(items)
    before = []
    theta = np.random.default_rng([1, 77]).uniform(-case["theta"], case["theta"], len(_rows(case)))
    keys, _ = _state(case, theta, before)
    return sum(len(k) for k, _ in before), len(keys)


def work(case):
    """Bytes and operations of one pass: 16 bytes for each stored (key,
    amplitude).  A chain reads the keys of every state it passes through once
    forward and once back, and touches few amplitudes; a sigma vector and the
    pool gradients read the state once and the integrals, and write their
    result; the network is counted in full."""
    K, n = len(_pool(case["n"])), case["n"]
    through, dets = _sizes(tuple(sorted((k, v) for k, v in case.items() if k not in ("name", "rows", "share", "kind"))))
    ints = 8 * (n ** 4 // 8 + n * n)
    kind = case["kind"]
    if kind == "evaluate":
        return {"bytes": 2 * 8 * through + 16 * dets + ints, "flops": 12 * through}
    if kind == "sigma":
        return {"bytes": 32 * dets + ints, "flops": 40 * dets}
    if kind == "screener":
        B, mac = case["rows"], 16 * 128 + 128 * 128 + 128
        return {"bytes": 16 * dets + K * (16 + 12 + 64 + 4 + 4) + B * (64 + 4 + 4 + 4) + 3 * 4 * 18817,
                "flops": 2 * mac * (K + 3 * B)}
    out = K if kind == "pool" else int(case["share"] * K)
    return {"bytes": 16 * dets + ints + 8 * out, "flops": 40 * dets}
