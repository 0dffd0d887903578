"""Cases that the product is timed on: what a program has this library do.

A case is a dict of plain values.  `kind` says which entry point it goes
through and `family` where its monomials come from:

  sparse5   (1+x+y+2z^2+3t^3+5u^5)^n times (1+u+t+2z^2+3y^3+5x^5)^n, 5 variables
  dense4    (1+x+y+z+t)^n times itself plus one, 4 variables
  random    distinct random exponent vectors, `nvars` variables, exponents 0..max_exp

A case's monomials are its own (by n, or by the sizes); the coefficients are
drawn from the seed, so that every seed's result has the same terms with other
coefficients.
"""
import math

import numpy as np
import torch

from paper_1303_7425_amd import polymul as pm
from paper_1303_7425_amd import workloads as W

# exponents 0..max_exp in fields of `bits` bits, by number of variables: the
# batched workload's own layout (6 variables) and generic ones around it, each
# with room for 20000 distinct monomials
RANDOM_LAYOUTS = {3: (16, 63), 4: (16, 31), 6: (10, 15), 8: (8, 7)}
MAX_RANDOM_TERMS = 20000


def _power(kind, family, n, ring, **more):
    return dict(kind=kind, family=family, n=n, ring=ring, **more)


def _random(kind, nvars, na, nb, ring):
    bits, max_exp = RANDOM_LAYOUTS[nvars]
    return dict(kind=kind, family="random", nvars=nvars, bits=bits, max_exp=max_exp, na=na, nb=nb, ring=ring)


def _batch(kind, count, size_seed, ring):
    return dict(kind=kind, family="random", count=count, size_seed=size_seed, ring=ring)


def listed():
    return [
        # the smallest products of the batched mix, one at a time: latency and launches
        dict(_random("mul", 6, 57, 61, "f64"), name="random6_57x61_f64"),
        # the smallest product of the serving mix
        dict(_power("mul", "sparse5", 6, "modp"), name="sparse5_n6_modp"),
        # a small dense product in machine integers (the smallest benchmark configuration)
        dict(_power("mul", "dense4", 10, "i64"), name="dense4_n10_i64"),
        # a ragged product of unlike operands, nearly no like terms
        dict(_random("mul", 6, 777, 12345, "modp"), name="random6_777x12345_modp"),
        # the large sparse product that the benchmark reports, exact and in FP64
        dict(_power("mul", "sparse5", 12, "modp"), name="sparse5_n12_modp"),
        dict(_power("mul", "sparse5", 12, "f64"), name="sparse5_n12_f64"),
        # dense products mod p: the benchmark's and the serving mix's largest
        dict(_power("mul", "dense4", 20, "modp"), name="dense4_n20_modp"),
        dict(_power("mul", "dense4", 30, "modp"), name="dense4_n30_modp"),
        # exact integers of three words
        dict(_power("mul", "sparse5", 10, "z192"), name="sparse5_n10_z192"),
        # products of very uneven sizes in one validated call, and as a prepared graph that is replayed
        dict(_batch("batch", 24, 4, "modp"), name="batch24_modp"),
        dict(_batch("graph", 24, 4, "f64"), name="batch24_graph_f64"),
        # a burst of serving requests: n = 6..12 in turn
        dict(kind="serve", family="sparse5", count=14, n_lo=6, n_hi=12, ring="modp", name="serve14_modp"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    exact = ("modp", "modp", "i64", "modq")
    kind = rng.choice(("sparse5", "sparse5", "random", "random", "random", "dense4", "dense4", "z192", "batch", "graph",
                       "serve"))
    if kind == "sparse5":
        return _power("mul", "sparse5", rng.randint(5, 12), rng.choice(exact + ("f64", "f64")))
    if kind == "random":
        na, nb = log_int(50, MAX_RANDOM_TERMS), log_int(50, MAX_RANDOM_TERMS)
        while na * nb > 100_000_000:
            na, nb = log_int(50, MAX_RANDOM_TERMS), log_int(50, MAX_RANDOM_TERMS)
        return _random("mul", rng.choice((3, 4, 6, 6, 8)), na, nb, rng.choice(exact + ("f64", "f64")))
    if kind == "dense4":
        ring = rng.choice(exact + ("f64",))
        return _power("mul", "dense4", rng.randint(8, 15 if ring == "f64" else 27), ring)
    if kind == "z192":
        return _power("mul", rng.choice(("sparse5", "dense4")), rng.randint(6, 11), "z192")
    if kind == "serve":
        return dict(kind="serve", family="sparse5", count=rng.randint(5, 16), n_lo=rng.randint(6, 8),
                    n_hi=rng.randint(9, 12), ring="modp")
    case = _batch(kind, rng.randint(5, 20), rng.randrange(1 << 20), rng.choice(("modp", "f64", "modp", "i64")))
    while sum(a * b for a, b in _sizes(case)) > 400_000_000:
        case["size_seed"] = rng.randrange(1 << 20)
    return case


# ----------------------------------------------------------------------------
# operands
# ----------------------------------------------------------------------------
_KEYS = {}


def _power_keys(family, n):
    """Both operands of a power family; their keys are what is used."""
    if (family, n) not in _KEYS:
        if family == "sparse5":
            _KEYS[family, n] = (W.sparse_power(n, "f"), W.sparse_power(n, "g"))
        else:
            f = W.dense_power(n)
            _KEYS[family, n] = (f, f)  # the constant term is there already: plus one keeps the monomials
    return _KEYS[family, n]


def _sizes(case):
    s, _ = W.config4_sizes(case["count"], case["size_seed"])
    return [(int(a), int(b)) for a, b in s]


def _coefs(p, rng, ring):
    """p's monomials with new coefficients, none of them zero (a zero's monomials would be missing from the result)."""
    q = W.with_random_coefs(p, rng, ring)
    if ring == "i64":
        q.coefs[q.coefs == 0] = 1
    return q


def _pairs(case, seed):
    """The products' operands on the host, as [(f, g)]."""
    if case["family"] == "random":
        lay = (case.get("nvars", 6), case.get("bits", 10), case.get("max_exp", 15))
        sizes = _sizes(case) if "size_seed" in case else [(case["na"], case["nb"])]
        at = (lay, tuple(sizes))
        if at not in _KEYS:
            keys = W.rng_for(sum(a * 20011 + b for a, b in sizes))
            _KEYS[at] = [tuple(W.random_sparse(keys, m, *lay) for m in s) for s in sizes]
        pairs = _KEYS[at]
    elif case["kind"] == "serve":
        ns = [case["n_lo"] + i % (case["n_hi"] - case["n_lo"] + 1) for i in range(case["count"])]
        pairs = [_power_keys(case["family"], n) for n in ns]
    else:
        pairs = [_power_keys(case["family"], case["n"])]
    rng = W.rng_for(seed)
    return [tuple(_coefs(p, rng, case["ring"]) for p in fg) for fg in pairs]


# ----------------------------------------------------------------------------
# the framework's part
# ----------------------------------------------------------------------------
class _Burst:
    """A server, a burst of requests and their result arrays (counts side by side)."""

    def __init__(self, layout, pairs):
        self.layout, self.pairs = layout, pairs
        self.server = pm.Server(6 << 30, 4)
        self.counts = torch.zeros(len(pairs), dtype=torch.int64, device="cuda")
        self.outs = []
        for i, (f, g) in enumerate(pairs):
            k, c, _ = pm.alloc_out(pm.bound(layout, f, g)[0], "modp")
            self.outs.append((k, c, self.counts[i:i + 1]))

    def run(self):
        s = self.server
        tickets = [s.submit(self.layout, f, g, o) for (f, g), o in zip(self.pairs, self.outs)]
        for t in tickets:
            if s.wait(t) != 0:
                raise RuntimeError("request %d failed" % t)
        return [(k[:m], c[:m]) for (k, c, _), m in zip(self.outs, self.counts.tolist())]


def prepare(case, seed):
    host = _pairs(case, seed)
    lay = host[0][0].layout
    layout = (lay.nvars, lay.bits, case["ring"])
    dev = [tuple(pm.to_device(p) for p in fg) for fg in host]
    kind = case["kind"]
    if kind == "mul":
        return kind, pm.MulCall(layout, *dev[0])
    if kind == "serve":
        return kind, _Burst(layout, dev)
    call = pm.BatchCall(layout, [f for f, _ in dev], [g for _, g in dev])
    if kind == "graph":
        call.prepare_graph()
    return kind, call


def run(state):
    """One product, batch or burst; results cut to their term counts, which the program reads to go on with them."""
    kind, call = state
    if kind == "mul":
        call.run()
        h = call.result()
        return h.keys[:h.n], h.coefs[:h.n]
    if kind == "serve":
        return call.run()
    call.run() if kind == "batch" else call.launch_graph()
    return [(call.out_k[o:o + n], call.out_c[o:o + n]) for o, n in zip(call.offsets.tolist(), call.out_n.tolist())]


# ----------------------------------------------------------------------------
# what a pass cannot do without, and its result in 64 bits
# ----------------------------------------------------------------------------
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _sums(f, g):
    """Exponent sums of all term pairs, row-major."""
    fk, gk = (torch.from_numpy(np.ascontiguousarray(p.keys).view(np.int64)).to(_device()) for p in (f, g))
    return (fk[:, None] + gk[None, :]).reshape(-1)


def _terms(f, g):
    """Distinct monomials of the product (exponent sums in rows of f, merged as they come)."""
    rows = max(1, (1 << 27) // max(1, len(g)))
    got = None
    for i in range(0, len(f), rows):
        part = W.Poly(f.layout, f.keys[i:i + rows], f.coefs[i:i + rows])
        u = torch.unique(_sums(part, g))
        got = u if got is None else torch.unique(torch.cat([got, u]))
    return int(got.numel())


_WORK = {}


def work(case):
    """Each operand term read once, each result term written once; one multiplication and one addition per term pair."""
    key = tuple(sorted((k, v) for k, v in case.items() if k not in ("name", "kind", "ring")))
    if key not in _WORK:
        one = {}
        for f, g in _pairs(dict(case, ring="modp"), 1):
            if case["family"] == "dense4":
                out = math.comb(2 * case["n"] + 4, 4)
            else:
                at = (len(f), len(g), case["family"])
                if case["family"] == "random":
                    out = _terms(f, g)
                else:
                    out = one[at] = one[at] if at in one else _terms(f, g)
            got = _WORK.setdefault(key, [0, 0, 0])
            got[0] += len(f) + len(g)
            got[1] += out
            got[2] += len(f) * len(g)
    ops, out, pairs = _WORK[key]
    size = 32 if case["ring"] == "z192" else 16
    return {"bytes": size * (ops + out), "flops": 2 * pairs}


def _exact_f64(f, g):
    s = _sums(f, g)
    fc, gc = (torch.from_numpy(np.ascontiguousarray(p.coefs)).to(s.device) for p in (f, g))
    keys, at = torch.unique(s, return_inverse=True)
    del s
    sums = torch.zeros(keys.numel(), dtype=torch.float64, device=at.device)
    sums.index_add_(0, at, (fc[:, None] * gc[None, :]).reshape(-1))
    return sums[sums != 0].cpu()


def exact(case, seed):
    """FP64 coefficients by a plain sum per monomial; the other rings and the keys are whole numbers."""
    if case["ring"] != "f64":
        return None
    got = [(None, _exact_f64(f, g)) for f, g in _pairs(case, seed)]
    return got if case["kind"] in ("batch", "graph") else got[0]
