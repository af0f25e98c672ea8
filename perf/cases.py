"""The library's everyday work as timed cases.

Each case is one pass through the public binding (paper_2511_09376_amd.wdf): rows
explained against a resident summary, a background summarised or refreshed,
interaction values, a burst of served requests.  The ensembles are the seeded
ones of paper_2511_09376_amd.synth; they are loaded once per process, as a program
that explains a trained model does, and the rows are drawn on the GPU from the
same column mix.  `exact` recomputes a case's outputs with plain torch and numpy in
64 bits from the definitions: decision patterns, the four cube rules and the
closed-form weights.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2511_09376_amd import synth, wdf

DEVICE = "cuda:0"
KINDS = {"shapley": wdf.SHAPLEY, "banzhaf": wdf.BANZHAF, "shapley_iv": wdf.SHAPLEY_IV, "banzhaf_iv": wdf.BANZHAF_IV}

# Most consumer and background rows per ensemble and kind of pass; the listed cases
# reach them.
MOST_ROWS = {"mid": 3_000_000, "uneven": 300_001, "small": 3_000_000}
MOST_BACKGROUND = {"mid": 5_000_000, "uneven": 1_000_000, "small": 1_000_000}
MOST_IV_ROWS = 8_192
MOST_GENERIC = (2_000, 20_000)   # consumer rows, background rows


def listed():
    return [
        # one row explained while its user waits: latency only
        {"name": "explain_1", "op": "explain", "model": "mid", "values": "shapley", "n": 1, "m": 20_000, "offset": 0},
        # the largest served request, explained by the covers alone
        {"name": "explain_4096", "op": "explain", "model": "mid", "values": "pathdep", "n": 4_096, "m": 0, "offset": 0},
        # a day's rows in one call (the mid workload's consumers), Banzhaf values
        {"name": "explain_100k", "op": "explain", "model": "mid", "values": "banzhaf", "n": 100_000, "m": 20_000,
         "offset": 0},
        # the whole data set of the paper-scale workload
        {"name": "explain_3m", "op": "explain", "model": "mid", "values": "shapley", "n": 3_000_000, "m": 20_000,
         "offset": 0},
        # pruned trees of depth 3..8, an odd row count, a column slice of a larger matrix
        {"name": "explain_uneven", "op": "explain", "model": "uneven", "values": "shapley", "n": 300_001, "m": 20_000,
         "offset": 1},
        # a toy model's step: refresh and explain are all launches
        {"name": "step_small", "op": "refresh", "model": "small", "values": "shapley", "n": 100, "m": 100, "offset": 0},
        # a rolling background refreshed and a monitoring sample explained, replayed as a graph
        {"name": "step_mid", "op": "graph", "model": "mid", "values": "shapley", "n": 1_000, "m": 100_000, "offset": 0},
        # the paper-scale background summarised anew
        {"name": "step_5m", "op": "graph", "model": "mid", "values": "shapley", "n": 1_000, "m": 5_000_000, "offset": 0},
        # a one-off run of a large ensemble without waiting for kernels to compile: load and explain
        {"name": "oneoff_generic", "op": "load", "model": "generic", "values": "shapley", "n": 2_000, "m": 20_000,
         "offset": 0},
        # interactions of a few rows on request
        {"name": "iv_64", "op": "iv", "model": "iv", "values": "shapley_iv", "n": 64, "m": 20_000, "offset": 0},
        # interactions of a sample, bound by its F x F output
        {"name": "iv_8192", "op": "iv", "model": "iv", "values": "shapley_iv", "n": 8_192, "m": 20_000, "offset": 0},
        # a burst of requests of log-uniform size on host rows, through the batching server
        {"name": "serve_burst", "op": "serve", "model": "mid", "values": "shapley", "n": 48, "m": 20_000, "offset": 0},
    ]


def _log(rng, lo, hi):
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["explain", "explain", "explain", "refresh", "graph", "load", "generic", "iv", "serve"])
    offset = rng.choice([0, 0, 1, 4])
    if op == "generic":
        return {"op": "load", "model": "generic", "values": rng.choice(["shapley", "banzhaf"]),
                "n": _log(rng, 1, MOST_GENERIC[0]), "m": _log(rng, 1, MOST_GENERIC[1]), "offset": offset}
    if op == "iv":
        return {"op": "iv", "model": "iv", "values": rng.choice(["shapley_iv", "banzhaf_iv"]),
                "n": _log(rng, 1, MOST_IV_ROWS), "m": _log(rng, 1, 20_000), "offset": offset}
    if op == "serve":
        return {"op": "serve", "model": "mid", "values": rng.choice(["shapley", "banzhaf"]), "n": rng.randint(1, 48),
                "m": _log(rng, 1, 20_000), "offset": 0}
    model = rng.choice(["mid", "mid", "uneven", "small"])
    if op == "explain":
        values = rng.choice(["shapley", "banzhaf", "pathdep"])
        return {"op": op, "model": model, "values": values, "n": _log(rng, 1, MOST_ROWS[model]),
                "m": 0 if values == "pathdep" else _log(rng, 1, 20_000), "offset": offset}
    return {"op": op, "model": model, "values": rng.choice(["shapley", "banzhaf"]),
            "n": _log(rng, 1, 10_000), "m": _log(rng, 1, MOST_BACKGROUND[model]), "offset": offset}


# ---------------------------------------------------------------------------
# Ensembles and rows
# ---------------------------------------------------------------------------

_ensembles, _models, _context = {}, {}, []


def ensemble(name):
    """mid and small: the workloads' own.  uneven: the first 100 trees of the uneven
    workload; generic: all 500 of them.  iv: the first 20 trees of mid."""
    if name not in _ensembles:
        w = synth.WORKLOADS["uneven" if name == "generic" else "mid" if name == "iv" else name]
        spec = w.model
        trees = {"uneven": 100, "iv": 20}.get(name, spec.n_trees)
        spec = synth.ModelSpec(trees, spec.depth_lo, spec.depth_hi, spec.prune_p, spec.n_features, spec.feature_pool)
        _ensembles[name] = (synth.make_ensemble(spec, w.data, w.seeds()[0]), w.data)
    return _ensembles[name]


def _model(name):
    if not _context:
        _context.append(wdf.Context(0))
    if name not in _models:
        kernel = wdf.KERNEL_GENERIC if name == "generic" else wdf.KERNEL_AUTO
        _models[name] = wdf.Model(_context[0], ensemble(name)[0], kernel=kernel)
    return _models[name]


def _rows(data, n, gen, offset=0):
    """float32 [F, n] rows of the workload's column mix; with an offset, a column
    slice of a wider matrix."""
    X = torch.empty((data.n_features, n + (offset + 3 if offset else 0)), dtype=torch.float32, device=DEVICE)
    X = X[:, offset:offset + n]
    for f, kind in enumerate(data.column_kinds()):
        if kind == 0:
            col = torch.randn(n, generator=gen, device=DEVICE)
        elif kind == 1:
            col = torch.randn(n, generator=gen, device=DEVICE).exp_()
        elif kind == 2:
            col = (torch.rand(n, generator=gen, device=DEVICE) < 0.3).float()
        else:
            col = torch.poisson(torch.full((n,), 3.0, device=DEVICE), generator=gen)
        if data.nan_rate > 0:
            col[torch.rand(n, generator=gen, device=DEVICE) < data.nan_rate] = float("nan")
        X[f] = col
    return X


def _inputs(case, seed):
    """(X, B, request sizes) of a case: X consumer rows, B background rows or None."""
    data = ensemble(case["model"])[1]
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed) * 7919 + case["n"])
    sizes = None
    n = case["n"]
    if case["op"] == "serve":
        sizes = synth.request_sizes(n, np.random.SeedSequence(n))  # the same sizes for every seed
        n = int(sizes.sum())
    B = _rows(data, case["m"], gen, case["offset"]) if case["m"] else None
    return _rows(data, n, gen, case["offset"]), B, sizes


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.op = case["op"]
    s.model = _model(case["model"])
    s.X, s.B, sizes = _inputs(case, seed)
    s.values = KINDS.get(case["values"], wdf.SHAPLEY)
    if s.op == "load":
        return s
    if case["values"] == "pathdep":
        s.bg = wdf.Background(s.model, values=wdf.SHAPLEY, pathdep=True)
    else:
        s.bg = wdf.Background(s.model, s.B, values=s.values)
    if s.op == "refresh":
        s.bg.refresh(s.B)  # the first refresh allocates the workspace the later ones reuse
    elif s.op == "graph":
        s.phi = torch.empty_like(s.X)
        s.graph = wdf.Graph(s.bg, s.X, s.phi, s.B)
    elif s.op == "serve":
        s.server = wdf.Server(s.bg, mem_budget=4 << 28)
        host = s.X.cpu().numpy()
        cuts = np.cumsum(sizes)[:-1]
        s.requests = [np.ascontiguousarray(x) for x in np.split(host, cuts, axis=1)]
        s.answers = [np.zeros_like(x) for x in s.requests]
        s.X = None
    return s


def run(s):
    if s.op == "explain":
        return s.bg.explain(s.X)
    if s.op == "refresh":
        s.bg.refresh(s.B)
        return s.bg.explain(s.X)
    if s.op == "graph":
        s.graph.launch()
        return s.phi
    if s.op == "load":
        bg = wdf.Background(s.model, s.B, values=s.values)
        return {"phi": bg.explain(s.X), "base": bg.base_value}
    if s.op == "iv":
        return s.bg.explain_iv(s.X)
    for ticket in [s.server.submit(x, phi) for x, phi in zip(s.requests, s.answers)]:
        s.server.wait(ticket)
    return s.answers


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

_shapes = {}


def _leaves(ens):
    """(value, [(node, goes right)]) of every leaf, trees concatenated, depth first."""
    for t in range(ens.n_trees):
        base = int(ens.node_offset[t])
        stack = [(base, [])]
        while stack:
            nd, path = stack.pop()
            if ens.feature[nd] < 0:
                yield float(ens.value[nd]), path
                continue
            stack.append((base + int(ens.right[nd]), path + [(nd, 1)]))
            stack.append((base + int(ens.left[nd]), path + [(nd, 0)]))


def _shape(name):
    """Inner nodes; per leaf summed: pattern bins, values added per row, pairs added
    per row, and the operations of one contraction."""
    if name not in _shapes:
        ens = ensemble(name)[0]
        bins = adds = pairs = flops = flops_iv = 0
        for _, path in _leaves(ens):
            d = len({int(ens.feature[nd]) for nd, _ in path})
            bins += 2 ** d if d else 0
            adds += d
            pairs += d * (d - 1)
            flops += 2 * d * 4 ** d
            flops_iv += d * (d - 1) * 4 ** d
        # sibling leaves share a pattern; about half of the leaves' values are added once per pair
        _shapes[name] = {"inner": int((ens.feature >= 0).sum()), "bins": bins // 2, "adds": adds // 2,
                         "pairs": pairs // 2, "flops": flops, "flops_iv": flops_iv}
    return _shapes[name]


def work(case):
    F, sh = ensemble(case["model"])[1].n_features, _shape(case["model"])
    n = case["n"]
    if case["op"] == "serve":
        n = int(synth.request_sizes(n, np.random.SeedSequence(n)).sum())
    table = 4 * sh["bins"] * 6
    if case["op"] == "iv":
        return {"bytes": 4 * F * n + 4 * F * F * n + 3 * table, "flops": n * (sh["inner"] + sh["pairs"])}
    nbytes, flops = 8 * F * n + table, n * (sh["inner"] + sh["adds"])
    if case["op"] in ("refresh", "graph", "load"):
        nbytes += 4 * F * case["m"]
        flops += case["m"] * (sh["inner"] + sh["adds"] // 3) + sh["flops"]
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# The same values in 64 bits
# ---------------------------------------------------------------------------

def _coefficients(d, values):
    """[positions or position pairs][2^d][2^d]: what the cube of consumer pattern c and
    background pattern b (first position in the top bit) gives each position, or each
    pair u < v of them."""
    P = 1 << d
    c, b = np.meshgrid(np.arange(P), np.arange(P), indexing="ij")
    bit = lambda x, k: (x >> (d - 1 - k)) & 1
    count = lambda x: sum(bit(x, k) for k in range(d))
    alive = (c | b) == P - 1
    a, g = count(c & ~b), count(~c & b)  # positive and negated literals
    s = a + g
    binom = np.array([[float(math.comb(i, j)) if 0 <= j <= i else 1.0 for j in range(d + 1)] for i in range(d + 1)])
    pos = [(bit(c, k) == 1) & (bit(b, k) == 0) for k in range(d)]
    neg = [(bit(c, k) == 0) & (bit(b, k) == 1) for k in range(d)]
    if values in ("shapley_iv", "banzhaf_iv"):
        out = []
        for u in range(d):
            for v in range(u + 1, d):
                both_pos, both_neg = pos[u] & pos[v], neg[u] & neg[v]
                mixed = (pos[u] & neg[v]) | (neg[u] & pos[v])
                if values == "banzhaf_iv":
                    w = 2.0 ** (-(s - 2.0))
                    m = np.where(both_pos | both_neg, w, 0.0) - np.where(mixed, w, 0.0)
                else:
                    at = lambda i, j: binom[np.maximum(i, 0), np.maximum(j, 0)]
                    m = np.where(both_pos, 1.0 / (np.maximum(a - 1, 1) * at(s - 1, a - 1)), 0.0)
                    m += np.where(both_neg, 1.0 / (np.maximum(g - 1, 1) * at(s - 1, g - 1)), 0.0)
                    m -= np.where(mixed, 1.0 / (np.maximum(a, 1) * at(s - 1, a)), 0.0)
                out.append(np.where(alive, m, 0.0))
        return np.stack(out) if out else np.zeros((0, P, P))
    if values == "banzhaf":
        wp = wn = 2.0 ** (-(s - 1.0))
    else:
        wp = 1.0 / (np.maximum(a, 1) * binom[s, a])
        wn = 1.0 / (np.maximum(g, 1) * binom[s, g])
    return np.stack([np.where(alive & pos[k], wp, 0.0) - np.where(alive & neg[k], wn, 0.0) for k in range(d)])


def _exact_rows(ens, X, B, values):
    """(phi or interaction values in float64 on the GPU, base value)."""
    F, n = X.shape
    iv = values.endswith("_iv")
    kind = "shapley" if values == "pathdep" else values
    out = torch.zeros((F, F, n) if iv else (F, n), dtype=torch.float64, device=DEVICE)
    coef, base = {}, 0.0

    def left_of(M, nd):
        col, thr = M[int(ens.feature[nd])], float(ens.threshold[nd])
        return torch.where(torch.isnan(col), bool(ens.default_left[nd]), col < thr).to(torch.int64)

    def frequencies(path, pat_b):
        """Share of the background per raw pattern of the path."""
        d = len(path)
        if B is not None:
            return torch.bincount(pat_b, minlength=1 << d).cpu().numpy().astype(np.float64) / B.shape[1]
        p, f = np.arange(1 << d), np.ones(1 << d)
        for k, (nd, right) in enumerate(path):
            child = tree + int((ens.right if right else ens.left)[nd])
            r = ens.cover[child] / ens.cover[nd] if ens.cover[nd] > 0 else 0.0
            f *= np.where((p >> (d - 1 - k)) & 1, r, 1.0 - r)
        return f

    def leaf(value, path, pat_c, freq):
        nonlocal base
        d = len(path)
        base += value * freq[-1]
        feats = []
        for nd, _ in path:
            if int(ens.feature[nd]) not in feats:
                feats.append(int(ens.feature[nd]))
        e = len(feats)
        p = np.arange(1 << d)
        merged = np.full(1 << d, (1 << e) - 1)  # a repeated feature follows where all its nodes do
        for k, (nd, _) in enumerate(path):
            place = e - 1 - feats.index(int(ens.feature[nd]))
            merged &= ~np.where((p >> (d - 1 - k)) & 1, 0, 1 << place)
        if e not in coef:
            coef[e] = _coefficients(e, kind)
        table = coef[e] @ (value * np.bincount(merged, weights=freq, minlength=1 << e))
        table = torch.from_numpy(np.ascontiguousarray(table[:, merged])).to(DEVICE)
        if iv:
            q = 0
            for u in range(e):
                for v in range(u + 1, e):
                    add = table[q][pat_c]
                    out[feats[u], feats[v]] += add
                    out[feats[v], feats[u]] += add
                    q += 1
        else:
            for k in range(e):
                out[feats[k]] += table[k][pat_c]

    def visit(nd, path, pat_c, pat_b):
        if ens.feature[nd] < 0:
            if path:
                leaf(float(ens.value[nd]), path, pat_c, frequencies(path, pat_b))
            else:
                nonlocal base
                base += float(ens.value[nd])
            return
        lc = left_of(X, nd)
        lb = left_of(B, nd) if B is not None else None
        for right in (0, 1):
            child = tree + int((ens.right if right else ens.left)[nd])
            step = lambda pat, l: None if pat is None else pat * 2 + (1 - l if right else l)
            visit(child, path + [(nd, right)], step(pat_c, lc), step(pat_b, lb))

    for t in range(ens.n_trees):
        tree = int(ens.node_offset[t])
        zero = lambda M: None if M is None else torch.zeros(M.shape[1], dtype=torch.int64, device=DEVICE)
        visit(tree, [], zero(X), zero(B))
    return out, base


def exact(case, seed):
    X, B, sizes = _inputs(case, seed)
    phi, base = _exact_rows(ensemble(case["model"])[0], X, B, case["values"])
    if case["op"] == "load":
        return {"phi": phi, "base": base}
    if case["op"] == "serve":
        return [np.ascontiguousarray(x) for x in np.split(phi.cpu().numpy(), np.cumsum(sizes)[:-1], axis=1)]
    return phi
