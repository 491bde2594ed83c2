"""Workloads the library's speed is judged on, each through the public entry points of paper_1806_11248_amd.

A case is a dict of plain values:

  kind      what one pass does
              round         one boosting iteration over the packed matrix (Context.boost_round), some rounds into a model
              tree          one tree on given gradient pairs, with the row order and the leaf of every row
              sparse_round  one boosting iteration over sparse rows: gradients, grow_tree_sparse, predict_sparse
              leafwise      one boosting iteration with loss-guided growth: gradients, grow_tree_lossguide, predict
              quantise      cuts, binning and packing of a dense float matrix (Context.quantise_packed)
              quantise_csr  the same from compressed sparse rows
              predict       margins of many trees on raw float rows
              steps         the calls a caller makes who drives a tree's first split by hand: fixed-point pairs, root
                            totals, histogram, split, partition, the smaller child's histogram, its sibling by
                            subtraction, the two children's splits
  data      which columns: uniform, normal, tabular (Zipf categories and heavy-tailed numbers), wide (a fifth of the
            columns are noisy copies of others), missing (mostly absent lognormal values)
  rows, cols, bins, depth, leaves, trees, objective, present (share of elements that are not missing)

All sums inside the library are exact integers and every result is reproducible to the last bit, whatever the
order of accumulation: outputs are compared exactly.
"""
from __future__ import annotations

import math

import torch

import paper_1806_11248_amd as g

DEV = "cuda"


def _case(name, kind, data, rows, cols, bins, depth=6, leaves=0, trees=0, objective="squared", present=1.0):
    return dict(name=name, kind=kind, data=data, rows=rows, cols=cols, bins=bins, depth=depth, leaves=leaves,
                trees=trees, objective=objective, present=present)


def listed():
    return [
        # the smallest: one shallow tree on a table of 10,000 rows, launches and waits are what it costs
        _case("tree_10k", "tree", "uniform", 10_000, 8, 16, depth=3),
        # an everyday table of odd sizes with some values missing (9-bit symbols)
        _case("round_50k_odd", "round", "normal", 50_021, 19, 256, depth=6, objective="logistic", present=0.9),
        # the ordinary case: binary classification, a million rows, 28 features
        _case("round_1m", "round", "normal", 1_000_000, 28, 256, depth=6, objective="logistic"),
        # regression on rows that are 80% empty, stored as a packed matrix ...
        _case("round_10m_missing", "round", "missing", 10_000_000, 50, 256, depth=8, present=0.2),
        # ... and in the sparse-row form
        _case("sparse_round_10m", "sparse_round", "missing", 10_000_000, 50, 256, depth=8, present=0.2),
        # many features, few bins, deep: histogram memory and subtraction
        _case("round_500k_wide", "round", "wide", 500_000, 2000, 64, depth=10),
        # the largest: 115 million rows of mixed categorical and numeric columns
        _case("round_115m", "round", "tabular", 115_000_000, 13, 256, depth=8, objective="logistic"),
        # best-first growth to a leaf budget
        _case("leafwise_10m", "leafwise", "tabular", 10_000_000, 13, 256, leaves=256, objective="logistic"),
        # from raw floats to the packed matrix, once per data set: the largest dense table, and sparse rows
        _case("quantise_115m", "quantise", "tabular", 115_000_000, 13, 256),
        _case("quantise_csr_10m", "quantise_csr", "missing", 10_000_000, 50, 256, present=0.2),
        # scoring new rows with a finished model
        _case("predict_1m_100_trees", "predict", "normal", 1_000_000, 28, 256, depth=6, trees=100, objective="logistic"),
        # a caller with a growth loop of its own
        _case("steps_1m", "steps", "normal", 1_000_000, 28, 256, objective="logistic"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    kind = rng.choice(["round"] * 5 + ["tree", "sparse_round", "leafwise", "quantise", "quantise_csr", "predict", "steps"])
    c = _case("", kind, "normal", 0, 0, rng.choice([16, 64, 128, 255, 256, 256]), depth=rng.randint(3, 9),
              objective=rng.choice(["squared", "logistic"]))
    rows_lo, rows_hi, cols_lo, cols_hi, most = 5_000, 50_000_000, 4, 1000, 400_000_000
    if kind in ("round", "steps"):
        c["data"] = rng.choice(["normal", "tabular", "tabular", "missing", "wide"])
    elif kind == "tree":
        c["data"], rows_lo, rows_hi, cols_hi = rng.choice(["uniform", "normal"]), 1_000, 2_000_000, 60
    elif kind == "sparse_round":
        c["data"], cols_hi, most = "missing", 200, 300_000_000
    elif kind == "leafwise":
        c["data"], cols_hi = rng.choice(["normal", "tabular"]), 100
        c["leaves"] = rng.randint(15, 300)
    elif kind == "quantise":
        c["data"] = rng.choice(["normal", "tabular", "wide"])
    elif kind == "quantise_csr":
        c["data"], cols_hi = "missing", 500
    elif kind == "predict":
        rows_lo, rows_hi, cols_hi, c["trees"], most = 1_000, 5_000_000, 200, rng.randint(10, 200), 50_000_000
    if c["data"] == "wide":
        cols_lo, cols_hi, rows_hi = 50, 2000, 2_000_000
    if c["data"] == "tabular":
        cols_hi = min(cols_hi, 40)
    if c["data"] == "missing":
        cols_hi = min(cols_hi, 500)
        c["present"] = rng.uniform(0.05, 0.5)
    elif c["data"] == "normal" and kind in ("round", "leafwise", "quantise", "steps") and rng.random() < 0.4:
        c["present"] = rng.uniform(0.7, 0.99)
    c["cols"] = _log_int(rng, cols_lo, cols_hi)
    c["rows"] = min(_log_int(rng, rows_lo, rows_hi), most // c["cols"])
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------ inputs

def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _matrix(c, gen):
    """The raw float matrix [rows, cols]; missing elements are NaN."""
    n, F = c["rows"], c["cols"]
    if c["data"] == "uniform":
        X = torch.rand((n, F), device=DEV, generator=gen)
    elif c["data"] == "tabular":
        X = torch.empty((n, F), device=DEV)
        n_cat = (F * 8 + 12) // 13
        for j in range(F):
            if j < n_cat:   # an integer category with P(k) ~ k^-1.2
                K = 7 + (j * 97 + 41) % 294
                cdf = torch.cumsum(torch.arange(1, K + 1, device=DEV, dtype=torch.float64) ** -1.2, 0)
                cdf = (cdf / cdf[-1]).to(torch.float32)
                u = torch.rand(n, device=DEV, generator=gen)
                X[:, j] = (torch.bucketize(u, cdf, out_int32=True, right=True).clamp_(max=K - 1) + 1).to(torch.float32)
            else:
                X[:, j] = torch.empty(n, device=DEV).log_normal_(0.0, 2.0, generator=gen)
    elif c["data"] == "wide":
        X = torch.randn((n, F), device=DEV, generator=gen)
        for j in range(4, F, 5):
            X[:, j] *= 0.05
            X[:, j] += X[:, (7 * j) % (F - F % 5) // 5 * 5]
    elif c["data"] == "missing":
        X = torch.empty((n, F), device=DEV).log_normal_(0.0, 1.0, generator=gen)
    else:
        X = torch.randn((n, F), device=DEV, generator=gen)
    if c["present"] < 1.0:
        step = max(1, (1 << 26) // F)
        for r in range(0, n, step):
            block = X[r:r + step]
            block[torch.rand(block.shape, device=DEV, generator=gen) >= c["present"]] = float("nan")
    return X


def _labels(c, X, gen):
    """Labels that depend on a few of the columns: a linear part, one product, noise."""
    n, F = X.shape
    z = torch.zeros(n, device=DEV)
    cols = []
    for k in range(min(6, F)):
        x = torch.nan_to_num(X[:, (k * 5 + 1) % F], nan=-0.5)
        if c["data"] in ("tabular", "missing"):
            x = torch.log1p(x)
        x = (x - x.mean()) / (x.std() + 1e-6)
        cols.append(x)
        z += (0.9, -0.7, 0.6, 0.5, -0.4, 0.3)[k] * x
    z += 0.8 * cols[0] * cols[-1]
    if c["objective"] == "logistic":
        return (torch.rand(n, device=DEV, generator=gen) < torch.sigmoid(z)).to(torch.float32)
    return z + 0.1 * torch.randn(n, device=DEV, generator=gen)


def _csr(X):
    present = ~torch.isnan(X)
    indptr = torch.zeros(X.shape[0] + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(present.sum(dim=1), 0, out=indptr[1:])
    indices = present.nonzero()[:, 1].to(torch.int32)
    return indptr, indices, X[present]


def _params(c, depth=None):
    return g.make_params(max_depth=c["depth"] if depth is None else depth, max_bins=c["bins"], eta=0.1,
                         objective=c["objective"])


def _first_rounds(s, rounds):
    """Some rounds of boosting from margin 0: the model a later pass goes on from."""
    s["margin"] = torch.zeros(s["n"], device=DEV)
    s["gpair"] = torch.empty((s["n"], 2), device=DEV)
    return [s["ctx"].boost_round(s["packed"], s["bits"], s["n"], s["F"], s["missing_sym"], s["nb"], s["cuts"], s["label"],
                                 s["margin"], s["margin"], s["gpair"], s["params"]) for _ in range(rounds)]


def prepare(case, seed):
    c, gen, ctx = case, _generator(seed), g.Context(0)
    n, F = c["rows"], c["cols"]
    s = dict(case=c, ctx=ctx, n=n, F=F)
    if c["kind"] == "predict":   # new rows, and a model trained on others of their kind
        s["X"] = _matrix(c, gen)
        c = dict(c, rows=50_000)
        s.update(n=50_000)
    X = _matrix(c, gen)
    if c["kind"] == "quantise":
        return dict(s, X=X)
    if c["kind"] == "quantise_csr":
        return dict(s, csr=_csr(X))
    s["label"] = _labels(c, X, gen)
    s["params"] = _params(c)
    if c["kind"] == "sparse_round":
        csr = _csr(X)
        del X
        s["cuts"], s["nb"], sym, _, ms = ctx.quantise(csr=csr, max_bins=c["bins"], n=n, F=F)
        del csr
        s["rowptr"], s["ent"], s["nnz"] = ctx.compress_sparse(sym, c["bins"], ms)
        s["margin_in"] = torch.zeros(n, device=DEV)
        s["margin"] = torch.empty_like(s["margin_in"])
        s["gpair"] = torch.empty((n, 2), device=DEV)
        for _ in range(2):
            _sparse_round(s)
            s["margin_in"].copy_(s["margin"])
        return s
    s["cuts"], s["nb"], s["packed"], s["bits"], _, s["missing_sym"] = ctx.quantise_packed(X, max_bins=c["bins"])
    del X
    if c["kind"] == "tree":
        s["gpair"] = torch.stack([torch.randn(n, device=DEV, generator=gen),
                                  0.1 + 0.9 * torch.rand(n, device=DEV, generator=gen)], 1)
        return s
    trees = _first_rounds(s, c["trees"] if c["kind"] == "predict" else 2)
    if c["kind"] == "predict":
        return dict(case=case, ctx=ctx, X=s["X"], trees=trees, margin=torch.zeros(case["rows"], device=DEV))
    s["margin_in"] = s.pop("margin")
    s["margin"] = torch.empty_like(s["margin_in"])
    if c["kind"] == "leafwise":
        s["params"] = _params(c, depth=64)
    if c["kind"] == "steps":
        s["gpair"] = ctx.gradients(c["objective"], s["margin_in"], s["label"])
        s["rows"] = torch.empty(n, dtype=torch.int32, device=DEV)
    return s


# ------------------------------------------------------------------------------------------------ passes

def _sparse_round(s):
    c, ctx = s["case"], s["ctx"]
    ctx.gradients(c["objective"], s["margin_in"], s["label"], out=s["gpair"])
    tree, _, _ = ctx.grow_tree_sparse(s["rowptr"], s["ent"], s["n"], s["nnz"], s["F"], s["nb"], s["cuts"], s["gpair"],
                                      s["params"], want_leaf=False, want_rows=False)
    s["margin"].copy_(s["margin_in"])
    ctx.predict_sparse([tree], s["margin"], 0.1, s["rowptr"], s["ent"], s["n"], s["F"], c["bins"])
    return {"tree": tree, "margin": s["margin"], "gpair": s["gpair"]}


def _steps(s):
    c, ctx, n, F = s["case"], s["ctx"], s["n"], s["F"]
    packed, bits, ms, B, p = s["packed"], s["bits"], s["missing_sym"], c["bins"], s["params"]
    gq, scale = ctx.gpair_fixed(s["gpair"])
    G, H = ctx.sum_gpair(gq)
    root = ctx.build_hist(packed, bits, n, F, B, ms, gq)
    best = ctx.eval_split(root, s["nb"], G, H, scale, p)
    out = {"root": root, "split": best, "totals": (G, H)}
    if not best["valid"]:
        return out
    rows = torch.arange(n, dtype=torch.int32, device=DEV, out=s["rows"])
    n_left = ctx.partition(packed, bits, n, F, rows, 0, n, best["feature"], best["bin"], best["default_left"], ms)
    small_left = n_left <= n - n_left
    small = rows[:n_left] if small_left else rows[n_left:]
    built = ctx.build_hist(packed, bits, n, F, B, ms, gq, row_idx=small)
    other = ctx.hist_subtract(root, built)
    left, right = (built, other) if small_left else (other, built)
    out["left"] = ctx.eval_split(left, s["nb"], best["GLq"], best["HLq"], scale, p)
    out["right"] = ctx.eval_split(right, s["nb"], G - best["GLq"], H - best["HLq"], scale, p)
    out.update(rows=rows, n_left=n_left, built=built, other=other)
    return out


def run(state):
    s, c, ctx = state, state["case"], state["ctx"]
    kind = c["kind"]
    if kind == "quantise":
        cuts, nb, packed, bits, max_value, missing = ctx.quantise_packed(s["X"], max_bins=c["bins"])
        return {"cuts": cuts, "nb": nb, "packed": packed, "bits": bits, "max_value": max_value, "missing": missing}
    if kind == "quantise_csr":
        cuts, nb, packed, bits, max_value, missing = ctx.quantise_packed(csr=s["csr"], max_bins=c["bins"], n=s["n"], F=s["F"])
        return {"cuts": cuts, "nb": nb, "packed": packed, "bits": bits, "max_value": max_value, "missing": missing}
    if kind == "predict":
        s["margin"].zero_()
        return ctx.predict(s["trees"], s["margin"], 0.1, X=s["X"])
    if kind == "sparse_round":
        return _sparse_round(s)
    if kind == "steps":
        return _steps(s)
    if kind == "tree":
        tree, rows, leaf = ctx.grow_tree(s["packed"], s["bits"], s["n"], s["F"], s["missing_sym"], s["nb"], s["cuts"],
                                         s["gpair"], s["params"])
        return {"tree": tree, "rows": rows, "leaf": leaf}
    if kind == "leafwise":
        ctx.gradients(c["objective"], s["margin_in"], s["label"], out=s["gpair"])
        tree, _, _ = ctx.grow_tree_lossguide(s["packed"], s["bits"], s["n"], s["F"], s["missing_sym"], s["nb"], s["cuts"],
                                             s["gpair"], s["params"], c["leaves"], want_leaf=False, want_rows=False)
        s["margin"].copy_(s["margin_in"])
        ctx.predict([tree], s["margin"], 0.1, packed=s["packed"], bits=s["bits"], missing_sym=s["missing_sym"], n=s["n"],
                    F=s["F"])
        return {"tree": tree, "margin": s["margin"], "gpair": s["gpair"]}
    tree = ctx.boost_round(s["packed"], s["bits"], s["n"], s["F"], s["missing_sym"], s["nb"], s["cuts"], s["label"],
                           s["margin_in"], s["margin"], s["gpair"], s["params"])
    return {"tree": tree, "margin": s["margin"], "gpair": s["gpair"]}


def work(case):
    """Bytes: each input read once, each output written once.  Operations: two additions for every present element of
    the root's histogram (deeper levels add at most half as much each), or one comparison per row, tree and level."""
    c = case
    n, F, B = c["rows"], c["cols"], c["bins"]
    present = n * F * c["present"]
    bits = max(1, (B if c["present"] < 1.0 else B - 1).bit_length())
    packed = n * F * bits / 8
    if c["kind"] == "quantise":
        return {"bytes": 4.0 * n * F + packed, "flops": float(n * F)}
    if c["kind"] == "quantise_csr":
        return {"bytes": 8.0 * present + 8.0 * n + packed, "flops": present}
    if c["kind"] == "predict":
        return {"bytes": n * (4.0 * F + 8.0), "flops": float(n) * c["trees"] * (c["depth"] + 1)}
    if c["kind"] == "tree":
        return {"bytes": packed + n * (8.0 + 8.0), "flops": 2.0 * present}
    if c["kind"] == "steps":
        return {"bytes": packed + n * (8.0 + 8.0 + 4.0) + 3 * F * B * 16.0, "flops": 3.0 * present}
    if c["kind"] == "sparse_round":
        return {"bytes": present * (2 if F * B <= 65536 else 4) + n * (4.0 + 4.0 + 4.0 + 8.0 + 4.0), "flops": 2.0 * present}
    return {"bytes": packed + n * (4.0 + 4.0 + 8.0 + 4.0), "flops": 2.0 * present}


def tolerance(case):
    # sums of fixed-point integers in any order, fp64 gains of those sums, comparisons and copies: no result depends on
    # how the work is divided
    return "exact"
