"""Prediction with many trees on raw floats (Sec. 2.4: trees in order, one instance per thread) in the
form that reads the rows once and takes the trees through LDS in groups (-m gpu).  The oracle walks
one tree at a time over the same floats; margins must be bit-identical (fp32 rounding after every
tree on both sides), on new data as well as on the training matrix."""
import numpy as np
import pytest
import torch

from gpu_util import dev
from test_host_rules import SHARED

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1806_11248_amd as g
    c = g.Context(0)
    yield c
    c.close()


def _boost(ctx, X, y, B, rounds, depth, lossguide_every=0):
    """rounds trees grown on the GPU (each judged elsewhere); returns trees as numpy dicts."""
    import paper_1806_11248_amd as g
    n, F = X.shape
    cuts, nb, sym, mv, ms = ctx.quantise(dev(X), max_bins=B)
    packed, bits = ctx.compress(sym, mv)
    margin = torch.zeros(n, device="cuda")
    trees = []
    for r in range(rounds):
        d = 1 + (r * 3) % depth                      # trees of different depths inside one group
        params = g.make_params(max_depth=d, max_bins=B, lam=1.0, eta=0.3, objective="logistic")
        gp = ctx.gradients("logistic", margin, dev(y))
        if lossguide_every and r % lossguide_every == 1:
            big = g.make_params(max_depth=12, max_bins=B, lam=1.0, eta=0.3, objective="logistic")
            t, _, _ = ctx.grow_tree_lossguide(packed, bits, n, F, ms, nb, cuts, gp, big, 24, want_rows=False,
                                              want_leaf=False)
        else:
            t, _, _ = ctx.grow_tree(packed, bits, n, F, ms, nb, cuts, gp, params, want_rows=False, want_leaf=False)
        ctx.predict([t], margin, 0.3, packed=packed, bits=bits, missing_sym=ms, n=n, F=F)
        trees.append(t)
    return trees, margin.cpu().numpy()


@pytest.mark.parametrize("n,F,B,rounds,depth,miss", [
    (30_011, 28, 256, 45, 6, 0.0),      # three groups of trees (2048 nodes of LDS each)
    (9_000, 7, 64, 20, 5, 0.3),         # missing values, an odd number of features
    (5_003, 95, 32, 6, 4, 0.1),         # the widest row tile the kernel takes
    (300, 3, 16, 2, 3, 0.0),            # two trees, one partial tile
])
def test_many_trees_on_raw_floats(ctx, oracle, n, F, B, rounds, depth, miss):
    rng = np.random.default_rng(n + F)
    X = rng.standard_normal((n, F)).astype(np.float32)
    X[:, 0] = np.round(X[:, 0] * 3)
    if miss:
        X[rng.random((n, F)) < miss] = np.nan
    y = (rng.random(n) < 1 / (1 + np.exp(-(X[:, 0] + np.nan_to_num(X[:, 1]))))).astype(np.float32)
    print(f"batched predict n={n} F={F} trees={rounds}", flush=True)
    trees, boosted = _boost(ctx, X, y, B, rounds, depth, lossguide_every=4)
    # the training matrix: the margins the boosting loop accumulated tree by tree over packed symbols
    got = ctx.predict(trees, dev(np.zeros(n, np.float32)), 0.3, X=dev(X)).cpu().numpy()
    assert np.array_equal(got, boosted)
    # new rows, with infinities and values equal to thresholds, against the oracle's walk
    m = 4_099
    Z = rng.standard_normal((m, F)).astype(np.float32) * 2
    Z[rng.random((m, F)) < 0.15] = np.nan
    Z[rng.random((m, F)) < 0.02] = np.inf
    Z[rng.random((m, F)) < 0.02] = -np.inf
    thr = np.concatenate([t["threshold"][:t["n_nodes"]][t["feature"][:t["n_nodes"]] >= 0] for t in trees])
    thr = thr[np.isfinite(thr)]
    if len(thr):
        Z[np.arange(0, m, 7), 0] = thr[np.arange(0, m, 7) % len(thr)]     # x == threshold goes right
    start = rng.standard_normal(m).astype(np.float32)
    ref = start.copy()
    for t in trees:
        ref = oracle.predict_raw(t, Z, 0.3, ref)
    got = ctx.predict(trees, dev(start), 0.3, X=dev(Z)).cpu().numpy()
    assert np.array_equal(got, ref)
    # one tree at a time through the single-tree kernels gives the same
    step = dev(start)
    for t in trees:
        ctx.predict([t], step, 0.3, X=dev(Z))
    assert np.array_equal(step.cpu().numpy(), ref)


@pytest.mark.parametrize("F", [1, 4, 64, 65, 128, 129, 300])   # the widths at which the rows per tile change, and four-feature chunks with and without a remainder
@pytest.mark.parametrize("n", [1, 255, 1_027])
def test_row_tiles_of_every_width(ctx, oracle, n, F):
    rng = np.random.default_rng(17 * n + F)
    X = rng.standard_normal((3_000, F)).astype(np.float32)
    X[rng.random(X.shape) < 0.1] = np.nan
    X[:, -1] = np.where(rng.random(3_000) < 0.5, -0.0, np.round(rng.standard_normal(3_000)))   # a threshold of zero, either sign
    y = (np.nan_to_num(X[:, 0]) + X[:, -1] > 0).astype(np.float32)
    print(f"row tiles n={n} F={F}", flush=True)
    trees, _ = _boost(ctx, X, y, 32, 5, 6)
    Z = X[rng.permutation(3_000)[:n]].copy()
    Z[rng.random(Z.shape) < 0.05] = 0.0
    start = rng.standard_normal(n).astype(np.float32)
    ref = start.copy()
    for t in trees:
        ref = oracle.predict_raw(t, Z, 0.3, ref)
    got = ctx.predict(trees, dev(start), 0.3, X=dev(Z)).cpu().numpy()
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("n,F,rounds", [(30_001, 300, 2), (30_001, 300, 12), (5_000, 300, 2), (9_000, 500, 3), (300, 129, 9)])
def test_few_trees_on_wide_rows(ctx, oracle, n, F, rounds):
    """Wide rows take one pass over the rows or a kernel per tree, by rows, columns and trees: the same margins."""
    rng = np.random.default_rng(n + F + rounds)
    X = rng.standard_normal((3_000, F)).astype(np.float32)
    y = (X[:, 0] + X[:, -1] * X[:, F // 2] > 0).astype(np.float32)
    print(f"wide rows n={n} F={F} trees={rounds}", flush=True)
    trees, _ = _boost(ctx, X, y, 32, rounds, 4)
    Z = rng.standard_normal((n, F)).astype(np.float32)
    Z[rng.random(Z.shape) < 0.05] = np.nan
    start = rng.standard_normal(n).astype(np.float32)
    ref = start.copy()
    for t in trees:
        ref = oracle.predict_raw(t, Z, 0.3, ref)
    assert np.array_equal(ctx.predict(trees, dev(start), 0.3, X=dev(Z)).cpu().numpy(), ref)


def test_few_trees_on_wide_rows_cost_no_more_than_one_by_one(ctx):
    """Two shallow trees on 1M x 300: a pass that stages whole rows took 12 times what the two walks take."""
    import time
    gen = torch.Generator(device="cuda").manual_seed(1)
    X = torch.randn((1_000_000, 300), device="cuda", generator=gen)
    head = X[:3_000].cpu().numpy()
    trees, _ = _boost(ctx, head, (head[:, 0] + head[:, 299] * head[:, 150] > 0).astype(np.float32), 32, 2, 3)
    margin = torch.zeros(1_000_000, device="cuda")

    def fastest(groups):
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for g in groups:
                ctx.predict(g, margin, 0.3, X=X)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best
    print("wide rows, two trees", flush=True)
    together, single = fastest([trees]), fastest([[t] for t in trees])
    assert together < 2 * single, (together, single)


def _made_tree(rng, F, n_splits, numbering):
    """A tree of n_splits splits made by hand.  numbering: where the pairs of children stand, "dense" (odd left ids, as
    grown trees have them), "gap" (an unused node behind the root: even left ids) or "mixed" (unused nodes in between)."""
    import paper_1806_11248_amd as g
    cap = 2 * n_splits + 1 + (0 if numbering == "dense" else n_splits + 1)
    t = {k: np.zeros(cap, v.dtype) for k, v in g.new_tree(0).items() if isinstance(v, np.ndarray)}
    t["feature"][:] = -1
    t["left"][:] = t["right"][:] = -1
    t["threshold"][:] = np.inf
    t["weight"][:] = rng.normal(0, 1, cap)
    open_, at = [0], 1 if numbering == "dense" else 2
    for _ in range(n_splits):
        i = open_.pop(rng.integers(0, len(open_)))
        if numbering == "mixed":
            at += int(rng.integers(0, 2))
        t["feature"][i], t["left"][i], t["right"][i] = rng.integers(0, F), at, at + 1
        t["threshold"][i] = np.float32(rng.choice([rng.normal(), 0.0, -0.0, 1e30]))
        t["default_left"][i] = rng.integers(0, 2)
        open_ += [at, at + 1]
        at += 2
    # children have to come after their parents for the one-pass form: they do, pairs are handed out in order
    t["n_nodes"], t["capacity"] = at, cap
    return t


@pytest.mark.parametrize("numbering", ["dense", "gap", "mixed"])
@pytest.mark.parametrize("sizes", [[3, 1, 0, 2], [766, 767, 768], [700, 60, 6, 1], [100] * 16, [2500, 5, 2500]])
@pytest.mark.parametrize("miss", [0.0, 0.1])
def test_groups_of_trees_and_their_numbering(ctx, oracle, numbering, sizes, miss):
    """Groups that end at, before and behind the 1536 places they have, trees of one node, ids with gaps; tiles of rows with
    and without a missing value."""
    rng = np.random.default_rng(sum(sizes) + len(numbering))
    F, n = 9, 700
    trees = [_made_tree(rng, F, k, numbering) for k in sizes]
    print(f"groups sizes={sizes} {numbering} missing={miss}", flush=True)
    Z = rng.standard_normal((n, F)).astype(np.float32)
    Z[rng.random(Z.shape) < 0.02] = np.inf
    Z[rng.random(Z.shape) < 0.05] = 0.0
    if miss:
        Z[:300][rng.random((300, F)) < miss] = np.nan   # (the rows behind are tiles without a missing value)
    start = rng.standard_normal(n).astype(np.float32)
    ref = start.copy()
    for t in trees:
        ref = oracle.predict_raw(t, Z, 0.3, ref)
    got = ctx.predict(trees, dev(start), 0.3, X=dev(Z)).cpu().numpy()
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("F,bits", [(3, 5), (9, 8), (28, 8), (57, 8)])
@pytest.mark.parametrize("name", SHARED)
def test_splits_that_share_children(ctx, oracle, name, F, bits):
    """Two splits may lead to the same node: many trees and one, on raw floats, packed symbols and sparse rows."""
    import paper_1806_11248_amd as g
    splits, n_nodes = SHARED[name]
    rng = np.random.default_rng(len(name) + F)
    t = {k: np.zeros(n_nodes, v.dtype) for k, v in g.new_tree(0).items() if isinstance(v, np.ndarray)}
    t["feature"][:], t["left"][:], t["right"][:] = -1, -1, -1
    t["weight"][:] = rng.normal(0, 1, n_nodes)
    for i, (f, l, r) in splits.items():
        t["feature"][i], t["left"][i], t["right"][i], t["bin"][i] = f, l, r, rng.integers(5, 25)
        t["threshold"][i], t["default_left"][i] = t["bin"][i] + 1, rng.integers(0, 2)   # (the values below are symbols)
    t["n_nodes"] = t["capacity"] = n_nodes
    n, missing = 3_001, 30
    sym = rng.integers(0, 31, (n, F)).astype(np.uint16)
    Z = np.where(sym == missing, np.nan, sym).astype(np.float32)
    start = rng.standard_normal(n).astype(np.float32)
    print(f"shared children {name} F={F} bits={bits}", flush=True)
    trees = [t, _made_tree(rng, F, 5, "gap"), t]
    ref = start
    for q in trees:
        ref = oracle.predict_raw(q, Z, 0.3, ref)
    assert np.array_equal(ctx.predict(trees, dev(start), 0.3, X=dev(Z)).cpu().numpy(), ref)
    ref = oracle.predict_raw(t, Z, 0.3, start)
    assert np.array_equal(ref, oracle.predict_sym(t, sym, missing, 0.3, start))
    assert np.array_equal(ctx.predict([t], dev(start), 0.3, X=dev(Z)).cpu().numpy(), ref)
    packed = dev(oracle.pack(sym, bits).view(np.int32))
    got = ctx.predict([t], dev(start), 0.3, packed=packed, bits=bits, missing_sym=missing, n=n, F=F).cpu().numpy()
    assert np.array_equal(got, ref)
    rowptr, ent, _ = ctx.compress_sparse(dev(sym), 32, missing)
    assert np.array_equal(ctx.predict_sparse([t], dev(start), 0.3, rowptr, ent, n, F, 32).cpu().numpy(), ref)


MANY = 6 << 20   # rows from which on trees past 3072 nodes are walked from LDS where the rows' own reads are few


@pytest.mark.parametrize("splits", [1535, 1536, 2457, 2458, 2559, 2560])   # 3071, 3073, 4915, 4917, 5119, 5121 nodes
@pytest.mark.parametrize("n,F,bits", [(2_001, 13, 8), (2_001, 14, 9), (2_001, 28, 8), (2_001, 57, 8), (MANY - 1, 5, 8), (MANY, 5, 8)])
def test_trees_around_the_sizes_kept_in_lds(ctx, oracle, n, F, bits, splits):
    """One tree at the sizes and row counts where a walk keeps its nodes in LDS or leaves them in the caches."""
    rng = np.random.default_rng(splits + F)
    t = _made_tree(rng, F, splits, "dense")
    t["bin"][:] = rng.integers(60, 190, len(t["bin"]))
    missing = (1 << bits) - 1
    sym = rng.integers(0, missing + 1, (n, F), dtype=np.uint16)
    start = rng.standard_normal(n).astype(np.float32)
    print(f"tree sizes n={n} F={F} bits={bits} nodes={t['n_nodes']}", flush=True)
    ref = oracle.predict_sym(t, sym, missing, 0.3, start)
    packed = dev(oracle.pack(sym, bits).view(np.int32))
    got = ctx.predict([t], dev(start), 0.3, packed=packed, bits=bits, missing_sym=missing, n=n, F=F).cpu().numpy()
    assert np.array_equal(got, ref)
    if n < MANY - 1:
        rowptr, ent, _ = ctx.compress_sparse(dev(sym), missing, missing)
        assert np.array_equal(ctx.predict_sparse([t], dev(start), 0.3, rowptr, ent, n, F, missing).cpu().numpy(), ref)


@pytest.mark.parametrize("n", [MANY - 1, MANY])
def test_rows_counted_by_the_walk_of_a_large_tree(ctx, n):
    """A boosting round of depth 11 (4095 nodes at most): its last level's rows are counted in the margin's walk, from 6M rows of
    bytes on, else by a pass of their own; the growth on its own counts them with the partition."""
    import paper_1806_11248_amd as g
    F, B = 6, 255
    gen = torch.Generator("cuda").manual_seed(2)
    sym = torch.randint(0, B, (n, F), device="cuda", generator=gen, dtype=torch.int16)
    y = torch.randn(n, device="cuda", generator=gen) * 0.01
    for f in range(F):
        y += (1 + 0.3 * f) * sym[:, f].float() / B   # (smooth: nodes split near the middle, down to the last level)
    packed, bits = ctx.compress(sym.view(torch.uint16), B)
    assert bits == 8
    nb = torch.full((F,), B, dtype=torch.int32, device="cuda")
    cuts = torch.arange(1, B, device="cuda", dtype=torch.float32).repeat(F, 1)
    params = g.make_params(max_depth=11, max_bins=B, eta=0.3, objective="squared")
    print(f"rows counted by the walk n={n}", flush=True)
    m, out, gp = torch.zeros(n, device="cuda"), torch.empty(n, device="cuda"), torch.empty((n, 2), device="cuda")
    t = ctx.boost_round(packed, bits, n, F, B, nb, cuts, y, m, out, gp, params)
    bare, _, leaf = ctx.grow_tree(packed, bits, n, F, B, nb, cuts, gp, params, want_rows=False)
    nn = t["n_nodes"]
    assert nn > 3072 and bare["n_nodes"] == nn
    for k in ("feature", "bin", "left", "n_rows", "weight"):
        assert np.array_equal(t[k][:nn], bare[k][:nn]), k
    count = torch.bincount(leaf, minlength=nn).cpu().numpy()
    leaves = t["feature"][:nn] < 0
    assert np.array_equal(t["n_rows"][:nn][leaves], count[leaves])
    w = torch.from_numpy(0.3 * t["weight"][:nn]).cuda()
    assert torch.equal(out, (m.double() + w[leaf.long()]).float())


# rows, bytes a row, splits: both sides of the rows, widths and tree sizes at which gathering walks change their blocks
GATHERED = [(262_144, 130, 200), (262_145, 130, 200), (704 << 10, 129, 300), ((704 << 10) + 1, 129, 300), (3 << 20, 129, 400),
            ((3 << 20) + 1, 129, 511), ((3 << 20) + 1, 129, 512), ((3 << 20) + 1, 129, 1023), (400_000, 32, 200), (400_000, 33, 200),
            (4 << 20, 33, 200), ((4 << 20) - 1, 40, 200), (400_000, 41, 200)]


@pytest.mark.parametrize("n,F,splits", GATHERED)
def test_gathered_rows_of_every_block_form(ctx, n, F, splits):
    """Byte rows and one tree: margins against the same walk in torch."""
    rng = np.random.default_rng(n % 1000 + F)
    t = _made_tree(rng, F, splits, "dense")
    t["bin"][:] = rng.integers(60, 190, len(t["bin"]))
    print(f"gathered rows n={n} F={F} nodes={t['n_nodes']}", flush=True)
    gen = torch.Generator("cuda").manual_seed(F)
    flat = torch.randint(0, 256, (n * F + 64,), dtype=torch.uint8, device="cuda", generator=gen)
    packed = flat[:(flat.numel() // 4) * 4].view(torch.int32)
    sym = flat[:n * F].view(n, F)
    at = {k: torch.from_numpy(t[k].astype(np.int64)).cuda() for k in ("feature", "bin", "default_left", "left", "right")}
    node = torch.zeros(n, dtype=torch.int64, device="cuda")
    while True:
        f = at["feature"][node]
        if not bool((f >= 0).any()):
            break
        s = sym.gather(1, f.clamp(min=0)[:, None])[:, 0].long()
        left = torch.where(s == 255, at["default_left"][node] != 0, s <= at["bin"][node])
        node = torch.where(f < 0, node, torch.where(left, at["left"][node], at["right"][node]))
    start = torch.randn(n, device="cuda", generator=gen)
    weight = torch.from_numpy(t["weight"]).cuda()
    got = ctx.predict([t], start.clone(), 0.3, packed=packed, bits=8, missing_sym=255, n=n, F=F)
    assert torch.equal(got, (start.double() + 0.3 * weight[node]).float())
