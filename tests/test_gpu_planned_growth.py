"""Depth-wise growth planned on the device (one wait per tree) against the same growth planned on the host: every array of
the tree, the margins, each row's leaf and the row order have to be the same (-m gpu).  The shapes sit where the planned
form can go wrong: trees that end early or never split, levels past the depth from which the host waits for a level's
splits, more nodes than one workgroup's prefix sum takes in a step, one row, trees walked from LDS and not."""
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TREE_KEYS = ("feature", "bin", "default_left", "left", "right", "n_rows", "threshold", "weight", "gain", "sumG", "sumH")


def _context(**env):
    import paper_1806_11248_amd as g
    old = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        return g.Context(0)
    finally:
        for k, v in old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v


@pytest.fixture(scope="module")
def contexts():
    pair = _context(GBT_TUNE_PLAN="1"), _context(GBT_TUNE_PLAN="0")
    yield pair
    for c in pair:
        c.close()


# rows, columns, bins, missing share, depth, labels
CASES = [
    (10_000, 8, 16, 0.0, 3, "noise"),       # rows of one word
    (1, 19, 256, 0.0, 4, "noise"),          # one row: no split
    (63, 19, 256, 0.3, 6, "noise"),         # less than a wave
    (4_097, 20, 200, 0.0, 1, "noise"),      # byte symbols; the root's children are the last level
    (30_011, 28, 256, 0.0, 6, "noise"),     # byte symbols, rows that are moved
    (30_011, 28, 256, 0.0, 6, "constant"),  # nothing to gain after the first rounding: the tree ends at once
    (20_000, 19, 256, 0.2, 9, "step"),      # 9 bits; ends after one level of nine
    (50_021, 19, 256, 0.1, 10, "noise"),    # the deepest tree walked without a wait
    (60_000, 20, 64, 0.0, 12, "noise"),     # deeper: levels of more than 1024 nodes
    (3_001, 50, 256, 0.8, 8, "noise"),      # rows that stay in place, ids partitioned
    (5_000, 200, 64, 0.1, 5, "noise"),      # the same, wide
    (20_000, 60, 128, 0.5, 11, "noise"),    # ... and deep
]


def _data(n, F, miss, labels):
    gen = np.random.default_rng(11 * n + F)
    X = gen.normal(0, 1, (n, F)).astype(np.float32)
    if miss > 0:
        X[gen.random(X.shape) < miss] = np.nan
    if labels == "constant":
        y = np.ones(n, np.float32)
    elif labels == "step":
        y = np.where(np.nan_to_num(X[:, 3], nan=-1.0) > 0, 3.0, -1.0).astype(np.float32)
    else:
        y = (np.nan_to_num(X[:, 0]) * 0.7 + gen.normal(0, 1, n)).astype(np.float32)
    return torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()


def _same_tree(a, b, what):
    assert a["n_nodes"] == b["n_nodes"], what
    for k in TREE_KEYS:
        assert np.array_equal(a[k][:a["n_nodes"]], b[k][:b["n_nodes"]]), (what, k)


@pytest.mark.parametrize("n,F,B,miss,depth,labels", CASES)
def test_planned_growth_equals_growth_planned_on_the_host(contexts, n, F, B, miss, depth, labels):
    import paper_1806_11248_amd as g
    print(f"planned growth n={n} F={F} B={B} missing={miss} depth={depth} labels={labels}", flush=True)
    X, y = _data(n, F, miss, labels)
    params = g.make_params(max_depth=depth, max_bins=B, eta=0.3, objective="squared", min_child_weight=1.0)
    cuts, nb, packed, bits, _, ms = contexts[0].quantise_packed(X, max_bins=B)
    margin0 = torch.full((n,), 0.25, device="cuda")
    gp = contexts[0].gradients("squared", margin0, y)
    gp[:, 1] += torch.rand(n, device="cuda", generator=torch.Generator("cuda").manual_seed(1))   # (pairs of unequal h)
    seen = []
    for c in contexts:
        rounds = []
        margin = margin0.clone()
        for _ in range(2):   # the second round's pairs follow from the first's tree
            gpair = torch.empty((n, 2), device="cuda")
            rounds.append(c.boost_round(packed, bits, n, F, ms, nb, cuts, y, margin, margin, gpair, params))
        full = c.grow_tree(packed, bits, n, F, ms, nb, cuts, gp, params)
        leaf_only = c.grow_tree(packed, bits, n, F, ms, nb, cuts, gp, params, want_rows=False)
        bare = c.grow_tree(packed, bits, n, F, ms, nb, cuts, gp, params, want_rows=False, want_leaf=False)
        torch.cuda.synchronize()
        seen.append((rounds, margin, full, leaf_only, bare))
    (ra, ma, fa, la, ba), (rb, mb, fb, lb, bb) = seen
    for k in range(2):
        _same_tree(ra[k], rb[k], f"round {k}")
    assert torch.equal(ma, mb)
    for what, a, b in (("full", fa, fb), ("leaf", la, lb), ("bare", ba, bb)):
        _same_tree(a[0], b[0], what)
        for k in (1, 2):
            assert (a[k] is None) == (b[k] is None) and (a[k] is None or torch.equal(a[k], b[k])), (what, k)


@pytest.mark.parametrize("n,F,B,miss,depth,labels", [c for c in CASES if c[3] > 0])
def test_planned_sparse_growth_equals_growth_planned_on_the_host(contexts, n, F, B, miss, depth, labels):
    import paper_1806_11248_amd as g
    print(f"planned sparse growth n={n} F={F} B={B} missing={miss} depth={depth} labels={labels}", flush=True)
    X, y = _data(n, F, miss, labels)
    params = g.make_params(max_depth=depth, max_bins=B, eta=0.3, objective="squared")
    cuts, nb, sym, _, ms = contexts[0].quantise(X, max_bins=B)
    rowptr, ent, nnz = contexts[0].compress_sparse(sym, B, ms)
    gp = contexts[0].gradients("squared", torch.zeros(n, device="cuda"), y)
    seen = []
    for c in contexts:
        seen.append((c.grow_tree_sparse(rowptr, ent, n, nnz, F, nb, cuts, gp, params),
                     c.grow_tree_sparse(rowptr, ent, n, nnz, F, nb, cuts, gp, params, want_leaf=False, want_rows=False)))
        torch.cuda.synchronize()
    for a, b in zip(*seen):
        _same_tree(a[0], b[0], "sparse")
        for k in (1, 2):
            assert (a[k] is None) == (b[k] is None) and (a[k] is None or torch.equal(a[k], b[k])), k


# Byte symbols of at most 16 features: few rows are planned on the device and moved (path 1), many take the passes that
# partition and build histograms at once, which the host plans (path 2, here for every size with GBT_TUNE_PLAN=0).
FEW = [
    (50, 13, 256, 0.0, 4, "noise"),
    (4_095, 4, 256, 0.0, 6, "noise"),
    (20_011, 13, 256, 0.0, 8, "noise"),
    (70_001, 16, 255, 0.1, 7, "noise"),
    (150_001, 13, 256, 0.0, 9, "noise"),
    (9_000, 5, 250, 0.0, 11, "noise"),
]


@pytest.mark.parametrize("env", [{}, {"GBT_TUNE_PART_NOMOVE": "0"}, {"GBT_TUNE_PART_NOMOVE": "1"}, {"GBT_TUNE_PART_CYCLE": "0"},
                                 {"GBT_TUNE_HIST8": "0"}])
def test_few_rows_of_bytes_equal_the_fused_passes(contexts, env):
    import paper_1806_11248_amd as g
    other = _context(GBT_TUNE_PLAN="0", **env)
    try:
        for n, F, B, miss, depth, labels in FEW:
            print(f"few rows of bytes n={n} F={F} B={B} missing={miss} depth={depth} {env}", flush=True)
            X, y = _data(n, F, miss, labels)
            params = g.make_params(max_depth=depth, max_bins=B, eta=0.3, objective="logistic")
            y = (y > 0).float()
            cuts, nb, packed, bits, _, ms = other.quantise_packed(X, max_bins=B)
            if n > 1000:
                assert bits == 8
            seen = []
            for c in (contexts[0], other):
                margin, trees = torch.zeros(n, device="cuda"), []
                for _ in range(2):
                    gpair = torch.empty((n, 2), device="cuda")
                    trees.append(c.boost_round(packed, bits, n, F, ms, nb, cuts, y, margin, margin, gpair, params))
                full = c.grow_tree(packed, bits, n, F, ms, nb, cuts, gpair, params)
                torch.cuda.synchronize()
                seen.append((trees, margin, full))
            (ta, ma, fa), (tb, mb, fb) = seen
            for k in range(2):
                _same_tree(ta[k], tb[k], k)
            _same_tree(fa[0], fb[0], "full")
            assert torch.equal(ma, mb) and torch.equal(fa[1], fb[1]) and torch.equal(fa[2], fb[2])
    finally:
        other.close()


@pytest.mark.parametrize("n,form", [((1 << 22) - 1, (1, True)), (1 << 22, (2, False))])
def test_both_sides_of_the_rows_at_which_bytes_take_the_fused_passes(contexts, n, form):
    import paper_1806_11248_amd as g
    F, B, depth = 5, 256, 6
    print(f"fused passes from 2^22 rows on, n={n}", flush=True)
    planned, host = contexts
    assert planned.grow_tree_form(n, F, 8, B, depth) == form and host.grow_tree_form(n, F, 8, B, depth) == (2, False)
    X, y = _data(n, F, 0.0, "noise")
    params = g.make_params(max_depth=depth, max_bins=B, eta=0.3, objective="squared")
    cuts, nb, packed, bits, _, ms = planned.quantise_packed(X, max_bins=B)
    assert bits == 8
    del X
    seen = []
    for c in contexts:
        margin, gpair = torch.zeros(n, device="cuda"), torch.empty((n, 2), device="cuda")
        tree = c.boost_round(packed, bits, n, F, ms, nb, cuts, y, margin, margin, gpair, params)
        full = c.grow_tree(packed, bits, n, F, ms, nb, cuts, gpair, params)
        torch.cuda.synchronize()
        seen.append((tree, margin, full))
    (ta, ma, fa), (tb, mb, fb) = seen
    _same_tree(ta, tb, "round")
    _same_tree(fa[0], fb[0], "full")
    assert torch.equal(ma, mb) and torch.equal(fa[1], fb[1]) and torch.equal(fa[2], fb[2])


def test_form_of_a_growth(contexts):
    """Which form a shape takes, at the edges of the rules."""
    planned, host = contexts
    assert planned.grow_tree_form(10_000, 28, 8, 256, 6) == (1, True) and host.grow_tree_form(10_000, 28, 8, 256, 6) == (1, False)
    assert planned.grow_tree_form(10_000, 50, 9, 256, 6) == (3, True) and host.grow_tree_form(10_000, 50, 9, 256, 6) == (3, False)
    assert planned.grow_tree_form(10_000, 13, 8, 256, 0) == (2, False)    # a single leaf
    assert planned.grow_tree_form(10_000, 13, 8, 256, 15) == (1, True)
    assert planned.grow_tree_form(10_000, 13, 8, 256, 16) == (2, False)   # more nodes than the read-back buffer holds
    for c in contexts:
        for bad in (dict(n=0), dict(F=0), dict(bits=17), dict(max_bins=1), dict(max_depth=17), dict(max_depth=-1)):
            with pytest.raises(Exception):
                c.grow_tree_form(**{**dict(n=100, F=4, bits=8, max_bins=16, max_depth=3), **bad})
