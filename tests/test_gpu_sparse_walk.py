"""Prediction over sparse rows of 16-bit entries against the packed walk, bit for bit (-m gpu).  Row lengths sit at the edges
of what a wave keeps in registers (8, 16, 24, 32, 48, ... 256 entries from the row's first word, rows at odd places included), past
it, and at none; id ranges end at 65536; trees are leaves only, shallow, and of more nodes than a workgroup's threads."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# rows, columns, bins, row lengths to draw from, depth
CASES = [
    (1, 4, 16, (0,), 2),
    (63, 4, 16, (0, 1, 2, 3, 4), 3),
    (1_000, 40, 256, (0, 1, 7, 8, 9), 4),
    (5_003, 60, 256, (15, 16, 17, 1), 6),
    (5_003, 60, 256, (23, 24, 25, 0), 6),
    (5_003, 90, 256, (31, 32, 33, 2), 6),
    (5_003, 63, 256, (46, 47, 48, 49, 63), 7),
    (5_003, 127, 256, (64, 65, 95, 96, 97, 127), 7),
    (5_003, 255, 256, (127, 128, 129, 191, 192, 193, 255), 8),
    (20_011, 256, 256, (3, 12, 47, 200, 256), 9),   # ids up to 65535
    (4_000, 16, 4095, (1, 5, 16), 5),
    (2_001, 400, 100, (255, 256, 257, 2, 400), 6),  # rows past the registers
]


@pytest.mark.parametrize("n,F,B,lengths,depth", CASES)
def test_sparse_walk_equals_packed_walk(n, F, B, lengths, depth):
    import paper_1806_11248_amd as g
    print(f"sparse walk n={n} F={F} B={B} lengths={lengths} depth={depth}", flush=True)
    gen = np.random.default_rng(n + F)
    missing = B
    sym = np.full((n, F), missing, np.uint16)
    for r in range(n):
        cols = gen.permutation(F)[:lengths[int(gen.integers(len(lengths)))]]
        sym[r, cols] = gen.integers(0, B, len(cols))
    if n > 10:
        sym[1, F - 1] = B - 1   # the largest id
        sym[2, 0] = 0           # the smallest
    ctx = g.Context(0)
    try:
        sym_d = torch.from_numpy(sym).cuda()
        packed, bits = ctx.compress(sym_d, missing)
        rowptr, ent, nnz = ctx.compress_sparse(sym_d, B, missing)
        assert ent.element_size() == 2
        cuts = torch.arange(B - 1, device="cuda", dtype=torch.float32).repeat(F, 1).contiguous()
        nb = torch.full((F,), B, dtype=torch.int32, device="cuda")
        margin = torch.zeros(n, device="cuda")
        y = torch.from_numpy(gen.normal(0, 1, n).astype(np.float32)).cuda()
        params = g.make_params(max_depth=depth, max_bins=B, min_child_weight=1.0)
        trees = []
        for k in range(3):
            gp = ctx.gradients("squared", margin, y)
            tree, _, leaf = ctx.grow_tree(packed, bits, n, F, missing, nb, cuts, gp, params)
            sp_tree, _, sp_leaf = ctx.grow_tree_sparse(rowptr, ent, n, nnz, F, nb, cuts, gp, params)
            assert sp_tree["n_nodes"] == tree["n_nodes"] and torch.equal(leaf, sp_leaf), k
            trees.append(tree)
            before = margin.clone()
            ctx.predict([tree], margin, 0.3, packed=packed, bits=bits, missing_sym=missing, n=n, F=F)
            ctx.predict_sparse([tree], before, 0.3, rowptr, ent, n, F, B)
            torch.cuda.synchronize()
            assert torch.equal(before, margin), k
        together = torch.zeros(n, device="cuda")
        ctx.predict_sparse(trees, together, 0.3, rowptr, ent, n, F, B)
        torch.cuda.synchronize()
        assert torch.equal(together, margin)
    finally:
        ctx.close()


# rows, columns, bins, share present, depth: both sides of the numbers of rows and of entries at which the walk bisects staged
# rows instead of keeping them in registers (more than 262,144 rows; 40 + 40 per level entries a row; 1,572,864 rows)
LONG = [
    (262_144, 100, 128, 0.95, 1),
    (262_145, 100, 128, 0.95, 1),
    (262_145, 100, 128, 0.5, 1),
    (300_001, 130, 128, 0.95, 2),    # 123 entries, from 120 on
    (300_001, 130, 128, 0.9, 2),     # 117
    (280_000, 300, 200, 0.99, 6),    # past the registers
    (1_572_864, 96, 64, 0.98, 1),
    (1_572_865, 96, 64, 0.98, 1),
]


@pytest.mark.parametrize("n,F,B,present,depth", LONG)
def test_walks_of_long_rows(n, F, B, present, depth):
    import paper_1806_11248_amd as g
    print(f"long sparse rows n={n} F={F} B={B} present={present} depth={depth}", flush=True)
    gen = torch.Generator("cuda").manual_seed(n + F)
    sym = torch.empty((n, F), dtype=torch.uint16, device="cuda")
    for a in range(0, n, 200_000):
        m = min(200_000, n - a)
        s = torch.randint(0, B, (m, F), device="cuda", generator=gen)
        s[torch.rand((m, F), device="cuda", generator=gen) >= present] = B
        sym[a:a + m] = s.to(torch.uint16)
    ctx = g.Context(0)
    try:
        packed, bits = ctx.compress(sym, B)
        rowptr, ent, nnz = ctx.compress_sparse(sym, B, B)
        assert ent.element_size() == 2
        cuts = torch.arange(B - 1, device="cuda", dtype=torch.float32).repeat(F, 1).contiguous()
        nb = torch.full((F,), B, dtype=torch.int32, device="cuda")
        y = torch.randn(n, device="cuda", generator=gen)
        margin = torch.randn(n, device="cuda", generator=gen)
        params = g.make_params(max_depth=depth, max_bins=B)
        gp = ctx.gradients("squared", margin, y)
        tree, _, leaf = ctx.grow_tree(packed, bits, n, F, B, nb, cuts, gp, params, want_rows=False)
        sp_tree, _, sp_leaf = ctx.grow_tree_sparse(rowptr, ent, n, nnz, F, nb, cuts, gp, params, want_rows=False)
        assert sp_tree["n_nodes"] == tree["n_nodes"] > 1 and torch.equal(leaf, sp_leaf)
        sparse = margin.clone()
        for _ in range(2):
            ctx.predict([tree], margin, 0.3, packed=packed, bits=bits, missing_sym=B, n=n, F=F)
        ctx.predict_sparse([tree, tree], sparse, 0.3, rowptr, ent, n, F, B)
        torch.cuda.synchronize()
        assert torch.equal(sparse, margin)
    finally:
        ctx.close()
