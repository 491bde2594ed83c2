"""The partition of sparse rows at every tile size, against growth over the packed matrix (-m gpu)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1806_11248_amd as g
    c = g.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n,F,B,present", [
    (262_145, 20, 256, 0.3),     # tiles of 1024 rows, one row in the last
    (262_999, 50, 64, 0.35),     # 512: 17 entries a row
    (131_073, 60, 256, 0.5),     # 256: 30 entries
    (66_001, 200, 256, 0.4),     # 128: 80 entries
    (40_001, 250, 250, 0.8),     # rows that do not fit 128 at a time
    (70_001, 300, 256, 0.1),     # ids of 32 bits
    (1_025, 30, 256, 0.3),       # few rows: the shortest tiles
])
def test_tiles(ctx, n, F, B, present):
    import paper_1806_11248_amd as g
    print(f"sparse tiles n={n} F={F} B={B} present={present}", flush=True)
    gen = torch.Generator("cuda").manual_seed(n)
    X = torch.randn((n, F), device="cuda", generator=gen)
    X[torch.rand((n, F), device="cuda", generator=gen) >= present] = float("nan")
    X[: n // 3, F // 2:] = float("nan")          # rows of unequal length, and tiles of such rows
    params = g.make_params(max_depth=5, max_bins=B, eta=0.3, objective="squared")
    cuts, nb, sym, _, ms = ctx.quantise(X, max_bins=B)
    packed, bits = ctx.compress(sym, ms)
    rowptr, ent, nnz = ctx.compress_sparse(sym, B, ms)
    gp = torch.stack([torch.randn(n, device="cuda", generator=gen) + torch.nan_to_num(X[:, 0], nan=1.0),
                      0.5 + torch.rand(n, device="cuda", generator=gen)], 1)
    a = ctx.grow_tree_sparse(rowptr, ent, n, nnz, F, nb, cuts, gp, params)
    b = ctx.grow_tree(packed, bits, n, F, ms, nb, cuts, gp, params)
    assert a[0]["n_nodes"] == b[0]["n_nodes"] > 8
    for k in ("feature", "bin", "default_left", "left", "right", "threshold", "weight", "gain", "sumG", "sumH", "n_rows"):
        assert np.array_equal(a[0][k][:a[0]["n_nodes"]], b[0][k][:b[0]["n_nodes"]]), k
    assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
