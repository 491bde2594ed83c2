"""Ids partitioned in one launch, at every tile size, against the stable partition in three launches (-m gpu)."""
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def contexts():
    import paper_1806_11248_amd as g
    ours = g.Context(0)
    os.environ["GBT_TUNE_PLAN"] = "0"
    try:
        host = g.Context(0)
    finally:
        del os.environ["GBT_TUNE_PLAN"]
    yield ours, host
    ours.close()
    host.close()


@pytest.mark.parametrize("n,F,B,miss,depth", [
    (131_071, 50, 256, 0.7, 6),    # tiles of 256 rows, 9 bits
    (131_072, 33, 256, 0.0, 5),    # 512, bytes: symbols that end a word
    (262_145, 64, 16, 0.0, 7),     # rows of eight words, which are moved
    (262_145, 65, 16, 0.0, 7),     # 1024, one row in the last
    (524_287, 40, 64, 0.3, 4),     # 1024, one row short of the next size
    (524_289, 40, 64, 0.3, 8),     # 2048, children that need not fill one
    (1_000_003, 50, 512, 0.5, 3),  # 2048, 10 bits across words
])
def test_ids(contexts, n, F, B, miss, depth):
    import paper_1806_11248_amd as g
    print(f"partition ids n={n} F={F} B={B} missing={miss} depth={depth}", flush=True)
    gen = torch.Generator("cuda").manual_seed(n)
    X = torch.randn((n, F), device="cuda", generator=gen)
    if miss:
        X[torch.rand((n, F), device="cuda", generator=gen) < miss] = float("nan")
    params = g.make_params(max_depth=depth, max_bins=B, eta=0.3, objective="squared")
    cuts, nb, packed, bits, _, ms = contexts[0].quantise_packed(X, max_bins=B)
    # rows of more than eight words are listed by id (path 3), with the levels planned on the device and, for comparison, on the host
    if F * bits > 8 * 32:
        assert [c.grow_tree_form(n, F, bits, B, depth, track_rows=False) for c in contexts] == [(3, True), (3, False)]
    gp = torch.stack([torch.randn(n, device="cuda", generator=gen) + torch.nan_to_num(X[:, F - 1], nan=1.0),
                      0.5 + torch.rand(n, device="cuda", generator=gen)], 1)
    (a, _, leaf), (b, _, leaf_host) = (c.grow_tree(packed, bits, n, F, ms, nb, cuts, gp, params, want_rows=False) for c in contexts)
    assert a["n_nodes"] == b["n_nodes"] > 4
    for k in ("feature", "bin", "default_left", "left", "right", "threshold", "weight", "gain", "sumG", "sumH", "n_rows"):
        assert np.array_equal(a[k][:a["n_nodes"]], b[k][:b["n_nodes"]]), k
    assert torch.equal(leaf, leaf_host)
