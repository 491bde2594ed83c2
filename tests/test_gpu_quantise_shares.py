"""Selection over columns of unequal work, shared out among the workgroups, against the library's sort, bit for bit (-m gpu)."""
import os

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctxs():
    import paper_1806_11248_amd as g
    sel = g.Context(0)
    os.environ["GBT_TUNE_QUANTISE_SORT"] = "1"
    try:
        srt = g.Context(0)
    finally:
        del os.environ["GBT_TUNE_QUANTISE_SORT"]
    yield sel, srt
    sel.close()
    srt.close()


# n numbers, c categories (no keys collected), d dates (sorted: no work in either kernel), m missing throughout; categories with one
# frequent key, counted by itself: h alone in its cell, x beside its neighbours among the floats, v an eighth of the column
@pytest.mark.parametrize("n,F,kinds", [
    (600_000, 32, "n"),
    (600_011, 32, "c"),              # nothing to collect
    (600_011, 32, "ncccccc"),
    (400_000, 67, "dcm" + 30 * "c" + "n" + 33 * "c"),   # one column of numbers, behind a word of the others
    (400_000, 67, "n" + 65 * "m" + "n"),
    (300_007, 64, "dnd"),
    (120_000, 200, 65 * "c" + "n" + 133 * "d" + "n"),
    (130_000, 128, "mndc"),          # fewer tiles than eight a workgroup on a large device
    (600_011, 32, "hxvn"),
    (5_001, 6, "hxv"),
    (40_000, 1024, 1023 * "c" + "n"),
    (40_000, 1025, 1000 * "c" + 25 * "n"),   # more columns than threads
])
def test_shares(ctxs, n, F, kinds):
    print(f"shares n={n} F={F} kinds={kinds[:8]}", flush=True)
    gen = torch.Generator("cuda").manual_seed(n + F)
    kinds = (kinds * F)[:F]
    X = torch.randn((n, F), device="cuda", generator=gen)
    for f, k in enumerate(kinds):
        if k == "c":
            X[:, f] = torch.floor(3 * X[:, f].abs())
        elif k == "d":
            X[:, f] = 20_150_000 + torch.floor(400 * X[:, f])
        elif k == "h":
            X[:, f] = torch.where(X[:, f] < 1.3, 0.0, torch.floor(30 * X[:, f]))
        elif k == "x":
            X[:, f] = 1.0 + torch.floor(3 * X[:, f].abs()) * 2.0 ** -23
            X[n // 5: n // 4, f] = float("nan")
        elif k == "v":
            X[:, f] = torch.floor(8 * torch.rand(n, device="cuda", generator=gen))
        elif k == "m":
            X[:, f] = float("nan")
    a, b = (c.quantise_packed(X, max_bins=64) for c in ctxs)
    assert all(torch.equal(x, y) if isinstance(x, torch.Tensor) else x == y for x, y in zip(a, b))
