"""The reductions over all rows (bounds of the pairs, totals of the fixed-point pairs) leave one partial result per
workgroup: row counts around a workgroup's share, one workgroup, all of them, and pairs that start on 8 bytes (-m gpu)."""
import numpy as np
import pytest
import torch

import grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1806_11248_amd as g
    c = g.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n", [1, 2, 63, 1023, 4097, 8191, 8193, 100_001, 512 * 1024 * 4 + 3, 512 * 1024 * 8 + 1])
@pytest.mark.parametrize("shift", [0, 1])
def test_totals_and_scales(ctx, n, shift):
    print(f"reductions n={n} shift={shift}", flush=True)
    rng = np.random.default_rng(n + shift)
    gp = np.stack([rng.normal(0, 3, n), rng.uniform(0.01, 1.0, n)], 1).astype(np.float32)
    at = rng.integers(0, n)   # the extremes anywhere: every row has to be looked at
    gp[at] = (-50.0, 7.0)
    buf = torch.empty((n + 1, 2), dtype=torch.float32, device="cuda")
    pairs = buf[shift:shift + n]
    pairs.copy_(torch.from_numpy(gp))
    gq, scale = ctx.gpair_fixed(pairs)
    q, want_scale = grid.fixed_point(gp)
    assert tuple(scale) == tuple(want_scale)
    assert np.array_equal(gq.cpu().numpy(), q)
    total = q.astype(np.int64).sum(0)
    assert ctx.sum_gpair(gq) == (int(total[0]), int(total[1]))
    rows = torch.from_numpy(rng.integers(0, n, min(n, 5000)).astype(np.int32)).cuda()
    part = q[rows.cpu().numpy()].astype(np.int64).sum(0)
    assert ctx.sum_gpair(gq, rows) == (int(part[0]), int(part[1]))


@pytest.mark.parametrize("objective", ["squared", "logistic"])
@pytest.mark.parametrize("n", [1, 4095, 4097, 512 * 1024 * 4 + 5])
def test_bounds_left_by_the_gradients(ctx, objective, n):
    """A round's tree follows from scales that the gradient kernel's bounds give: its root totals are the pairs' own."""
    import paper_1806_11248_amd as g
    print(f"bounds n={n} {objective}", flush=True)
    gen = torch.Generator("cuda").manual_seed(n)
    X = torch.randn((n, 3), device="cuda", generator=gen)
    y = (torch.rand(n, device="cuda", generator=gen) < 0.5).float()
    margin = torch.randn(n, device="cuda", generator=gen)
    cuts, nb, packed, bits, _, ms = ctx.quantise_packed(X, max_bins=16)
    params = g.make_params(max_depth=1, max_bins=16, objective=objective)
    gpair = torch.empty((n, 2), device="cuda")
    tree = ctx.boost_round(packed, bits, n, 3, ms, nb, cuts, y, margin, margin.clone(), gpair, params)
    gq, scale = ctx.gpair_fixed(gpair)
    G, H = ctx.sum_gpair(gq)
    assert tree["sumG"][0] == G / scale[0] and tree["sumH"][0] == H / scale[1]
