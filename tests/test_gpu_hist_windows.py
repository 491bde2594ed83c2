"""Histograms of every symbol width at the edges of the register windows, against sums of the same integers (-m gpu)."""
import numpy as np
import pytest
import torch

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1806_11248_amd as g
    c = g.Context(0)
    yield c
    c.close()


def _window(bits):   # whole symbols in sixteen bytes that start at the first one's byte
    first = 0 if bits % 8 == 0 else 4 if bits % 4 == 0 else 6 if bits % 2 == 0 else 7
    return min(32, (128 - first) // bits)


def _reference(sym, gq, B, missing, rows):
    n, F = sym.shape
    out = np.zeros((F, B, 2), np.int64)
    rows = rows[rows < n]
    for f in range(F):
        s = sym[rows, f].astype(np.int64)
        live = (s < B) & (s != missing)
        np.add.at(out[f, :, 0], s[live], gq[rows[live], 0].astype(np.int64))
        np.add.at(out[f, :, 1], s[live], gq[rows[live], 1].astype(np.int64))
    return out


@pytest.mark.parametrize("bits", range(1, 17))
@pytest.mark.parametrize("columns", ["one", "under", "window", "over", "two", "over_two", "four", "over_four"])
def test_windows(ctx, oracle, bits, columns):
    """Tiles of one, two and four windows and one column more or less; tables with a row for every symbol and with one for what is
    no bin; a missing symbol among the bins and behind them; matrices down to less than sixteen bytes, whose first and last
    rows end at the buffer's edges; row lists in any order with ids that name no row."""
    E = _window(bits)
    F = {"one": 1, "under": E - 1, "window": E, "over": E + 1, "two": 2 * E, "over_two": 2 * E + 3, "four": 4 * E,
         "over_four": 4 * E + 1}[columns]
    rng = np.random.default_rng(1000 * bits + F)
    for n, B, missing in ((1, 1 << bits, 1 << bits), (3, max(2, (1 << bits) - 1), 0), (1037, 1 << bits, 1 << bits),
                          (2500, max(2, (2 << bits) // 3), 1), (700, max(2, 1 << (bits - 1)), (1 << bits) - 1)):
        B = min(B, 4096)
        if B < 2:
            continue
        sym = rng.integers(0, 1 << bits, (n, F)).astype(np.uint16)
        sym[rng.random((n, F)) < 0.3] = min(B - 1, 1)
        gq = np.stack([rng.integers(-(1 << 26), (1 << 26) + 1, n), rng.integers(0, (1 << 22) + 1, n)], 1).astype(np.int32)
        gq[rng.random(n) < 0.5] = (1 << 26, 1 << 22)      # sums that pass the fields' ends
        packed = dev(oracle.pack(sym, bits).view(np.int32))
        print(f"bits={bits} n={n} F={F} B={B} missing={missing}", flush=True)
        got = ctx.build_hist(packed, bits, n, F, B, missing, dev(gq)).cpu().numpy().reshape(F, B, 2)
        assert np.array_equal(got, _reference(sym, gq, B, missing, np.arange(n)))
        rows = rng.permutation(n)[: max(1, n // 2)].astype(np.int64)
        rows[rng.random(len(rows)) < 0.1] = n
        got = ctx.build_hist(packed, bits, n, F, B, missing, dev(gq), row_idx=torch.from_numpy(rows.astype(np.int32)).cuda())
        assert np.array_equal(got.cpu().numpy().reshape(F, B, 2), _reference(sym, gq, B, missing, rows))


def _check_equal_hessians(ctx, oracle, sym, bits, B, missing, columns, rng, depth=1):
    """Rows of one hessian are counted, not summed.  For each of `columns` gradients that make it the split: the sums of the
    nodes under it are those of its bins up to a drawn one, and of the rest."""
    import paper_1806_11248_amd as g
    n, F = sym.shape
    packed = dev(oracle.pack(sym, bits).view(np.int32))
    nb = torch.full((F,), B, dtype=torch.int32, device="cuda")
    cuts = torch.arange(B - 1, dtype=torch.float32, device="cuda").repeat(F, 1).contiguous()
    params = g.make_params(max_depth=depth, max_bins=B, eta=0.3, objective="squared")
    for f in columns:
        s = sym[:, f].astype(np.int64)
        live = (s < B) & (s != missing)
        bins = np.unique(s[live])
        if len(bins) < 2:
            continue
        t = int(bins[rng.integers(0, len(bins) - 1)])
        grad = (np.where(live & (s <= t), -64.0, 64.0) + rng.integers(-3, 4, n)) / 8.0
        gp = torch.from_numpy(np.stack([grad, np.full(n, 0.5)], 1).astype(np.float32)).cuda()
        tree, _, _ = ctx.grow_tree(packed, bits, n, F, missing, nb, cuts, gp, params, want_rows=False)
        assert (tree["feature"][0], tree["bin"][0]) == (f, t), (f, t, tree["feature"][0], tree["bin"][0])
        left = (s <= t) & (s != missing) if not tree["default_left"][0] else (s <= t) | (s == missing)
        for node, rows in ((tree["left"][0], left), (tree["right"][0], ~left)):
            assert tree["n_rows"][node] == rows.sum()
            assert (tree["sumG"][node], tree["sumH"][node]) == (grad[rows].sum(), 0.5 * rows.sum()), (f, t)


@pytest.mark.parametrize("bits", range(10, 17))
def test_short_windows(ctx, oracle, bits):
    """Columns that one load of eight bytes holds, and one more; tables of few and of many bins; rows that end the buffer."""
    rng = np.random.default_rng(bits)
    for F in range(1, 57 // bits + 2):
        for n, B, missing in ((5, 16, 16), (37, 16, 3), (1037, 16, 16), (2048, min(4096, 1 << bits), 7), (1500, 300, 1)):
            sym = rng.integers(0, 1 << bits, (n, F)).astype(np.uint16)
            few = rng.random((n, F)) < 0.8
            sym[few] = rng.integers(0, min(B + 2, 1 << bits), int(few.sum()))
            gq = np.stack([rng.integers(-(1 << 26), (1 << 26) + 1, n), rng.integers(0, (1 << 22) + 1, n)], 1).astype(np.int32)
            packed = dev(oracle.pack(sym, bits).view(np.int32))
            print(f"short bits={bits} n={n} F={F} B={B} missing={missing}", flush=True)
            got = ctx.build_hist(packed, bits, n, F, B, missing, dev(gq)).cpu().numpy().reshape(F, B, 2)
            assert np.array_equal(got, _reference(sym, gq, B, missing, np.arange(n)))
            rows = rng.permutation(n)[: max(1, n // 2)].astype(np.int64)
            got = ctx.build_hist(packed, bits, n, F, B, missing, dev(gq), row_idx=torch.from_numpy(rows.astype(np.int32)).cuda())
            assert np.array_equal(got.cpu().numpy().reshape(F, B, 2), _reference(sym, gq, B, missing, rows))
            sym[sym >= B] = missing   # (a tree's symbols are bins or the missing one)
            if n > 1000:
                _check_equal_hessians(ctx, oracle, sym, bits, B, missing, range(F), rng)
