"""Histograms of every symbol width at the edges of the register windows, against sums of the same integers (-m gpu)."""
import numpy as np
import pytest
import torch

import hist_tiles
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
    """The general form (of bytes: the byte kernel).  Columns around one, two and four windows, in tiles as the rule cuts them; tables
    with a row for every symbol and with one for what is no bin; a missing symbol among the bins and behind them; matrices down to
    less than sixteen bytes, whose first and last rows end at the buffer's edges; row lists in any order with ids that name no
    row."""
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
        gq[rng.random(n) < 0.5] = (1 << 26, 1 << 22)
        packed = dev(oracle.pack(sym, bits).view(np.int32))
        print(f"bits={bits} n={n} F={F} B={B} missing={missing}", flush=True)
        got = ctx.build_hist(packed, bits, n, F, B, missing, dev(gq)).cpu().numpy().reshape(F, B, 2)
        assert np.array_equal(got, _reference(sym, gq, B, missing, np.arange(n)))
        rows = rng.permutation(n)[: max(1, n // 2)].astype(np.int64)
        rows[rng.random(len(rows)) < 0.1] = n
        got = ctx.build_hist(packed, bits, n, F, B, missing, dev(gq), row_idx=torch.from_numpy(rows.astype(np.int32)).cuda())
        assert np.array_equal(got.cpu().numpy().reshape(F, B, 2), _reference(sym, gq, B, missing, rows))


def _symbols(rng, n, F, bits, B):
    """Mostly bins, some symbols that are none."""
    sym = rng.integers(0, 1 << bits, (n, F)).astype(np.uint16)
    few = rng.random((n, F)) < 0.8
    sym[few] = rng.integers(0, min(B + 2, 1 << bits), int(few.sum()))
    return sym


def _pairs(rng, n):
    return np.stack([rng.integers(-(1 << 26), (1 << 26) + 1, n), rng.integers(0, (1 << 22) + 1, n)], 1).astype(np.int32)


@pytest.mark.parametrize("bits,F", [(b, F) for table in (hist_tiles.TWO, hist_tiles.FOUR) for b, F in table.items()])
def test_tiles_of_several_windows(ctx, oracle, bits, F):
    """Rows whose windows go to two and four lanes, full and not (the last tile)."""
    rng = np.random.default_rng(F)
    B = min(16, 1 << bits)
    for n, missing in ((700, B), (901, 1)):
        sym, gq = _symbols(rng, n, F, bits, B), _pairs(rng, n)
        packed = dev(oracle.pack(sym, bits).view(np.int32))
        print(f"windows bits={bits} n={n} F={F} B={B} missing={missing}", flush=True)
        got = ctx.build_hist(packed, bits, n, F, B, missing, dev(gq)).cpu().numpy().reshape(F, B, 2)
        assert np.array_equal(got, _reference(sym, gq, B, missing, np.arange(n)))
        rows = rng.permutation(n)[: n // 2].astype(np.int64)
        got = ctx.build_hist(packed, bits, n, F, B, missing, dev(gq), row_idx=torch.from_numpy(rows.astype(np.int32)).cuda())
        assert np.array_equal(got.cpu().numpy().reshape(F, B, 2), _reference(sym, gq, B, missing, rows))


@pytest.mark.parametrize("bits,F", hist_tiles.FOUR_GATHERED.items())
def test_tiles_of_four_windows_gathered(ctx, bits, F):
    """A few rows listed of a matrix that the caches do not hold, its first and its last among them."""
    gen = torch.Generator("cuda").manual_seed(bits)
    n = -(-hist_tiles.GATHERED_BYTES * 8 // (F * bits))
    words = (n * F * bits + 31) // 32 + 1
    packed = torch.randint(-(1 << 31), 1 << 31, (words,), dtype=torch.int32, device="cuda", generator=gen)
    gq = torch.stack([torch.randint(-(1 << 26), (1 << 26) + 1, (n,), device="cuda", generator=gen),
                      torch.randint(0, (1 << 22) + 1, (n,), device="cuda", generator=gen)], 1).to(torch.int32)
    rows = torch.randint(0, n, (3000,), device="cuda", generator=gen)
    rows[:2] = torch.tensor([0, n - 1], device="cuda")
    first = rows * (F * bits)                                      # bits and words of the listed rows, unpacked here
    at = (first >> 5)[:, None] + torch.arange((F * bits + 62) // 32, device="cuda")
    mine = packed[at.clamp(max=words - 1)].cpu().numpy().view(np.uint32)
    bit = (first & 31).cpu().numpy()[:, None] + np.arange(F * bits)
    field = (np.take_along_axis(mine, bit >> 5, 1) >> (bit & 31).astype(np.uint32)) & 1
    sym = (field.reshape(len(rows), F, bits).astype(np.uint32) << np.arange(bits, dtype=np.uint32)).sum(2)
    B = min(16, 1 << bits)
    print(f"gathered bits={bits} n={n} F={F} B={B}", flush=True)
    for missing in (B, 1):
        got = ctx.build_hist(packed, bits, n, F, B, missing, gq, row_idx=rows.to(torch.int32)).cpu().numpy().reshape(F, B, 2)
        assert np.array_equal(got, _reference(sym, gq[rows].cpu().numpy(), B, missing, np.arange(len(rows))))


@pytest.mark.parametrize("bits", range(1, 17))
def test_sums_that_leave_their_fields(ctx, oracle, bits):
    """Columns of one symbol and the largest pairs: in any 256 rows, the fewest of a job, the h of a bin passes 2^30, and its g 2^33
    upwards in one half of the rows and downwards in the other."""
    rng = np.random.default_rng(bits)
    B = min(16, 1 << bits)
    for F in (1, 3, _window(bits), hist_tiles.TWO.get(bits, 40), hist_tiles.FOUR.get(bits, 64)):
        n = 3000 if F < 500 else 1100
        sym = rng.integers(0, B, (n, F)).astype(np.uint16)
        sym[:, ::2] = rng.integers(0, B, (F + 1) // 2)
        gq = np.tile(np.array([[1 << 26, 1 << 22]], np.int32), (n, 1))
        gq[n // 2:, 0] = -(1 << 26)
        block = gq[:256].astype(np.int64).sum(0)
        assert block[1] >= 1 << 30 and block[0] > 1 << 33
        packed = dev(oracle.pack(sym, bits).view(np.int32))
        print(f"fields bits={bits} n={n} F={F} B={B}", flush=True)
        got = ctx.build_hist(packed, bits, n, F, B, B, dev(gq)).cpu().numpy().reshape(F, B, 2)
        assert np.array_equal(got, _reference(sym, gq, B, B, np.arange(n)))
        rows = np.concatenate([rng.permutation(n // 2), n // 2 + rng.permutation(n - n // 2)])
        got = ctx.build_hist(packed, bits, n, F, B, B, dev(gq), row_idx=torch.from_numpy(rows.astype(np.int32)).cuda())
        assert np.array_equal(got.cpu().numpy().reshape(F, B, 2), _reference(sym, gq, B, B, rows))


@pytest.mark.parametrize("bits", range(1, 17))
def test_equal_hessians(ctx, oracle, bits):
    """The form that counts rows, at the same edges, bytes among them: splits at the first and last columns of windows and tiles, and
    under the root with rows that were moved or listed."""
    rng = np.random.default_rng(100 + bits)
    E, B = _window(bits), min(16, 1 << bits)
    wide = (17, 32, 33, 64, 65, 127) if bits == 8 else (hist_tiles.TWO[bits], hist_tiles.FOUR.get(bits, 2 * E + 3))
    for F in (2, E - 1, E, E + 1, *wide):
        n = 1201 if F < 500 else 603
        missing = int(rng.choice([B, 1] if B > 2 else [B]))
        sym = _symbols(rng, n, F, bits, B)
        sym[sym >= B] = missing if missing < 1 << bits else 0   # (a tree's symbols are bins or the missing one)
        edges = {c for t in range(0, F, E) for c in (t - 1, t, t + 1)} | {F // 2, F - 1} | set(rng.integers(0, F, 4).tolist())
        print(f"equal hessians bits={bits} n={n} F={F} B={B} missing={missing}", flush=True)
        _check_equal_hessians(ctx, oracle, sym, bits, B, missing, sorted(c for c in edges if 0 <= c < F), rng, depth=2)


def _check_equal_hessians(ctx, oracle, sym, bits, B, missing, columns, rng, depth=1):
    """Rows of one hessian are counted, not summed.  For each of `columns` gradients that make it the root's split, at a drawn bin: the
    sums of every node are those of its rows."""
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
        open_ = [(0, np.ones(n, bool))]
        while open_:
            node, rows = open_.pop()
            assert tree["n_rows"][node] == rows.sum()
            assert (tree["sumG"][node], tree["sumH"][node]) == (grad[rows].sum(), 0.5 * rows.sum()), (f, t, node)
            if tree["feature"][node] >= 0:
                v = sym[:, tree["feature"][node]].astype(np.int64)
                left = np.where(v == missing, tree["default_left"][node] != 0, v <= tree["bin"][node])
                open_ += [(tree["left"][node], rows & left), (tree["right"][node], rows & ~left)]


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
