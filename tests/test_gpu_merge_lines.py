"""Histograms that begin anywhere in a line of memory, of any number of bins: sums of the same integers, nothing around them
touched (-m gpu)."""
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


def _sums(sym, gq, B, missing):
    out = np.zeros((sym.shape[1], B, 2), np.int64)
    for f in range(sym.shape[1]):
        live = sym[:, f] != missing
        np.add.at(out[f], sym[live, f], gq[live].astype(np.int64))
    return out


# columns, bins, rows: columns of less than a line, of whole lines and of some more; bytes and other widths; one job and several
@pytest.mark.parametrize("F,B,n", [(1, 2, 50), (5, 7, 900), (3, 8, 900), (40, 9, 900), (1, 31, 3000), (13, 33, 3000), (19, 255, 3000),
                                   (28, 256, 9000), (300, 63, 900), (90, 300, 20000)])
def test_lines(ctx, oracle, F, B, n):
    rng = np.random.default_rng(F * B)
    missing = B
    sym = rng.integers(0, B, (n, F)).astype(np.uint16)
    sym[rng.random((n, F)) < 0.4] = missing
    gq = np.stack([rng.integers(-(1 << 26), (1 << 26) + 1, n), rng.integers(0, (1 << 22) + 1, n)], 1).astype(np.int32)
    want = torch.from_numpy(_sums(sym, gq, B, missing)).cuda()
    bits = oracle.bits_for(B)
    packed = dev(oracle.pack(sym, bits).view(np.int32))
    full = np.where(sym == missing, 0, sym).astype(np.uint16)   # bytes of 256 bins leave no symbol to be missing
    rowptr, ent, nnz = ctx.compress_sparse(dev(sym), B, missing)
    rows = torch.arange(n, dtype=torch.int32, device="cuda")
    words = F * B * 2
    for at in (0, 1, 2, 6, 14, 16, 30):   # words of eight bytes: the middle of a bin as well
        buf = torch.full((words + 64,), -7, dtype=torch.int64, device="cuda")
        out = buf[at:at + words].view(F, B, 2)
        print(f"merge lines F={F} B={B} n={n} bits={bits} at={at}", flush=True)
        for build in (lambda: ctx.build_hist(packed, bits, n, F, B, missing, dev(gq), out=out),
                      lambda: ctx.build_hist(packed, bits, n, F, B, missing, dev(gq), row_idx=rows, out=out),
                      lambda: ctx.build_hist_sparse(rowptr, ent, n, F, B, dev(gq), out=out)):
            out.fill_(-7)
            build()
            assert torch.equal(out, want)
            assert (buf[:at] == -7).all() and (buf[at + words:] == -7).all()
        if B <= 256:
            eight = dev(oracle.pack(full, 8).view(np.int32))
            ctx.build_hist(eight, 8, n, F, B, 256, dev(gq), out=out)
            assert torch.equal(out, torch.from_numpy(_sums(full, gq, B, 256)).cuda())
            assert (buf[:at] == -7).all() and (buf[at + words:] == -7).all()
