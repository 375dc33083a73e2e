"""Passes of dense width 1 (SpMV, its transpose and VJP, the SMVM loss) at
the edges of their dispatch and tiles: one entry, the sizes up to which a pass
is complete in one launch of 512-entry tiles (16,384 entries; 8,192 with a loss
that gathers both vectors), tiles of 512 and 2,048 above (from 2^20 entries on),
patterns of short segments only, complete in one launch below 2^23 entries,
segments that cross no tile, some and all, runs of empty segments; against
64-bit sums of the same products.

Bound, additions a product passes through.  Complete in one launch: 6 over the
wave and 8 over the waves of its tile, 2 that join them, at most 9 strided ones of
the segment's rest (4,096 entries by 512 threads), 6 and 8 to sum those, 1.  With
a combine: 7 in the thread, 6, 4 and 2, then ceil(tiles / 64) + 7 over the tiles
that a segment crosses, at most 2,048 here: 58.  Each is within 2^-24 of the sum
of magnitudes; with the rounded products and the scale 61, below the 66 used."""
import numpy as np
import pytest
import torch

from helpers import assert_mag_close

pytestmark = pytest.mark.gpu

TOL = 66 * 2.0 ** -24


@pytest.fixture(scope="module")
def operand():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_07030_amd.operand import DeviceCsr
    return DeviceCsr


def pattern(kind, nnz, rng):
    """rowptr, colind, ncols: consecutive columns from a random start."""
    if kind == "one":  # a single row holds everything, other rows are empty
        lengths, ncols = np.array([0, 0, nnz, 0]), nnz + 5
    elif kind == "column":  # a single column holds everything
        lengths, ncols = np.ones(nnz, dtype=np.int64), 3
    else:
        mean = {"short": 4, "crossing": 1500}[kind]
        lengths = rng.integers(0, 2 * mean + 1, max(4, int(1.2 * nnz / mean) + 8))
        lengths[rng.random(len(lengths)) < 0.3] = 0
        lengths[10:40] = 0
        cut = np.searchsorted(np.cumsum(lengths), nnz)
        while cut >= len(lengths):
            lengths = np.concatenate([lengths, lengths])
            cut = np.searchsorted(np.cumsum(lengths), nnz)
        lengths = lengths[:cut + 1]
        lengths[-1] -= lengths.sum() - nnz
        lengths = np.concatenate([lengths, [0, 0]])
        ncols = max(int(lengths.max()) * 3, 50)
    rowptr = np.concatenate([[0], np.cumsum(lengths)])
    start = (rng.integers(0, max(ncols - int(lengths.max()), 1), len(lengths))
             if kind != "column" else np.ones(len(lengths), dtype=np.int64))
    col = np.repeat(start, lengths) + np.arange(nnz) - np.repeat(rowptr[:-1], lengths)
    return rowptr.astype(np.int32), col.astype(np.int32), ncols


@pytest.mark.parametrize("kind", ["short", "crossing", "one", "column"])
@pytest.mark.parametrize("nnz", [1, 7, 16383, 16384, 16385, 100_001, (1 << 18) + 1,
                                 (1 << 20) - 1, (1 << 20) + 2049])
@pytest.mark.parametrize("plans", [False, True])
def test_width_one(operand, kind, nnz, plans):
    from paper_2303_07030_amd import nsd
    rng = np.random.default_rng(nnz)
    rowptr, col, ncols = pattern(kind, nnz, rng)
    nrows = len(rowptr) - 1
    row = np.repeat(np.arange(nrows), np.diff(rowptr))
    val = rng.standard_normal(nnz).astype(np.float32)
    x, gy = (rng.standard_normal(n).astype(np.float32) for n in (ncols, nrows))
    A = operand(nrows, ncols, rowptr, col, val, k_hint=1, perm_plans=plans)
    ws = A.workspace(1)
    xd, gd = torch.from_numpy(x).cuda(), torch.from_numpy(gy).cuda()

    def out(n, dtype=torch.float32):
        return torch.full((n,), float("nan"), dtype=dtype, device="cuda")

    def close(got, dst, prod, n, what):
        ref = np.bincount(dst, prod, n)
        assert_mag_close(got.cpu().numpy(), ref, np.bincount(dst, np.abs(prod), n), TOL, what)

    v64, x64, g64 = val.astype(np.float64), x.astype(np.float64), gy.astype(np.float64)
    y = out(nrows)
    nsd.nsd_spmv(A.desc, xd, y, ws)
    close(y, row, v64 * x64[col], nrows, "y")
    dA, dx = out(nnz), out(ncols)
    nsd.nsd_spmv_vjp(A.desc, A.csc, xd, gd, dA, dx, ws)
    close(dx, col, v64 * g64[row], ncols, "dx")
    assert np.array_equal(dA.cpu().numpy(), gy[row] * x[col])
    loss, dA, dx = out(1, torch.float64), out(nnz), out(ncols)
    nsd.nsd_loss_sum_spmv(A.desc, A.csc, xd, 0.5, loss, dA, dx, ws)
    close(dx, col, 0.5 * v64, ncols, "column sums")
    assert np.array_equal(dA.cpu().numpy(), np.float32(0.5) * x[col])
    terms = v64 * x64[col]
    # fp64 sums: 2^-53 per addition
    assert abs(loss.item() - terms.sum()) <= 1e-12 * np.abs(terms).sum()
    loss2 = out(1, torch.float64)
    nsd.nsd_loss_bilinear(A.desc, A.csc, xd, gd, 1, 1.0, loss2, dA, dx, ws)
    assert np.array_equal(dA.cpu().numpy(), gy[row] * x[col])
    # d is rounded to 32 bits before the sum
    t2 = v64 * x64[col] * g64[row]
    assert abs(loss2.item() - t2.sum()) <= 2.0 ** -23 * np.abs(t2).sum()
    close(dx, col, v64 * g64[row], ncols, "dH")


@pytest.mark.parametrize("kind", ["short", "crossing", "one", "column"])
@pytest.mark.parametrize("nnz", [4095, 4097, 8191, 8192, 8193, 12_289])
def test_width_one_of_few_entries(operand, kind, nnz):
    test_width_one(operand, kind, nnz, False)


@pytest.mark.parametrize("nnz", [(1 << 23) - 1, (1 << 23) + 1])
def test_width_one_of_short_rows(operand, nnz):
    test_width_one(operand, "short", nnz, False)
