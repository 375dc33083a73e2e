"""Widths that are no multiple of four: the last lane of a slot steps back to
the row's last four columns and shares some with the lane before.  Every
remainder at the narrowest widths, at the edges of each slot size and past a
wave's chunk, against the fp64 oracle; and a shared column that is infinite.
The matrix passes take widths up to 16 that are not of whole quads one column
per lane, and so do others by the number of entries: the last tests are on the
sizes past those lines.
"""
import numpy as np
import pytest
import torch

from helpers import assert_mag_close
from test_gpu_parity import (check_cp, check_cpn, check_frob, dev, edge_pattern, host,
                             in_input_order, oracle_dok, run_bilinear, run_cp, run_cpn,
                             run_frob)
from test_gpu_wide import check_mf_all, cp_case, dev_offset, empty_offset, mf_case

pytestmark = pytest.mark.gpu

# 2, 3: below one quad; then lanes * 4 - 3 .. - 1 around the slots of 2 to 64
WIDTHS = [2, 3, 5, 6, 7, 9, 10, 15, 17, 31, 35, 63, 66, 127, 130, 255]


@pytest.fixture(scope="module")
def nsd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_07030_amd import nsd as m
    return m


def operand_of(seed, k):
    from paper_2303_07030_amd.operand import DeviceCsr
    pat = edge_pattern(seed)
    return pat, DeviceCsr(*pat, k_hint=k)


@pytest.mark.parametrize("k", WIDTHS)
def test_matrix_losses(nsd, orc, k):
    (nrows, ncols, rowptr, colind, val), A = operand_of(31, k)
    rng = np.random.default_rng(k)
    H = rng.standard_normal((ncols, k)).astype(np.float32)
    G = rng.standard_normal((nrows, k)).astype(np.float32)
    check_frob(orc, nrows, ncols, rowptr, colind, val, H, k, run_frob(nsd, A, H, k, seed=2.0),
               seed=2.0)
    Lg, dAg, dHg = run_bilinear(nsd, A, H, G, k, seed=0.25)
    D = oracle_dok(orc, nrows, ncols, rowptr, colind, val)
    rows = np.repeat(np.arange(nrows, dtype=np.int32), np.diff(rowptr))
    L, Lm = orc.loss_bilinear(D, G, H, k)
    dA, dAm = orc.sddmm(D, G, H, k, rows, colind, alpha=0.25)
    dH, dHm = orc.spmm_t(D, G, k, alpha=0.25)
    assert_mag_close(Lg, L, Lm, what="loss")
    assert_mag_close(dAg, dA, dAm, what="dA")
    assert_mag_close(dHg, dH, dHm, what="dH")
    # the sampled product by itself, its rows at odd addresses
    out = torch.full((A.nnz,), np.nan, dtype=torch.float32, device="cuda")
    nsd.nsd_sddmm(A.desc, dev_offset(G), dev_offset(H), k, 0.25, out)
    assert_mag_close(host(out), dA, dAm, what="sddmm")


@pytest.mark.parametrize("k", WIDTHS)
def test_factorisation(nsd, orc, k):
    from paper_2303_07030_amd.operand import DeviceCsr
    nrows, ncols, rowptr, colind, val, U, V = mf_case(k)
    A = DeviceCsr(nrows, ncols, rowptr, colind, val, k_hint=k)
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    dU, dV = empty_offset((nrows, k)), empty_offset((ncols, k))
    nsd.nsd_loss_mf(A.desc, A.csc, None, dev_offset(U), dev(V), k, 0.5, loss, dU, dV,
                    A.workspace(k))
    D = oracle_dok(orc, nrows, ncols, rowptr, colind, val)
    check_mf_all(orc, D, U, V, k, host(loss)[0], host(dU), host(dV), 0.5)


@pytest.mark.parametrize("rank", WIDTHS)
def test_cp(nsd, orc, rank):
    from paper_2303_07030_amd.operand import DeviceCoo3, DeviceCooN
    dims, i, j, l, val, F = cp_case(rank)
    X = DeviceCoo3(dims, i, j, l, val, rank_hint=rank)
    check_cp(orc, dims, i, j, l, val, F, rank, run_cp(nsd, X, F, rank, seed=0.75), seed=0.75)
    # with fibers (two long modes, short others) and without
    for dims in ((6, 5, 40, 3), (9, 8, 7, 6)):
        rng = np.random.default_rng(rank)
        nnz = int(np.prod(dims)) // 2
        keys = rng.choice(2 * nnz, size=nnz, replace=False)
        coords = [c.astype(np.int32) for c in np.unravel_index(keys, dims)]
        val = rng.standard_normal(nnz).astype(np.float32)
        F = [(0.3 * rng.standard_normal((d, rank))).astype(np.float32) for d in dims]
        X = DeviceCooN(dims, coords, val, rank_hint=rank, item_len=16)
        check_cpn(orc, dims, coords, val, F, rank, run_cpn(nsd, X, F, rank, seed=0.5), seed=0.5)


@pytest.mark.parametrize("k", WIDTHS + [258, 515])
def test_tangents(nsd, orc, k):
    (nrows, ncols, rowptr, colind, val), A = operand_of(33, k)
    rng = np.random.default_rng(k)
    m = 5
    B, dB = (rng.standard_normal(s).astype(np.float32) for s in ((ncols, k), (m, ncols, k)))
    dval = rng.standard_normal((m, A.nnz)).astype(np.float32)
    C = torch.full((nrows, k), np.nan, device="cuda")
    dC = torch.full((m, nrows, k), np.nan, device="cuda")
    ws = torch.empty(nsd.nsd_spmm_jvp_batch_workspace_size(A.desc, k), dtype=torch.uint8,
                     device="cuda")
    nsd.nsd_spmm_jvp_batch(A.desc, m, dev(dval), dev(B), dev(dB), k, C, dC, ws)
    D = oracle_dok(orc, nrows, ncols, rowptr, colind, val)
    assert_mag_close(host(C), *orc.spmm(D, B, k), what="C")
    for t in range(m):
        Dt = oracle_dok(orc, nrows, ncols, rowptr, colind, dval[t])
        (r1, m1), (r2, m2) = orc.spmm(Dt, B, k), orc.spmm(D, dB[t], k)
        assert_mag_close(host(dC[t]), r1 + r2, m1 + m2, what=f"dC[{t}]")


@pytest.mark.parametrize("k", [5, 6, 7, 63, 258])
def test_infinite_shared_column(nsd, k):
    """Column k - 4 is the last lane's and the lane before's: an infinity
    there reaches a product once, and stays an infinity of its sign."""
    from paper_2303_07030_amd.operand import DeviceCsr
    A = DeviceCsr(2, 2, np.array([0, 1, 2], np.int32), np.array([0, 1], np.int32),
                  np.ones(2, np.float32), k_hint=k)
    X, Y = torch.ones((2, k), device="cuda"), torch.ones((2, k), device="cuda")
    X[0, k - 4] = float("inf")
    Y[1, k - 4] = float("-inf")
    out = torch.empty(2, device="cuda")
    nsd.nsd_sddmm(A.desc, X, Y, k, 1.0, out)
    assert host(out).tolist() == [np.inf, -np.inf]
    dA, dY, loss = torch.empty(2, device="cuda"), torch.empty((2, k), device="cuda"), \
        torch.empty(1, dtype=torch.float64, device="cuda")
    nsd.nsd_loss_bilinear(A.desc, A.csc, Y, X, k, 1.0, loss, dA, dY, A.workspace(k))
    assert host(dA).tolist() == [np.inf, -np.inf]


@pytest.mark.parametrize("perm_plans", [False, True])
@pytest.mark.parametrize("k", [257, 258, 260, 512, 513, 1027])
def test_column_slices(nsd, orc, k, perm_plans):
    """Rows wider than a slot: column passes of at most 256 columns that add
    up the sampled products, in A's order and in CSC order."""
    from paper_2303_07030_amd.operand import DeviceCsr
    nrows, ncols, rowptr, colind, val = edge_pattern(35)
    A = DeviceCsr(nrows, ncols, rowptr, colind, val, k_hint=k, perm_plans=perm_plans)
    rng = np.random.default_rng(k)
    X = rng.standard_normal((ncols, k)).astype(np.float32)
    G = rng.standard_normal((nrows, k)).astype(np.float32)
    D = oracle_dok(orc, nrows, ncols, rowptr, colind, val)
    rows = np.repeat(np.arange(nrows, dtype=np.int32), np.diff(rowptr))
    dA, dAm = orc.sddmm(D, G, X, k, rows, colind)
    dX, dXm = orc.spmm_t(D, G, k)
    got, gotX = torch.full((A.nnz,), np.nan, device="cuda"), empty_offset((ncols, k))
    nsd.nsd_spmm_vjp(A.desc, A.csc, dev_offset(X), dev(G), k, got, gotX, A.workspace(k))
    assert_mag_close(host(got), dA, dAm, what="vjp dA")
    assert_mag_close(host(gotX), dX, dXm, what="vjp dX")
    L, Lm = orc.loss_bilinear(D, G, X, k)
    Lg, dAg, dHg = run_bilinear(nsd, A, X, G, k, seed=-0.5)
    assert_mag_close(Lg, L, Lm, what="loss")
    assert_mag_close(dAg, -0.5 * dA, 0.5 * dAm, what="dA")
    assert_mag_close(dHg, -0.5 * dX, 0.5 * dXm, what="dH")
    check_frob(orc, nrows, ncols, rowptr, colind, val, X, k, run_frob(nsd, A, X, k, seed=3.0),
               seed=3.0)


@pytest.mark.parametrize("perm_plans", [False, True])
@pytest.mark.parametrize("k", [257, 260, 512, 1027])
def test_column_slices_of_larger_patterns(nsd, k, perm_plans):
    """Patterns of which a slice gathers at least 20 * 2**20 floats are taken
    in column slices (above: a sampled product and a gather-reduce of their
    own); against dense products in 64 bits."""
    from paper_2303_07030_amd.operand import DeviceCsr
    rng = np.random.default_rng(k)
    nrows, ncols = 420, 500
    dense = rng.standard_normal((nrows, ncols)) * (rng.random((nrows, ncols)) < 0.8)
    dense[:, [0, 77]], dense[5] = 0.0, 0.0  # empty columns and an empty row
    rows, cols = np.nonzero(dense)
    rowptr = np.concatenate([[0], np.cumsum((dense != 0).sum(1))]).astype(np.int32)
    val = dense[rows, cols].astype(np.float32)
    assert len(val) * (k // -(-k // 256)) >= 20 << 20
    dense[rows, cols] = val
    A = DeviceCsr(nrows, ncols, rowptr, cols.astype(np.int32), val, k_hint=k,
                  perm_plans=perm_plans)
    X = rng.standard_normal((ncols, k)).astype(np.float32)
    G = rng.standard_normal((nrows, k)).astype(np.float32)
    x, g = X.astype(np.float64), G.astype(np.float64)
    dA, dAm = (g @ x.T)[rows, cols], (abs(g) @ abs(x).T)[rows, cols]
    dX, dXm = dense.T @ g, abs(dense).T @ abs(g)
    got, gotX = torch.full((A.nnz,), np.nan, device="cuda"), empty_offset((ncols, k))
    nsd.nsd_spmm_vjp(A.desc, A.csc, dev_offset(X), dev(G), k, got, gotX, A.workspace(k))
    assert_mag_close(host(got), dA, dAm, what="vjp dA")
    assert_mag_close(host(gotX), dX, dXm, what="vjp dX")
    Lg, dAg, dHg = run_bilinear(nsd, A, X, G, k, seed=-0.5)
    assert_mag_close(Lg, (val * dA).sum(), (abs(val) * dAm).sum(), what="loss")
    assert_mag_close(dAg, -0.5 * dA, 0.5 * dAm, what="dA")
    assert_mag_close(dHg, -0.5 * dX, 0.5 * dXm, what="dH")
    C, Cm = dense @ x, abs(dense) @ abs(x)
    Cf, Lf, dAf, dBf = run_frob(nsd, A, X, k)
    assert_mag_close(Cf, C, Cm, what="C")
    assert_mag_close(Lf, 0.5 * (C * C).sum(), 0.5 * (Cm * Cm).sum(), what="frob loss")
    assert_mag_close(dAf, (C @ x.T)[rows, cols], (Cm @ abs(x).T)[rows, cols], what="frob dA")
    assert_mag_close(dBf, dense.T @ C, abs(dense).T @ Cm, what="frob dB")


def large_pattern(rng, nrows, ncols, nnz):
    key = np.unique(rng.integers(0, nrows * ncols, nnz + nnz // 8))
    key = np.sort(rng.permutation(key)[:nnz])
    rows, cols = (key // ncols).astype(np.int32), (key % ncols).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=nrows))]).astype(np.int32)
    return rows, rowptr, cols, rng.standard_normal(nnz).astype(np.float32)


@pytest.mark.parametrize("nnz", [(1 << 15) + 5, (1 << 18) + 5])
@pytest.mark.parametrize("rank", [5, 7, 9, 15, 21])
def test_cp_of_more_entries(nsd, orc, rank, nnz):
    """Ragged ranks in quads: from 2^15 entries on above eight, from 2^18 on
    below (items of eight entries)."""
    from paper_2303_07030_amd.operand import DeviceCoo3, DeviceCooN
    dims, i, j, l, val, F = cp_case(rank, dims=(90, 70, 120), nnz=nnz)
    X = DeviceCoo3(dims, i, j, l, val, item_len=8)
    check_cp(orc, dims, i, j, l, val, F, rank, run_cp(nsd, X, F, rank, seed=0.75), seed=0.75)
    if nnz < 1 << 18:
        return
    dims = (60, 50, 40, 9)
    key = np.random.default_rng(rank).choice(int(np.prod(dims)), nnz, replace=False)
    coords = [c.astype(np.int32) for c in np.unravel_index(key, dims)]
    F = [(0.3 * np.random.default_rng(n).standard_normal((d, rank))).astype(np.float32)
         for n, d in enumerate(dims)]
    X = DeviceCooN(dims, coords, val, item_len=8, fibers=True)
    check_cpn(orc, dims, coords, val, F, rank, run_cpn(nsd, X, F, rank, seed=0.5), seed=0.5)


@pytest.mark.parametrize("rank", [4, 8, 12])
def test_cp_off_lines_of_more_entries(nsd, orc, rank):
    """Rows of whole quads off their 16-byte lines: one column a lane at ranks 4
    and 8, quads at 12."""
    from paper_2303_07030_amd.operand import DeviceCoo3
    dims, i, j, l, val, F = cp_case(rank, dims=(90, 70, 120), nnz=(1 << 18) + 5)
    X = DeviceCoo3(dims, i, j, l, val, rank_hint=rank)
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    dX, dF = torch.full((X.nnz,), np.nan, device="cuda"), [empty_offset((d, rank)) for d in dims]
    nsd.nsd_loss_cp(X.desc, *[dev_offset(f) for f in F], rank, 0.75, loss, dX, *dF,
                    X.workspace(rank))
    got = host(loss)[0], in_input_order(X, host(dX)), [host(t) for t in dF]
    check_cp(orc, dims, i, j, l, val, F, rank, got, seed=0.75)


@pytest.mark.parametrize("k", [17, 31, 32])
def test_sampled_product_of_more_entries(nsd, k):
    """From 2^22 entries on up to 32 columns take one lane each (32: of rows
    off their 16-byte lines)."""
    from paper_2303_07030_amd.operand import DeviceCsr
    rng = np.random.default_rng(k)
    rows, rowptr, cols, val = large_pattern(rng, 3000, 2500, (1 << 22) + 3)
    A = DeviceCsr(3000, 2500, rowptr, cols, val, k_hint=k, build_csc=False)
    X = rng.standard_normal((3000, k)).astype(np.float32)
    Y = rng.standard_normal((2500, k)).astype(np.float32)
    out = torch.full((A.nnz,), np.nan, device="cuda")
    nsd.nsd_sddmm(A.desc, dev_offset(X), dev_offset(Y), k, -2.0, out)
    x, y = X.astype(np.float64), Y.astype(np.float64)
    assert_mag_close(host(out), -2.0 * (x @ y.T)[rows, cols], 2.0 * (abs(x) @ abs(y).T)[rows, cols])


@pytest.mark.parametrize("perm_plans", [False, True])
@pytest.mark.parametrize("k", [2, 3, 4])
def test_frob_of_more_entries(nsd, k, perm_plans):
    """Up to four columns (4: of rows off their 16-byte lines) go in separate
    passes from 3 * 2^17 entries on, unless the values move to CSC order."""
    import scipy.sparse as sp
    from paper_2303_07030_amd.operand import DeviceCsr
    rng = np.random.default_rng(k)
    nrows, ncols = 9000, 7000
    rows, rowptr, cols, val = large_pattern(rng, nrows, ncols, (3 << 17) + 7)
    A = DeviceCsr(nrows, ncols, rowptr, cols, val, k_hint=k, perm_plans=perm_plans)
    B = rng.standard_normal((ncols, k)).astype(np.float32)
    C, dB = empty_offset((nrows, k)), empty_offset((ncols, k))
    dA, loss = torch.full((A.nnz,), np.nan, device="cuda"), \
        torch.empty(1, dtype=torch.float64, device="cuda")
    nsd.nsd_loss_frob_spmm(A.desc, A.csc, dev_offset(B), k, 0.5, C, loss, dA, dB, A.workspace(k))
    S, b = sp.csr_matrix((val.astype(np.float64), cols, rowptr), (nrows, ncols)), B.astype(float)
    c, cm = S @ b, abs(S) @ abs(b)
    assert_mag_close(host(C), c, cm, what="C")
    assert_mag_close(host(loss)[0], 0.5 * (c * c).sum(), 0.5 * (cm * cm).sum(), what="loss")
    assert_mag_close(host(dA), 0.5 * (c[rows] * b[cols]).sum(1),
                     0.5 * (cm[rows] * abs(b[cols])).sum(1), what="dA")
    assert_mag_close(host(dB), 0.5 * (S.T @ c), 0.5 * (abs(S).T @ cm), what="dB")


@pytest.mark.parametrize("nnz", [(1 << 14) - 1, (1 << 14) + 1, (1 << 17) + 1])
@pytest.mark.parametrize("k", [17, 31])
def test_tangents_of_more_entries(nsd, k, nnz):
    """One column a lane up to 32 columns below 2^14 entries and from 2^17 on."""
    import scipy.sparse as sp
    from paper_2303_07030_amd.operand import DeviceCsr
    rng = np.random.default_rng(k)
    nrows, ncols, m = 1500, 1300, 3
    rows, rowptr, cols, val = large_pattern(rng, nrows, ncols, nnz)
    A = DeviceCsr(nrows, ncols, rowptr, cols, val, k_hint=k, build_csc=False)
    B, dB = (rng.standard_normal(s).astype(np.float32) for s in ((ncols, k), (m, ncols, k)))
    dval = rng.standard_normal((m, nnz)).astype(np.float32)
    C = torch.full((nrows, k), np.nan, device="cuda")
    dC = torch.full((m, nrows, k), np.nan, device="cuda")
    ws = torch.empty(nsd.nsd_spmm_jvp_batch_workspace_size(A.desc, k), dtype=torch.uint8,
                     device="cuda")
    nsd.nsd_spmm_jvp_batch(A.desc, m, dev(dval), dev(B), dev(dB), k, C, dC, ws)

    def mat(v):
        return sp.csr_matrix((v.astype(np.float64), cols, rowptr), (nrows, ncols))

    S, b = mat(val), B.astype(np.float64)
    assert_mag_close(host(C), S @ b, abs(S) @ abs(b), what="C")
    for t in range(m):
        D, d = mat(dval[t]), dB[t].astype(np.float64)
        assert_mag_close(host(dC[t]), D @ b + S @ d, abs(D) @ abs(b) + abs(S) @ abs(d),
                         what=f"dC[{t}]")


@pytest.mark.parametrize("k, over", [(31, -9), (31, 9), (17, 9)])
def test_cold_operands(nsd, k, over):
    """One column a lane up to 32 columns from 2^28 gathered floats on, in every
    pass of a matrix."""
    from paper_2303_07030_amd.operand import DeviceCsr
    rng = np.random.default_rng(k)
    nrows, ncols, nnz = 300_000, 250_000, (1 << 28) // k + over
    rows, rowptr, cols, val = large_pattern(rng, nrows, ncols, nnz)
    A = DeviceCsr(nrows, ncols, rowptr, cols, val, k_hint=k)
    H, G = (rng.standard_normal((n, k)).astype(np.float32) for n in (ncols, nrows))
    r, c, v, h, g = (torch.from_numpy(x).cuda() for x in (rows, cols, val, H, G))
    r, c = r.long(), c.long()

    def reduce(n, at, w, x, idx):  # sum of w_p x[idx_p] at at_p, and its magnitude, in fp64
        s, m = (torch.zeros((n, k), dtype=torch.float64, device="cuda") for _ in range(2))
        for p in torch.arange(nnz, device="cuda").split(1 << 20):
            t = w[p].double()[:, None] * x[idx[p]].double()
            s.index_add_(0, at[p], t)
            m.index_add_(0, at[p], t.abs())
        return host(s), host(m)

    def dots(x, y):
        s, m = (torch.empty(nnz, dtype=torch.float64, device="cuda") for _ in range(2))
        for p in torch.arange(nnz, device="cuda").split(1 << 20):
            t = x[r[p]].double() * y[c[p]].double()
            s[p], m[p] = t.sum(1), t.abs().sum(1)
        return s, m

    ws, loss = A.workspace(k), torch.empty(1, dtype=torch.float64, device="cuda")
    C, dC, dH = (empty_offset((n, k)) for n in (nrows, nrows, ncols))
    dA = torch.full((nnz,), np.nan, device="cuda")
    d, dm = dots(g, h)
    fwd, col = reduce(nrows, r, v, h, c), reduce(ncols, c, v, g, r)

    nsd.nsd_loss_bilinear(A.desc, A.csc, dev_offset(H), dev_offset(G), k, 0.5, loss, dA, dH, ws)
    assert_mag_close(host(loss)[0], host((v * d).sum()), host((v.abs() * dm).sum()), what="loss")
    assert_mag_close(host(dA), 0.5 * host(d), 0.5 * host(dm), what="dA")
    assert_mag_close(host(dH), 0.5 * col[0], 0.5 * col[1], what="dH")

    nsd.nsd_spmm(A.desc, h, k, C, ws)
    assert_mag_close(host(C), *fwd, what="spmm")

    wj = torch.empty(nsd.nsd_spmm_jvp_batch_workspace_size(A.desc, k), dtype=torch.uint8,
                     device="cuda")
    nsd.nsd_spmm_jvp_batch(A.desc, 1, v.neg()[None], h, 2 * h[None], k, C, dC[None], wj)
    assert_mag_close(host(C), *fwd, what="C")
    assert_mag_close(host(dC), fwd[0], 3 * fwd[1], what="dC")

    B, dB = dev_offset(H), empty_offset((ncols, k))
    nsd.nsd_loss_frob_spmm(A.desc, A.csc, B, k, 1.0, C, loss, dA, dB, ws)
    cd = C.double()
    assert_mag_close(host(C), *fwd, what="C of the loss")
    assert_mag_close(host(loss)[0], host(0.5 * (cd * cd).sum()), host(0.5 * (cd * cd).sum()),
                     what="half square")
    s, m = dots(C, h)
    assert_mag_close(host(dA), host(s), host(m), what="dA of the half square")
    assert_mag_close(host(dB), *reduce(ncols, c, v, C, r), what="dB of the half square")

    dU, dV = (empty_offset((n, k)) for n in (nrows, ncols))
    nsd.nsd_loss_mf(A.desc, A.csc, A.values_in_csc_order(), dev_offset(G), dev_offset(H), k, 1.0,
                    loss, dU, dV, ws)
    res, mag = v - d, v.abs() + dm
    assert_mag_close(host(loss)[0], host((res * res).sum()), host((mag * mag).sum()), what="squares")
    for got, n, at, x, idx in ((dU, nrows, r, h, c), (dV, ncols, c, g, r)):
        assert_mag_close(host(got), -2 * reduce(n, at, res, x, idx)[0],
                         2 * reduce(n, at, mag, x.abs(), idx)[1], what="factor gradient")
