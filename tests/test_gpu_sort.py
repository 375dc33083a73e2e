"""The radix sort of the builders at the edges of its digits (8 bits, or 9 and
10 where they save a third of the passes) and of its tiles (4,096 elements, 8,192
from 8M on), bit for bit against a stable sort; and the pair key of the COO
builder with digits that straddle column and row.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nsd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_07030_amd import nsd as m
    return m


def keys_of(n, dim, seed, skew):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    k = torch.randint(dim, (n,), generator=g, device="cuda", dtype=torch.int32)
    if skew and n:  # most keys equal, the extremes present
        k = torch.where(torch.rand(n, generator=g, device="cuda") < 0.9, k[0], k)
        k[n // 2], k[-1] = dim - 1, 0
    return k


@pytest.mark.parametrize("n", [1, 63, 4095, 4096, 4097, 100_003])
@pytest.mark.parametrize("bits", [1, 8, 9, 10, 11, 16, 17, 19, 20, 21, 24, 27])
def test_mode_index_order(nsd, n, bits):
    dim = 1 << bits
    for skew in (False, True):
        key = keys_of(n, dim, bits, skew)
        segptr = torch.empty(dim + 1, dtype=torch.int32, device="cuda")
        segidx, perm = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
        ws = torch.empty(nsd.nsd_build_workspace_size(n, dim), dtype=torch.uint8, device="cuda")
        nsd.nsd_coo_mode_index(n, dim, key, segptr, segidx, perm, ws)
        want, order = torch.sort(key, stable=True)
        assert torch.equal(segidx, want) and torch.equal(perm, order.int())


@pytest.mark.parametrize("n", [(1 << 23) - 1, 1 << 23, (1 << 23) + 1, (1 << 23) + 8191])
@pytest.mark.parametrize("dim", [200, 1000, 500_000, 1_100_000])
def test_mode_index_order_large(nsd, n, dim):
    key = keys_of(n, dim, n % 97, dim == 1000)
    segptr = torch.empty(dim + 1, dtype=torch.int32, device="cuda")
    segidx, perm = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.empty(nsd.nsd_build_workspace_size(n, dim), dtype=torch.uint8, device="cuda")
    nsd.nsd_coo_mode_index(n, dim, key, segptr, segidx, perm, ws)
    want, order = torch.sort(key, stable=True)
    assert torch.equal(segidx, want) and torch.equal(perm, order.int())


@pytest.mark.parametrize("nrows,ncols", [(3, 1), (200, 5), (1000, 3), (700, 900), (90_000, 11),
                                         (5, 90_000), (1_000_000, 500_000)])
@pytest.mark.parametrize("n", [5000, 1 << 23])
def test_coo_to_csr_pair_keys(nsd, nrows, ncols, n):
    """Duplicates summed away or not, the sorted pairs and their first
    occurrences are those of a stable sort by row * ncols + col."""
    row, col = keys_of(n, nrows, 1, False), keys_of(n, ncols, 2, False)
    val = torch.ones(n, device="cuda")
    rowptr = torch.empty(nrows + 1, dtype=torch.int32, device="cuda")
    out = [torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(3)]
    vout = torch.empty(n, device="cuda")
    ws = torch.empty(nsd.nsd_build_workspace_size(n, max(nrows, ncols)), dtype=torch.uint8,
                     device="cuda")
    rowidx, colind, perm = out
    m = nsd.nsd_coo_to_csr(nrows, ncols, n, row, col, val, nsd.NSD_DUP_SUM, rowptr, rowidx, colind,
                           vout, perm, ws)
    key, order = torch.sort(row.long() * ncols + col, stable=True)
    first = torch.ones(n, dtype=torch.bool, device="cuda")
    first[1:] = key[1:] != key[:-1]
    assert m == int(first.sum())
    assert torch.equal(rowidx[:m].long() * ncols + colind[:m], key[first])
    assert torch.equal(perm[:m], order[first].int())
    counts = torch.unique_consecutive(key, return_counts=True)[1]
    assert torch.equal(vout[:m], counts.float())


@pytest.mark.parametrize("nrows,ncols", [(8000, 4097), (5000, 16_000), (100_000, 120_000),
                                         (200_000, 250_000)])
@pytest.mark.parametrize("n", [5000, 1 << 23])
def test_coo_to_csr_nine_bit_digits(nsd, nrows, ncols, n):
    """Pairs of 26, 27, 34 and 36 bits: digits of nine bits save a pass."""
    test_coo_to_csr_pair_keys(nsd, nrows, ncols, n)
