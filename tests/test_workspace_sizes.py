"""Size queries (host only): a workspace sized for one input serves every
smaller one of its kind."""
import pytest

from paper_2303_07030_amd import nsd

# around the sizes at which the sort, its scans and its tiles change
SIZES = sorted({max(n + d, 0) for n in (0, 4096, 2048 * 2048, 1 << 22, 1 << 23, 1 << 24, 50_000_000)
                for d in (-8193, -1, 0, 1, 4097)})


@pytest.mark.parametrize("query", [
    lambda n: nsd.nsd_build_workspace_size(n, 1000),
    lambda n: nsd.nsd_build_workspace_size(n, 2**30),
    lambda n: nsd.nsd_ttv_build_workspace_size(3, (1000, 1000, 1000), n),
    lambda n: nsd.nsd_validate_coo_workspace_size((1000, 1000, 1000), n),
    nsd.nsd_perm_plan_workspace_size,
], ids=["build", "build_wide_keys", "ttv_build", "validate_coo", "perm_plan"])
def test_builders_workspace_grows_with_the_entries(query):
    sizes = [query(n) for n in SIZES]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("csc", [False, True])
@pytest.mark.parametrize("item_len, nitems", [(2, 2**29), (16, 2**26), (256, 2**22)])
def test_width_one_partials_follow_the_entries(item_len, nitems, csc):
    """The tiles of a width-1 pass are of entries (2,048 each of this many):
    two floats and a loss partial a tile whatever the plan's items, beside
    what the other passes of the width need."""
    nnz, ptr = 2**29, 0x1000  # no pointer is read
    plan = nsd.nsd_plan(item_len, nitems, 0, 0, 0, 0, ptr, 0, 0, 0, 0, 0)
    A = nsd.nsd_csr(nitems, nitems, nnz, ptr, ptr, ptr, ptr)
    At = nsd.nsd_csc(nitems, nitems, nnz, ptr, ptr, ptr, ptr)
    A.plan = At.plan = plan
    one, two = (nsd.nsd_workspace_size(A, At if csc else None, k) for k in (1, 2))
    assert one <= two + 2 * 16 * (nnz // 2048) + 1024


def test_item_length_hint():
    """Items of the narrow slots of widths that are no multiple of four stay
    short; those of wider ones and of one column a lane go with the entries."""
    for k in range(1, 65):
        lens = [nsd.nsd_plan_item_len(1 << p, k) for p in range(31)]
        assert min(lens) >= 2 and max(lens) <= 256
        assert nsd.nsd_plan_item_len(2**30, k) == (32 if k > 32 and k % 4 else 256)
    # one column a lane from 2^28 gathered floats on
    assert nsd.nsd_plan_item_len((1 << 28) // 31, 31) == 24
    assert nsd.nsd_plan_item_len((1 << 28) // 31 + 1, 31) == 128
