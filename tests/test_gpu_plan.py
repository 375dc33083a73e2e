"""Work plans (nsd_plan_build) against the definition evaluated segment by
segment on the host, bit for bit: at the edges of the builder's steps (1,024
segments) and block ranges, with empty, short, long and huge segments, runs
of empty segments across steps, and one segment holding everything."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nsd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2303_07030_amd import nsd as m
    return m


def reference(lengths, L):
    S = L + min(L, 32)
    out = dict(item_ptr=[], long_seg=[], long_first=[], huge_idx=[], chunk_item=[], chunk_ord=[],
               empty_seg=[])
    beg = pos = 0
    prev = None  # (window, long) of the nonempty segment before
    longest = 0
    for r, n in enumerate(lengths):
        n = int(n)
        if n == 0:
            out["empty_seg"].append(r)
            continue
        if n > S:
            chunks = -(-n // L)
            longest = max(longest, chunks)
            if chunks > 64:
                out["huge_idx"].append(len(out["long_seg"]))
            out["long_seg"].append(r)
            out["long_first"].append(len(out["item_ptr"]))
            for c in range(chunks):
                out["chunk_ord"].append(len(out["chunk_item"]))
                out["chunk_item"].append(len(out["item_ptr"]))
                out["item_ptr"].append(beg + c * L)
            prev = (None, True)
            pos += L
        else:
            if prev is None or prev[1] or prev[0] != pos // L:
                out["chunk_ord"].append(-1)
                out["item_ptr"].append(beg)
            prev = (pos // L, False)
            pos += n + 1
        beg += n
    nitems = len(out["item_ptr"])
    out["item_ptr"].append(beg)
    return out, nitems, longest


def lengths_of(kind, nseg, rng):
    if kind == "mixed":
        x = np.minimum((4 * rng.pareto(0.9, nseg)).astype(np.int64), 9000)
        x[rng.random(nseg) < 0.3] = 0
        return x
    if kind == "gaps":  # nonempty segments far apart
        x = np.zeros(nseg, dtype=np.int64)
        x[::997] = 3
        return x
    if kind == "long":  # every segment a few chunks
        return rng.integers(20, 200, nseg)
    x = np.zeros(nseg, dtype=np.int64)  # "one": everything in one segment
    x[nseg // 2] = 300_000
    return x


@pytest.mark.parametrize("kind", ["mixed", "gaps", "long", "one"])
@pytest.mark.parametrize("nseg,L", [(1, 16), (3, 2), (1023, 16), (1024, 16), (1025, 64),
                                    (5000, 2), (70_001, 16)])
def test_plan_matches_definition(nsd, kind, nseg, L):
    from paper_2303_07030_amd.operand import build_plan
    lengths = lengths_of(kind, nseg, np.random.default_rng(nseg + L))
    segptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    nnz = int(segptr[-1])
    plan = build_plan(nseg, nnz, torch.from_numpy(segptr).cuda(), L, "cuda")
    ref, nitems, longest = reference(lengths, L)
    assert plan.nitems == nitems and plan.longest_chunks == longest
    for field, count in (("long_seg", plan.nlong), ("huge_idx", plan.nhuge),
                         ("chunk_item", plan.nchunks), ("empty_seg", plan.nempty)):
        assert count == len(ref[field]), field
    for field, want in ref.items():
        got = plan._keep[field].cpu().numpy()[:len(want)]
        assert np.array_equal(got, np.asarray(want, dtype=np.int32)), field
