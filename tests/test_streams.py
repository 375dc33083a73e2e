"""Calls that enqueue work on a stream given to them: their scratch belongs to
that stream, so nothing else gets its memory while the work runs."""
import contextlib
import types

import numpy as np
import pytest
import torch

from paper_2303_07030_amd import nsd, operand


@pytest.fixture
def owners(monkeypatch):
    """On the CPU: which stream owned each allocation (None: the current one),
    by the allocation's address."""
    active, owner, keep = [None], {}, []

    @contextlib.contextmanager
    def stream(s):
        active.append(s)
        yield
        active.pop()

    def recorded(f):
        def g(*a, **kw):
            t = f(*a, **kw)
            owner[t.data_ptr()] = active[-1]
            keep.append(t)  # so that no address comes up twice
            return t
        return g

    monkeypatch.setattr(torch.cuda, "stream", stream)
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda h, device=None: ("external", h))
    monkeypatch.setattr(torch.cuda, "default_stream", lambda device=None: ("external", 0))
    monkeypatch.setattr(torch, "empty", recorded(torch.empty))
    monkeypatch.setattr(torch, "empty_like", recorded(torch.empty_like))
    return owner


@pytest.mark.parametrize("stream, owner", [(None, None), (0, ("external", 0)),
                                           (0x77, ("external", 0x77)), ("side", "side")])
def test_staging_of_values_in_csc_order_belongs_to_the_call(owners, monkeypatch, stream, owner):
    A = object.__new__(operand.DeviceCsr)
    A.nnz, A.val = 5, torch.arange(5, dtype=torch.float32)
    A.csc = types.SimpleNamespace(to_csc=types.SimpleNamespace(n=5))
    A.to_csc = A.csc.to_csc
    seen = []

    def permute(plan, src, dst, staging, s):
        seen.append((owners[staging.data_ptr()], s))

    monkeypatch.setattr(nsd, "nsd_permute_f32", permute)
    A.values_in_csc_order(stream)
    assert seen == [(owner, stream)]


@pytest.mark.parametrize("stream, owner", [(None, None), ("side", "side")])
def test_arrays_of_lex_order_belong_to_the_call(owners, monkeypatch, stream, owner):
    """Every array that a gather still reads or writes when lex_order returns."""
    coords = [torch.zeros(4, dtype=torch.int32) for _ in range(3)]
    held = {c.data_ptr() for c in coords}
    seen = []

    def gather(n, perm, src, dst, s):
        seen.extend(owners[t.data_ptr()] for t in (perm, src, dst) if t.data_ptr() not in held)

    monkeypatch.setattr(nsd, "nsd_gather_i32", gather)
    monkeypatch.setattr(nsd, "nsd_coo_mode_index", lambda *a: None)
    operand.lex_order(coords, (2, 2, 2), None, stream)
    assert len(seen) == 10 and set(seen) == {owner}


@pytest.mark.gpu
@pytest.mark.parametrize("raw", [False, True])
def test_values_in_csc_order_on_a_side_stream(raw):
    """The move runs while the current stream takes and writes memory of the
    staging's size."""
    rng = np.random.default_rng(3)
    n, nnz = 3000, 200_000
    key = np.sort(rng.choice(n * n, nnz, replace=False))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=n))]).astype(np.int32)
    val = rng.standard_normal(nnz).astype(np.float32)
    A = operand.DeviceCsr(n, n, rowptr, (key % n).astype(np.int32), val, perm_plans=True)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):  # the move waits behind some milliseconds of work
        x = torch.ones(2048, 2048, device="cuda")
        for _ in range(40):
            x = (x @ x).clamp_(max=1.0)
    valT = A.values_in_csc_order(side.cuda_stream if raw else side)
    taken = [torch.full((nnz,), float("nan"), device="cuda") for _ in range(4)]
    torch.cuda.synchronize()
    assert np.array_equal(valT.cpu().numpy(), val[A.perm.cpu().numpy()])
    assert all(torch.isnan(t).all().item() for t in taken)


@pytest.mark.gpu
def test_lex_order_on_a_side_stream():
    """The current stream takes memory of the sorts' arrays' size at once."""
    rng = np.random.default_rng(4)
    n, dims = 300_000, (70, 40, 500)
    key = rng.choice(int(np.prod(dims)), n, replace=False)
    coords = [c.astype(np.int32) for c in np.unravel_index(key, dims)]
    dev = [torch.from_numpy(c).cuda() for c in coords]
    ws = torch.empty(nsd.nsd_build_workspace_size(n, max(dims)), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    perm = operand.lex_order(dev, dims, ws, side)
    taken = [torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(6)]
    torch.cuda.synchronize()
    assert np.array_equal(perm.cpu().numpy(), np.argsort(key, kind="stable"))
    assert all((t == -1).all().item() for t in taken)
