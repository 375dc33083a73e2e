#!/usr/bin/env python3
"""Benchmark of the sparse-gradient hot path on one MI355X.

A step is one pass of the whole path over one batch of inputs already
resident in HBM.  The default workload is the largest one, the GNN-layer
gradient (CSR adjacency of a 2.4M-node power-law graph with 60M weighted
edges, node features H and upstream G of 2.4M x 256): the loss
L = sum((A H) o G), the SDDMM gradient dA = <G_i, H_j> on A's pattern and
dH = A^T G, through nsd_loss_bilinear.  --workload selects the others (spmm:
the SpMM gradient 1/2 ||A B||^2; mf: sparse factorisation; cp: CP
decomposition; spmv: SMVM; and the pattern builders, the BATAX Jacobian, the
SpMM tangent and the order-4 CP).
Pattern-only preprocessing (row expansion, CSR -> CSC, work plans, mode
indexes) is timed separately and is not part of a step.

Prints one JSON line: the metric (gradient nonzeros per second), the roofline
of the step's dominant kernel (its algorithmic bytes over its average launch
duration, from HIP events recorded around every launch of that kernel during
the timed steps, against 8 TB/s), the same step replayed from a HIP graph
(beside the eager value, for the paths that need no host round trip), and
the fp64 oracle timed on this host on a bounded sample of the workload, as a
reported baseline.
"""
import argparse
import hashlib
import json
import os
import re
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
ITEM_LEN = None  # work-plan item length; None = the library's choice
CP_FIBERS = False  # order-N CP with its fiber level
PROBE_EVERY = 4  # timed steps per step whose dominant-kernel launches are bracketed
WORKLOAD_NAMES = {
    "spmm": "spmm_grad_100k_1M_zipf1.1_k64",
    "gnn": "gnn_bilinear_2.4M_60M_zipf1.05_k256",
    "mf": "mf_1M_500k_50M_zipf1.1_k128",
    "cp": "cp_10k3_20M_rank32",
    "spmv": "spmv_sum_1k_10k",
    "build": "build_coo_to_csr_csc_1M_500k_50M",
    "batax": "batax_jacobian_100k_1M_uniform",
    "jvp": "spmm_jvp_100k_1M_zipf1.1_k64",
    "cp4": "cp_order4_1000^4_20M_rank32",
}


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="gnn", choices=list(WORKLOAD_NAMES))
    ap.add_argument("--size", default="full")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cold-steps", type=int, default=10,
                    help="steps timed one by one after writing a 512 MiB buffer (no cached "
                         "operand left in L2 or the 256 MB MALL); 0 to skip")
    ap.add_argument("--item-len", type=int, default=None,
                    help="work-plan item length (default: the library's choice)")
    ap.add_argument("--replicate", type=int, default=0,
                    help="input replicate (0: the headline inputs; 1, 2: same recipe, other "
                         "seeds, for variance)")
    ap.add_argument("--cp-fibers", action="store_true",
                    help="order-N CP with its fiber level (the factor row of each run of equal "
                         "coordinate gathered once)")
    ap.add_argument("--tangents", type=int, default=1, metavar="M",
                    help="jvp workload: M tangents per step, in one nsd_spmm_jvp_batch call "
                         "(J V for a batch of M directions) when M > 1")
    ap.add_argument("--cpu-seconds", type=float, default=12.0)
    ap.add_argument("--profile-only", action="store_true",
                    help="warmup + steps only (for rocprofv3), no JSON line")
    ap.add_argument("--calibrate-copy", type=int, default=0, metavar="BYTES",
                    help="with --profile-only: also copy a buffer of BYTES once (a plain copy "
                         "kernel of known size, to scale the HBM counters)")
    return ap.parse_args()


# The source file that holds each probed kernel; a kernel's digest covers
# that file, every shared header and the public header.
KERNEL_SOURCE = {"frob_row": "segreduce.hip", "sgr_main": "segreduce.hip",
                 "sddmm": "segreduce.hip", "frob_col": "dual.hip", "dual": "dual.hip",
                 "mf": "dual.hip", "cp": "cp.hip", "sort": "build.hip", "jvp": "jvp.hip",
                 "cpn": "cpn.hip", "perm": "perm.hip", "batax_rows": "batax.hip"}
# Passes of one column (the spmv workload) have kernels of their own.
WIDTH_ONE_SOURCE = {k: "vec1.hip" for k in ("sgr_main", "sddmm", "dual")}


def source_digest(kernel=None, workload=None):
    """Digest of the sources a kernel is built from (all sources if None)."""
    h = hashlib.sha256()
    d = os.path.join(ROOT, "paper_2303_07030_amd", "csrc")
    files = sorted(os.listdir(d))
    if kernel is not None:
        own = KERNEL_SOURCE[kernel]
        if workload == "spmv":
            own = WIDTH_ONE_SOURCE.get(kernel, own)
        files = [f for f in files if f.endswith(".hpp") or f == own]
    paths = [os.path.join(d, f) for f in files] + [os.path.join(ROOT, "include", "nsd.h")]
    for path in paths:
        with open(path, "r", encoding="utf-8") as fh:
            h.update(_code_only(fh.read()).encode())
    return h.hexdigest()[:16]


def _code_only(text):
    """Source text without comments and blank space, so that edits to
    comments alone keep a kernel's digest."""
    text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
    text = re.sub(r"//[^\n]*", " ", text)
    return " ".join(text.split())


def committed_traffic(kernel, workload):
    """HBM bytes per launch from the committed counter summary, if it was
    taken on the current kernel sources (else None)."""
    path = os.path.join(ROOT, "profiles", f"{kernel}_{workload}_counters.md")
    if not os.path.exists(path):
        return None
    text = open(path).read()
    m = re.search(r"traffic_bytes_per_launch:\s*([0-9.eE+]+)", text)
    s = re.search(r"source_digest:\s*([0-9a-f]+)", text)
    if not m or not s or s.group(1) != source_digest(kernel, workload):
        return None
    return float(m.group(1))


# ----------------------------------------------------------------- setups

class Setup:
    """Operands in HBM, one step function and the kernels worth a roofline:
    name -> (kernel id, algorithmic bytes per launch).  `graphable`: the
    step is launches only (no host synchronisation), so it can be captured
    in a HIP graph."""
    graphable = True


def setup_spmm(d, dev, torch, nsd, ops):
    A = ops.DeviceCsr(d["nrows"], d["ncols"], d["rowptr"], d["colind"], d["val"], device=dev,
                      k_hint=d["k"], item_len=ITEM_LEN)
    k, nnz, nr, nc = d["k"], A.nnz, A.nrows, A.ncols
    B = torch.from_numpy(d["B"]).to(dev)
    C = torch.empty((nr, k), dtype=torch.float32, device=dev)
    dB = torch.empty((nc, k), dtype=torch.float32, device=dev)
    dA = torch.empty(nnz, dtype=torch.float32, device=dev)
    loss = torch.empty(1, dtype=torch.float64, device=dev)
    ws = A.workspace(k)
    S = Setup()
    S.A, S.nnz, S.k = A, nnz, k
    S.step = lambda: nsd.nsd_loss_frob_spmm(A.desc, A.csc, B, k, 1.0, C, loss, dA, dB, ws)
    S.kernels = {
        # rowidx, colind, val in; B read once, C written once
        "frob_row": 3 * 4 * nnz + 4 * k * (nr + nc),
        # colidx, rowind, perm, val (through perm) in, dA out; C and B read
        # once, dB written once
        "frob_col": 5 * 4 * nnz + 4 * k * (nr + 2 * nc),
    }
    return S


def setup_gnn(d, dev, torch, nsd, ops):
    A = ops.DeviceCsr(d["nrows"], d["ncols"], d["rowptr"], d["colind"], d["val"], device=dev,
                      k_hint=d["k"], item_len=ITEM_LEN)
    k, nnz, nr, nc = d["k"], A.nnz, A.nrows, A.ncols
    H = torch.from_numpy(d["H"]).to(dev)
    G = torch.from_numpy(d["G"]).to(dev)
    dH = torch.empty((nc, k), dtype=torch.float32, device=dev)
    dA = torch.empty(nnz, dtype=torch.float32, device=dev)
    loss = torch.empty(1, dtype=torch.float64, device=dev)
    ws = A.workspace(k)
    S = Setup()
    S.A, S.nnz, S.k = A, nnz, k
    S.step = lambda: nsd.nsd_loss_bilinear(A.desc, A.csc, H, G, k, 1.0, loss, dA, dH, ws)
    if A.csc.to_csc.n:
        S.kernels = {
            # one column pass: colidx, rowind, the values in CSC order in and
            # dA in CSC order out; G and H read once, dH written once
            "dual": 4 * 4 * nnz + 4 * k * (nr + 2 * nc),
            # each move of nnz values (before and after the pass): read once,
            # written once
            "perm": 2 * 4 * nnz,
        }
    else:
        S.kernels = {
            # one column pass: colidx, rowind, perm, val (through perm) in, dA
            # out; G and H read once, dH written once
            "dual": 5 * 4 * nnz + 4 * k * (nr + 2 * nc),
        }
    return S


def setup_mf(d, dev, torch, nsd, ops):
    A = ops.DeviceCsr.from_coo(d["nrows"], d["ncols"], d["row"], d["col"], d["val"], device=dev,
                               k_hint=d["k"], item_len=ITEM_LEN)
    valT = A.values_in_csc_order()
    k, nnz, nr, nc = d["k"], A.nnz, A.nrows, A.ncols
    U = torch.from_numpy(d["U"]).to(dev)
    V = torch.from_numpy(d["V"]).to(dev)
    dU = torch.empty((nr, k), dtype=torch.float32, device=dev)
    dV = torch.empty((nc, k), dtype=torch.float32, device=dev)
    loss = torch.empty(1, dtype=torch.float64, device=dev)
    ws = A.workspace(k)
    S = Setup()
    S.A, S.nnz, S.k = A, nnz, k
    S.step = lambda: nsd.nsd_loss_mf(A.desc, A.csc, valT, U, V, k, 1.0, loss, dU, dV, ws)
    S.kernels = {
        # both passes: (segment, gathered index, value) in per entry per pass;
        # U and V read once, dU and dV written once
        "mf": 2 * 3 * 4 * nnz + 2 * 4 * k * (nr + nc),
    }
    return S


def setup_cp(d, dev, torch, nsd, ops):
    X = ops.DeviceCoo3(d["dims"], d["i"], d["j"], d["k"], d["val"], device=dev,
                       rank_hint=d["rank"], item_len=ITEM_LEN)
    R, nnz = d["rank"], X.nnz
    F = [torch.from_numpy(d[f]).to(dev) for f in ("F1", "F2", "F3")]
    dF = [torch.empty((X.dims[m], R), dtype=torch.float32, device=dev) for m in range(3)]
    dX = torch.empty(nnz, dtype=torch.float32, device=dev)
    loss = torch.empty(1, dtype=torch.float64, device=dev)
    ws = X.workspace(R)
    S = Setup()
    S.A, S.nnz, S.k = X, nnz, R
    S.step = lambda: nsd.nsd_loss_cp(X.desc, *F, R, 1.0, loss, dX, *dF, ws)
    fac = 4 * R * sum(X.dims)
    S.kernels = {
        # three passes of (mode coordinate, two coordinates, value); the
        # first also reads perm and writes the residual; factors read and
        # gradients written once
        "cp": 3 * 4 * 4 * nnz + 2 * 4 * nnz + 2 * fac,
    }
    return S


def setup_spmv(d, dev, torch, nsd, ops):
    A = ops.DeviceCsr(d["nrows"], d["ncols"], d["rowptr"], d["colind"], d["val"], device=dev,
                      k_hint=1, item_len=ITEM_LEN)
    nnz, nr, nc = A.nnz, A.nrows, A.ncols
    x = torch.from_numpy(d["x"]).to(dev)
    dx = torch.empty(nc, dtype=torch.float32, device=dev)
    dA = torch.empty(nnz, dtype=torch.float32, device=dev)
    loss = torch.empty(1, dtype=torch.float64, device=dev)
    ws = A.workspace(1)
    S = Setup()
    S.A, S.nnz, S.k = A, nnz, 1
    S.step = lambda: nsd.nsd_loss_sum_spmv(A.desc, A.csc, x, 1.0, loss, dA, dx, ws)
    S.kernels = {
        # one column pass: colidx, rowind, perm, val (through perm) in, dA
        # out; x read once, dx written once
        "dual": 5 * 4 * nnz + 2 * 4 * nc,
    }
    return S


def _sort_passes(*max_keys):
    """Digit passes of the library's radix sort by keys < max_keys together:
    8 bits a pass, 9 where they save one, 10 where they save a third of them."""
    bits = sum(max(m - 1, 0).bit_length() for m in max_keys)
    narrow, nine, wide = (max(1, -(-bits // b)) for b in (8, 9, 10))
    return nine if nine < narrow else wide if 3 * wide <= 2 * narrow else narrow


def setup_build(d, dev, torch, nsd, ops):
    """Pattern preparation of the factorisation input (50M unsorted COO
    entries): COO -> CSR (a1), CSR -> CSC (a2) and the value permute (a3)."""
    nr, nc = d["nrows"], d["ncols"]
    row, col = (torch.from_numpy(d[x]).to(dev) for x in ("row", "col"))
    val = torch.from_numpy(d["val"]).to(dev)
    n = int(row.numel())

    def i32(m):
        return torch.empty(max(m, 1), dtype=torch.int32, device=dev)

    rowptr, rowidx, colind, perm = i32(nr + 1), i32(n), i32(n), i32(n)
    colptr, colidx, rowind, permc = i32(nc + 1), i32(n), i32(n), i32(n)
    vout = torch.empty(n, dtype=torch.float32, device=dev)
    valT = torch.empty(n, dtype=torch.float32, device=dev)
    ws = torch.empty(max(nsd.nsd_build_workspace_size(n, max(nr, nc)),
                         nsd.nsd_build_workspace_size(n, nc)), dtype=torch.uint8, device=dev)

    def step():
        m = nsd.nsd_coo_to_csr(nr, nc, n, row, col, val, nsd.NSD_DUP_ERROR, rowptr, rowidx,
                               colind, vout, perm, ws)
        A = nsd.csr_desc(nr, nc, rowptr, rowidx[:m], colind[:m], vout[:m])
        nsd.nsd_csr_to_csc(A, colptr, colidx, rowind, permc, ws)
        nsd.nsd_gather_f32(m, permc, vout, valT)

    S = Setup()
    S.A, S.nnz, S.k, S.step = None, n, 0, step
    S.graphable = False  # the builders read counts back to the host
    # scatter passes: by the pair (row, column) (COO -> CSR), each carrying the
    # input position, the row and the value (32 B per entry read and written);
    # by column (CSR -> CSC) carrying the CSR slot and the row (24 B); a sort's
    # first pass reads no position (its own index): 4 B less
    pairs, cols = _sort_passes(nr, nc), _sort_passes(nc)
    launches = pairs + cols
    total = (32 * n * pairs - 4 * n) + (24 * n * cols - 4 * n)
    S.kernels = {"sort": total / launches}
    return S


def setup_batax(d, dev, torch, nsd, ops):
    """Jacobian of the BATAX kernel, J = beta A^T A (an output pattern that
    is not an input's): A's CSC, then each row of J gathered, sorted in LDS
    and summed in fixed order (rows of at most 512 terms; else every product
    expanded and sorted twice through HBM)."""
    A = ops.DeviceCsr(d["nrows"], d["ncols"], d["rowptr"], d["colind"], d["val"], device=dev,
                      build_csc=False)
    ws0 = torch.empty(256, dtype=torch.uint8, device=dev)
    P = nsd.nsd_batax_pairs(A.desc, ws0)  # depends on the pattern only
    ws = torch.empty(nsd.nsd_batax_workspace_size(A.desc, P), dtype=torch.uint8, device=dev)
    n = A.ncols
    jrowptr = torch.empty(n + 1, dtype=torch.int32, device=dev)
    jcol = torch.empty(max(P, 1), dtype=torch.int32, device=dev)
    jval = torch.empty(max(P, 1), dtype=torch.float32, device=dev)
    S = Setup()
    S.graphable = False  # the key count comes back to the host
    nk = nsd.nsd_batax_jacobian(A.desc, d["beta"], P, jrowptr, jcol, jval, ws)
    S.A, S.nnz, S.k = A, nk, 0
    S.step = lambda: nsd.nsd_batax_jacobian(A.desc, d["beta"], P, jrowptr, jcol, jval, ws)
    S.pairs = P
    nnz = A.nnz
    # the CSC of A: a radix sort of the nnz column indices carrying each
    # entry's row and value (key and two payloads read and written per pass)
    S.kernels = {"sort": 24 * nnz,
                 # per stored entry: the CSC slot's row and value and the
                 # row's bounds (16 B); per product: k and a_ik (8 B); per
                 # key of J: its column and value (8 B); per row of J: its
                 # column bounds and key count
                 "batax_rows": 16 * nnz + 8 * P + 8 * nk + 12 * n}
    return S


def setup_jvp(d, dev, torch, nsd, ops):
    """Forward-mode tangent of C = A B on the SpMM workload: C and
    dC = dA B + A dB in one pass (tangents dA on A's keys and dB ~ N(0,1),
    drawn from the workload's fourth stream)."""
    A = ops.DeviceCsr(d["nrows"], d["ncols"], d["rowptr"], d["colind"], d["val"], device=dev,
                      k_hint=d["k"], item_len=ITEM_LEN, build_csc=False)
    k, nnz, nr, nc = d["k"], A.nnz, A.nrows, A.ncols
    B = torch.from_numpy(d["B"]).to(dev)
    dA = torch.from_numpy(d["dval"]).to(dev)
    dB = torch.from_numpy(d["dB"]).to(dev)
    C = torch.empty((nr, k), dtype=torch.float32, device=dev)
    dC = torch.empty((nr, k), dtype=torch.float32, device=dev)
    ws = A.workspace(2 * k)
    S = Setup()
    S.A, S.nnz, S.k = A, nnz, k
    M = d.get("tangents", 1)
    if M == 1:
        S.step = lambda: nsd.nsd_spmm_jvp(A.desc, dA, B, dB, k, C, dC, ws)
        # rowidx, colind, val, dA in; B and dB read once, C and dC written once
        S.kernels = {"jvp": 4 * 4 * nnz + 2 * 4 * k * (nr + nc)}
        return S
    # a batch of M tangents: groups of four per launch, each reading A's
    # entries and B once and, per tangent, dA_t and dB_t once and writing
    # dC_t once (C with the first group)
    dC = torch.empty((M, nr, k), dtype=torch.float32, device=dev)
    ws = torch.empty(nsd.nsd_spmm_jvp_batch_workspace_size(A.desc, k), dtype=torch.uint8,
                     device=dev)
    S.nnz = nnz * M
    S.step = lambda: nsd.nsd_spmm_jvp_batch(A.desc, M, dA, B, dB, k, C, dC, ws)
    groups = [min(4, M - g) for g in range(0, M, 4)]
    per = [3 * 4 * nnz + 4 * k * nc + g * (4 * nnz + 4 * k * (nc + nr)) for g in groups]
    S.kernels = {"jvp": (sum(per) + 4 * k * nr) / len(groups)}
    return S


def setup_cp4(d, dev, torch, nsd, ops):
    """CP gradient of an order-4 tensor through the order-N entry point."""
    X = ops.DeviceCooN(d["dims"], d["coords"], d["val"], device=dev, rank_hint=d["rank"],
                       item_len=ITEM_LEN, fibers=CP_FIBERS)
    R, nnz, N = d["rank"], X.nnz, len(d["dims"])
    F = [torch.from_numpy(f).to(dev) for f in d["F"]]
    dF = [torch.empty((X.dims[m], R), dtype=torch.float32, device=dev) for m in range(N)]
    dX = torch.empty(nnz, dtype=torch.float32, device=dev)
    loss = torch.empty(1, dtype=torch.float64, device=dev)
    ws = X.workspace(R)
    S = Setup()
    S.A, S.nnz, S.k = X, nnz, R
    S.step = lambda: nsd.nsd_loss_cpn(X.desc, F, R, 1.0, loss, dX, dF, ws)
    # N passes of (mode coordinate, N-1 coordinates, value); the first also
    # reads perm and writes the residual; factors read and gradients
    # written once
    S.kernels = {"cpn": N * (N + 1) * 4 * nnz + 2 * 4 * nnz + 2 * 4 * R * sum(X.dims)}
    return S


SETUPS = {"spmm": setup_spmm, "gnn": setup_gnn, "mf": setup_mf, "cp": setup_cp,
          "spmv": setup_spmv, "build": setup_build, "batax": setup_batax, "jvp": setup_jvp,
          "cp4": setup_cp4}


# ------------------------------------------------------------ measurement

def probe_events(torch, n):
    """n (start, stop) HIP event pairs, created (recorded once) before they
    are handed to the library."""
    starts = [torch.cuda.Event(enable_timing=True) for _ in range(n)]
    stops = [torch.cuda.Event(enable_timing=True) for _ in range(n)]
    for e in starts + stops:
        e.record()
    return starts, stops


def probe_durations(torch, nsd, kernel, step, n_events):
    """Sets a probe on `kernel`: the library records HIP event pair i % n_events
    around its i-th launch from now on (collect() reads them back)."""
    # events are created lazily by torch: record once before handing them over
    starts, stops = probe_events(torch, n_events)
    torch.cuda.synchronize()
    nsd.nsd_probe_set(nsd.KERNEL_IDS[kernel], [e.cuda_event for e in starts],
                      [e.cuda_event for e in stops])
    return starts, stops


def collect(torch, nsd, starts, stops):
    torch.cuda.synchronize()
    n = nsd.nsd_probe_count()
    nsd.nsd_probe_clear()
    m = min(n, len(starts))
    if m == 0:
        return None, 0
    return float(np.mean([starts[i].elapsed_time(stops[i]) for i in range(m)])), n


def main():
    args = parse()
    global ITEM_LEN, CP_FIBERS
    ITEM_LEN = args.item_len
    CP_FIBERS = args.cp_fibers
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}): the library measures "
              "one GPU's share; a multi-GPU layout is described, not implemented",
              file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2303_07030_amd import nsd, synth
    from paper_2303_07030_amd import operand as ops

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)

    synth.VERBOSE = True  # progress lines on stderr while the inputs are drawn
    t0 = time.perf_counter()
    d = synth.make({"build": "mf", "jvp": "spmm"}.get(args.workload, args.workload), args.size,
                   replicate=args.replicate)
    if args.workload == "jvp":
        g = synth.streams("spmm", args.replicate)[3]  # the fourth stream: the tangents
        M = d["tangents"] = args.tangents
        lead = () if M == 1 else (M,)
        d["dval"] = g.standard_normal(lead + (len(d["val"]),), dtype=np.float32)
        d["dB"] = g.standard_normal(lead + d["B"].shape, dtype=np.float32)
    gen_s = time.perf_counter() - t0
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    S = SETUPS[args.workload](d, dev, torch, nsd, ops)
    torch.cuda.synchronize()
    prep_ms = (time.perf_counter() - t0) * 1e3

    for _ in range(args.warmup):
        S.step()
    torch.cuda.synchronize()
    if args.profile_only:
        if args.calibrate_copy:
            n = args.calibrate_copy // 4
            src = torch.ones(n, dtype=torch.float32, device=dev)
            dst = torch.empty_like(src)
            torch.cuda.synchronize()
            dst.copy_(src)
            torch.cuda.synchronize()
            del src, dst
        for _ in range(args.steps):
            S.step()
        torch.cuda.synchronize()
        return

    # which kernel dominates a step: probe each candidate over a few steps
    per_kernel, per_step_launches = {}, {}
    for name in S.kernels:
        starts, stops = probe_durations(torch, nsd, name, S.step, 32)
        for _ in range(4):
            S.step()
        ms, n = collect(torch, nsd, starts, stops)
        per_kernel[name] = ms
        per_step_launches[name] = max(1, -(-n // 4))
    dom = max(per_kernel, key=lambda n: per_kernel[n] or 0.0)

    # timed region: exactly K steps; in every PROBE_EVERY-th step the library
    # records HIP events around each launch of the dominant kernel (a bracket
    # costs a few microseconds of event processing on the stream, so not
    # every step carries one)
    m = per_step_launches[dom]
    probed = [i for i in range(args.steps) if i % PROBE_EVERY == 0]
    brackets = {i: probe_events(torch, m) for i in probed}
    counts = {}
    kid = nsd.KERNEL_IDS[dom]
    torch.cuda.synchronize()
    t_start = torch.cuda.Event(enable_timing=True)
    t_end = torch.cuda.Event(enable_timing=True)
    t_start.record()
    for i in range(args.steps):
        if i in brackets:
            a, b = brackets[i]
            nsd.nsd_probe_set(kid, [e.cuda_event for e in a], [e.cuda_event for e in b])
        S.step()
        if i in brackets:
            counts[i] = nsd.nsd_probe_count()
            nsd.nsd_probe_clear()
    t_end.record()
    torch.cuda.synchronize()
    ms_per_step = t_start.elapsed_time(t_end) / args.steps
    durs = [brackets[i][0][j].elapsed_time(brackets[i][1][j])
            for i in probed for j in range(min(counts[i], m))]
    dom_ms, dom_launches = (float(np.mean(durs)) if durs else None), len(durs)

    algo = S.kernels[dom]
    achieved = algo / (dom_ms * 1e-3) / 1e9
    # the committed counters were taken on the workload's default inputs and
    # arguments; any other configuration has none
    default_config = (args.size == "full" and args.item_len is None and args.replicate == 0
                      and args.tangents == 1 and not args.cp_fibers)
    traffic = committed_traffic(dom, args.workload) if default_config else None
    roofline = {
        "bound": "hbm", "kernel": dom, "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS,
        "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4),
        "traffic": traffic,
        # the counters' bytes (FETCH_SIZE + WRITE_SIZE, scaled by a plain
        # copy) over the same average launch duration
        "traffic_GBps": None if traffic is None else round(traffic / (dom_ms * 1e-3) / 1e9, 1),
        "traffic_frac": None if traffic is None else
        round(traffic / (dom_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
        "algo_bytes_per_launch": int(algo), "avg_launch_ms": round(dom_ms, 5),
        "launches_timed": dom_launches,
    }
    kernels = {n: {"ms": None if v is None else round(v, 5), "algo_bytes": int(S.kernels[n]),
                   "GBps": None if not v else round(S.kernels[n] / (v * 1e-3) / 1e9, 1)}
               for n, v in per_kernel.items()}

    per_step = single_steps(torch, S, args.steps)
    cold = cold_steps(torch, dev, S, args) if args.cold_steps else None
    graph = graph_steps(torch, S, args.steps) if S.graphable else None
    stream = stream_copy(torch, dev)
    stream["frac"] = round(achieved / stream["copy_GBps"], 4)

    cpu = None
    if not args.no_cpu_baseline:
        cpu = cpu_baseline(args, d)

    build = args.workload == "build"
    metric = {"build": "pattern entries/sec (COO->CSR, CSR->CSC, value permute)",
              "batax": "Jacobian nonzeros/sec (BATAX, beta A^T A)"}.get(
                  args.workload, "gradient nonzeros/sec (forward+backward)")
    if args.workload == "jvp":
        metric = "tangent nonzeros/sec (forward-mode dC = dA B + A dB)"
        if args.tangents > 1:
            metric = (f"tangent nonzeros/sec (J V for a batch of {args.tangents} tangents "
                      "dC_t = dA_t B + A dB_t; nnz x tangents per step)")
    out = {
        "metric": metric,
        "value": round(S.nnz / (ms_per_step * 1e-3), 1),
        "unit": "entries/s" if build else "nnz/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 5),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": WORKLOAD_NAMES[args.workload] if args.size == "full"
                   else f"{args.workload}_{args.size}", "replicate": args.replicate,
                   "nnz": S.nnz, "k": S.k,
                   "item_len": S.A.item_len if S.A is not None else None,
                   **({"tangents": args.tangents} if args.workload == "jvp" else {})},
        "roofline": roofline,
        "kernels": kernels,
        "preprocess_ms": round(prep_ms, 2), "generate_s": round(gen_s, 1),
        "per_step": per_step,
        "cold": cold,
        "graph": graph,
        "achievable": stream,
        "cpu_baseline": cpu,
        "inputs": {"numpy": np.__version__, "index_sha256": index_digest(d),
                   "seeds": f"PCG64 from SeedSequence(entropy={synth.ENTROPY}, "
                            f"spawn_key=(workload, replicate={args.replicate}))"},
        "source_digest": source_digest(),
    }
    print(json.dumps(out))


def index_digest(d):
    """sha256 of the workload's index arrays (every integer array, in key
    order), so that runs on different hosts can be checked for identical
    patterns."""
    h = hashlib.sha256()
    for key in sorted(d):
        v = d[key]
        for a in (v if isinstance(v, (list, tuple)) else [v]):
            if isinstance(a, np.ndarray) and a.dtype.kind in "iu":
                h.update(key.encode())
                h.update(memoryview(np.ascontiguousarray(a)).cast("B"))
    return h.hexdigest()[:16]


def cpu_model():
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def single_steps(torch, S, steps):
    """Each of `steps` warm steps between its own pair of HIP events (queued
    back to back, one synchronisation at the end): median and minimum."""
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
          for _ in range(steps)]
    torch.cuda.synchronize()
    for a, b in ev:
        a.record()
        S.step()
        b.record()
    torch.cuda.synchronize()
    t = [a.elapsed_time(b) for a, b in ev]
    return {"median_ms": round(float(np.median(t)), 5), "min_ms": round(float(min(t)), 5),
            "steps": steps}


def graph_steps(torch, S, steps, per_graph=10):
    """The step captured `per_graph` times in a row in one HIP graph, the
    graph replayed until `steps` steps ran, between HIP events: the host's
    per-call cost (argument marshalling, launch) leaves the step.  The
    eager steps stay the reported value."""
    per = per_graph if steps % per_graph == 0 else 1
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        S.step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        for _ in range(per):
            S.step()
    g.replay()
    torch.cuda.synchronize()
    a = torch.cuda.Event(enable_timing=True)
    b = torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(steps // per):
        g.replay()
    b.record()
    torch.cuda.synchronize()
    ms = a.elapsed_time(b) / steps
    return {"ms_per_step": round(ms, 5), "value": round(S.nnz / (ms * 1e-3), 1),
            "steps": steps, "steps_per_graph": per,
            "note": "consecutive steps captured in one HIP graph, replayed"}


def stream_copy(torch, dev, nbytes=1 << 30, reps=10):
    """Achievable streaming rate on this GPU: a plain device-to-device copy
    of 1 GiB (read + write bytes over time, median of reps), beside which the
    dominant kernel's algorithmic rate is also given as a fraction."""
    n = nbytes // 4
    src = torch.ones(n, dtype=torch.float32, device=dev)
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    times = []
    for _ in range(reps):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        dst.copy_(src)
        e1.record()
        torch.cuda.synchronize()
        times.append(e0.elapsed_time(e1))
    ms = float(np.median(times))
    del src, dst
    return {"copy_GBps": round(2 * nbytes / (ms * 1e-3) / 1e9, 1), "copy_bytes": nbytes,
            "note": "plain device copy, read + write bytes; frac = roofline.achieved / copy"}


def cold_steps(torch, dev, S, args):
    """Steps with cold caches: before each, a 512 MiB buffer is rewritten
    (untimed), then the step alone is timed between HIP events."""
    flush = torch.empty(128 << 20, dtype=torch.float32, device=dev)
    times = []
    for _ in range(args.cold_steps):
        flush.fill_(1.0)
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        a.record()
        S.step()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    del flush
    ms = float(np.median(times))
    return {"ms_per_step": round(ms, 5), "value": round(S.nnz / (ms * 1e-3), 1),
            "steps": args.cold_steps, "note": "median step after a 512 MiB cache flush"}


# ------------------------------------------------------------ CPU baseline

def _sample(args, d):
    """A bounded sample of the workload for the oracle: the whole input when
    it is small, else a prefix (leading rows / entries) of it."""
    w = args.workload
    if w in ("spmm", "spmv", "jvp"):
        return d, "the full workload"
    if w == "gnn":
        # leading rows; the columns they touch are renumbered so that only
        # the needed rows of H and of dH are formed
        rp = d["rowptr"]
        nr = int(np.searchsorted(rp, 150_000, side="right")) - 1
        e = int(rp[nr])
        cols, colind = np.unique(d["colind"][:e], return_inverse=True)
        s = dict(d, nrows=nr, ncols=len(cols), rowptr=rp[: nr + 1],
                 colind=colind.astype(np.int32), val=d["val"][:e], G=d["G"][:nr],
                 H=d["H"][cols])
        return s, f"rows 0..{nr - 1} ({e} nnz) of the workload with the {len(cols)} columns they use"
    if w == "cp4":
        e = 1_000_000
        return dict(d, coords=[c[:e] for c in d["coords"]], val=d["val"][:e]), \
            f"the first {e} COO entries of the workload, full factors"
    if w == "batax":
        rp = d["rowptr"]
        nr = 12_000
        e = int(rp[nr])
        return dict(d, nrows=nr, rowptr=rp[: nr + 1], colind=d["colind"][:e], val=d["val"][:e]), \
            f"rows 0..{nr - 1} ({e} entries) of the workload"
    if w == "build":
        e = 4_000_000
        return dict(d, row=d["row"][:e], col=d["col"][:e], val=d["val"][:e]), \
            f"the first {e} COO entries of the workload"
    if w == "mf":
        e = 400_000
        rows, row = np.unique(d["row"][:e], return_inverse=True)
        cols, col = np.unique(d["col"][:e], return_inverse=True)
        s = dict(d, nrows=len(rows), ncols=len(cols), row=row.astype(np.int32),
                 col=col.astype(np.int32), val=d["val"][:e], U=d["U"][rows], V=d["V"][cols])
        return s, f"the first {e} COO entries of the workload with their rows of U and V"
    e = 1_000_000
    return dict(d, i=d["i"][:e], j=d["j"][:e], k=d["k"][:e], val=d["val"][:e]), \
        f"the first {e} COO entries of the workload, full factors"


def cpu_baseline(args, d):
    """The fp64 oracle, unchanged, on a bounded sample of the workload, on
    every host CPU visible to the process (its gradient loops split their
    outputs by owner, its loss scans by fixed chunks) and on one thread (the
    paper's own protocol): whole passes (DOK build + every output) repeated
    for about cpu_seconds each."""
    import oracle
    ncpu = len(os.sched_getaffinity(0))
    try:
        oracle.set_threads(ncpu)
        leg = _cpu_leg(args, d, ncpu)
        oracle.set_threads(1)
        leg["single_thread"] = _cpu_leg(args, d, 1)
    finally:
        oracle.set_threads(1)
    return leg


def _cpu_leg(args, d, threads):
    import oracle
    s, what = _sample(args, d)
    w = args.workload

    if w in ("spmm", "spmv", "gnn", "batax", "jvp"):
        nrows, ncols = s["nrows"], s["ncols"]
        rows = np.repeat(np.arange(nrows, dtype=np.int32), np.diff(s["rowptr"]))
        nnz = len(s["colind"]) * s.get("tangents", 1)
    elif w in ("mf", "build"):
        nnz = len(s["row"])
    elif w == "cp4":
        nnz = len(s["val"])
    else:
        nnz = len(s["i"])

    dok_s = [0.0]

    def dok(*a):
        t = time.perf_counter()
        D = oracle.Dok(*a)
        dok_s[0] += time.perf_counter() - t
        return D

    def one_pass():
        if w == "spmm":
            D = dok((nrows, ncols), (rows, s["colind"]), s["val"])
            k = s["k"]
            Cr, Cm = oracle.spmm(D, s["B"], k)
            oracle.loss_half_sq(Cr, Cm)
            oracle.sddmm(D, Cr, s["B"], k, rows, s["colind"], Xmag=Cm)
            oracle.spmm_t(D, Cr, k, Gmag=Cm)
        elif w == "spmv":
            D = dok((nrows, ncols), (rows, s["colind"]), s["val"])
            oracle.loss_sum_spmv(D, s["x"])
            oracle.sddmm(D, None, s["x"].reshape(-1, 1), 1, rows, s["colind"])
            oracle.spmm_t(D, None, 1)
        elif w == "gnn":
            D = dok((nrows, ncols), (rows, s["colind"]), s["val"])
            k = s["k"]
            oracle.loss_bilinear(D, s["G"], s["H"], k)
            oracle.sddmm(D, s["G"], s["H"], k, rows, s["colind"])
            oracle.spmm_t(D, s["G"], k)
        elif w == "cp4":
            D = dok(s["dims"], s["coords"], s["val"])
            oracle.cpn_loss(D, s["F"], s["rank"])
            oracle.cpn_resid(D, s["F"], s["rank"], s["coords"])
            for m in range(len(s["dims"])):
                oracle.cpn_grad(D, s["F"], s["rank"], m)
        elif w == "jvp":
            D = dok((nrows, ncols), (rows, s["colind"]), s["val"])
            M = s.get("tangents", 1)
            for t in range(M):
                dv, dB = (s["dval"], s["dB"]) if M == 1 else (s["dval"][t], s["dB"][t])
                dD = dok((nrows, ncols), (rows, s["colind"]), dv)
                oracle.spmm_jvp(D, dD, s["B"], dB, s["k"])
        elif w == "batax":
            D = dok((nrows, ncols), (rows, s["colind"]), s["val"])
            one_pass.nk = len(oracle.batax_jacobian(D, s["beta"])[1])
        elif w == "build":
            D = dok((s["nrows"], s["ncols"]), (s["row"], s["col"]), s["val"])
            _, ci, _, _ = oracle.coo_to_csr(D)
            oracle.stable_sort_by_key(ci, s["ncols"])
        elif w == "mf":
            D = dok((s["nrows"], s["ncols"]), (s["row"], s["col"]), s["val"])
            k = s["k"]
            oracle.mf_loss(D, s["U"], s["V"], k)
            oracle.mf_grad(D, s["U"], s["V"], k, 0)
            oracle.mf_grad(D, s["U"], s["V"], k, 1)
        else:
            D = dok(s["dims"], (s["i"], s["j"], s["k"]), s["val"])
            F = (s["F1"], s["F2"], s["F3"])
            oracle.cp_loss(D, *F, s["rank"])
            oracle.cp_resid(D, *F, s["rank"], s["i"], s["j"], s["k"])
            for m in range(3):
                oracle.cp_grad(D, *F, s["rank"], m)

    one_pass()  # warm-up pass, untimed (first touch of the host arrays)
    dok_s[0] = 0.0
    passes, t0 = 0, time.perf_counter()
    while True:
        one_pass()
        passes += 1
        el = time.perf_counter() - t0
        if el >= args.cpu_seconds or passes >= 1000:
            break
    done = {"build": "DOK build + CSR emission + stable column sort",
            "jvp": "DOK builds + C and its tangent",
            "batax": "DOK build + the Jacobian's outer products + CSR emission"}.get(
                w, "DOK build + loss + all gradients")
    if w == "batax":
        nnz = one_pass.nk  # the metric counts the Jacobian's keys
    on = "one thread" if threads == 1 else f"{threads} threads"
    return {"value": round(nnz * passes / el, 1), "unit": "entries/s" if w == "build" else "nnz/s",
            "cores": threads, "kind": "oracle",
            "sample": f"{what}: {passes} pass(es) of {done}, {el:.1f} s on {on}",
            "dok_build_s": round(dok_s[0], 3), "compute_s": round(el - dok_s[0], 3),
            "host_cpus_visible": len(os.sched_getaffinity(0)), "cpu_model": cpu_model()}


if __name__ == "__main__":
    main()
