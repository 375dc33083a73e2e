"""Workloads by which the library's speed is judged from one version to the next.

Each case is one call (or the calls of one training step) that a program
makes through the public binding on operands already in HBM: the fused losses
with their gradients, a layer's forward product and its vector-Jacobian
product, the forward-mode tangents, the construction of an operand from COO
input and the BATAX Jacobian.  `listed` names twelve of them, from a call
that is all launch latency to the largest layer that the benchmark runs;
`draw` gives more of the same kinds over the ranges between, odd widths and
uneven shapes among them.

All inputs are drawn on the GPU from a seed: row and column popularity from a
truncated Zipf profile (s = 0: uniform), distinct keys, dense operands normal.
"""
import math

import torch

from paper_2303_07030_amd import nsd
from paper_2303_07030_amd import operand as ops

DEV = "cuda"


# ------------------------------------------------------------------ cases

def listed():
    return [
        # the sum of a sparse matrix-vector product at the small end of the
        # paper's synthetic sweep: a call of microseconds, all latency
        dict(name="smvm_1k_10k", kind="smvm", nrows=1000, ncols=1000, nnz=10_000, s=0.0, cap=0),
        # the same loss on a large uneven matrix
        dict(name="smvm_1m_20m", kind="smvm", nrows=1_000_000, ncols=800_000, nnz=20_000_000,
             s=1.05, cap=100_000),
        # gradient of 1/2 ||A B||^2, the ordinary SpMM training step
        dict(name="spmm_100k_1m_k64", kind="spmm", nrows=100_000, ncols=100_000, nnz=1_000_000,
             s=1.1, cap=5000, k=64),
        # the same at a width that is no multiple of four (latent sizes are
        # often round decimal numbers), rectangular, odd sizes
        dict(name="spmm_70k_1m5_k50", kind="spmm", nrows=70_001, ncols=40_003, nnz=1_500_007,
             s=1.1, cap=5000, k=50),
        # a GNN layer's bilinear loss with both gradients: the largest step
        dict(name="gnn_2m4_60m_k256", kind="gnn", nrows=2_400_000, ncols=2_400_000,
             nnz=60_000_000, s=1.05, cap=2_400_000, k=256),
        # forward product and its VJP at a wide hidden size
        dict(name="layer_200k_4m_k512", kind="layer", nrows=200_000, ncols=200_000,
             nnz=4_000_000, s=1.05, cap=20_000, k=512),
        # sparse matrix factorisation, popularity skewed on both axes
        dict(name="mf_1m_500k_50m_k128", kind="mf", nrows=1_000_000, ncols=500_000,
             nnz=50_000_000, s=1.1, k=128),
        # CP gradient of a large order-3 tensor
        dict(name="cp_10k3_20m_r32", kind="cp", dims="10000 10000 10000", nnz=20_000_000, rank=32),
        # CP gradient of an order-4 tensor with uneven modes at rank ten
        dict(name="cp4_uneven_3m_r10", kind="cp", dims="6000 1500 220 31", nnz=3_000_000, rank=10),
        # an operand built from unsorted COO input: CSR, CSC, work plans and
        # the values in CSC order (each new matrix pays this once)
        dict(name="build_1m_500k_50m", kind="build", nrows=1_000_000, ncols=500_000,
             nnz=50_000_000, s=1.1, k=128, dups=False),
        # Jacobian of the BATAX kernel, an output pattern of its own
        dict(name="batax_100k_1m", kind="batax", nrows=100_000, ncols=100_000, nnz=1_000_000),
        # forward mode: four tangents of C = A B at once
        dict(name="jvp_100k_1m_k64_x4", kind="jvp", nrows=100_000, ncols=100_000, nnz=1_000_000,
             s=1.1, cap=5000, k=64, m=4),
    ]


def _log(rng, lo, hi):
    """A whole number spread evenly over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, nnz, lo_deg, hi_deg):
    """Rows and columns of a matrix of nnz entries with lo_deg to hi_deg
    entries per row and per column on average."""
    return tuple(max(64, int(nnz / math.exp(rng.uniform(math.log(lo_deg), math.log(hi_deg)))))
                 for _ in range(2))


def _width(rng, lo, hi):
    """Half of the widths are the usual powers of two, half anything."""
    if rng.random() < 0.5:
        return rng.choice([w for w in (8, 16, 32, 64, 128, 256, 512) if lo <= w <= hi])
    return _log(rng, lo, hi)


def draw(rng):
    kind = rng.choice(["smvm", "spmm", "gnn", "layer", "mf", "cp", "build", "batax", "jvp"])
    if kind == "smvm":
        nnz = _log(rng, 10_000, 20_000_000)
        nr, nc = _shape(rng, nnz, 5, 40)
        return dict(kind=kind, nrows=nr, ncols=nc, nnz=nnz, s=rng.choice([0.0, 1.05]),
                    cap=max(64, nc // 8))
    if kind == "spmm":
        nnz = _log(rng, 30_000, 4_000_000)
        nr, nc = _shape(rng, nnz, 5, 40)
        return dict(kind=kind, nrows=nr, ncols=nc, nnz=nnz, s=rng.choice([0.0, 1.1]),
                    cap=max(64, nc // 16), k=_width(rng, 8, 256))
    if kind == "gnn":
        nnz = _log(rng, 70_000, 30_000_000)
        n = _shape(rng, nnz, 8, 40)[0]
        return dict(kind=kind, nrows=n, ncols=n, nnz=nnz, s=1.05, cap=n, k=_width(rng, 16, 256))
    if kind == "layer":
        nnz = _log(rng, 50_000, 6_000_000)
        nr, nc = _shape(rng, nnz, 8, 40)
        return dict(kind=kind, nrows=nr, ncols=nc, nnz=nnz, s=1.05, cap=max(64, nc // 10),
                    k=_width(rng, 16, 512))
    if kind == "mf":
        nnz = _log(rng, 60_000, 30_000_000)
        nr, nc = _shape(rng, nnz, 40, 120)
        return dict(kind=kind, nrows=nr, ncols=nc, nnz=nnz, s=1.1, k=_width(rng, 8, 128))
    if kind == "cp":
        nnz = _log(rng, 25_000, 20_000_000)
        order = rng.choice([3, 3, 4])
        dims = [_log(rng, 20, 10_000) for _ in range(order)]
        while math.prod(dims) < 16 * nnz:
            dims[dims.index(min(dims))] *= 4
        return dict(kind=kind, dims=" ".join(map(str, dims)), nnz=nnz, rank=_width(rng, 8, 64))
    if kind == "build":
        nnz = _log(rng, 60_000, 50_000_000)
        nr, nc = _shape(rng, nnz, 20, 120)
        return dict(kind=kind, nrows=nr, ncols=nc, nnz=nnz, s=rng.choice([0.0, 1.1]),
                    k=_width(rng, 8, 128), dups=rng.random() < 0.5)
    if kind == "batax":
        nnz = _log(rng, 20_000, 2_000_000)
        nr, nc = _shape(rng, nnz, 5, 20)
        return dict(kind=kind, nrows=nr, ncols=nc, nnz=nnz)
    nnz = _log(rng, 30_000, 2_000_000)
    nr, nc = _shape(rng, nnz, 5, 40)
    return dict(kind=kind, nrows=nr, ncols=nc, nnz=nnz, s=rng.choice([0.0, 1.1]),
                cap=max(64, nc // 16), k=_width(rng, 8, 128), m=rng.choice([1, 2, 4, 7]))


# ----------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _ids(g, n, size, s, cap_share=1.0):
    """`size` draws from [0, n): uniform (s = 0), or by a Zipf(s) popularity
    over a random ranking, no id more popular than cap_share."""
    if s == 0.0:
        return torch.randint(n, (size,), generator=g, device=DEV)
    w = torch.arange(1, n + 1, device=DEV, dtype=torch.float64) ** (-s)
    w = w / w.sum()
    for _ in range(30):  # the share cut off the top goes to all others
        w = torch.clamp(w, max=cap_share)
        w = w / w.sum()
    cdf = torch.cumsum(w, 0)
    u = torch.rand(size, generator=g, device=DEV, dtype=torch.float64)
    rank = torch.searchsorted(cdf, u, right=True).clamp_(max=n - 1)
    return torch.randperm(n, generator=g, device=DEV)[rank]


def _distinct(g, nnz, draw_keys):
    """nnz distinct int64 keys in increasing order."""
    keys = torch.unique(draw_keys(nnz + nnz // 16 + 64))
    while keys.numel() < nnz:
        keys = torch.unique(torch.cat([keys, draw_keys(nnz // 2 + 64)]))
    m = keys.numel()  # thin evenly to exactly nnz
    return keys[torch.arange(nnz, device=DEV) * m // nnz] if m > nnz else keys


def _csr(g, c, s_cols=0.0):
    """(rowptr, row, col) of a pattern: rows by the case's profile."""
    nr, nc, nnz, s = c["nrows"], c["ncols"], c["nnz"], c.get("s", 0.0)
    cap = c.get("cap") or nc
    keys = _distinct(g, nnz, lambda m: _ids(g, nr, m, s, cap / nnz) * nc
                     + _ids(g, nc, m, s_cols))
    row, col = keys // nc, keys % nc
    rowptr = torch.zeros(nr + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(torch.bincount(row, minlength=nr), 0)
    return rowptr.int(), row, col


def _normal(g, *shape, std=1.0):
    x = torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32)
    return x if std == 1.0 else x.mul_(std)


def _inputs(c, seed):
    """Plain tensors of the case."""
    g = _gen(seed)
    kind = c["kind"]
    if kind == "cp":
        dims = [int(d) for d in c["dims"].split()]

        def keys(m):
            key = torch.zeros(m, dtype=torch.int64, device=DEV)
            for d in dims:
                key = key * d + _ids(g, d, m, 0.0)
            return key

        key = _distinct(g, c["nnz"], keys)
        coords = []
        for d in reversed(dims):
            coords.append((key % d).int())
            key = key // d
        return dict(dims=dims, coords=coords[::-1], val=_normal(g, c["nnz"]),
                    F=[_normal(g, d, c["rank"], std=0.1) for d in dims])
    if kind in ("mf", "build"):
        nr, nc, nnz = c["nrows"], c["ncols"], c["nnz"]
        again = nnz // 20 if c.get("dups") else 0  # coordinates given twice, as unclean data has
        keys = _distinct(g, nnz - again,
                         lambda m: _ids(g, nr, m, c["s"]) * nc + _ids(g, nc, m, c["s"]))
        if again:
            twice = torch.randint(nnz - again, (again,), generator=g, device=DEV)
            keys = torch.cat([keys, keys[twice]])
        keys = keys[torch.randperm(nnz, generator=g, device=DEV)]
        d = dict(row=(keys // nc).int(), col=(keys % nc).int(),
                 val=1.0 + 4.0 * torch.rand(nnz, generator=g, device=DEV))
        if kind == "mf":
            d.update(U=_normal(g, nr, c["k"], std=0.1), V=_normal(g, nc, c["k"], std=0.1))
        return d
    # the BATAX pattern is the case's (the Jacobian's size follows from it),
    # its values the seed's
    rowptr, row, col = _csr(_gen(1) if kind == "batax" else g, c)
    nr, nc, nnz = c["nrows"], c["ncols"], c["nnz"]
    d = dict(rowptr=rowptr, row=row, col=col.int())
    d["val"] = (torch.rand(nnz, generator=g, device=DEV) if kind in ("gnn", "layer")
                else _normal(g, nnz))
    if kind == "smvm":
        d["x"] = _normal(g, nc)
    elif kind == "spmm":
        d["B"] = _normal(g, nc, c["k"])
    elif kind in ("gnn", "layer"):
        d["H"], d["G"] = _normal(g, nc, c["k"]), _normal(g, nr, c["k"])
    elif kind == "jvp":
        d["B"] = _normal(g, nc, c["k"])
        d["dval"], d["dB"] = _normal(g, c["m"], nnz), _normal(g, c["m"], nc, c["k"])
    return d


def _empty(*shape, dtype=torch.float32):
    return torch.empty(*shape, dtype=dtype, device=DEV)


def _operand(c, d, **kw):
    return ops.DeviceCsr(c["nrows"], c["ncols"], d["rowptr"], d["col"], d["val"], device=DEV,
                         k_hint=c.get("k", 1), **kw)


def prepare(case, seed):
    c, d = case, _inputs(case, seed)
    kind, nnz, S = c["kind"], c["nnz"], dict(c=case, d=d)
    S["loss"] = _empty(1, dtype=torch.float64)
    if kind == "build":
        return S
    if kind == "cp":
        R = c["rank"]
        dims = d["dims"]
        if len(dims) == 3:
            X = ops.DeviceCoo3(dims, *d["coords"], d["val"], device=DEV, rank_hint=R)
        else:
            X = ops.DeviceCooN(dims, d["coords"], d["val"], device=DEV, rank_hint=R)
        S.update(X=X, ws=X.workspace(R), dX=_empty(nnz), dF=[_empty(n, R) for n in dims])
        return S
    if kind == "mf":
        A = ops.DeviceCsr.from_coo(c["nrows"], c["ncols"], d["row"], d["col"], d["val"],
                                   device=DEV, k_hint=c["k"])
        S.update(A=A, valT=A.values_in_csc_order(), ws=A.workspace(c["k"]),
                 dU=_empty(c["nrows"], c["k"]), dV=_empty(c["ncols"], c["k"]))
        return S
    if kind in ("batax", "jvp"):
        A = _operand(c, d, build_csc=False)
    else:
        A = _operand(c, d)
    S["A"] = A
    nr, nc, k = c["nrows"], c["ncols"], c.get("k", 1)
    if kind == "batax":
        P = nsd.nsd_batax_pairs(A.desc, torch.empty(256, dtype=torch.uint8, device=DEV))
        S.update(P=P, ws=_empty(nsd.nsd_batax_workspace_size(A.desc, P), dtype=torch.uint8),
                 jrowptr=_empty(nc + 1, dtype=torch.int32), jcol=_empty(P, dtype=torch.int32),
                 jval=_empty(P))
    elif kind == "jvp":
        S.update(ws=_empty(nsd.nsd_spmm_jvp_batch_workspace_size(A.desc, k), dtype=torch.uint8),
                 C=_empty(nr, k), dC=_empty(c["m"], nr, k))
    else:
        S.update(ws=A.workspace(k), dA=_empty(nnz))
        if kind in ("spmm", "layer"):
            S["C"] = _empty(nr, k)
        S["dB"] = _empty(nc) if kind == "smvm" else _empty(nc, k)
    return S


def run(S):
    c, d, kind = S["c"], S["d"], S["c"]["kind"]
    k, A = c.get("k", 1), S.get("A")
    if kind == "smvm":
        nsd.nsd_loss_sum_spmv(A.desc, A.csc, d["x"], 1.0, S["loss"], S["dA"], S["dB"], S["ws"])
        return {"loss": S["loss"], "dA": S["dA"], "dx": S["dB"]}
    if kind == "spmm":
        nsd.nsd_loss_frob_spmm(A.desc, A.csc, d["B"], k, 1.0, S["C"], S["loss"], S["dA"],
                               S["dB"], S["ws"])
        return {"C": S["C"], "loss": S["loss"], "dA": S["dA"], "dB": S["dB"]}
    if kind == "gnn":
        nsd.nsd_loss_bilinear(A.desc, A.csc, d["H"], d["G"], k, 1.0, S["loss"], S["dA"], S["dB"],
                              S["ws"])
        return {"loss": S["loss"], "dA": S["dA"], "dH": S["dB"]}
    if kind == "layer":
        nsd.nsd_spmm(A.desc, d["H"], k, S["C"], S["ws"])
        nsd.nsd_spmm_vjp(A.desc, A.csc, d["H"], d["G"], k, S["dA"], S["dB"], S["ws"])
        return {"C": S["C"], "dA": S["dA"], "dX": S["dB"]}
    if kind == "mf":
        nsd.nsd_loss_mf(A.desc, A.csc, S["valT"], d["U"], d["V"], k, 1.0, S["loss"], S["dU"],
                        S["dV"], S["ws"])
        return {"loss": S["loss"], "dU": S["dU"], "dV": S["dV"]}
    if kind == "cp":
        X, R = S["X"], c["rank"]
        if len(d["dims"]) == 3:
            nsd.nsd_loss_cp(X.desc, *d["F"], R, 1.0, S["loss"], S["dX"], *S["dF"], S["ws"])
        else:
            nsd.nsd_loss_cpn(X.desc, d["F"], R, 1.0, S["loss"], S["dX"], S["dF"], S["ws"])
        return {"loss": S["loss"], "dX": S["dX"], "dF": S["dF"]}
    if kind == "build":
        A = ops.DeviceCsr.from_coo(c["nrows"], c["ncols"], d["row"], d["col"], d["val"],
                                   device=DEV, k_hint=k)
        return {"rowptr": A.rowptr, "rowidx": A.rowidx, "colind": A.colind, "val": A.val,
                "coo_perm": A.coo_perm, "colptr": A.colptr, "rowind": A.rowind, "perm": A.perm,
                "valT": A.values_in_csc_order()}
    if kind == "batax":
        nk = nsd.nsd_batax_jacobian(A.desc, 1.5, S["P"], S["jrowptr"], S["jcol"], S["jval"],
                                    S["ws"])
        return {"rowptr": S["jrowptr"], "colind": S["jcol"][:nk], "val": S["jval"][:nk]}
    nsd.nsd_spmm_jvp_batch(A.desc, c["m"], d["dval"], d["B"], d["dB"], k, S["C"], S["dC"],
                           S["ws"])
    return {"C": S["C"], "dC": S["dC"]}


# ------------------------------------------------------- work and accuracy

def work(case):
    c, kind, nnz = case, case["kind"], case["nnz"]
    if kind == "cp":
        dims = [int(d) for d in c["dims"].split()]
        N, R = len(dims), c["rank"]
        # coordinates and value in, residual out; factors in, gradients out
        return dict(bytes=4 * nnz * (N + 2) + 8 * R * sum(dims), flops=nnz * R * (4 * N + 2))
    nr, nc, k = c["nrows"], c["ncols"], c.get("k", 1)
    if kind == "smvm":
        return dict(bytes=12 * nnz + 8 * nc, flops=3 * nnz)
    if kind == "spmm":
        return dict(bytes=12 * nnz + 4 * k * (nr + 2 * nc), flops=6 * nnz * k)
    if kind == "gnn":
        return dict(bytes=12 * nnz + 4 * k * (nr + 2 * nc), flops=4 * nnz * k)
    if kind == "layer":
        return dict(bytes=12 * nnz + 4 * k * (2 * nr + 2 * nc), flops=6 * nnz * k)
    if kind == "mf":
        return dict(bytes=8 * nnz + 8 * k * (nr + nc), flops=6 * nnz * k)
    if kind == "build":
        # row, column, value in; two index arrays, values and the permutation
        # of the CSR, three arrays of the CSC and the values in its order out
        return dict(bytes=44 * nnz + 4 * (nr + nc), flops=0)
    if kind == "batax":
        pairs = nnz * (1 + nnz / nr)
        return dict(bytes=8 * nnz + 8 * max(pairs - nnz, nc), flops=2 * pairs)
    m = c["m"]
    return dict(bytes=(8 + 4 * m) * nnz + 4 * k * (1 + m) * (nr + nc),
                flops=2 * nnz * k * (1 + 2 * m))


def tolerance(case):
    if case["kind"] == "build" and not case["dups"]:
        return "exact"
    return {"rel": 2e-6}


def _rows_of(idx, val, X, n, chunk=1 << 21):
    """sum over p of val[p] X[src[p]] into row dst[p], in 64 bits."""
    dst, src = idx
    out = torch.zeros(n, X.shape[1], dtype=torch.float64, device=DEV)
    for a in range(0, dst.numel(), chunk):
        b = a + chunk
        out.index_add_(0, dst[a:b], X[src[a:b]].double().mul_(val[a:b].double()[:, None]))
    return out


def _dots(r, X, c, Y, chunk=1 << 21):
    return torch.cat([(X[r[a:a + chunk]].double() * Y[c[a:a + chunk]].double()).sum(1)
                      for a in range(0, r.numel(), chunk)])


def exact(case, seed):
    c, d, kind = case, _inputs(case, seed), case["kind"]
    val = d["val"]
    if kind == "cp":
        co = [x.long() for x in d["coords"]]
        F = d["F"]
        res = torch.empty(c["nnz"], dtype=torch.float64, device=DEV)
        dF = [torch.zeros(f.shape, dtype=torch.float64, device=DEV) for f in F]
        for a in range(0, c["nnz"], 1 << 21):
            b = a + (1 << 21)
            rows = [f[i[a:b]].double() for f, i in zip(F, co)]
            prod = rows[0]
            for x in rows[1:]:
                prod = prod * x
            r = val[a:b].double() - prod.sum(1)
            res[a:b] = r
            for n in range(len(F)):
                t = -r[:, None]
                for m in range(len(F)):
                    if m != n:
                        t = t * rows[m]
                dF[n].index_add_(0, co[n][a:b], t)
        return {"loss": (0.5 * (res * res).sum()).reshape(1), "dX": res, "dF": dF}
    nr, nc, k = c["nrows"], c["ncols"], c.get("k", 1)
    if kind == "build":
        key = d["row"].long() * nc + d["col"].long()
        skey, order = torch.sort(key, stable=True)
        v = val[order].double()
        if c["dups"]:
            skey, run, cnt = torch.unique_consecutive(skey, return_inverse=True,
                                                      return_counts=True)
            v = torch.zeros(skey.numel(), dtype=torch.float64, device=DEV).index_add_(0, run, v)
            order = order[torch.cumsum(cnt, 0) - cnt]
        row, col = skey // nc, skey % nc

        def ptr(x, n):
            return torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV),
                              torch.cumsum(torch.bincount(x, minlength=n), 0)])

        scol, perm = torch.sort(col, stable=True)
        return {"rowptr": ptr(row, nr), "rowidx": row, "colind": col, "val": v,
                "coo_perm": order, "colptr": ptr(scol, nc), "rowind": row[perm], "perm": perm,
                "valT": v[perm]}
    if kind == "mf":
        row, col = d["row"].long(), d["col"].long()
        r = val.double() - _dots(row, d["U"], col, d["V"])
        return {"loss": (r * r).sum().reshape(1), "dU": _rows_of((row, col), -2 * r, d["V"], nr),
                "dV": _rows_of((col, row), -2 * r, d["U"], nc)}
    row, col = d["row"], d["col"].long()
    if kind == "smvm":
        x = d["x"].double()[col]
        return {"loss": (val.double() * x).sum().reshape(1), "dA": x,
                "dx": torch.zeros(nc, dtype=torch.float64,
                                  device=DEV).index_add_(0, col, val.double())}
    if kind == "spmm":
        C = _rows_of((row, col), val, d["B"], nr)
        return {"C": C, "loss": (0.5 * (C * C).sum()).reshape(1),
                "dA": _dots(row, C, col, d["B"]), "dB": _rows_of((col, row), val, C, nc)}
    if kind == "gnn":
        dA = _dots(row, d["G"], col, d["H"])
        return {"loss": (val.double() * dA).sum().reshape(1), "dA": dA,
                "dH": _rows_of((col, row), val, d["G"], nc)}
    if kind == "layer":
        return {"C": _rows_of((row, col), val, d["H"], nr),
                "dA": _dots(row, d["G"], col, d["H"]),
                "dX": _rows_of((col, row), val, d["G"], nc)}
    if kind == "batax":
        rp = d["rowptr"].long()
        n = rp[1:] - rp[:-1]
        reps = n[row]  # every entry p meets the entries of its row
        p = torch.repeat_interleave(torch.arange(c["nnz"], device=DEV), reps)
        first = torch.cumsum(reps, 0) - reps
        q = rp[row[p]] + torch.arange(p.numel(), device=DEV) - first[p]
        keys, run = torch.unique(col[p] * nc + col[q], return_inverse=True)
        v = torch.zeros(keys.numel(), dtype=torch.float64, device=DEV)
        v.index_add_(0, run, 1.5 * val[p].double() * val[q].double())
        jr = torch.zeros(nc + 1, dtype=torch.int64, device=DEV)
        jr[1:] = torch.cumsum(torch.bincount(keys // nc, minlength=nc), 0)
        return {"rowptr": jr, "colind": keys % nc, "val": v}
    C = _rows_of((row, col), val, d["B"], nr)
    dC = torch.stack([_rows_of((row, col), d["dval"][t], d["B"], nr)
                      + _rows_of((row, col), val, d["dB"][t], nr) for t in range(c["m"])])
    return {"C": C, "dC": dC}
