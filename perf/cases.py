"""The work that is timed: products of sparse with dense operands through the entry points of the package.

Every case is a matrix (or tensor) pattern with its sizes, a value type and an operation.  Patterns: `uniform` (random
columns, equal rows), `zipf` (row lengths from a truncated Zipf law), `stencil` (27 neighbours on a grid).  Inputs are
made on the GPU from the seed alone.  A program that multiplies by one matrix many times keeps the operands, the output
and the workspace, and asks the library once how to multiply (column passes, column-slab copy): that is prepare().
"""
from __future__ import annotations

import math

import torch

import paper_2001_00532_amd as psk

ZIPF_ALPHA = 1.8
SLAB_ARRAYS = ("slab_chunk", "qpos")      # the parts of the copy whose size does not depend on where the entries fall


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # a small system solved over and over (10 entries per row): launch latency and the host side of a call
        {"name": "spmv_small", "op": "spmv", "pattern": "uniform", "rows": 1024, "cols": 1024, "per_row": 10, "dtype": "f32"},
        # four million random nonzeros: a medium graph, where three launches are a visible share
        {"name": "spmv_medium", "op": "spmv", "pattern": "uniform", "rows": 250_000, "cols": 1_000_000, "per_row": 16, "dtype": "f32"},
        # 27-point stencil on 160^3 (a discretised PDE): one product per solver iteration
        {"name": "spmv_stencil", "op": "spmv", "pattern": "stencil", "grid": 160, "dtype": "f32"},
        # power-law graph of two million vertices, scattered columns: the product over the column-slab copy
        {"name": "slab_powerlaw", "op": "slab", "pattern": "zipf", "rows": 2_000_000, "cols": 2_000_000, "max_row": 200_000, "dtype": "f32"},
        # the same in the value type of the paper's own schedules
        {"name": "slab_powerlaw_f64", "op": "slab", "pattern": "zipf", "rows": 2_000_000, "cols": 2_000_000, "max_row": 200_000, "dtype": "f64"},
        # a matrix that changes: the column-slab copy is made anew, then one product
        {"name": "slab_build", "op": "slab_build", "pattern": "zipf", "rows": 2_000_000, "cols": 2_000_000, "max_row": 200_000, "dtype": "f32"},
        # hypersparse operand: a million stored rows out of 2^26
        {"name": "dcsr_hypersparse", "op": "dcsr", "pattern": "zipf", "rows": 1 << 26, "cols": 1 << 21, "stored": 1_000_000, "max_row": 50_000, "dtype": "f32"},
        # feature propagation over a graph with 16 neighbours: 128 dense columns
        {"name": "spmm_k128", "op": "spmm", "pattern": "uniform", "rows": 1_000_000, "cols": 1_000_000, "per_row": 16, "k": 128, "dtype": "f32"},
        # long rows times a narrow dense operand (100k x 100k, 1000 per row, 32 columns)
        {"name": "spmm_k32", "op": "spmm", "pattern": "uniform", "rows": 100_000, "cols": 100_000, "per_row": 1000, "k": 32, "dtype": "f32"},
        # 4x4 blocks (several unknowns per grid point): product with a vector and with 64 columns
        {"name": "bcsr_spmv", "op": "bcsr_spmv", "pattern": "uniform", "rows": 250_000, "cols": 250_000, "per_row": 8, "bs": 4, "dtype": "f32"},
        {"name": "bcsr_spmm_n64", "op": "bcsr_spmm", "pattern": "uniform", "rows": 250_000, "cols": 250_000, "per_row": 8, "bs": 4, "k": 64, "dtype": "f32"},
        # one mode of a CP decomposition of a three-way tensor, rank 64
        {"name": "mttkrp_j64", "op": "mttkrp", "I": 500_000, "K": 100_000, "L": 100_000, "fibers": 8, "max_leaves": 4096, "k": 64, "dtype": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["spmv", "spmv", "spmv", "slab", "slab_build", "dcsr", "spmm", "spmm", "bcsr_spmv", "bcsr_spmm", "mttkrp"])
    dtype = "f64" if op in ("spmv", "slab", "slab_build") and rng.random() < 0.3 else "f32"
    if op == "spmv":
        pattern = rng.choice(["uniform", "zipf", "stencil"])
        if pattern == "stencil":
            return {"op": op, "pattern": pattern, "grid": _log(rng, 6, 150), "dtype": dtype}
        nnz, mean = _log(rng, 2_000, 30_000_000), _log(rng, 3, 200)
        rows = max(16, nnz // mean)
        if pattern == "zipf":
            rows = max(16, nnz // 28)
            return {"op": op, "pattern": pattern, "rows": rows, "cols": max(256, rows), "max_row": max(64, rows // 10), "dtype": dtype}
        return {"op": op, "pattern": pattern, "rows": rows, "cols": max(4 * mean, _log(rng, 1_000, 1_500_000)), "per_row": mean, "dtype": dtype}
    if op in ("slab", "slab_build"):
        rows = _log(rng, 150_000, 1_900_000)
        if rng.random() < 0.5:
            return {"op": op, "pattern": "zipf", "rows": rows, "cols": _log(rng, 1_600_000, 4_000_000), "max_row": rows // 10, "dtype": dtype}
        per = rng.randint(5, 28)
        return {"op": op, "pattern": "uniform", "rows": rows, "cols": _log(rng, 1_600_000, 4_000_000), "per_row": per, "dtype": dtype}
    if op == "dcsr":
        stored = _log(rng, 2_000, 900_000)
        return {"op": op, "pattern": "zipf", "rows": min(1 << 26, stored * _log(rng, 10, 1000)), "cols": _log(rng, 10_000, 1 << 21),
                "stored": stored, "max_row": _log(rng, 200, 50_000), "dtype": "f32"}
    if op == "spmm":
        k = _log(rng, 3, 256)
        per = _log(rng, 6, 1000)
        nnz = min(_log(rng, 50_000, 80_000_000), 1_900_000_000 // max(32, k))
        rows = max(64, nnz // per)
        return {"op": op, "pattern": "uniform", "rows": rows, "cols": max(4 * per, min(1_000_000, rows)), "per_row": per, "k": k, "dtype": "f32"}
    if op in ("bcsr_spmv", "bcsr_spmm"):
        bs = rng.choice([2, 4, 8])
        rows, per = _log(rng, 2_000, 900_000 // bs), rng.randint(4, 32 // bs + 4)
        c = {"op": op, "pattern": "uniform", "rows": rows, "cols": rows, "per_row": per, "bs": bs, "dtype": "f32"}
        return dict(c, k=_log(rng, 8, 128)) if op == "bcsr_spmm" else c
    return {"op": op, "I": _log(rng, 5_000, 250_000), "K": _log(rng, 5_000, 100_000), "L": _log(rng, 5_000, 100_000),
            "fibers": rng.randint(2, 8), "max_leaves": 4096, "k": _log(rng, 6, 96), "dtype": "f32"}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1_000_003 + 17)
    return g


def _uniform(n, dtype, g, lo=-1.0, hi=1.0):
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float64 if dtype == "f64" else torch.float32) * (hi - lo) + lo


def _zipf(n, kmax, g):
    """n draws from the law k^-ZIPF_ALPHA on [1, kmax]."""
    w = torch.arange(1, kmax + 1, device="cuda", dtype=torch.float64).pow(-ZIPF_ALPHA).cumsum(0)
    u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * w[-1]
    return torch.searchsorted(w, u).clamp_(max=kmax - 1) + 1


def _csr(lengths, cols, g):
    """(pos, crd): random distinct columns, sorted in each row; a column drawn twice in a row is kept once."""
    rows = lengths.numel()
    key = torch.repeat_interleave(torch.arange(rows, device="cuda"), lengths) * cols
    key += torch.randint(cols, (key.numel(),), generator=g, device="cuda")
    key = torch.unique_consecutive(key.sort()[0])
    row = key // cols
    crd = (key - row * cols).to(torch.int32)
    pos = torch.zeros(rows + 1, dtype=torch.int32, device="cuda")
    pos[1:] = torch.bincount(row, minlength=rows).cumsum(0)
    return pos, crd


def _stencil(n, dtype, g):
    r = torch.arange(n ** 3, device="cuda")
    x, y, z = r % n, (r // n) % n, r // (n * n)
    d = torch.tensor([(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)], device="cuda")
    ok = torch.ones((n ** 3, 27), dtype=torch.bool, device="cuda")
    for v, j in ((z, 0), (y, 1), (x, 2)):
        t = v[:, None] + d[None, :, j]
        ok &= (t >= 0) & (t < n)
    pos = torch.zeros(n ** 3 + 1, dtype=torch.int32, device="cuda")
    pos[1:] = ok.sum(1).cumsum(0)
    off = (d[:, 0] * n + d[:, 1]) * n + d[:, 2]
    crd = (r[:, None] + off[None, :])[ok].to(torch.int32)
    vals = _uniform(crd.numel(), dtype, g, 0.5, 1.5)
    centre = torch.zeros((n ** 3, 27), dtype=torch.bool, device="cuda")
    centre[:, 13] = True
    vals[centre[ok]] = 27.0
    return pos, crd, vals


def _inputs(case, seed):
    """The operands of a case as a dict of device tensors."""
    g, op, dt = _gen(seed), case["op"], case["dtype"]
    if op == "mttkrp":
        fibers = torch.randint(2 * case["fibers"] + 1, (case["I"],), generator=g, device="cuda").clamp_(max=case["K"])
        pos_k, crd_k = _csr(fibers, case["K"], g)
        pos_l, crd_l = _csr(_zipf(crd_k.numel(), min(case["max_leaves"], case["L"]), g), case["L"], g)
        return {"pos_k": pos_k, "crd_k": crd_k, "pos_l": pos_l, "crd_l": crd_l, "vals": _uniform(crd_l.numel(), dt, g),
                "C": _uniform(case["K"] * case["k"], dt, g).view(case["K"], case["k"]),
                "D": _uniform(case["L"] * case["k"], dt, g).view(case["L"], case["k"])}
    bs = case.get("bs", 1)
    d = {}
    if case.get("pattern") == "stencil":
        d["pos"], d["crd"], d["vals"] = _stencil(case["grid"], dt, g)
        cols = case["grid"] ** 3
    else:
        cols = case["cols"]
        n = case["rows"]
        if op == "dcsr":
            d["crd_i"] = _csr(torch.tensor([case["stored"]], device="cuda"), n, g)[1]
            n = d["crd_i"].numel()
        if case["pattern"] == "zipf":
            lengths = _zipf(n, min(case["max_row"], cols), g)
        else:
            lengths = torch.full((n,), case["per_row"], device="cuda")
        d["pos"], d["crd"] = _csr(lengths, cols, g)
        d["vals"] = _uniform(d["crd"].numel() * bs * bs, dt, g)
    if "k" in case:
        d["B"] = _uniform(cols * bs * case["k"], dt, g).view(cols * bs, case["k"])
    else:
        d["x"] = _uniform(cols * bs, dt, g)
    return d


def _sizes(case):
    n = case["grid"] ** 3 if "grid" in case else 0
    return (case.get("rows", n), case.get("cols", n)) if "I" not in case else (case["I"], case["L"])


def prepare(case, seed):
    s, op, f64 = _inputs(case, seed), case["op"], case["dtype"] == "f64"
    rows, cols = _sizes(case)
    s.update(op=op, f64=f64, rows=rows, cols=cols)
    if op == "mttkrp":
        s["dims"] = (case["I"], case["K"], case["L"])
        s["out"] = torch.empty((case["I"], case["k"]), device="cuda")
        s["ws"] = psk.workspace(psk.PSK_OP_MTTKRP_CSF3, case["I"], s["crd_l"].numel(), k=case["k"])
        return s
    nnz = s["nnz"] = s["crd"].numel()
    bs = s["bs"] = case.get("bs", 1)
    if op == "spmv":
        s["out"] = torch.empty(rows, dtype=s["vals"].dtype, device="cuda")
        s["passes"] = psk.psk_analyze_csr(rows, cols, nnz, s["pos"], s["crd"])
        s["ws"] = psk.workspace(psk.PSK_OP_SPMV_CSR_F64 if f64 else psk.PSK_OP_SPMV_CSR, rows, nnz)
    elif op == "dcsr":
        s["out"] = torch.empty(rows, device="cuda")
        stored = s["pos"].numel() - 1
        s["passes"] = psk.psk_analyze_csr(stored, cols, nnz, s["pos"], s["crd"])
        s["ws"] = psk.workspace(psk.PSK_OP_SPMV_CSR, stored, nnz)
    elif op == "slab":
        build = psk.psk_slab_build_csr_f64 if f64 else psk.psk_slab_build_csr
        s["out"] = torch.empty(rows, dtype=s["vals"].dtype, device="cuda")
        s["slab"] = build(rows, cols, nnz, s["pos"], s["crd"], s["vals"])
        s["ws"] = psk.psk_slab_spmv_workspace(s["slab"])
    elif op == "slab_build":
        s["out"] = torch.empty(rows, dtype=s["vals"].dtype, device="cuda")
        mem, ws = ((psk.psk_slab_mem_bytes_f64, psk.psk_slab_build_workspace_bytes_f64) if f64 else
                   (psk.psk_slab_mem_bytes, psk.psk_slab_build_workspace_bytes))
        s["mem"] = torch.empty(mem(rows, cols, nnz), dtype=torch.uint8, device="cuda")
        s["ws"] = torch.empty(ws(rows, cols, nnz), dtype=torch.uint8, device="cuda")
    elif op == "bcsr_spmv":
        s["out"] = torch.empty(rows * bs, device="cuda")
        s["ws"] = psk.workspace(psk.PSK_OP_SPMV_BCSR, rows, nnz, bs=bs)
    else:
        s["out"] = torch.empty((rows * bs, case["k"]), device="cuda")
        s["ws"] = psk.workspace(psk.PSK_OP_SPMM_CSR if op == "spmm" else psk.PSK_OP_SPMM_BCSR, rows, nnz, k=case["k"], bs=bs)
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    op = s["op"]
    if op == "mttkrp":
        return psk.psk_mttkrp_csf3(s["dims"], None, s["pos_k"], s["crd_k"], s["pos_l"], s["crd_l"], s["vals"], s["C"], s["D"],
                                   s["out"], ws=s["ws"])
    rows, cols, nnz = s["rows"], s["cols"], s["nnz"]
    if op == "spmv":
        f = psk.psk_spmv_csr_f64 if s["f64"] else psk.psk_spmv_csr
        return f(rows, cols, nnz, s["pos"], s["crd"], s["vals"], s["x"], s["out"], col_passes=s["passes"], ws=s["ws"])
    if op == "dcsr":
        return psk.psk_spmv_dcsr(rows, cols, nnz, s["crd_i"], s["pos"], s["crd"], s["vals"], s["x"], s["out"],
                                 col_passes=s["passes"], ws=s["ws"])
    if op == "slab":
        return (psk.psk_spmv_slab_f64 if s["f64"] else psk.psk_spmv_slab)(s["slab"], s["x"], s["out"], ws=s["ws"])
    if op == "slab_build":
        build, product = (psk.psk_slab_build_csr_f64, psk.psk_spmv_slab_f64) if s["f64"] else (psk.psk_slab_build_csr, psk.psk_spmv_slab)
        S = build(rows, cols, nnz, s["pos"], s["crd"], s["vals"], mem=s["mem"], ws=s["ws"])
        return dict({"y": product(S, s["x"], s["out"])}, **{a: S.array(a) for a in SLAB_ARRAYS})
    if op == "spmm":
        return psk.psk_spmm_csr(rows, cols, nnz, s["pos"], s["crd"], s["vals"], s["B"], s["out"], ws=s["ws"])
    if op == "bcsr_spmv":
        return psk.psk_spmv_bcsr(rows, cols, nnz, s["bs"], s["pos"], s["crd"], s["vals"], s["x"], s["out"], ws=s["ws"])
    return psk.psk_spmm_bcsr(rows, cols, nnz, s["bs"], s["pos"], s["crd"], s["vals"], s["B"], s["out"], ws=s["ws"])


# ------------------------------------------------------------------ what a pass cannot do without
def _expected_zipf(kmax):
    k = range(1, kmax + 1)
    return sum(i ** (1.0 - ZIPF_ALPHA) for i in k) / sum(i ** -ZIPF_ALPHA for i in k)


def work(case):
    """Every input read once, every output written once (sizes that depend on the seed: their expected value)."""
    v, rows, cols = (8 if case["dtype"] == "f64" else 4), *_sizes(case)
    if case["op"] == "mttkrp":
        fibers = case["I"] * case["fibers"]
        nnz, j = fibers * _expected_zipf(min(case["max_leaves"], case["L"])), case["k"]
        return {"bytes": 8 * nnz + 8 * fibers + 4 * case["I"] + 4 * j * (case["K"] + case["L"] + case["I"]),
                "flops": 2 * j * nnz + 2 * j * fibers}
    bs, k, stored = case.get("bs", 1), case.get("k", 1), case.get("stored", rows)
    if case.get("pattern") == "stencil":
        nnz = (3 * case["grid"] - 2) ** 3
    elif case.get("pattern") == "zipf":
        nnz = stored * _expected_zipf(min(case["max_row"], cols))
    else:
        nnz = rows * case["per_row"]
    moved = nnz * (4 + v * bs * bs) + 4 * stored * (2 if case["op"] == "dcsr" else 1) + v * k * bs * (rows + cols)
    if case["op"] == "slab_build":
        moved += nnz * (2 + v)            # the copy is written: value and 16-bit column
    return {"bytes": moved, "flops": 2 * nnz * bs * bs * k}


def tolerance(case):
    # against the sums in 64 bits the products are 6e-8 to 2.8e-7 off (fp64: 5e-15, most of it the reference's own)
    return {"rel": 2e-14, "max": 1e-12} if case["dtype"] == "f64" else {"rel": 1e-6, "max": 5e-5}


# ------------------------------------------------------------------ the same in 64 bits
def _segments(pos):
    return torch.repeat_interleave(torch.arange(pos.numel() - 1, device="cuda"), (pos[1:] - pos[:-1]).long())


def _times(pos, crd, vals, B):
    """The CSR matrix (pos, crd, vals) times the dense B."""
    A = torch.sparse_csr_tensor(pos, crd, vals.double(), (pos.numel() - 1, B.shape[0]))
    return A @ B.double()


def exact(case, seed):
    d, op = _inputs(case, seed), case["op"]
    if op == "mttkrp":
        fibers = _times(d["pos_l"], d["crd_l"], d["vals"], d["D"]) * d["C"].double()[d["crd_k"].long()]
        return torch.zeros((case["I"], case["k"]), dtype=torch.float64, device="cuda").index_add_(0, _segments(d["pos_k"]), fibers)
    rows, _ = _sizes(case)
    if op == "spmm":
        return _times(d["pos"], d["crd"], d["vals"], d["B"])
    row, col, bs, k = _segments(d["pos"]), d["crd"].long(), case.get("bs", 1), case.get("k", 1)
    if op == "dcsr":
        row = d["crd_i"].long()[row]
    if bs == 1:
        terms = d["vals"].double() * d["x"].double()[col]
        y = torch.zeros(rows, dtype=torch.float64, device="cuda").index_add_(0, row, terms)
        return dict({"y": y}, **{a: None for a in SLAB_ARRAYS}) if op == "slab_build" else y
    B = (d["B"] if op == "bcsr_spmm" else d["x"]).double().view(-1, bs, k)
    terms = torch.bmm(d["vals"].double().view(-1, bs, bs), B[col]).view(-1, bs * k)
    out = torch.zeros((rows, bs * k), dtype=torch.float64, device="cuda").index_add_(0, row, terms)
    return out.view(rows * bs, k) if op == "bcsr_spmm" else out.view(-1)
