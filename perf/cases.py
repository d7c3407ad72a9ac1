"""The work a user of spk has it do, as cases that can be timed and compared.

Each case is one call (or one closed round of calls) of the public binding
``paper_1309_1894_amd.spk`` on inputs made from a seed:

* ``vec``    WAXPY or dot on vectors of n elements (the vector sweep covers
             n = 1e4 .. 2^27 in both dtypes);
* ``spmv``   a registered matrix: y = A x, or the fused Krylov step
             y = A x, w = 0.5 y + x;
* ``csr``    y = A x on a CSR matrix the caller holds on the device;
* ``batch``  thousands of independent banded matrices in one launch;
* ``cg``     a conjugate-gradient solve of a fixed number of iterations;
* ``serve``  a closed round of requests through the serving loop, vectors in
             pinned host memory, as a serving front end holds them.

``plan`` says what the program has in its tuning database before the call:
``default`` nothing (the library's own dispatch), ``recorded`` the winners a
tuning run left for such matrices (a program in production loads them; here
they are put in directly, so that every run times the same variants).
"""
from __future__ import annotations

import functools
import math
import types
import weakref

import numpy as np
import torch

from paper_1309_1894_amd import inputs as I
from paper_1309_1894_amd import spk

ALPHA = 0.5                       # step coefficient of the batched, served and 2-D steps
DTYPES = {"f64": torch.float64, "f32": torch.float32}


def listed():
    return [
        # the 2-D Krylov step, 65,536 rows: a few microseconds of GPU work, so
        # the call itself, its launch and the two output allocations count
        dict(name="step_lap2d_256", kind="spmv", matrix="lap2d", size=256, dtype="f64", fused=True, plan="default"),
        # a reduction inside an iterative solver on an ordinary vector, odd length
        dict(name="dot_f64_1m", kind="vec", op="dot", n=1_000_003, dtype="f64"),
        # a vector update that streams from memory, odd length
        dict(name="waxpy_f64_20m", kind="vec", op="waxpy", n=20_000_003, dtype="f64"),
        # the large grid operator (2,097,152 rows), untuned program
        dict(name="spmv_lap3d_128", kind="spmv", matrix="lap3d", size=128, dtype="f64", fused=False, plan="default"),
        # the large random-column matrix (1,000,000 rows, about 16.2 M entries)
        # with the form its tuning records: x staged in LDS by window
        dict(name="spmv_zipf_1m_recorded", kind="spmv", matrix="zipf", size=1_000_000, dtype="f64", fused=False,
             plan="recorded"),
        # the same kind of matrix in single precision, odd size, untuned, fused
        dict(name="step_zipf_f32_300k", kind="spmv", matrix="zipf", size=300_001, dtype="f32", fused=True,
             plan="default"),
        # a banded matrix the caller keeps on the device itself
        dict(name="csr_banded_200k", kind="csr", size=200_003, half_band=16, dtype="f64"),
        # the batched workload (4,096 instances, 12.2 M rows), tuned launch
        dict(name="batch_4096_recorded", kind="batch", count=4096, dtype="f64", plan="recorded"),
        # a small batch in single precision, constructed with the binding's defaults
        dict(name="batch_96_f32", kind="batch", count=96, dtype="f32", plan="default"),
        # a small solve: every iteration is launch latency
        dict(name="cg_lap2d_48", kind="cg", matrix="lap2d", size=48, iters=50, plan="default"),
        # the large solve on the grid operator, tuned
        dict(name="cg_lap3d_128_recorded", kind="cg", matrix="lap3d", size=128, iters=20, plan="recorded"),
        # a closed round of the serving pool: rows log-uniform, banded and Zipf, both dtypes
        dict(name="serve_64", kind="serve", requests=64, matrices=16, rows_max=100_000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["vec", "vec", "spmv", "spmv", "spmv", "csr", "batch", "cg", "cg", "serve"])
    dtype = rng.choice(["f64", "f64", "f32"])
    if kind == "vec":
        return dict(kind=kind, op=rng.choice(["dot", "waxpy"]), n=_log_int(rng, 10_000, 50_000_000), dtype=dtype)
    if kind == "spmv":
        matrix = rng.choice(["lap2d", "lap3d", "zipf"])
        size = {"lap2d": _log_int(rng, 64, 1400), "lap3d": _log_int(rng, 24, 128),
                "zipf": _log_int(rng, 5_000, 1_000_000)}[matrix]
        # the recorded form of a random-column matrix is for x beyond an L2 (4 MiB)
        big = matrix == "zipf" and size * (8 if dtype == "f64" else 4) > (4 << 20)
        return dict(kind=kind, matrix=matrix, size=size, dtype=dtype, fused=rng.random() < 0.4,
                    plan="recorded" if matrix == "lap3d" and rng.random() < 0.5 or big else "default")
    if kind == "csr":
        return dict(kind=kind, size=_log_int(rng, 1_000, 600_000), half_band=rng.randint(1, 32), dtype=dtype)
    if kind == "batch":
        return dict(kind=kind, count=_log_int(rng, 16, 512), dtype=dtype, plan=rng.choice(["default", "recorded"]))
    if kind == "cg":
        matrix = rng.choice(["lap2d", "lap3d", "spd_zipf"])
        size = {"lap2d": _log_int(rng, 16, 512), "lap3d": _log_int(rng, 12, 112),
                "spd_zipf": _log_int(rng, 1_000, 60_000)}[matrix]
        return dict(kind=kind, matrix=matrix, size=size, iters=8 if matrix == "spd_zipf" else rng.randint(10, 40),
                    plan=rng.choice(["default", "recorded"]) if matrix == "lap3d" else "default")
    return dict(kind=kind, requests=_log_int(rng, 4, 64), matrices=rng.randint(2, 16),
                rows_max=_log_int(rng, 5_000, 100_000))


# ------------------------------------------------------------------ inputs --

class State(types.SimpleNamespace):
    """What the program holds before the call; the library's objects are
    released when it is dropped."""


def _gen(seed):
    return torch.Generator("cuda").manual_seed(int(seed))


def _uniform(n, dtype, g):
    """Uniform in [-1, 1), as the library's own seeded inputs."""
    return torch.rand(n, dtype=dtype, device="cuda", generator=g) * 2 - 1


@functools.lru_cache(maxsize=4)
def _laplacian(matrix, size):
    """A grid operator: its entries do not depend on a seed."""
    return I.lap2d(size) if matrix == "lap2d" else I.lap3d(size)


def _from_keys(m, n, key, dtype, g):
    """Host CSR of the sorted distinct positions row*n + col, values uniform."""
    rows, cols = torch.div(key, n, rounding_mode="floor"), key % n
    rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.bincount(rows, minlength=m).cumsum(0)
    val = _uniform(key.numel(), dtype, g)
    return I.CSR(m, n, rp.int().cpu().numpy(), cols.int().cpu().numpy(), val.cpu().numpy())


def _zipf_keys(m, g):
    """Positions of a matrix with truncated-Zipf row lengths (mean 16, one row
    of 4,096) and uniform columns."""
    kmax = min(4096, m)
    cdf = (torch.arange(1, kmax + 1, dtype=torch.float64, device="cuda") ** -I.ZIPF_S_MEAN16).cumsum(0)
    length = torch.searchsorted(cdf / cdf[-1], torch.rand(m, dtype=torch.float64, device="cuda", generator=g)) + 1
    length = length.clamp_(max=kmax)
    length[torch.randint(m, (1,), device="cuda", generator=g)] = kmax
    rows = torch.repeat_interleave(torch.arange(m, device="cuda"), length)
    return torch.unique(rows * m + torch.randint(m, (rows.numel(),), device="cuda", generator=g))


def _zipf(m, dtype, g):
    return _from_keys(m, m, _zipf_keys(m, g), dtype, g)


def _spd_zipf(m, g):
    """The Zipf pattern made symmetric, strictly diagonally dominant."""
    key = _zipf_keys(m, g)
    r, c = torch.div(key, m, rounding_mode="floor"), key % m
    key = torch.unique(torch.minimum(r, c) * m + torch.maximum(r, c))
    lo, hi = torch.div(key, m, rounding_mode="floor"), key % m
    lo, hi = lo[lo != hi], hi[lo != hi]
    v = _uniform(lo.numel(), torch.float64, g)
    diag = torch.arange(m, device="cuda")
    rows, cols = torch.cat([lo, hi, diag]), torch.cat([hi, lo, diag])
    val = torch.cat([v, v, 1.0 + torch.bincount(torch.cat([lo, hi]), minlength=m)])
    order = torch.argsort(rows * m + cols)
    rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.bincount(rows, minlength=m).cumsum(0)
    return I.CSR(m, m, rp.int().cpu().numpy(), cols[order].int().cpu().numpy(), val[order].cpu().numpy())


def _banded(sizes, bands, dtype, g):
    """Banded matrices stored back to back (fill 0.6): device arrays of local
    row_ptr (one extra entry per matrix), columns and values, and the host
    sizes and offsets."""
    m, b = torch.tensor(sizes, device="cuda"), torch.tensor(bands, device="cuda")
    total = int(m.sum())
    inst = torch.repeat_interleave(torch.arange(len(sizes), device="cuda"), m)
    vec_off = m.cumsum(0) - m
    local = torch.arange(total, device="cuda") - vec_off[inst]
    width = 2 * b[inst] + 1
    start = width.cumsum(0) - width
    row = torch.repeat_interleave(torch.arange(total, device="cuda"), width)
    col = torch.arange(row.numel(), device="cuda") - start[row] - b[inst[row]] + local[row]
    keep = (torch.rand(row.numel(), device="cuda", generator=g) < 0.6) & (col >= 0) & (col < m[inst[row]])
    row, col = row[keep], col[keep].int()
    count = torch.bincount(row, minlength=total)
    nnz = torch.zeros_like(m).index_add_(0, inst, count)
    nz_off, rp_off = nnz.cumsum(0) - nnz, vec_off + torch.arange(len(sizes), device="cuda")
    ends = count.cumsum(0)
    rp = torch.zeros(total + len(sizes), dtype=torch.int32, device="cuda")
    rp[torch.arange(total, device="cuda") + inst + 1] = (ends - nz_off[inst]).int()
    rp[rp_off] = 0
    val = _uniform(col.numel(), dtype, g)
    host = types.SimpleNamespace(count=len(sizes), **{k: v.cpu().numpy() for k, v in dict(
        m=m, nnz=nnz, rp_off=rp_off, nz_off=nz_off, vec_off=vec_off, row_ptr=rp).items()})
    return rp, col, val, host


def _batch_inputs(case, seed):
    """Rows log-uniform in 64..16384 and half-bands 1..32, as the batched workload."""
    g, dtype = _gen(seed), DTYPES[case["dtype"]]
    # the sizes are the workload's own; the pattern, values and x follow the seed
    sizes, bands = I.batch_sizes(case["count"])
    rp, ci, val, host = _banded(sizes.tolist(), bands.tolist(), dtype, g)
    return rp, ci, val, host, _uniform(int(host.m.sum()), dtype, g)


def _spmv_inputs(case, seed):
    g, dtype = _gen(seed), DTYPES[case["dtype"]]
    if case["matrix"] == "zipf":
        A = _zipf(case["size"], dtype, g)
    else:
        A = _laplacian(case["matrix"], case["size"])
        A = A if dtype is torch.float64 else A.astype(np.float32)
    return A, _uniform(A.ncols, dtype, g)


def _cg_inputs(case, seed):
    g = _gen(seed)
    A = _spd_zipf(case["size"], g) if case["matrix"] == "spd_zipf" else _laplacian(case["matrix"], case["size"])
    return A, _uniform(A.nrows, torch.float64, g)


def _vec_inputs(case, seed):
    g, dtype = _gen(seed), DTYPES[case["dtype"]]
    return _uniform(case["n"], dtype, g), _uniform(case["n"], dtype, g)


def _csr_inputs(case, seed):
    g, dtype = _gen(seed), DTYPES[case["dtype"]]
    rp, ci, val, _ = _banded([case["size"]], [min(case["half_band"], case["size"] - 1)], dtype, g)
    return rp, ci, val, _uniform(case["size"], dtype, g)


def _serve_inputs(case, seed):
    """The pool (rows log-uniform from 1,000, half banded, half Zipf, 70%
    FP64) and one x per request in pinned host memory."""
    g = _gen(seed)
    rows = I.log_uniform_int(1000, case["rows_max"], 51, 0, case["matrices"])
    pool = []
    for i, m in enumerate(int(v) for v in rows):
        dtype = torch.float32 if i % 10 in (2, 5, 8) else torch.float64
        if i % 2:
            pool.append(_zipf(m, dtype, g))
        else:
            rp, ci, val, _ = _banded([m], [1 + 7 * i % 32], dtype, g)
            pool.append(I.CSR(m, m, rp.cpu().numpy(), ci.cpu().numpy(), val.cpu().numpy()))
    order = [(5 * i + 3) % case["matrices"] for i in range(case["requests"])]
    xs = [_uniform(pool[k].ncols, torch.from_numpy(pool[k].val).dtype, g).cpu().pin_memory() for k in order]
    return pool, order, xs


# ----------------------------------------------------------------- prepare --

@functools.lru_cache(maxsize=None)
def _handle(plan):
    """One handle per tuning database: without records, and with them."""
    return spk.Handle(torch.cuda.current_device())


def _record_batch(h, dtype):
    """What spk_batch_tune records on the batched workload: one-wavefront
    workgroups, 1,024-entry tiles, compact columns in every class."""
    spk.spk_plan_put(f"batch:{dtype}:launch", spk.make_variant(block=64, lds=1024, unroll=256, grid=0), h)
    for c in range(8):
        spk.spk_plan_put(f"batch:{dtype}:c{c}", spk.make_variant(group=3), h)


def _record_spmv(h, A, case, op, x, y, w):
    """What spk_tune records: x windows in LDS for random columns, row blocks
    with two-byte columns for the grid operators."""
    key = spk.spk_class_key(spk.problem(op, A=A, x=x, y=y, w=w), h)
    if case["matrix"] == "zipf":
        v = spk.make_variant(format=spk.SPK_FMT_XWIN, block=768, group=128, unroll=1, grid=1, streams=1, lds=256)
    else:
        v = spk.make_variant(format=spk.SPK_FMT_ADAPTIVE, block=256, group=1, unroll=1, vec=2, streams=1, lds=256)
    spk.spk_plan_put(key, v, h)


def _owned(state, *objects):
    for o in objects:
        weakref.finalize(state, getattr(o, "release", None) or getattr(o, "free", None) or o.close)
    return state


def prepare(case, seed):
    kind = case["kind"]
    h = _handle(case.get("plan", "default"))
    if kind == "vec":
        x, y = _vec_inputs(case, seed)
        out = torch.empty(1, dtype=torch.float64, device="cuda") if case["op"] == "dot" else torch.empty_like(x)
        return State(kind=case["op"], h=h, x=x, y=y, out=out)
    if kind == "spmv":
        csr, x = _spmv_inputs(case, seed)
        A = spk.Matrix(csr, h)
        op = spk.SPK_OP_SPMV_WAXPY if case["fused"] else spk.SPK_OP_SPMV
        y, w = torch.empty_like(x), torch.empty_like(x) if case["fused"] else None
        if case["plan"] == "recorded":
            _record_spmv(h, A, case, op, x, y, w)
        return _owned(State(kind="step" if case["fused"] else "spmv", A=A, x=x, y=y), A)
    if kind == "csr":
        rp, ci, val, x = _csr_inputs(case, seed)
        return State(kind=kind, h=h, rp=rp, ci=ci, val=val, x=x, y=torch.empty_like(x))
    if kind == "batch":
        rp, ci, val, host, x = _batch_inputs(case, seed)
        if case["plan"] == "recorded":
            _record_batch(h, case["dtype"])
            b = spk.Batch(host, (rp, ci, val), block=0, handle=h)
        else:
            b = spk.Batch(host, (rp, ci, val), handle=h)
        return _owned(State(kind=kind, b=b, x=x, y=torch.empty_like(x), w=torch.empty_like(x)), b)
    if kind == "cg":
        csr, rhs = _cg_inputs(case, seed)
        A = spk.Matrix(csr, h)
        if case["plan"] == "recorded":
            key = spk.spk_class_key(spk.problem(spk.SPK_OP_SPMV, A=A, x=rhs, y=rhs), h)
            spk.spk_plan_put("cg:" + key, spk.make_variant(format=spk.SPK_FMT_ADAPTIVE, block=512, group=1, unroll=1,
                                                           vec=2, streams=1, lds=512), h)
        hist = torch.empty(case["iters"] + 1, dtype=torch.float64, device="cuda")
        return _owned(State(kind=kind, A=A, b=rhs, x=torch.empty_like(rhs), hist=hist, iters=case["iters"]), A)
    pool, order, xs = _serve_inputs(case, seed)
    srv = spk.Server(hbm_budget=int(20e9), alpha=ALPHA, handle=h)
    ids = [srv.add_matrix(A) for A in pool]
    ys, ws = ([torch.empty_like(x).pin_memory() for x in xs] for _ in range(2))
    host = [tuple(t.numpy() for t in xyw) for xyw in zip(xs, ys, ws)]
    return _owned(State(kind=kind, srv=srv, ids=[ids[k] for k in order], host=host, keep=(xs, ys, ws)), srv)


# --------------------------------------------------------------------- run --

def run(s):
    if s.kind == "dot":
        return spk.spk_dot(s.x, s.y, s.out, handle=s.h)
    if s.kind == "waxpy":
        return spk.spk_waxpy(1.5, s.x, s.y, s.out, handle=s.h)
    if s.kind == "spmv":
        return spk.spk_spmv_mat(s.A, s.x, s.y)
    if s.kind == "step":
        return spk.spk_spmv_waxpy(s.A, ALPHA, s.x)
    if s.kind == "csr":
        return spk.spk_spmv_csr(s.rp, s.ci, s.val, s.x, s.y, handle=s.h)
    if s.kind == "batch":
        s.b.run(ALPHA, s.x, s.y, s.w)
        return s.y, s.w
    if s.kind == "cg":
        s.x.zero_()
        spk.spk_cg(s.A, s.b, s.x, s.iters, s.hist)
        return s.x, s.hist
    for mid, (x, y, w) in zip(s.ids, s.host):
        s.srv.submit(mid, x, y, w)
    s.srv.drain()
    # both dtypes' results, whole: one array of each vector and dtype
    return [np.concatenate([v[k] for v in s.host if v[k].dtype == t] or [np.zeros(0, t)])
            for t in (np.float64, np.float32) for k in (1, 2)]


# -------------------------------------------------------------------- work --

def _zipf_mean(m):
    return I.zipf_mean(I.ZIPF_S_MEAN16, min(4096, m))


def _spmv_work(m, nnz, s, fused):
    return dict(bytes=nnz * (s + 4) + 4 * (m + 1) + (3 if fused else 2) * m * s, flops=2 * nnz + (2 * m if fused else 0))


def _lap(matrix, size):
    return (size ** 2, I.expected_lap_nnz(size, 2)) if matrix == "lap2d" else (size ** 3, I.expected_lap_nnz(size, 3))


def _sum(parts):
    parts = list(parts)
    return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}


def work(case):
    kind, s = case["kind"], 4 if case.get("dtype") == "f32" else 8
    if kind == "vec":
        return dict(bytes=case["n"] * s * (2 if case["op"] == "dot" else 3), flops=2 * case["n"])
    if kind == "spmv":
        m, nnz = ((case["size"], int(case["size"] * _zipf_mean(case["size"]))) if case["matrix"] == "zipf"
                  else _lap(case["matrix"], case["size"]))
        return _spmv_work(m, nnz, s, case["fused"])
    if kind == "csr":
        m = case["size"]
        return _spmv_work(m, int(0.6 * m * (2 * case["half_band"] + 1)), s, False)
    if kind == "batch":
        sizes, bands = I.batch_sizes(case["count"])
        return _sum(_spmv_work(int(m), int(0.6 * m * (2 * b + 1)), s, True) for m, b in zip(sizes, bands))
    if kind == "cg":
        if case["matrix"] == "spd_zipf":
            m, nnz = case["size"], int(case["size"] * (2 * _zipf_mean(case["size"]) + 1))
        else:
            m, nnz = _lap(case["matrix"], case["size"])
        # the solve reads the matrix and moves its vectors in every iteration
        return dict(bytes=case["iters"] * (12 * nnz + 4 * (m + 1) + 72 * m), flops=case["iters"] * (2 * nnz + 10 * m))
    rows = [int(v) for v in I.log_uniform_int(1000, case["rows_max"], 51, 0, case["matrices"])]
    parts = []
    for i in range(case["requests"]):
        k = (5 * i + 3) % case["matrices"]
        m, w = rows[k], 4 if k % 10 in (2, 5, 8) else 8
        nnz = m * _zipf_mean(m) if k % 2 else 0.6 * m * (2 * (1 + 7 * k % 32) + 1)
        parts.append(_spmv_work(m, int(nnz), w, True))
    return _sum(parts)


# ------------------------------------------------------------------- exact --

def _product(rp, ci, val, x):
    """A x in 64 bits: row_ptr, columns and values on any device."""
    rp, ci, val = (torch.as_tensor(v).cuda() for v in (rp, ci, val))
    n = (rp[1:] - rp[:-1]).long()
    rows = torch.repeat_interleave(torch.arange(n.numel(), device="cuda"), n)
    return torch.zeros(n.numel(), dtype=torch.float64, device="cuda").index_add_(
        0, rows, val.double() * x.double()[ci.long()])


def exact(case, seed):
    kind = case["kind"]
    if kind == "vec":
        x, y = (v.double() for v in _vec_inputs(case, seed))
        return (x * y).sum().reshape(1) if case["op"] == "dot" else 1.5 * x + y
    if kind == "spmv":
        A, x = _spmv_inputs(case, seed)
        y = _product(A.row_ptr, A.col_idx, A.val, x)
        return (y, ALPHA * y + x.double()) if case["fused"] else y
    if kind == "csr":
        return _product(*_csr_inputs(case, seed))
    if kind == "batch":
        rp, ci, val, host, x = _batch_inputs(case, seed)
        m, nnz = (torch.as_tensor(v).cuda() for v in (host.m, host.nnz))
        inst = torch.repeat_interleave(torch.arange(host.count, device="cuda"), m)
        at = torch.arange(inst.numel(), device="cuda") + inst
        length = (rp[at + 1] - rp[at]).long()
        rows = torch.repeat_interleave(torch.arange(inst.numel(), device="cuda"), length)
        cols = ci.long() + torch.as_tensor(host.vec_off).cuda()[inst[rows]]
        y = torch.zeros(inst.numel(), dtype=torch.float64, device="cuda").index_add_(
            0, rows, val.double() * x.double()[cols])
        return y, ALPHA * y + x.double()
    if kind == "cg":
        A, b = _cg_inputs(case, seed)
        x, r, p = torch.zeros_like(b), b.clone(), b.clone()
        rr = [r.dot(r)]
        for _ in range(case["iters"]):
            q = _product(A.row_ptr, A.col_idx, A.val, p)
            a = rr[-1] / p.dot(q)
            x, r = x + a * p, r - a * q
            rr.append(r.dot(r))
            p = r + (rr[-1] / rr[-2]) * p
        return x, torch.stack(rr)
    pool, order, xs = _serve_inputs(case, seed)
    out = [([], []), ([], [])]
    for k, x in zip(order, xs):
        y = _product(pool[k].row_ptr, pool[k].col_idx, pool[k].val, x.cuda())
        for to, v in zip(out[0 if x.dtype is torch.float64 else 1], (y, ALPHA * y + x.cuda().double())):
            to.append(v)
    return [torch.cat(v) if v else torch.zeros(0, dtype=torch.float64) for pair in out for v in pair]
