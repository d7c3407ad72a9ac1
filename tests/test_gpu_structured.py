"""GPU parity of the structured SpMV formats (DIA, matrix-free stencil)
against the oracle.  Both add a row's products in ascending column order
with fused multiply-adds -- the oracle's order on rows with sorted columns
-- so on the generators' matrices the product is bit-exact (FP32: the
oracle's double result rounded once)."""
import numpy as np
import pytest
import torch

import oracle as O
from conftest import say
from paper_1309_1894_amd import inputs as I

pytestmark = pytest.mark.gpu

NP = {0: np.float32, 1: np.float64}
DIA, STENCIL = 5, 6


def tridiag(n):
    r = np.concatenate([np.arange(1, n), np.arange(n), np.arange(n - 1)])
    c = np.concatenate([np.arange(n - 1), np.arange(n), np.arange(1, n)])
    v = np.concatenate([np.full(n - 1, -1.25), np.full(n, 2.5), np.full(n - 1, 0.5)])
    order = np.lexsort((c, r))
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, r + 1, 1)
    return I.CSR(n, n, np.cumsum(rp).astype(np.int32), c[order].astype(np.int32), v[order])


CASES = {
    "lap2d_33": (lambda: I.lap2d(33), {DIA, STENCIL}),
    "lap3d_20": (lambda: I.lap3d(20), {DIA, STENCIL}),
    "lap3d_5x_odd": (lambda: I.lap3d(5), {DIA, STENCIL}),
    "tridiag_4099": (lambda: tridiag(4099), {DIA, STENCIL}),
    "banded_b5_full": (lambda: I.banded(3001, 5, 1.0, stream=6), {DIA}),
    "banded_b3_fill06": (lambda: I.banded(2999, 3, 0.6, stream=7), {DIA}),   # absent slots inside the band
}


# compiled structured variants: (threads, rows per lane, x staged in LDS)
SHAPES = {DIA: [(bs, r, 0) for bs in (128, 256, 512) for r in (1, 2)],
          STENCIL: [(bs, r, 0) for bs in (128, 256) for r in (1, 2, 4, 8)] + [(512, r, 0) for r in (1, 2, 4)]
          + [(bs, r, 1) for bs in (256, 512) for r in (2, 4)]}


def _variants(spk, fmt):
    return [spk.make_variant(format=fmt, block=bs, group=1, unroll=r, streams=1, lds=l) for bs, r, l in SHAPES[fmt]]


def _expect(A, x, dt):
    ref, _ = O.spmv(A, x)
    return ref.astype(NP[dt])


@pytest.mark.parametrize("dt", [1, 0])
@pytest.mark.parametrize("name", list(CASES))
def test_structured_formats_bit_exact(spk, dev, name, dt):
    make, fmts = CASES[name]
    A = make().astype(NP[dt])
    M = spk.Matrix(A)
    try:
        mask = M.formats()
        assert {f for f in (DIA, STENCIL) if mask & (1 << f)} == fmts
        x = I.uniform(41, 0, A.ncols, NP[dt])
        xd = torch.from_numpy(x).to(dev)
        y = torch.empty(A.nrows, dtype=M.torch_dtype, device=dev)
        w = torch.empty_like(y)
        yref = _expect(A, x, dt)
        wref = O.waxpy(0.5, yref, x)
        for fmt in sorted(fmts):
            for v in _variants(spk, fmt):
                say(f"structured {name} dt={dt} format={fmt} block={v.block} rows={v.unroll} lds={v.lds}")
                y.fill_(float("nan"))
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
                assert np.array_equal(y.cpu().numpy(), yref), (fmt, v.block, v.unroll, v.lds)
                y.fill_(float("nan"))
                w.fill_(float("nan"))
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV_WAXPY, A=M, x=xd, y=y, w=w, alpha=0.5), v)
                assert np.array_equal(y.cpu().numpy(), yref)
                # FP32: the oracle's w is rounded twice (double, then float)
                d, at = O.max_ulp(w.cpu().numpy(), wref)
                assert d <= (0 if dt == 1 else 1), (fmt, v.block, d, at)
    finally:
        M.release()


def test_absent_slots_do_not_touch_inf(spk, dev):
    """DIA padding is skipped, not multiplied: Inf/NaN in x reach exactly
    the rows that store an entry in their column."""
    A = I.banded(2000, 3, 0.6, stream=8)
    x = I.uniform(42, 0, A.ncols)
    x[[5, 700, 1999]] = [np.inf, np.nan, -np.inf]
    M = spk.Matrix(A)
    try:
        xd = torch.from_numpy(x).to(dev)
        y = torch.empty(A.nrows, dtype=torch.float64, device=dev)
        ref, _ = O.spmv(A, x)
        for v in _variants(spk, DIA):
            spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
            yg = y.cpu().numpy()
            assert np.array_equal(np.isnan(yg), np.isnan(ref))
            fin = np.isfinite(ref)
            assert np.array_equal(yg[~fin & ~np.isnan(ref)], ref[~fin & ~np.isnan(ref)])
            assert np.array_equal(yg[fin], ref[fin])
    finally:
        M.release()


def test_format_not_applicable_is_an_error(spk, dev):
    A = I.zipf(3000, seed_struct=9, seed_val=10)
    M = spk.Matrix(A)
    try:
        assert not (M.formats() & ((1 << DIA) | (1 << STENCIL)))
        xd = torch.from_numpy(I.uniform(43, 0, A.ncols)).to(dev)
        y = torch.empty(A.nrows, dtype=torch.float64, device=dev)
        for fmt in (DIA, STENCIL):
            with pytest.raises(spk.SpkError, match="SPK_ERR_ARG"):
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), _variants(spk, fmt)[0])
            with pytest.raises(spk.SpkError, match="SPK_ERR_ARG"):
                M.format_bytes(fmt)
    finally:
        M.release()


def test_staged_stencil_needs_short_grid_lines(spk, dev):
    """A 2-D stencil whose grid lines are too long for the LDS budget
    (64 KiB: block*rows + 2*N3 values) rejects the staged variants and the
    tuner leaves them out; the unstaged ones still run."""
    N = 6000   # 2*6000*8 bytes of halo + the rows exceed 64 KiB
    rows, cols, vals = [], [], []
    # a 2-D Laplacian on a 3 x N grid (N3 = N)
    n = 3 * N
    r = np.arange(n)
    k, j = r % N, r // N
    for off, ok, v in ((-N, j > 0, -1.0), (-1, k > 0, -1.0), (0, np.ones(n, bool), 4.0), (1, k < N - 1, -1.0),
                       (N, j < 2, -1.0)):
        rows.append(r[ok]); cols.append(r[ok] + off); vals.append(np.full(ok.sum(), v))
    rows, cols, vals = (np.concatenate(t) for t in (rows, cols, vals))
    order = np.lexsort((cols, rows))
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, rows + 1, 1)
    A = I.CSR(n, n, np.cumsum(rp).astype(np.int32), cols[order].astype(np.int32), vals[order])
    M = spk.Matrix(A)
    try:
        assert M.formats() & (1 << STENCIL)
        x = I.uniform(45, 0, n)
        xd = torch.from_numpy(x).to(dev)
        y = torch.empty(n, dtype=torch.float64, device=dev)
        ref, _ = O.spmv(A, x)
        staged = spk.make_variant(format=STENCIL, block=512, group=1, unroll=4, streams=1, lds=1)
        with pytest.raises(spk.SpkError, match="SPK_ERR_ARG"):
            spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), staged)
        plain = spk.make_variant(format=STENCIL, block=256, group=1, unroll=2, streams=1)
        spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), plain)
        assert np.array_equal(y.cpu().numpy(), ref)
        rep = spk.spk_tune(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), reps=2, warmup=1, record=False,
                           formats=1 << STENCIL)
        assert rep.tried == len([s for s in SHAPES[STENCIL] if s[2] == 0]) and rep.best.lds == 0
    finally:
        M.release()


def test_format_bytes(spk, dev):
    A = I.lap3d(16)
    M = spk.Matrix(A)
    try:
        n, nnz = A.nrows, A.nnz
        assert M.format_bytes(spk.SPK_FMT_ADAPTIVE) == 12 * nnz + 4 * (n + 1) + 16 * n
        assert M.format_bytes(DIA) == 7 * 8 * n + 2 * n + 16 * n
        assert M.format_bytes(STENCIL) == 16 * n
        assert M.format_bytes(STENCIL, fused=True) == 24 * n
    finally:
        M.release()


def test_tuner_searches_structured_formats(spk, dev):
    """spk_tune validates and times DIA and stencil variants when the matrix
    admits them, and leaves them out when the format mask does."""
    A = I.lap3d(48)
    H = spk.Handle()
    try:
        M = spk.Matrix(A, handle=H)
        xd = torch.from_numpy(I.uniform(44, 0, A.ncols)).to(dev)
        y = torch.empty(A.nrows, dtype=torch.float64, device=dev)
        say("tune lap3d 48, all formats")
        rep = spk.spk_tune(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), reps=3, warmup=1, record=False, handle=H)
        assert rep.rejected == 0
        ref, absum = O.spmv(A, I.uniform(44, 0, A.ncols))
        assert O.check_rows(y.cpu().numpy(), ref, absum, O.TAU_F64)[0] == 0
        say("tune lap3d 48, CSR formats only")
        rep2 = spk.spk_tune(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), reps=3, warmup=1, record=False,
                            formats=spk.CSR_FORMATS, handle=H)
        assert rep2.best.format not in (DIA, STENCIL)
        # every structured variant more; the stream refinement (two more
        # timed runs) follows a CSR winner only
        ns = len(SHAPES[DIA]) + len(SHAPES[STENCIL])
        structured_won = rep.best.format in (DIA, STENCIL)
        assert rep.tried - rep2.tried == (ns - 2 if structured_won else ns)
        M.release()
    finally:
        H.close()


def test_full_size_lap3d_128(spk, dev):
    A = I.lap3d(128)
    x = I.uniform(31, 0, A.ncols)
    M = spk.Matrix(A)
    try:
        xd = torch.from_numpy(x).to(dev)
        y = torch.empty(A.nrows, dtype=torch.float64, device=dev)
        ref, _ = O.spmv(A, x)
        for fmt in (DIA, STENCIL):
            say(f"full-size lap3d 128 format {fmt}")
            for v in _variants(spk, fmt):
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
                assert np.array_equal(y.cpu().numpy(), ref), (fmt, v.block, v.unroll, v.lds)
    finally:
        M.release()


def grid_stencil(dims, coef):
    """The constant-coefficient stencil on a grid of `dims` lines (slowest
    first), `coef` per offset in ascending column order, columns of each row
    in descending order (storage order is the caller's)."""
    n = int(np.prod(dims))
    strides = [int(np.prod(dims[d + 1:])) for d in range(len(dims))]
    r = np.arange(n)
    rows, cols, vals = [], [], []
    steps = [(-s, (r // s) % d > 0) for s, d in zip(strides, dims)] + [(0, np.ones(n, bool))]
    steps += [(s, (r // s) % d < d - 1) for s, d in list(zip(strides, dims))[::-1]]
    for (off, ok), v in zip(steps, coef):
        rows.append(r[ok])
        cols.append(r[ok] + off)
        vals.append(np.full(int(ok.sum()), v))
    rows, cols, vals = map(np.concatenate, (rows, cols, vals))
    order = np.lexsort((-cols, rows))
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, rows + 1, 1)
    return I.CSR(n, n, np.cumsum(rp).astype(np.int32), cols[order].astype(np.int32), vals[order])


COEF = (-0.75, 0.3125, -1.1, 4.7, 0.9, -2.3, 0.55)
GRIDS = {1: (4099,), 2: (61, 67), 3: (17, 5, 23)}
BIG = {1: ((1 << 20) - 1, 1 << 20), 2: (1023, 1024), 3: (127, 128)}


@pytest.mark.parametrize("dt", [1, 0])
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("dims", list(GRIDS.values()) + [(b,) for b in BIG[1]] + [(b, 1024) for b in BIG[2]]
                         + [(b, 128, 64) for b in BIG[3]], ids=str)
def test_default_of_grid_stencils_is_the_matrix_free_form(spk, dev, dims, fused, dt):
    """The default product of grid stencils in one, two and three dimensions,
    on both sides of the 2^20 rows where its shape changes: the bits of the
    matrix-free form, within rounding of the row blocks' (at most 7 products
    and 6 additions in FP64 each way, one rounding to the result's type), with
    Inf and NaN in x reaching the same rows, and x and y off 16-byte alignment.
    With one value changed in its last bit, A is no stencil and takes the row
    blocks."""
    say("default stencil", dims, fused, dt)
    npt = NP[dt]
    A = grid_stencil(dims, COEF[3 - len(dims):4 + len(dims)]).astype(npt)
    n = A.nrows
    h = spk.Handle(0)
    try:
        op = spk.SPK_OP_SPMV_WAXPY if fused else spk.SPK_OP_SPMV
        alpha = 0.625
        tiles = spk.make_variant(format=spk.SPK_FMT_ADAPTIVE, block=256, group=1, unroll=1, streams=1, lds=512)
        free = spk.make_variant(format=STENCIL, block=256, group=1, unroll=1, streams=1)

        def product(M, x, v):
            y = torch.full((n + 1,), 7.0, dtype=M.torch_dtype, device=dev)[1:]
            w = torch.full((n + 1,), 7.0, dtype=M.torch_dtype, device=dev)[1:]
            spk.spk_run(spk.problem(op, A=M, x=x, y=y, alpha=alpha, **({"w": w} if fused else {})), v, handle=h)
            return [t.double().cpu().numpy() for t in ((y, w) if fused else (y,))]

        x = torch.from_numpy(I.uniform(77, 0, n + 1, npt)).to(dev)[1:]
        M = spk.Matrix(A, handle=h)
        assert M.formats() & (1 << STENCIL)
        absx = np.abs(x.double().cpu().numpy())
        bound = 26 * 2.0 ** -53 * sum(abs(c) for c in COEF) * absx.max()
        eps = 2.0 ** -52 if dt == 1 else 2.0 ** -23
        for special in (False, True):
            if special:
                x[n // 3] = float("inf")
                x[n // 2] = float("nan")
            got, same, ref = (product(M, x, v) for v in (None, free, tiles))
            for g, s, r in zip(got, same, ref):
                assert np.array_equal(g, s, equal_nan=True)
                fin = np.isfinite(r)
                assert np.array_equal(np.isnan(g), np.isnan(r))
                assert np.array_equal(g[~fin], r[~fin], equal_nan=True)
                # w = alpha*y + x: one more rounding of each, of at most |w|
                lim = bound + eps * np.abs(r[fin]) + (eps * np.abs(r[fin]) + eps * bound * 4 if fused else 0.0)
                if fused and dt == 0:
                    lim = lim + 2 * eps * alpha * sum(abs(c) for c in COEF) * absx.max()
                assert np.all(np.abs(g[fin] - r[fin]) <= lim)
        M.release()
        x = torch.from_numpy(I.uniform(78, 0, n, npt)).to(dev)
        val = A.val.copy()
        val[A.nnz // 2] = np.nextafter(val[A.nnz // 2], npt(np.inf))
        M = spk.Matrix(I.CSR(n, n, A.row_ptr, A.col_idx, val), handle=h)
        assert not M.formats() & (1 << STENCIL)
        for g, r in zip(product(M, x, None), product(M, x, tiles)):
            assert np.array_equal(g, r)
        M.release()
    finally:
        h.close()
