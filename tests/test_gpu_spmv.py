"""GPU parity of CSR SpMV (y = A*x) and the fused step (w = alpha*y + x)
against the oracle, for every compiled variant (scalar, G lanes per row,
sliced ELL, LDS row blocks), FP64 and FP32, on structural edge cases and on
the workload matrices."""
import numpy as np
import pytest
import torch

import oracle as O
from conftest import say
from paper_1309_1894_amd import inputs as I

pytestmark = pytest.mark.gpu

NP = {0: np.float32, 1: np.float64}


def csr_from_entries(m, n, entries, dtype=np.float64):
    entries = sorted(entries, key=lambda e: e[0])
    rp = np.zeros(m + 1, np.int64)
    for r, _, _ in entries:
        rp[r + 1] += 1
    rp = np.cumsum(rp).astype(np.int32)
    return I.CSR(m, n, rp, np.array([c for _, c, _ in entries], np.int32),
                 np.array([v for _, _, v in entries], dtype))


def edge_cases():
    rng = np.random.default_rng(11)
    out = {
        "m0": csr_from_entries(0, 5, []),                 # no rows: nothing to write
        "m0_n0": csr_from_entries(0, 0, []),
        "n0": csr_from_entries(6, 0, []),                 # no columns: y = 0, x never read
        "1x1": csr_from_entries(1, 1, [(0, 0, 2.5)]),
        "empty_rows": csr_from_entries(7, 5, [(1, 0, 1.25), (1, 4, -3.0), (5, 2, 0.5)]),
        "all_empty": csr_from_entries(300, 300, []),
        "rect_wide": csr_from_entries(5, 900, [(r, int(c), float(rng.uniform(-1, 1)))
                                               for r in range(5) for c in rng.choice(900, 300, replace=False)]),
        "rect_tall": csr_from_entries(700, 3, [(r, r % 3, float(rng.uniform(-1, 1))) for r in range(700)]),
        "duplicates_unsorted": csr_from_entries(4, 6, [(0, 5, 1.0), (0, 0, -0.75), (0, 5, 0.1), (1, 4, 3.0),
                                                       (3, 1, -0.3), (3, 1, 0.3), (3, 0, 0.0)]),
        "lap2d_33": I.lap2d(33),
        "banded_b7": I.banded(5000, 7, 0.6, stream=1),
        "zipf_6000": I.zipf(6000, seed_struct=8, seed_val=9),     # rows up to 4096 entries
    }
    # one dense row longer than every LDS tile, among short rows
    ents = [(r, r, 1.0 + r) for r in range(50)] + [(25, c, float(rng.uniform(-1, 1))) for c in range(50, 9050)]
    out["long_row"] = csr_from_entries(50, 9050, ents)
    return out


CASES = edge_cases()


def _check(A, x, y_gpu, w_gpu=None, alpha=None, dt=1):
    ref, absum = O.spmv(A, x)
    yg = y_gpu.cpu().numpy()
    assert yg.size == A.nrows
    bad, worst, at = O.check_rows(yg.astype(np.float64), ref, absum, O.tau_for(NP[dt]))
    assert bad == 0, f"{bad} rows outside tolerance (worst {worst:g} at row {at})"
    empty = np.diff(A.row_ptr) == 0
    assert np.all(yg[empty] == 0)
    if w_gpu is not None:
        wg = w_gpu.cpu().numpy()
        # the step's w from the GPU's own y: one fused rounding
        wr = O.waxpy(alpha, yg, x[:A.nrows])
        d, at = O.max_ulp(wg, wr)
        assert d <= (0 if dt == 1 else 1), (d, at)
        # end to end against the oracle's step: |w - w_ref| <= |alpha|*tau*sum|a x| + 1 ulp of w
        w_ref = O.waxpy(alpha, ref, x[:A.nrows].astype(np.float64))
        fin = np.isfinite(w_ref)
        inf = np.isinf(w_ref)
        assert np.array_equal(np.isnan(wg), np.isnan(w_ref)), "NaN positions of w"
        assert np.array_equal(wg[inf], w_ref[inf].astype(wg.dtype)), "Inf of w"
        err = np.abs(wg[fin].astype(np.float64) - w_ref[fin])
        bound = abs(alpha) * O.tau_for(NP[dt]) * absum[fin] + np.spacing(np.abs(wg[fin])).astype(np.float64)
        assert np.all(err <= bound), f"w end to end: worst excess {np.max(err - bound):g}"


@pytest.mark.parametrize("dt", [1, 0])
@pytest.mark.parametrize("name", list(CASES))
def test_every_variant(spk, dev, name, dt):
    A = CASES[name].astype(NP[dt])
    M = spk.Matrix(A)
    x = I.uniform(31, 0, A.ncols, NP[dt])
    xd = torch.from_numpy(x).to(dev)
    y = torch.empty(A.nrows, dtype=M.torch_dtype, device=dev)
    vs = spk.variants(spk.SPK_OP_SPMV, dt)
    say(f"spmv {name} dtype={dt}: {len(vs)} variants, m={A.nrows} nnz={A.nnz}")
    try:
        for v in vs:
            for streams in ((1, 2) if v.format != spk.SPK_FMT_SELL else (1,)):
                v.streams = streams
                y.fill_(float("nan"))
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
                try:
                    _check(A, x, y, dt=dt)
                except AssertionError as e:
                    raise AssertionError(f"{v}: {e}")
    finally:
        M.release()


@pytest.mark.parametrize("dt", [1, 0])
@pytest.mark.parametrize("name", ["lap2d_33", "banded_b7", "zipf_6000", "empty_rows", "long_row"])
def test_fused_step_every_variant(spk, dev, name, dt):
    A = CASES[name].astype(NP[dt])
    if A.nrows != A.ncols:
        A = I.CSR(A.nrows, A.nrows, A.row_ptr, np.minimum(A.col_idx, A.nrows - 1).astype(np.int32), A.val)
    M = spk.Matrix(A)
    x = I.uniform(32, 0, A.ncols, NP[dt])
    xd = torch.from_numpy(x).to(dev)
    y = torch.empty(A.nrows, dtype=M.torch_dtype, device=dev)
    w = torch.empty_like(y)
    say(f"spmv_waxpy {name} dtype={dt}")
    try:
        for v in spk.variants(spk.SPK_OP_SPMV_WAXPY, dt):
            y.fill_(float("nan"))
            w.fill_(float("nan"))
            spk.spk_run(spk.problem(spk.SPK_OP_SPMV_WAXPY, A=M, x=xd, y=y, w=w, alpha=0.5), v)
            try:
                _check(A, x, y, w, 0.5, dt)
            except AssertionError as e:
                raise AssertionError(f"{v}: {e}")
    finally:
        M.release()


def test_bit_exact_cases(spk, dev):
    """Identity, diagonal and the Laplacian on polynomials are exact in FP64
    for every variant (integer values, or one rounding)."""
    n = 4099
    rp = np.arange(n + 1, dtype=np.int32)
    ci = np.arange(n, dtype=np.int32)
    d = I.uniform(2, 0, n)
    x = I.uniform(1, 0, n)
    cases = [(I.CSR(n, n, rp, ci, np.ones(n)), x, x),
             (I.CSR(n, n, rp, ci, d), x, d * x)]
    N = 45
    L = I.lap2d(N)
    ii, jj = np.meshgrid(np.arange(N), np.arange(N), indexing="ij")
    ii, jj = ii.ravel().astype(np.float64), jj.ravel().astype(np.float64)
    p = lambda a, b: a * a + b * b
    yexp = np.full(N * N, -4.0)
    for di, dj in ((-1, 0), (1, 0), (0, -1), (0, 1)):
        a, b = ii + di, jj + dj
        out = (a < 0) | (a >= N) | (b < 0) | (b >= N)
        yexp += np.where(out, p(a, b), 0.0)
    cases.append((L, p(ii, jj), yexp))
    for A, xv, yv in cases:
        M = spk.Matrix(A)
        xd = torch.from_numpy(xv).to(dev)
        y = torch.empty(A.nrows, dtype=torch.float64, device=dev)
        try:
            for v in spk.variants(spk.SPK_OP_SPMV, 1):
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
                assert np.array_equal(y.cpu().numpy(), yv), v
        finally:
            M.release()


@pytest.mark.parametrize("dt", [1, 0])
def test_nan_inf_positions(spk, dev, dt):
    A = I.banded(3000, 4, 0.8, stream=2).astype(NP[dt])
    x = I.uniform(3, 0, 3000, NP[dt])
    x[[10, 500, 2999]] = [np.nan, np.inf, -np.inf]
    M = spk.Matrix(A)
    xd = torch.from_numpy(x).to(dev)
    y = torch.empty(3000, dtype=M.torch_dtype, device=dev)
    w = torch.empty_like(y)
    say(f"NaN/Inf in x, dtype={dt}")
    try:
        for v in spk.variants(spk.SPK_OP_SPMV, dt):
            y.fill_(0.0)
            spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
            try:
                _check(A, x, y, dt=dt)
            except AssertionError as e:
                raise AssertionError(f"{v}: {e}")
        for v in spk.variants(spk.SPK_OP_SPMV_WAXPY, dt):
            y.fill_(0.0)
            w.fill_(0.0)
            spk.spk_run(spk.problem(spk.SPK_OP_SPMV_WAXPY, A=M, x=xd, y=y, w=w, alpha=0.5), v)
            try:
                _check(A, x, y, w, 0.5, dt)
            except AssertionError as e:
                raise AssertionError(f"{v}: {e}")
    finally:
        M.release()


@pytest.mark.parametrize("dt", [1, 0])
@pytest.mark.parametrize("name", ["m0", "m0_n0", "n0"])
def test_degenerate_shapes_default_entry_points(spk, dev, name, dt):
    """No rows or no columns through the borrowed-CSR call, the registered
    call and (square shapes) the fused step: OK, nothing written for m = 0,
    y = 0 for n = 0."""
    A = CASES[name].astype(NP[dt])
    say(f"degenerate {name} dtype={dt}")
    x = torch.from_numpy(I.uniform(5, 0, A.ncols, NP[dt])).to(dev)
    rp, ci, val = spk.to_device_csr(A, dev)
    y = torch.full((A.nrows,), float("nan"), dtype=val.dtype, device=dev)
    spk.spk_spmv_csr(rp, ci, val, x, y, nrows=A.nrows, ncols=A.ncols)
    _check(A, x.cpu().numpy(), y, dt=dt)
    M = spk.Matrix(A)
    try:
        y.fill_(float("nan"))
        spk.spk_spmv_mat(M, x, y)
        _check(A, x.cpu().numpy(), y, dt=dt)
        if A.nrows == A.ncols:
            w = torch.empty_like(y)
            spk.spk_spmv_waxpy(M, 0.5, x, y, w)
            _check(A, x.cpu().numpy(), y, w, 0.5, dt)
    finally:
        M.release()


def test_borrowed_csr_and_default_dispatch(spk, dev):
    A = I.zipf(20000, seed_struct=4, seed_val=5)
    x = I.uniform(6, 0, A.ncols)
    rp, ci, val = spk.to_device_csr(A, dev)
    xd = torch.from_numpy(x).to(dev)
    y = spk.spk_spmv_csr(rp, ci, val, xd)
    _check(A, x, y)
    M = spk.Matrix(A)
    try:
        y2 = spk.spk_spmv_mat(M, xd)
        _check(A, x, y2)
        y3, w3 = spk.spk_spmv_waxpy(M, 0.5, xd)
        _check(A, x, y3, w3, 0.5)
        # the same variant gives the same bits every time
        y4 = spk.spk_spmv_mat(M, xd)
        assert torch.equal(y2, y4)
    finally:
        M.release()


def test_register_validation(spk, dev):
    A = I.lap2d(8)
    bad = I.CSR(A.nrows, A.ncols, A.row_ptr.copy(), A.col_idx.copy(), A.val)
    bad.col_idx[5] = 64
    with pytest.raises(spk.SpkError) as e:
        spk.Matrix(bad)
    assert e.value.name == "SPK_ERR_CSR"
    bad2 = I.CSR(A.nrows, A.ncols, A.row_ptr.copy(), A.col_idx, A.val)
    bad2.row_ptr[3] = bad2.row_ptr[4] + 1
    with pytest.raises(spk.SpkError):
        spk.Matrix(bad2)


@pytest.mark.parametrize("which", ["lap3d_128", "zipf_1M"])
def test_full_size_workloads(spk, dev, which):
    """Workload matrices at full size, with the default and the plain
    kernels, then tuned as the bench tunes them (CSR formats, cold cache):
    the winner and the default dispatch that follows its recorded plan."""
    A = I.lap3d(128) if which == "lap3d_128" else I.zipf(1000000)
    say(f"full-size {which}: m={A.nrows} nnz={A.nnz}")
    x = I.uniform(31 if which == "lap3d_128" else 34, 0, A.ncols)
    h = spk.Handle(0)
    M = spk.Matrix(A, handle=h)
    xd = torch.from_numpy(x).to(dev)
    y = torch.empty(A.nrows, dtype=torch.float64, device=dev)
    try:
        p = spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y)
        for v in [None, spk.spk_plain_variant(spk.SPK_OP_SPMV, 0), spk.spk_plain_variant(spk.SPK_OP_SPMV, 1)]:
            y.fill_(float("nan"))
            spk.spk_run(p, v, handle=h)
            _check(A, x, y)
        rep = spk.spk_tune(p, reps=10, warmup=2, flush=True, record=True, formats=spk.CSR_FORMATS, handle=h)
        say(f"full-size {which}: tuned {rep.best}")
        assert rep.rejected == 0
        for v in [rep.best, None]:
            y.fill_(float("nan"))
            spk.spk_run(p, v, handle=h)
            _check(A, x, y)
    finally:
        M.release()
        h.close()


def test_krylov_step_lap2d_256_as_benched(spk, dev):
    """The 2-D step (lap2d(256), w = 0.5*y + x) tuned as the bench tunes it:
    the CSR winner through the default dispatch, the structured winner, and
    1,000 captured steps replayed from a HIP graph, all against the oracle."""
    A = I.lap2d(256)
    x = I.uniform(11, 0, A.nrows)
    say("krylov step lap2d(256) as benched")
    h = spk.Handle(0)
    M = spk.Matrix(A, handle=h)
    xd = torch.from_numpy(x).to(dev)
    y = torch.empty(A.nrows, dtype=torch.float64, device=dev)
    w = torch.empty_like(y)
    try:
        p = spk.problem(spk.SPK_OP_SPMV_WAXPY, A=M, x=xd, y=y, w=w, alpha=0.5)
        rep = spk.spk_tune(p, reps=20, warmup=3, formats=spk.CSR_FORMATS, handle=h)
        assert rep.rejected == 0
        for v in (rep.best, None):
            y.fill_(float("nan"))
            w.fill_(float("nan"))
            spk.spk_run(p, v, handle=h)
            _check(A, x, y, w, 0.5)
        mask = M.formats() & ((1 << spk.SPK_FMT_DIA) | (1 << spk.SPK_FMT_STENCIL))
        st = spk.spk_tune(p, reps=20, warmup=3, record=False, formats=mask, handle=h)
        y.fill_(float("nan"))
        w.fill_(float("nan"))
        spk.spk_run(p, st.best, handle=h)
        yr, wr, _ = O.spmv_waxpy(A, x, 0.5)
        assert np.array_equal(y.cpu().numpy(), yr) and np.array_equal(w.cpu().numpy(), wr)   # sorted rows: exact
        # graph replay of the recorded plan, as the bench times it
        cs = torch.cuda.Stream()
        cs.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(cs):
            spk.spk_spmv_waxpy(M, 0.5, xd, y, w)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=cs):
            for _ in range(1000):
                spk.spk_spmv_waxpy(M, 0.5, xd, y, w)
        y.fill_(float("nan"))
        w.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        _check(A, x, y, w, 0.5)
        del g
    finally:
        M.release()
        h.close()


@pytest.mark.parametrize("dt", [1, 0])
def test_row_blocks_with_x_window_equal_plain_row_blocks(spk, dev, dt):
    """The row-block kernel with room for x in LDS (group 256) gives the bits
    of the same kernel without it on a banded matrix (every row-stream block's
    window fits) and on a 2-D Laplacian of 256 columns per grid line (the
    windows do not fit, x is read from memory), plain and fused."""
    for A in (I.banded(20000, 12, 0.6, stream=3), I.lap2d(256)):
        A = A.astype(NP[dt])
        M = spk.Matrix(A)
        x = I.uniform(41, 0, A.ncols, NP[dt])
        xd = torch.from_numpy(x).to(dev)
        say(f"row blocks with x window: m={A.nrows} dtype={dt}")
        try:
            for bs, e in ((128, 256), (256, 256), (256, 512), (512, 256)):
                outs = []
                for g in (1, 256):
                    v = spk.make_variant(format=spk.SPK_FMT_ADAPTIVE, block=bs, group=g, unroll=1, streams=1, lds=e)
                    y = torch.full((A.nrows,), float("nan"), dtype=M.torch_dtype, device=dev)
                    w = torch.full_like(y, float("nan"))
                    spk.spk_run(spk.problem(spk.SPK_OP_SPMV_WAXPY, A=M, x=xd, y=y, w=w, alpha=0.5), v)
                    _check(A, x, y, w, 0.5, dt)
                    outs.append((y, w))
                assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1]), (bs, e)
        finally:
            M.release()


@pytest.mark.parametrize("dt", [1, 0])
def test_row_blocks_two_byte_columns_equal_four_byte(spk, dev, dt):
    """The row-block kernel reading two-byte column offsets (vec 2) gives the
    bits of the same kernel reading the CSR's columns, plain and fused, with
    and without room for x in LDS: on a banded matrix (every block's window
    fits the room), a 3-D Laplacian (blocks span one grid plane each way:
    offsets fit two bytes, windows do not fit the room), and a random-column
    matrix over 200,000 columns (most blocks span more than 65,536 columns
    and keep the four-byte columns; a few short ones take offsets)."""
    cases = (I.banded(20000, 12, 0.6, stream=5), I.lap3d(40),
             I.zipf(30000, n=200000, kmax=600, seed_struct=61, seed_val=62))
    for A in cases:
        A = A.astype(NP[dt])
        M = spk.Matrix(A)
        x = I.uniform(43, 0, A.ncols, NP[dt])
        xd = torch.from_numpy(x).to(dev)
        say(f"row blocks, two-byte columns: m={A.nrows} n={A.ncols} nnz={A.nnz} dtype={dt}")
        try:
            for bs, g, e in ((64, 1, 256), (64, 1, 512), (64, 1, 1024), (128, 1, 256), (128, 1, 512),
                             (256, 1, 256), (256, 1, 512), (512, 1, 256), (256, 256, 256), (64, 256, 256)):
                outs = []
                for vec in (0, 2):
                    v = spk.make_variant(format=spk.SPK_FMT_ADAPTIVE, block=bs, group=g, unroll=1, streams=1, lds=e,
                                         vec=vec)
                    y = torch.full((A.nrows,), float("nan"), dtype=M.torch_dtype, device=dev)
                    if A.nrows == A.ncols:
                        w = torch.full_like(y, float("nan"))
                        spk.spk_run(spk.problem(spk.SPK_OP_SPMV_WAXPY, A=M, x=xd, y=y, w=w, alpha=0.5), v)
                        _check(A, x, y, w, 0.5, dt)
                    else:   # the fused step needs a square matrix
                        w = y
                        spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
                        _check(A, x, y, None, None, dt)
                    outs.append((y, w))
                assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1]), (bs, g, e)
        finally:
            M.release()


@pytest.mark.parametrize("dt", [1, 0])
def test_row_blocks_two_byte_columns_at_the_width_limit(spk, dev, dt):
    """Two-byte row-block columns at their limit: the first block of a
    70,000-row diagonal matrix also holds column 65,535 (span 65,536:
    offsets up to 65,535) or column 65,536 (span 65,537: that block keeps
    the four-byte columns); bit-equal to the four-byte kernel and against
    the oracle."""
    for far in (65535, 65536):
        m = 70000
        ents = [(i, i, float(v)) for i, v in enumerate(I.uniform(44, 0, m))] + [(0, far, 0.75), (1, 0, -0.5)]
        A = csr_from_entries(m, m, ents, NP[dt])
        M = spk.Matrix(A)
        x = I.uniform(45, 0, m, NP[dt])
        xd = torch.from_numpy(x).to(dev)
        say(f"row blocks, two-byte columns at the limit: far column {far}, dtype={dt}")
        try:
            outs = []
            for vec in (0, 2):
                v = spk.make_variant(format=spk.SPK_FMT_ADAPTIVE, block=256, group=1, unroll=1, streams=1, lds=256,
                                     vec=vec)
                y = torch.full((m,), float("nan"), dtype=M.torch_dtype, device=dev)
                w = torch.full_like(y, float("nan"))
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV_WAXPY, A=M, x=xd, y=y, w=w, alpha=0.5), v)
                _check(A, x, y, w, 0.5, dt)
                outs.append((y, w))
            assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1]), far
        finally:
            M.release()


@pytest.mark.parametrize("dt", [1, 0])
def test_row_tiles_at_the_length_limits(spk, dev, dt):
    """Row lengths on both sides of every limit of the row-block tiles (one
    lane, 16 lanes, a wavefront, a workgroup per row), mixed, every row-block
    variant, plain and fused, on one, two and four streams.  Integer data:
    every sum is exact, so the outputs are compared bit for bit."""
    lens = [0, 1, 95, 96, 97, 3, 128, 255, 256, 257, 0, 511, 512, 513, 5, 600, 1023, 1024, 1025, 2, 2047, 2048, 2049,
            4096, 4097, 1, 0, 98, 99, 100, 101, 130, 1, 1, 4700, 513, 514] + [97] * 9 + [2] * 150 + [1025]
    n = 4800
    rng = np.random.default_rng(5)
    rp = np.concatenate([[0], np.cumsum(lens + [0] * (n - len(lens)))]).astype(np.int32)
    A = I.CSR(n, n, rp, rng.integers(0, n, rp[-1]).astype(np.int32), rng.integers(-8, 9, rp[-1]).astype(NP[dt]))
    x = rng.integers(-8, 9, n).astype(NP[dt])
    ref, _ = O.spmv(A, x)
    M = spk.Matrix(A)
    xd = torch.from_numpy(x).to(dev)
    y, w = torch.empty_like(xd), torch.empty_like(xd)
    vs = [v for v in spk.variants(spk.SPK_OP_SPMV, dt) if v.format == spk.SPK_FMT_ADAPTIVE]
    say(f"row tiles at their limits dtype={dt}: {len(vs)} variants")
    try:
        for v in vs:
            for streams in (1, 2, 4):
                v.streams = streams
                y.fill_(float("nan"))
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
                assert np.array_equal(y.cpu().numpy(), ref.astype(NP[dt])), v
                y.fill_(float("nan"))
                w.fill_(float("nan"))
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV_WAXPY, A=M, x=xd, y=y, w=w, alpha=0.5), v)
                assert np.array_equal(y.cpu().numpy(), ref.astype(NP[dt])), v
                assert np.array_equal(w.cpu().numpy(), (0.5 * ref + x).astype(NP[dt])), v
    finally:
        M.release()


@pytest.mark.parametrize("dt", [1, 0])
@pytest.mark.parametrize("m,mean", [(8191, 20), (8192, 20), (8193, 79), (8200, 82), (20001, 5), (70001, 9), (70001, 11),
                                    (140001, 9), (140001, 0)])
def test_borrowed_csr_default_on_both_sides_of_its_rules(spk, dev, m, mean, dt):
    """spk_spmv_csr's default kernel around its limits (rows, mean length),
    ragged last wavefronts, empty rows, rows longer than a chunk and rows that
    end exactly at one.  Integer data: exact, compared bit for bit."""
    rng = np.random.default_rng(m + mean)
    lens = rng.integers(0, 2 * mean + 1, m)
    lens[[0, m // 2, m - 1]] = [2000, 512, 1500]
    lens[1:4] = 0
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    A = I.CSR(m, 4099, rp, rng.integers(0, 4099, rp[-1]).astype(np.int32), rng.integers(-8, 9, rp[-1]).astype(NP[dt]))
    x = rng.integers(-8, 9, 4099).astype(NP[dt])
    ref, _ = O.spmv(A, x)
    say(f"borrowed csr m={m} mean={mean} dtype={dt}")
    d = [torch.from_numpy(v).to(dev) for v in (A.row_ptr, A.col_idx, A.val, x)]
    y = torch.full((m + 64,), float("nan"), dtype=d[3].dtype, device=dev)
    spk.spk_spmv_csr(*d, y[:m])
    got = y.cpu().numpy()
    assert np.array_equal(got[:m], ref.astype(NP[dt])) and np.all(np.isnan(got[m:]))
    # arrays that are only element-aligned
    o = [torch.cat([t[:1], t])[1:] for t in d[1:3]]
    y.fill_(float("nan"))
    spk.spk_spmv_csr(d[0], o[0], o[1], d[3], y[:m])
    assert np.array_equal(y.cpu().numpy()[:m], ref.astype(NP[dt]))


@pytest.mark.parametrize("dt", [1, 0])
@pytest.mark.parametrize("group,unroll", [(8, 1), (4, 3), (16, 1), (4, 5), (8, 3), (4, 7), (32, 1), (16, 3), (64, 1)])
@pytest.mark.parametrize("mean", [1, 19, 70])
def test_row_stream_shapes(spk, dev, group, unroll, mean, dt):
    """Every row stream shape (rows per wavefront, powers of two or not) on
    rows that leave the last wavefront ragged, empty rows, rows longer than a
    chunk, and chunks that end at and inside a row.  Integer data: exact."""
    rows = group * unroll
    m = 37 * rows + rows // 2 + 1
    rng = np.random.default_rng(rows * 100 + mean)
    lens = rng.integers(0, 2 * mean + 1, m)
    lens[[0, m // 2, m - 1]] = [1100, 512, 700]
    lens[rows:2 * rows] = 512 // rows                   # a wavefront whose rows fill one chunk at most
    lens[2 * rows:3 * rows] = 0                         # and one without entries
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n = 1009
    A = I.CSR(m, n, rp, rng.integers(0, n, rp[-1]).astype(np.int32), rng.integers(-8, 9, rp[-1]).astype(NP[dt]))
    x = rng.integers(-8, 9, n).astype(NP[dt])
    ref = O.spmv(A, x)[0].astype(NP[dt])
    M = spk.Matrix(A)
    try:
        xd = torch.from_numpy(x).to(dev)
        y = torch.full((m + 64,), float("nan"), dtype=xd.dtype, device=dev)
        v = spk.make_variant(format=2, block=256, group=group, unroll=unroll, lds=512, streams=1)
        spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y[:m]), v)
        got = y.cpu().numpy()
        assert np.array_equal(got[:m], ref) and np.all(np.isnan(got[m:]))
    finally:
        M.release()


@pytest.mark.parametrize("dt", [1, 0])
@pytest.mark.parametrize("extra", [0, 1])
def test_matrices_on_both_sides_of_the_cache_rule(spk, dev, extra, dt):
    """A matrix of exactly 80 MB of values and columns and one of an entry
    more (where the values' loads change), by row blocks and by the row stream.
    Integer data: exact."""
    nnz = (80 << 20) // (np.dtype(NP[dt]).itemsize + 4) + extra
    m = nnz // 21
    lens = np.full(m, nnz // m)
    lens[:nnz - int(lens.sum())] += 1
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    assert rp[-1] == nnz
    n = 4096
    k = np.arange(nnz, dtype=np.int64)
    A = I.CSR(m, n, rp, ((k * 2654435761) % n).astype(np.int32), ((k % 17) - 8).astype(NP[dt]))
    x = (np.arange(n) % 13 - 6).astype(NP[dt])
    ref = np.add.reduceat((A.val.astype(np.float64) * x[A.col_idx]), rp[:-1])
    say(f"cache rule nnz={nnz} dtype={dt}")
    M = spk.Matrix(A)
    try:
        xd = torch.from_numpy(x).to(dev)
        y = torch.empty(m, dtype=xd.dtype, device=dev)
        spk.spk_spmv_mat(M, xd, y)
        assert np.array_equal(y.cpu().numpy(), ref.astype(NP[dt]))
        d = [torch.from_numpy(t).to(dev) for t in (A.row_ptr, A.col_idx, A.val)]
        y.fill_(float("nan"))
        spk.spk_spmv_csr(*d, xd, y)
        assert np.array_equal(y.cpu().numpy(), ref.astype(NP[dt]))
    finally:
        M.release()


@pytest.mark.parametrize("dt", [1, 0])
@pytest.mark.parametrize("left", [1, 64, 127, 128, 129, 255, 256, 257, 511, 512, 513, 640, 641, 768, 769, 1025])
def test_row_stream_chunk_tails(spk, dev, left, dt):
    """The row stream's chunks have forms for at most 128, at most 256 and more
    entries: wavefronts whose rows hold `left` entries, as one row among empty
    ones or spread over all, every shape, plain and fused.  Integer data: sums
    are exact, so the outputs are compared bit for bit."""
    rng = np.random.default_rng(left)
    for rows in (8, 12, 16, 20, 24, 28, 32, 48, 64):
        runs = []
        for i in range(40):
            n = np.zeros(rows, np.int64)
            if i % 2:
                n[rng.integers(rows)] = left
            else:
                n += np.bincount(rng.integers(0, rows, left), minlength=rows)
            runs.append(n)
        lens = np.concatenate(runs)
        m = lens.size
        rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        A = I.CSR(m, m, rp, rng.integers(0, m, rp[-1]).astype(np.int32), rng.integers(-8, 9, rp[-1]).astype(NP[dt]))
        x = rng.integers(-8, 9, m).astype(NP[dt])
        ref, _ = O.spmv(A, x)
        say(f"row stream chunk tails left={left} rows={rows} dtype={dt}")
        M = spk.Matrix(A)
        xd = torch.from_numpy(x).to(dev)
        y, w = torch.full_like(xd, float("nan")), torch.full_like(xd, float("nan"))
        try:
            g, u = {8: (8, 1), 12: (4, 3), 16: (16, 1), 20: (4, 5), 24: (8, 3), 28: (4, 7), 32: (32, 1), 48: (16, 3),
                    64: (64, 1)}[rows]
            v = spk.make_variant(format=spk.SPK_FMT_VECTOR, block=256, group=g, unroll=u, lds=512, streams=1)
            spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
            assert np.array_equal(y.cpu().numpy(), ref.astype(NP[dt]))
            y.fill_(float("nan"))
            spk.spk_run(spk.problem(spk.SPK_OP_SPMV_WAXPY, A=M, x=xd, y=y, w=w, alpha=0.5), v)
            assert np.array_equal(y.cpu().numpy(), ref.astype(NP[dt]))
            assert np.array_equal(w.cpu().numpy(), (0.5 * ref + x).astype(NP[dt]))
        finally:
            M.release()


@pytest.mark.parametrize("length", [8, 16, 20, 39, 60, 79])
def test_borrowed_csr_is_as_accurate_as_lanes_per_row(spk, dev, length):
    """FP64 products of a borrowed CSR (the row stream rounds a product before
    it adds it) have no larger rms error than one lane per entry and a tree
    (G lanes per row), both against sums in 80-bit floats."""
    m = 40000
    rng = np.random.default_rng(length)
    ci = np.sort(rng.integers(0, m, (m, length)), axis=1).astype(np.int32)
    val, x = rng.random((m, length)) * 2 - 1, rng.random(m) * 2 - 1
    # products exactly (Dekker's split), summed in 80 bits
    def split(v):
        t = 134217729.0 * v
        hi = t - (t - v)
        return hi, v - hi
    xs = x[ci]
    (vh, vl), (xh, xl) = split(val), split(xs)
    p = val * xs
    e = ((vh * xh - p) + vh * xl + vl * xh) + vl * xl
    exact = p.astype(np.longdouble).sum(1) + e.astype(np.longdouble).sum(1)
    A = I.CSR(m, m, (np.arange(m + 1) * length).astype(np.int32), ci.ravel(), val.ravel())
    say(f"accuracy of the borrowed CSR product, rows of {length}")
    xd = torch.from_numpy(x).to(dev)

    def rms(y):
        return float(np.sqrt(np.mean((y.cpu().numpy().astype(np.longdouble) - exact) ** 2)))

    stream = rms(spk.spk_spmv_csr(*spk.to_device_csr(A, dev), xd))
    M = spk.Matrix(A)
    try:
        g = min(64, 1 << (length - 1).bit_length())
        y = torch.empty_like(xd)
        v = spk.make_variant(format=spk.SPK_FMT_VECTOR, block=256, group=g, unroll=1, streams=1)
        spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
        lanes = rms(y)
    finally:
        M.release()
    assert stream <= lanes, (stream, lanes)


@pytest.mark.parametrize("length,rows", [(300, 12000), (512, 8000), (800, 1500), (1100, 1500)])
def test_wide_rows_are_as_accurate_as_lanes_per_row(spk, dev, length, rows):
    """FP64 row blocks (a product is rounded on its way through LDS) have no
    larger rms error than a wavefront per row with four sums to a lane, both
    against sums in 80-bit floats; the rows of one length, signs mixed."""
    rng = np.random.default_rng(length)
    n = 8000
    ci = rng.integers(0, n, (rows, length)).astype(np.int32)
    val = rng.random((rows, length)) * 2 - 1
    A = I.CSR(rows, n, (np.arange(rows + 1) * length).astype(np.int32), ci.ravel(), val.ravel())
    say(f"accuracy of rows of {length}")

    def split(v):                       # Dekker's: exact products
        t = 134217729.0 * v
        hi = t - (t - v)
        return hi, v - hi

    M = spk.Matrix(A)
    square = {None: 0.0, 64: 0.0}
    try:
        for _ in range(max(1, 12000 // rows)):
            x = rng.random(n) * 2 - 1
            xs = x[ci]
            (vh, vl), (xh, xl) = split(val), split(xs)
            p = val * xs
            e = ((vh * xh - p) + vh * xl + vl * xh) + vl * xl
            exact = p.astype(np.longdouble).sum(1) + e.astype(np.longdouble).sum(1)
            xd = torch.from_numpy(x).to(dev)
            for g in square:
                y = torch.empty(rows, dtype=torch.float64, device=dev)
                v = g and spk.make_variant(format=spk.SPK_FMT_VECTOR, block=256, group=g, unroll=4, streams=1)
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
                square[g] += float(np.sum((y.cpu().numpy().astype(np.longdouble) - exact) ** 2))
    finally:
        M.release()
    assert square[None] <= square[64], (square[None] / square[64]) ** 0.5


@pytest.mark.parametrize("dt", [1, 0])
def test_row_blocks_either_side_of_the_kept_size(spk, dev, dt):
    """Row blocks have a form whose values may stay in the last-level cache
    (matrices up to 80 MB of values and columns) and one whose values may not:
    sizes on both sides of the line, four- and two-byte columns, with and
    without room for x.  Integer data: bit for bit."""
    per = 10
    line = (80 << 20) // (12 if dt else 8) // per      # rows of `per` entries that reach it
    rng = np.random.default_rng(5)
    for m in (line, line + 1):
        start = np.minimum(np.arange(m), m - 20)
        ci = (start[:, None] + np.arange(0, 20, 2)[None, :]).astype(np.int32)
        A = I.CSR(m, m, (np.arange(m + 1) * per).astype(np.int32), ci.ravel(),
                  rng.integers(-8, 9, m * per).astype(NP[dt]))
        x = rng.integers(-8, 9, m).astype(NP[dt])
        ref, _ = O.spmv(A, x)
        M = spk.Matrix(A)
        xd = torch.from_numpy(x).to(dev)
        y, w = torch.empty_like(xd), torch.empty_like(xd)
        try:
            for group, vec in ((1, 0), (1, 2), (256, 0), (256, 2)):
                say(f"row blocks m={m} dtype={dt} group={group} vec={vec}")
                v = spk.make_variant(format=spk.SPK_FMT_ADAPTIVE, block=256, group=group, unroll=1, streams=1, lds=256,
                                     vec=vec)
                y.fill_(float("nan"))
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
                assert np.array_equal(y.cpu().numpy(), ref.astype(NP[dt]))
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV_WAXPY, A=M, x=xd, y=y, w=w, alpha=0.5), v)
                assert np.array_equal(w.cpu().numpy(), (0.5 * ref + x).astype(NP[dt]))
        finally:
            M.release()
