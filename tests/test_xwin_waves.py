"""The x-window form's wavefront ranges: on the CPU, a check program replays the
first pass's walk (marks, tiles, carried sums, aligned groups of partials) for
random matrices, chunkings and workgroup sizes; on the GPU, pairs of every
length around the lanes', rows' and tiles' edges give exact sums."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle as O
from conftest import say
from paper_1309_1894_amd import inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_xwin_waves_on_the_cpu(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = tmp_path / "xwin_waves_check"
    build = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                            "-I", os.path.join(ROOT, "paper_1309_1894_amd", "csrc"),
                            os.path.join(ROOT, "tests", "cpp", "xwin_waves_check.cpp"), "-o", str(exe)],
                           capture_output=True, text=True)
    if build.returncode != 0 and "sanitize" in build.stderr:
        pytest.skip("sanitizer runtime not available")
    assert build.returncode == 0, build.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=600,
                         env=dict(os.environ, UBSAN_OPTIONS="halt_on_error=1"))
    assert run.returncode == 0, run.stdout[-4000:] + run.stderr[-4000:]
    assert run.stdout.strip().endswith("ok")


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [1, 0])
@pytest.mark.parametrize("order", ["ascending", "shuffled"])
def test_xwin_pair_lengths(spk, dev, order, dt):
    """Rows of 0 to 70 entries and lengths around a lane's four, a row of
    lanes' 64, a tile's 128 and 256 and several tiles, all in one window of
    three, every kernel, plain and fused.  Integer data: every partial and sum
    is exact, so the outputs are compared bit for bit."""
    np_t = np.float64 if dt else np.float32
    rng = np.random.default_rng(9)
    lens = list(range(71)) + [120, 127, 128, 129, 191, 192, 193, 255, 256, 257, 511, 513, 1000, 3000] + [1] * 700 + [0] * 5
    if order == "shuffled":
        rng.shuffle(lens)
    n = 70000
    rp = np.concatenate([[0], np.cumsum(lens), np.full(n - len(lens), sum(lens))]).astype(np.int32)
    ci = np.concatenate([rng.integers(33000, 40000, rp[-1])]).astype(np.int32)
    ci[::97] = rng.integers(0, 16000, ci[::97].size)          # some pairs in another window
    A = I.CSR(n, n, rp, ci, rng.integers(-8, 9, rp[-1]).astype(np_t))
    x = rng.integers(-8, 9, n).astype(np_t)
    ref, _ = O.spmv(A, x)
    M = spk.Matrix(A)
    xd = torch.from_numpy(x).to(dev)
    y, w = torch.empty_like(xd), torch.empty_like(xd)
    try:
        for bs, kib, e in ((512, 128, 256), (1024, 128, 128), (768, 128, 256), (256, 64, 256), (512, 64, 256)):
            for grid in (1, 2, 4):
                v = spk.make_variant(format=spk.SPK_FMT_XWIN, block=bs, group=kib, lds=e, grid=grid, unroll=1, streams=1)
                say(f"x-window pair lengths {order} dtype={dt} {bs}/{kib}/{e} grid {grid}")
                y.fill_(float("nan"))
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV, A=M, x=xd, y=y), v)
                assert np.array_equal(y.cpu().numpy(), ref.astype(np_t)), v
                w.fill_(float("nan"))
                spk.spk_run(spk.problem(spk.SPK_OP_SPMV_WAXPY, A=M, x=xd, y=y, w=w, alpha=0.5), v)
                assert np.array_equal(w.cpu().numpy(), (0.5 * ref + x).astype(np_t)), v
    finally:
        M.release()
