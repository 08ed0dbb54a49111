"""Every extent that a corrector accepts has its transform passes, and a length
without one is an error instead of a launch left out.

A host program over the library's own header (msc_linefft.h) lists, per family
of passes, the lengths that the launches' dispatch reaches and what it does with
the others; the test compares the accepted shapes with the corrector's domain,
stated here by the LDS its lines take (128 KiB, two buffers per line).  The
values at the limits are compared with the oracle on the GPU.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_39474_amd", "csrc")

SRC = r"""
#include <cstdio>
#include "msc_linefft.h"
using namespace msc;
template <int HI> void reach(const char* name, int w) {
  for (int lg = 2; lg <= 16; ++lg) {
    int got = -1;
    try {
      with_lg<2, HI>(lg, [&](auto c) { got = c.value; });
    } catch (const DeviceError&) {
      got = -2;
    }
    std::printf("%s %d %d %d\n", name, w, lg, got);
  }
}
template <class CT> void all(int w) {
  using M = LineMax<CT>;
  reach<M::rows2>("rows2", w);
  reach<M::cols2>("cols2", w);
  reach<M::line3>("line3", w);
  reach<M::fs_rows>("fs_rows", w);
  reach<M::fs_cols>("fs_cols", w);
  if (w == 8) {
    reach<M::wall_rows>("wall_rows", w);
    reach<M::wall_cols>("wall_cols", w);
  }
}
int main() {
  all<double>(8);
  all<float>(4);
}
"""

# 128 KiB over the bytes of one site of a block's lines (real type of w bytes)
FITS = {
    "rows2": lambda n, w: 4 * n * 2 * w <= 131072,    # two lines of a row
    "cols2": lambda n, w: 6 * n * 2 * w <= 131072,    # three fields of a column
    "line3": lambda n, w: 8 * n * 2 * w <= 131072,    # four fields
    "fs_rows": lambda n, w: 10 * n * 2 * w <= 131072,  # five lines of a row
    "fs_cols": lambda n, w: 18 * n * 2 * w <= 131072,  # nine fields of a column
    "wall_rows": lambda n, w: 10 * n * 2 * w <= 131072,
    "wall_cols": lambda n, w: 18 * n * 2 * w <= 131072,
}


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
def test_accepted_lengths_are_dispatched(tmp_path):
    from paper_2609_39474_amd import build

    src, exe = str(tmp_path / "lines.hip"), str(tmp_path / "lines")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run([build.HIPCC, "-std=c++17", "-O1", "--offload-host-only", "-I", CSRC, src, "-o", exe], check=True,
                   capture_output=True, text=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout
    rows = [line.split() for line in out.splitlines()]
    assert len(rows) == 15 * (7 + 5)
    for name, w, lg, got in rows:
        w, lg, got = int(w), int(lg), int(got)
        assert got == (lg if FITS[name](1 << lg, w) else -2), (name, w, lg, got)


# ------------------------------------------------------------------- GPU --
@pytest.fixture(scope="module")
def M():
    from paper_2609_39474_amd import msc
    msc.lib()
    return msc


# bars: those of the shorter lines (test_gpu_fullsym, test_gpu_cavity)
@pytest.mark.gpu
@pytest.mark.parametrize("shape,storage", [((4, 512), "fp64"), ((256, 512), "fp64"), ((4, 512), "fp32"),
                                           ((8, 1024), "fp32"), ((512, 1024), "fp32")])
def test_longest_rows_full_symbol(M, orc, shape, storage):
    import test_gpu_fullsym as TF

    print("longest rows, full symbol", shape, storage, flush=True)
    f, h = TF._state(orc, shape, seed=35 + sum(shape))
    a = 3.0 / 128.0
    h[0] = a
    if storage == "fp32":
        f = f.astype(np.float32).astype(np.float64)  # the stored input
    s = TF._solver(M, shape, storage=storage, tau=(1.0, 1 / 0.8))
    fn, _, R = s.correct(f, h, a)
    s.close()
    ofn, _, oR = orc.full_symbol_iteration(f, h, a, 1.0, 0.8)
    if storage == "fp64":
        assert np.max(np.abs(fn - ofn)) <= 1e-11 * np.max(np.abs(ofn - f))
        assert abs(R - oR) <= 1e-12 * oR
    else:
        assert np.max(np.abs(fn - ofn)) <= 2e-6 * np.max(np.abs(ofn))
        assert abs(R - oR) <= 1e-3 * oR


@pytest.mark.gpu
@pytest.mark.parametrize("shape,storage", [((16, 512), "fp64"), ((64, 512), "fp64"), ((16, 1024), "fp32")])
def test_longest_rows_full_symbol_march(M, shape, storage):
    """The decision and the reconstruction in the rows pass: a call of four
    steps converges, and a replay of its counts one step per call gives the same
    state."""
    import test_gpu_fullsym as TF
    from paper_2609_39474_amd import workloads as W

    print("longest rows, full-symbol march", shape, storage, flush=True)
    n = min(shape)
    p0, u0 = W.random_field_2d(n, 1.0 / 6.0 / n, seed=5, jmax=min(4, n // 4))
    reps = tuple(k // n for k in shape)
    p0, u0 = np.tile(p0, reps), np.tile(u0, (1,) + reps)
    kw = dict(storage=storage, tau=(1.0, 1 / 0.8), eps=1e-10 if storage == "fp64" else 1e-6, p0=p0, u0=u0)
    s = TF._solver(M, shape, **kw)
    rc, stats = s.bdf2_step(4)
    assert rc == 0
    m, K = s.moments(), [x["iters"] for x in stats]
    s.close()
    print("  counts", K, flush=True)
    s = TF._solver(M, shape, **kw)
    s.set_schedule(K)
    for _ in range(4):
        s.bdf2_step(1)
    assert np.isfinite(m).all()
    np.testing.assert_array_equal(s.moments(), m)
    s.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(4, 512), (16, 512)])
def test_longest_rows_walls(M, orc, shape):
    import test_gpu_cavity as TC

    TC.test_wall_corrected_iteration(M, orc, shape, 32.0)


@pytest.mark.gpu
def test_longest_rows_walls_restarts(M, orc):
    """Short restarts and a loose tolerance at rows of 512 (more than one cycle,
    the FP32 basis), by the solve's own residual."""
    import test_gpu_cavity as TC

    for restart, tol in ((6, 1e-10), (50, 1e-4)):
        p = M.make_params(2, 4, dt=32.0, eps=1e-10, corrector="wall_kinetic", n_min=1, k_max=600, boundary="cavity",
                          u_lid=0.04, wall_restart=restart, krylov_tol=tol)
        p.n[0], p.n[1] = 8, 512
        s = M.Solver(p, np.zeros((8, 512)), np.zeros((2, 8, 512)))
        f, h = TC._state(orc, (8, 512), seed=12)
        s.correct(f, h, 1.0 / 32.0)
        solves, iters, _, worst = s.krylov_stats()
        print("walls 8 x 512: restart", restart, "tol", tol, "iterations", iters, "worst", worst, flush=True)
        assert solves == 1 and iters >= 1 and worst <= tol * (1.0 + 1e-6)
        s.close()


@pytest.mark.gpu
def test_longer_rows_are_refused(M):
    for shape, kw in (((4, 1024), dict(corrector="full_symbol")), ((512, 4), dict(corrector="full_symbol")),
                      ((4, 2048), dict(corrector="full_symbol", storage="fp32")),
                      ((1024, 4), dict(corrector="full_symbol", storage="fp32")),
                      ((4, 1024), dict(corrector="wall_kinetic", boundary="cavity")),
                      ((512, 4), dict(corrector="wall_kinetic", boundary="cavity"))):
        p = M.make_params(2, 4, dt=64.0, eps=1e-10, **kw)
        p.n[0], p.n[1] = shape
        with pytest.raises(M.MscError) as ei:
            M.Solver(p, np.zeros(shape), np.zeros((2,) + shape))
        assert ei.value.status == M.MSC_ERR_UNSUPPORTED, (shape, kw)
