"""Every line length of the transforms in registers, at the extremes of the
extents: one corrected iteration against the oracle, in 2D, 3D, with the
full-symbol corrector and with the wall corrector.  Bars: those of the other
extents (test_gpu_parity, test_gpu_fullsym, test_gpu_cavity): 1e-12 relative in
FP64; FP32 2e-6 of max |f| and 1e-5 of the correction."""
import numpy as np
import pytest

import test_gpu_cavity as TC
import test_gpu_fullsym as TF
import test_gpu_parity as TP

pytestmark = pytest.mark.gpu

NU = 1.0 / 6.0


@pytest.fixture(scope="module")
def M():
    from paper_2609_39474_amd import msc
    msc.lib()
    return msc


# each extent from 4 to the limit along x and along y (both storages), with
# rows inside the sweep (y <= 256) and as passes of their own
SHAPES_2D = [(4, 4), (4, 512), (8, 4), (8, 1024), (16, 2048), (1024, 4), (512, 8), (256, 16), (64, 32), (32, 1024),
             (2048, 4), (4, 4096)]


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES_2D)
def test_lines_2d(M, orc, shape, storage):
    if storage == "fp64" and (shape[0] > 1024 or shape[1] > 2048):
        pytest.skip("beyond the FP64 transforms")
    print("lines 2D", shape, storage, flush=True)
    _check(M, orc, 2, shape, storage)


SHAPES_3D = [(4, 4, 4), (4, 8, 16), (16, 4, 8), (8, 16, 4), (4, 4, 256), (4, 256, 4), (256, 4, 4), (4, 32, 512),
             (512, 4, 8), (8, 512, 4), (4, 4, 1024), (1024, 4, 4)]


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES_3D)
def test_lines_3d(M, orc, shape, storage):
    print("lines 3D", shape, storage, flush=True)
    _check(M, orc, 3, shape, storage)


def _check(M, orc, d, shape, storage):
    f, h = TP._rand_state(orc, d, shape, seed=31 + sum(shape))
    a = 3.0 / 128.0
    if storage == "fp32":
        f = f.astype(np.float32).astype(np.float64)  # the stored input
    s = TP._solver(M, shape, storage=storage)
    fn, dm, R = s.correct(f, h, a)
    s.close()
    ofn, _, _, odm, oR = orc.corrected_iteration(f, h, a, 1.0, 1.0, NU)
    if storage == "fp64":
        assert TP.rel_fields(dm, odm) <= 1e-12
        assert TP.rel(fn, ofn) <= 1e-12
        assert abs(R - oR) <= 1e-12 * oR
    else:
        assert np.max(np.abs(fn - ofn)) <= 2e-6 * np.max(np.abs(ofn))
        assert TP.rel(dm, odm) <= 1e-5
        assert abs(R - oR) <= 1e-3 * oR


@pytest.mark.parametrize("shape", [(4, 4), (4, 256), (256, 4), (8, 16), (16, 32), (64, 8), (32, 64), (128, 128)])
def test_lines_full_symbol(M, orc, shape):
    print("lines full symbol", shape, flush=True)
    f, h = TF._state(orc, shape, seed=33 + sum(shape))
    a = 3.0 / 128.0
    h[0] = a
    s = TF._solver(M, shape, tau=(1.0, 1 / 0.8))
    fn, _, R = s.correct(f, h, a)
    s.close()
    ofn, _, oR = orc.full_symbol_iteration(f, h, a, 1.0, 0.8)
    assert np.max(np.abs(fn - ofn)) <= 1e-11 * np.max(np.abs(ofn - f))
    assert abs(R - oR) <= 1e-12 * oR


@pytest.mark.parametrize("shape", [(4, 4), (8, 4), (4, 128), (128, 8), (256, 4), (4, 256)])
def test_lines_walls(M, orc, shape):
    TC.test_wall_corrected_iteration(M, orc, shape, 32.0)
