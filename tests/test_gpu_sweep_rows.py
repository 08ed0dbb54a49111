"""The 2D sweep with its three source rows in parallel (one-plane strips of
tiles that span whole rows) against the plane-by-plane sweep (two-plane
strips, msc_set_tuning key 1) on the same inputs: same inner counts replayed,
populations bit-exact (the arithmetic is the same code).

Shapes: rows below a wavefront, of one wavefront, and of the widest tile, the
fewest rows.  Corrected marches (first and lift sweeps, paper and linear trial),
Picard (the plain dual-time sweep), the cavity's wall rows and the tiled
explicit sweep.
"""
import numpy as np
import pytest

from test_gpu_aa import _rand_f, say

pytestmark = pytest.mark.gpu
KEY_STRIP, KEY_EXPLICIT_AA = 1, 10


@pytest.fixture(scope="module")
def M():
    from paper_2609_39474_amd import msc
    msc.lib()
    return msc


def _run(M, shape, storage, f0, strip, corrector, extrap, boundary, explicit):
    p = M.make_params(2, shape[0], dt=4.0, eps=1e-10, storage=storage, corrector=corrector, tau_plus=0.9,
                      tau_minus=1.2, extrap_states=extrap, boundary=boundary, u_lid=0.01)
    p.n[0], p.n[1] = shape
    s = M.Solver(p, np.zeros(shape), np.zeros((2,) + shape))
    s.set_tuning(KEY_STRIP, strip)
    s.set_tuning(KEY_EXPLICIT_AA, 0)
    s.set_populations(f0)
    if explicit:
        s.explicit_step(5)
        out = s.populations()
    else:
        s.set_schedule([3, 2, 1, 3, 2])
        s.bdf2_step(5)
        out = s.get_state()[0]
    s.close()
    return out


@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16dev"])
@pytest.mark.parametrize("shape", [(4, 4), (16, 8), (8, 32), (4, 64), (64, 128), (32, 256)])
def test_rows_in_parallel_bit_exact(M, orc, shape, storage):
    f0 = _rand_f(orc, shape, 31)
    for case in (("shadow", 2, "periodic", False), ("shadow", 0, "periodic", False),
                 ("picard", 0, "periodic", False), ("picard", 2, "cavity", False), ("picard", 2, "cavity", True),
                 ("picard", 2, "periodic", True)):
        say("rows in parallel", shape, storage, *case)
        a = _run(M, shape, storage, f0, 1, *case)
        b = _run(M, shape, storage, f0, 2, *case)
        assert np.isfinite(a).all()
        np.testing.assert_array_equal(a, b)
