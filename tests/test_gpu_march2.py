"""Several explicit steps per launch (2D): against the library's two-buffer
sweep on the same state, bit-exact (the collision is the same code; only the
number of steps between loads and stores differs).

Shapes: the smallest grids of each tile (a tile's halo then wraps around the
domain more than once), grids on both sides of the site counts where the tile
changes, elongated ones, and extents below a tile (the single-step kernels).
Step counts: one launch, a launch and what is left of the count (pairs, an odd
step), graph-captured chunks with both.
"""
import numpy as np
import pytest

from test_gpu_aa import _march, _rand_f, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    from paper_2609_39474_amd import msc
    msc.lib()
    return msc


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(8, 16), (4, 16), (8, 8), (16, 64), (256, 16), (128, 256), (256, 256), (16, 4096),
                                   (256, 512), (512, 512), (32, 8192), (8192, 32), (16, 16384)])
def test_steps_per_launch_bit_exact(M, orc, shape, storage):
    f0 = _rand_f(orc, shape, 21)
    for steps, graph in ((8, False), (15, False), (75, True), (134, True)):
        say("steps per launch", shape, storage, "steps", steps, "graph", graph)
        fa = _march(M, shape, storage, f0, steps, True, graph)
        fb = _march(M, shape, storage, f0, steps, False, graph)
        np.testing.assert_array_equal(fa, fb)


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("taus", [(1.0, 1.0), (1.0, 0.8), (0.7, 1.0)])
@pytest.mark.parametrize("shape", [(16, 16), (256, 256), (512, 512)])
def test_operating_point_update_bit_exact(M, orc, shape, taus, storage):
    """The update without populations (both rates 1) and the general one, per
    tile, against the single-step kernels."""
    from test_gpu_aa import KEY_EXPLICIT_AA

    f0 = _rand_f(orc, shape, 22)
    out = []
    for aa in (1, 0):
        p = M.make_params(2, shape[0], dt=64.0, eps=1e-6, storage=storage, tau_plus=taus[0], tau_minus=taus[1])
        p.n[0], p.n[1] = shape
        s = M.Solver(p, np.zeros(shape), np.zeros((2,) + shape))
        s.set_tuning(KEY_EXPLICIT_AA, aa)
        s.set_populations(f0)
        s.explicit_step(18)
        out.append(s.populations())
        s.close()
    np.testing.assert_array_equal(out[0], out[1])
