"""A step's first sweep taking the decision on the step before it (2D, rows of
at least 64 sites, several steps in one call) against calls of one step each,
whose decisions are launches of their own: the same populations and counts bit
for bit, the residuals to the order of their sum (1e-14).

Cases: rows of 64, 128 and 256 sites; every storage; trials from one to three
states; no corrector; counts that fall, rise and stay from step to step
(decisions that come early, go on, or end where predicted); a scheduled replay
with single sweeps; a step that fails in the middle of a call.
"""
import numpy as np
import pytest

from paper_2609_39474_amd import workloads as W

pytestmark = pytest.mark.gpu

NU = 1.0 / 6.0


@pytest.fixture(scope="module")
def M():
    from paper_2609_39474_amd import msc
    msc.lib()
    return msc


def _solver(M, shape, **kw):
    N = min(shape)
    p0, u0 = W.random_field_2d(N, 0.05 * NU * 16 / N, seed=8, jmax=4)
    reps = tuple(n // N for n in shape)
    p = M.make_params(2, shape[0], **kw)
    p.n[0], p.n[1] = shape
    return M.Solver(p, np.tile(p0, reps), np.tile(u0, (1,) + reps))


def _run(M, shape, cuts, sched=None, **kw):
    s = _solver(M, shape, **kw)
    if sched:
        s.set_schedule(sched)
    stats = []
    for c in cuts:
        rc, st = s.bdf2_step(c)
        assert rc == 0
        stats += st
    out = s.get_state()[0], s.moments(), stats
    s.close()
    return out


@pytest.mark.parametrize("shape,kw,sched", [
    ((16, 64), dict(dt=24.0, eps=1e-9), None),
    ((64, 64), dict(dt=64.0, eps=1e-7, storage="fp32", extrap_states=2), None),
    ((128, 128), dict(dt=256.0, eps=1e-8, extrap_states=2), None),
    ((32, 256), dict(dt=16.0, eps=1e-6, storage="fp16dev", extrap_states=1), None),
    ((256, 256), dict(dt=64.0, eps=1e-6, storage="fp32"), None),
    ((64, 128), dict(dt=4.0, eps=1e-9, corrector="picard"), None),
    ((512, 64), dict(dt=24.0, eps=1e-9, tau_plus=0.8, extrap_states=2), None),
    ((64, 64), dict(dt=24.0, eps=1e-9), [4, 1, 1, 2, 3, 1, 5, 2, 1, 1, 3, 2] * 2),
])
def test_merged_decisions(M, shape, kw, sched):
    n = 24
    a = _run(M, shape, [n], sched, **kw)
    b = _run(M, shape, [1] * n, sched, **kw)
    ka, kb = [x["iters"] for x in a[2]], [x["iters"] for x in b[2]]
    print("merged decisions", shape, kw, "K", ka, flush=True)
    assert ka == kb
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])
    for x, y in zip(a[2], b[2]):
        assert x["q"] == y["q"] and x["converged"] == y["converged"]
        assert abs(x["R_final"] - y["R_final"]) <= 1e-14 * y["R_final"]
        assert abs(x["R_first"] - y["R_first"]) <= 1e-14 * y["R_first"]


def test_failing_step_in_a_call(M):
    """K_max below what the second BDF order needs: both forms stop at the
    same step with the same statistics, and the state is the last accepted."""
    shape, out = (64, 64), []
    ref = _run(M, shape, [12], dt=64.0, eps=1e-9)
    K = [x["iters"] for x in ref[2]]
    print("counts", K, flush=True)
    kmax = max(K) - 1
    for cuts in ([12], [1] * 12):
        s = _solver(M, shape, dt=64.0, eps=1e-9, k_max=kmax)
        done, rc = [], 0
        for c in cuts:
            rc, st = s.bdf2_step(c, raise_on_fail=False)
            done += [x["iters"] for x in st if x["converged"]]
            if rc != 0:
                break
        assert rc == 5
        out.append((done, s.get_state()[0]))
        s.close()
    assert out[0][0] == out[1][0]
    assert out[0][0] == K[:K.index(max(K))]
    np.testing.assert_array_equal(out[0][1][:9 * 64 * 64], out[1][1][:9 * 64 * 64])
