"""The fused transposed sweeps of the adjoint (per site, and per row with the
row transforms inside) at the edges of their range, and records made over one
or several calls.

Bars: against the FP64 oracle per part of the state, ten times the oracle's own
response to a one-ulp change of the output adjoint, at least 1e-10 (the sums of
a sweep and of a transform of length <= 1024 round in another order there);
records of one batched call against records of single-step calls 1e-13 (the
same populations and history terms reversed by the same launches).
"""
import numpy as np
import pytest

from paper_2609_39474_amd import workloads as W

import parity_bars as PB

pytestmark = pytest.mark.gpu

NU = 1.0 / 6.0
KEY_FUSE_ROWS = 6


def rel(a, b):
    den = np.max(np.abs(b))
    return float(np.max(np.abs(a - b)) / (den if den > 0 else 1.0))


@pytest.fixture(scope="module")
def M():
    from paper_2609_39474_amd import msc
    msc.lib()
    return msc


def _solver(M, shape, *, dt=24.0, storage="fp64", corrector="shadow", extrap=0, eps=1e-10):
    d, N = len(shape), min(shape)
    U = 0.05 * NU * 16 / N
    if N < 8:
        rng = np.random.default_rng(21)
        p0, u0 = np.zeros(shape), U * rng.normal(size=(d,) + shape)
    else:
        if d == 2:
            p0, u0 = W.random_field_2d(N, U, seed=5, jmax=min(4, N // 4))
        else:
            p0, u0 = np.zeros((N,) * 3), W.random_perturbation_3d(N, U, seed=5, jmax=min(3, N // 4))
        reps = tuple(n // N for n in shape)
        p0, u0 = np.tile(p0, reps), np.tile(u0, (1,) + reps)
    p = M.make_params(d, shape[0], dt=dt, eps=eps, storage=storage, corrector=corrector, extrap_states=extrap)
    for a in range(d):
        p.n[a] = shape[a]
    return M.Solver(p, p0, u0)


@pytest.mark.parametrize("shape,fuse,corr,nsteps", [
    ((4, 4), 2, "shadow", 3), ((64, 4), 2, "shadow", 3), ((8, 8), 2, "shadow", 3), ((4, 16), 2, "shadow", 2),
    ((16, 32), 2, "shadow", 3), ((32, 64), 2, "shadow", 3), ((8, 128), 2, "shadow", 2),
    ((128, 256), 2, "shadow", 2), ((16, 256), 2, "picard", 2), ((32, 64), 1, "shadow", 3),
    ((32, 64), 0, "shadow", 3), ((4, 512), 2, "shadow", 2), ((1024, 8), 2, "shadow", 2), ((4, 8, 16), 2, "shadow", 2),
])
def test_adjoint_edges_vs_oracle(M, orc, shape, fuse, corr, nsteps):
    print("adjoint edges", shape, fuse, corr, flush=True)
    d = len(shape)
    Q, NS = (9 if d == 2 else 19), int(np.prod(shape))
    s = _solver(M, shape, corrector=corr)
    s.set_tuning(KEY_FUSE_ROWS, fuse)
    st0, bc0 = s.get_state()
    s.set_recording(True)
    if min(shape) < 8:  # too few modes for the march to converge: fixed counts
        s.set_schedule([3] * nsteps)
    rc, stats = s.bdf2_step(nsteps)
    assert rc == 0 and s.recorded_steps() == nsteps
    lam = np.random.default_rng(3).normal(size=s.state_size())
    g = s.bdf2_adjoint(nsteps, lam)
    s.close()
    kw = dict(dt=24.0, eps=1e-10, corrector=1 if corr == "shadow" else 0, extrap_states=0,
              nmin=2 if d == 2 else 1, kmax=300, schedule=[x["iters"] for x in stats])
    ref = orc.march_adjoint(st0, bc0, shape, lam, **kw)
    alt = orc.march_adjoint(st0, bc0, shape, PB.ulp_perturbed(lam, 1), **kw)
    FQ = Q * NS

    def parts(x):
        return [x[i * FQ:(i + 1) * FQ] for i in range(3)] + [x[3 * FQ + i * NS:3 * FQ + (i + 1) * NS]
                                                             for i in range(2 * (d + 1))]

    keep = [i for i, b in enumerate(parts(ref)) if np.max(np.abs(b)) > 0]
    errs = [rel(parts(g)[i], parts(ref)[i]) for i in keep]
    sens = [rel(parts(alt)[i], parts(ref)[i]) for i in keep]
    PB.check_fields(errs, PB.sensitivity_bars(sens, floor=1e-10), f"adjoint {shape}")
    assert np.array_equal(np.flatnonzero([np.max(np.abs(b)) > 0 for b in parts(g)]), keep)


@pytest.mark.parametrize("shape,storage,extrap,calls", [
    ((16, 16), "fp64", 0, [37]), ((32, 16), "fp32", 2, [1, 2, 40]), ((16, 32), "fp16dev", 0, [3, 1, 5]),
    ((8, 8, 8), "fp32", 0, [4, 3]), ((16, 16), "fp64", 1, [6]),
])
def test_records_of_batched_calls(M, shape, storage, extrap, calls):
    """Records share populations within a call; the reversed march is the same
    however it was cut into calls."""
    print("records", shape, storage, extrap, calls, flush=True)
    n = sum(calls)
    kw = dict(dt=16.0, storage=storage, extrap=extrap, eps=1e-6)
    a, b = _solver(M, shape, **kw), _solver(M, shape, **kw)
    lam = np.random.default_rng(4).normal(size=a.state_size())
    out = []
    for s, cut in ((a, calls), (b, [1] * n)):
        s.set_recording(True)
        K = []
        for c in cut:
            rc, stats = s.bdf2_step(c)
            assert rc == 0
            K += [x["iters"] for x in stats]
        assert s.recorded_steps() == n
        first = s.bdf2_adjoint(n - n // 3, lam)
        assert s.recorded_steps() == n // 3
        out.append((K, first, s.bdf2_adjoint(n // 3, first)))
        # recording goes on from where the march is
        s.bdf2_step(2)
        assert s.recorded_steps() == 2
        s.close()
    assert out[0][0] == out[1][0]
    assert rel(out[0][1], out[1][1]) <= 1e-13 and rel(out[0][2], out[1][2]) <= 1e-13


def test_failed_call_keeps_accepted_records(M):
    s = _solver(M, (16, 16), dt=24.0)
    ok = s.get_state()
    s.set_recording(True)
    s.set_schedule([3, 3, 3])
    rc, _ = s.bdf2_step(3)
    assert rc == 0 and s.recorded_steps() == 3
    bad = ok[0].copy()
    bad[5] = np.nan
    s.set_state(bad, ok[1])
    try:
        rc, _ = s.bdf2_step(4)
    except M.MscError:
        rc = -1
    assert rc != 0 and s.recorded_steps() == 3
    s.close()
