"""How many steps a call of the march enqueues before it first waits, seen in
the trace of its launches: one step where what the context has learnt about its
steps does not hold."""
import numpy as np
import pytest

from paper_2609_39474_amd import workloads as W

pytestmark = pytest.mark.gpu

N = 32


@pytest.fixture(scope="module")
def M():
    from paper_2609_39474_amd import msc
    msc.lib()
    return msc


def trace(fn):
    """The runtime calls and kernels of fn(), in order of their start."""
    import torch
    from torch.profiler import ProfilerActivity, profile

    torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as p:
        fn()
        torch.cuda.synchronize()
    ev = sorted(p.events(), key=lambda e: e.time_range.start)
    if not any("Launch" in e.name for e in ev):
        pytest.skip("torch's profiler records no launches here (another tracer at work)")
    return ev


def _launches(fn):
    """Kernel launches before each wait of the host in fn()."""
    out, n = [], 0
    for e in trace(fn):
        if "LaunchKernel" in e.name:
            n += 1
        elif e.name == "hipStreamSynchronize":
            out.append(n)
            n = 0
    assert out, "no calls traced"
    return out


def _marched(M, schedule):
    """A context that has marched 63 steps by a schedule (batches of up to 32)."""
    p0, u0 = W.random_field_2d(N, 0.1 / 6.0 / N, seed=8)
    s = M.Solver(M.make_params(2, N, dt=4.0, eps=1e-8, extrap_states=1), p0, u0)
    s.set_schedule(schedule)
    s.bdf2_step(63)
    return s


@pytest.mark.parametrize("what", ["nothing", "set_populations", "set_state", "explicit_step", "schedule ends"])
def test_first_batch(M, what):
    s = _marched(M, [3] * (63 if what == "schedule ends" else 70))
    if what == "set_populations":
        s.set_populations(s.populations())
    elif what == "set_state":
        s.set_state(*s.get_state())
    elif what == "explicit_step":
        s.explicit_step(2)
    waits = _launches(lambda: s.bdf2_step(7))
    s.close()
    print("launches before each wait:", what, waits, flush=True)
    # a step of three sweeps: the sweeps, two corrections, the decision
    if what == "nothing":
        assert waits[0] >= 7 * 5 and len(waits) == 1
    else:
        assert waits[0] <= 8


@pytest.mark.parametrize("steps,want", [(1, 7), (3, 3), (64, 1)])
def test_steps_per_wait_from_the_next_call(M, steps, want):
    """Tuning key 2 holds from the next call, also below what was reached."""
    s = _marched(M, [3] * 70)
    s.set_tuning(2, steps)
    waits = _launches(lambda: s.bdf2_step(7))
    s.close()
    print("launches before each wait: key 2 =", steps, waits, flush=True)
    assert len(waits) == want


@pytest.mark.parametrize("shape,steps,storage,aa", [((128, 128), 72, "fp64", 1), ((512, 512), 100, "fp32", 1),
                                                    ((16, 16), 65, "fp64", 1), ((16, 16, 16), 65, "fp32", 1),
                                                    ((64, 64), 65, "fp64", 0), ((64, 64), 65, "fp16dev", 1)])
def test_explicit_chunks_captured_once(M, shape, steps, storage, aa):
    """Calls of one length whose launches behind the graph's chunks exchange the
    two buffers: after two calls no chunk is captured again, and the state is
    that of one call without graphs."""
    d, n = len(shape), min(shape)
    p0, u0 = (W.random_field_2d(n, 0.1 / 6.0 / n, seed=8) if d == 2 else
              (np.zeros(shape), W.random_perturbation_3d(n, 0.1 / 6.0 / n, seed=8, jmax=3)))
    s, r = [M.Solver(M.make_params(d, n, dt=4.0, eps=1e-8, storage=storage), p0, u0) for _ in range(2)]
    s.set_tuning(10, aa)
    s.explicit_step(steps)
    s.explicit_step(steps)
    names = [e.name for e in trace(lambda: [s.explicit_step(steps) for _ in range(4)])]
    print("explicit", shape, steps, storage, "graph launches", names.count("hipGraphLaunch"), "captures",
          names.count("hipGraphInstantiate"), flush=True)
    assert names.count("hipGraphLaunch") >= 4 and names.count("hipGraphInstantiate") == 0
    r.set_tuning(10, aa)
    r.set_tuning(4, 0)
    r.explicit_step(6 * steps)
    np.testing.assert_array_equal(s.populations(), r.populations())
    # marches between explicit calls, in other buffers
    for x in (s, r):
        x.bdf2_step(1)
        x.explicit_step(steps)
    np.testing.assert_array_equal(s.populations(), r.populations())
    s.close()
    r.close()


@pytest.mark.parametrize("rows,folded", [(4096, False), (8192, True)])
def test_many_partials_are_folded_first(M, rows, folded):
    """One-row blocks on more than 4096 rows (tuning key 1): one launch folds the
    partials of each sweep, not every block of the next step's first sweep."""
    shape = (rows, 64)
    p0, u0 = W.random_field_2d(64, 1.0 / 6.0 / 64, seed=8)
    p = M.make_params(2, 64, dt=2.0, eps=1e-3, corrector="picard")
    p.n[0] = rows
    s = M.Solver(p, np.tile(p0, (rows // 64, 1)), np.tile(u0, (1, rows // 64, 1)))
    s.set_tuning(1, 1)
    s.bdf2_step(31)
    st = []
    ev = trace(lambda: st.extend(s.bdf2_step(8)[1]))
    s.close()
    n = sum("k_presum" in e.name for e in ev)
    print("many partials", shape, "counts", [x["iters"] for x in st], "folds", n, flush=True)
    assert n >= sum(x["iters"] for x in st) if folded else n == 0
