"""A recording march whose allocator runs out: the context stands at the last
accepted step with the records up to it, a call that goes on later continues
both, and where only small pieces are to be had the records lie in those.

Bar: bit for bit the march and the adjoint of a context that was not disturbed
(cut into calls of one step, so that every m^n is formed by its own step)."""
import numpy as np
import pytest

from paper_2609_39474_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    from paper_2609_39474_amd import msc
    msc.lib()
    return msc


class Alloc:
    """alloc_fn / free_fn over torch's caching allocator: refuses requests above
    `largest` bytes, and after `left` more requests any."""

    def __init__(self, M):
        import torch

        self.largest = self.left = None
        self.live = 0
        self.torch = torch
        self.alloc = M.ALLOC_FN(self._a)
        self.free = M.FREE_FN(self._f)

    def _a(self, nbytes, user):
        if self.largest is not None and nbytes > self.largest:
            return None
        if self.left is not None:
            if self.left == 0:
                return None
            self.left -= 1
        self.live += 1
        return int(self.torch.cuda.caching_allocator_alloc(int(nbytes)))

    def _f(self, ptr, user):
        if ptr:
            self.live -= 1
            self.torch.cuda.caching_allocator_delete(int(ptr))


def _solver(M, shape, alloc=None, **kw):
    d, n = len(shape), min(shape)
    if d == 2:
        p0, u0 = W.random_field_2d(n, 0.05 / 6.0 * 16 / n, seed=9, jmax=4)
    else:
        p0, u0 = np.zeros((n,) * 3), W.random_perturbation_3d(n, 0.05 / 6.0 * 16 / n, seed=9, jmax=3)
    reps = tuple(k // n for k in shape)
    p = M.make_params(d, shape[0], **kw)
    for i, k in enumerate(shape):
        p.n[i] = k
    if alloc is not None:
        p.alloc_fn, p.free_fn = alloc.alloc, alloc.free
    return M.Solver(p, np.tile(p0, reps), np.tile(u0, (1,) + reps))


def _reference(M, shape, n, kw):
    s = _solver(M, shape, **kw)
    s.set_recording(True)
    states, K = [s.get_state()], []
    for _ in range(n):
        K += [x["iters"] for x in s.bdf2_step(1)[1]]
        states.append(s.get_state())
    lam = np.random.default_rng(6).normal(size=s.state_size())
    adj = s.bdf2_adjoint(n, lam)
    s.close()
    return states, K, lam, adj


CASES = [((64, 64), dict(dt=24.0, eps=1e-9)), ((32, 32), dict(dt=24.0, eps=1e-9, extrap_states=1)),
         ((64, 64), dict(dt=24.0, eps=1e-6, storage="fp32")), ((32, 512), dict(dt=16.0, eps=1e-5, storage="fp16dev")),
         ((16, 16, 16), dict(dt=8.0, eps=1e-8))]


@pytest.mark.parametrize("shape,kw", CASES)
@pytest.mark.parametrize("left", [0, 1, 3, 5])
def test_memory_ends_in_a_call(M, shape, kw, left):
    n = 8
    states, K, lam, adj = _reference(M, shape, n, kw)
    a = Alloc(M)
    s = _solver(M, shape, a, **kw)
    s.get_state()  # (its staging buffer is there)
    s.set_recording(True)
    NS = int(np.prod(shape))
    # one record to a piece at most times, two where the first keeps more
    a.largest, a.left = 3 * (19 if len(shape) == 3 else 9) * NS * 8, left
    rc, st = s.bdf2_step(n, raise_on_fail=False)
    done = s.recorded_steps()
    print("memory ends", shape, kw, "pieces", left, "steps", done, flush=True)
    assert rc == (M.MSC_ERR_OUT_OF_MEMORY if done < n else 0) and done >= left
    assert (done == 0) == (left == 0)
    assert [x["iters"] for x in st[:done]] == K[:done]
    got, want = s.get_state(), states[done]
    np.testing.assert_array_equal(got[0], want[0])
    assert got[1] == want[1]
    # the march and its records go on
    a.largest = a.left = None
    rc, st = s.bdf2_step(n - done)
    assert rc == 0 and [x["iters"] for x in st[:n - done]] == K[done:]
    assert s.recorded_steps() == n
    np.testing.assert_array_equal(s.get_state()[0], states[n][0])
    np.testing.assert_array_equal(s.bdf2_adjoint(n, lam), adj)
    s.close()
    assert a.live == 0


@pytest.mark.parametrize("shape,kw", CASES)
def test_records_in_small_pieces(M, shape, kw):
    n = 8
    states, K, lam, adj = _reference(M, shape, n, kw)
    a = Alloc(M)
    s = _solver(M, shape, a, **kw)
    s.get_state()
    s.set_recording(True)
    a.largest = 3 * (19 if len(shape) == 3 else 9) * int(np.prod(shape)) * 8
    rc, st = s.bdf2_step(n)
    assert rc == 0 and [x["iters"] for x in st] == K and s.recorded_steps() == n
    a.largest = None
    np.testing.assert_array_equal(s.get_state()[0], states[n][0])
    np.testing.assert_array_equal(s.bdf2_adjoint(n, lam), adj)
    s.close()
    assert a.live == 0


def test_memory_ends_in_a_replay(M):
    """The replayed schedule goes on behind the accepted steps."""
    n, shape, kw = 8, (64, 64), dict(dt=24.0, eps=1e-9)
    K = [5, 4, 3, 4, 3, 5, 4, 3]
    r = _solver(M, shape, **kw)
    r.set_schedule(K)
    r.bdf2_step(n)
    a = Alloc(M)
    s = _solver(M, shape, a, **kw)
    s.set_recording(True)
    s.set_schedule(K)
    s.bdf2_step(1)  # (the schedule's device array)
    a.largest, a.left = 3 * 9 * 64 * 64 * 8, 4
    rc, _ = s.bdf2_step(n - 1, raise_on_fail=False)
    done = s.recorded_steps()
    print("replay: steps", done, flush=True)
    a.largest = a.left = None
    if rc != 0:
        assert rc == M.MSC_ERR_OUT_OF_MEMORY and done < n
        rc, st = s.bdf2_step(n - done)
        assert rc == 0 and [x["iters"] for x in st[:n - done]] == K[done:]
    np.testing.assert_array_equal(s.get_state()[0], r.get_state()[0])
    s.close()
    r.close()
