"""Device tensors that are still being filled when they are passed: a context
without a caller's stream works on a stream of its own and has to wait for the
default stream, where torch fills them (inputs, adjoints) and where memory
that torch's allocator hands out again may still be in use.

The default stream is kept busy by a chain of large products for some
milliseconds; the fields are written behind it.
"""
import numpy as np
import pytest

from test_gpu_aa import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    from paper_2609_39474_amd import msc
    msc.lib()
    return msc


def _busy(torch, a):
    for _ in range(20):
        a = a @ a
    return a


@pytest.mark.parametrize("torch_alloc", [False, True])
def test_inputs_still_being_filled(M, torch_alloc):
    import torch
    from paper_2609_39474_amd import workloads as W

    torch.cuda.set_device(0)
    N = 64
    p0, u0 = W.tgv2d(N, 1.0 / 6.0 / N)
    hp, hu = torch.from_numpy(p0), torch.from_numpy(u0)
    a = torch.eye(4096, device="cuda")

    def run(busy):
        tmp = torch.full((1 << 22,), float("nan"), device="cuda", dtype=torch.float64)
        torch.cuda.synchronize()
        p = torch.full(p0.shape, float("nan"), device="cuda", dtype=torch.float64)
        u = torch.full(u0.shape, float("nan"), device="cuda", dtype=torch.float64)
        dp, du = hp.cuda(), hu.cuda()
        torch.cuda.synchronize()
        if busy:
            _busy(torch, a)
            tmp.fill_(float("nan"))
            del tmp  # its memory may be handed to the context while the fill is pending
        p.copy_(dp)
        u.copy_(du)
        q = M.make_params(2, N, dt=16.0, eps=1e-8)
        s = M.Solver(q, p, u, torch_alloc=torch_alloc)
        s.bdf2_step(3)
        m = torch.empty((3, N, N), device="cuda", dtype=torch.float64)
        s.moments_device(m.data_ptr(), m[1:].data_ptr())
        out = m.cpu().numpy()
        s.close()
        return out

    want, got = run(False), run(True)
    say("inputs behind a busy default stream: max diff", float(np.max(np.abs(want - got))))
    assert np.isfinite(got).all()
    np.testing.assert_array_equal(got, want)
