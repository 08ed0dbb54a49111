"""msc_sweep_noalloc's residual formed in the sweep's own launch (2D, one row
per block): the smallest and largest rows and row counts, blocks of less than a
wavefront, more calls than arrival counters, calls of both forms in turn and a
captured graph.  Bar: the sums of a context's sweep in another order, 1e-13."""
import numpy as np
import pytest

from test_zz_no_alloc import _state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    from paper_2609_39474_amd import msc
    msc.lib()
    return msc


def _device(shape, storage, seed):
    import torch

    tdt = torch.float64 if storage == "fp64" else torch.float32
    f, h = _state(2, shape, seed)
    fd = torch.tensor(f, dtype=tdt, device="cuda").contiguous()
    hd = torch.tensor(h, dtype=torch.float64, device="cuda").contiguous()
    return f, h, fd, hd, torch.empty_like(fd), torch.empty((3,) + shape, dtype=tdt, device="cuda")


def _reference(M, shape, storage, f, h, a):
    p = M.make_params(2, shape[0], dt=64.0, eps=1e-10, storage=storage, corrector="picard")
    p.n[0], p.n[1] = shape
    s = M.Solver(p, np.zeros(shape), np.zeros((2,) + shape))
    R = s.sweep(f, h, a)[2]
    s.close()
    return R


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(4, 4), (512, 4), (8, 8), (64, 16), (4, 32), (512, 32), (4, 64), (64, 64),
                                   (256, 128), (512, 256), (1024, 64), (64, 512)])
def test_residual_of_one_launch(M, shape, storage):
    import torch

    a = 3.0 / 128.0
    f, h, fd, hd, fT, Pr = _device(shape, storage, 5 + sum(shape))
    ref = _reference(M, shape, storage, f, h, a)
    R = torch.zeros(300, dtype=torch.float64, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    for i in range(300):
        M.sweep_noalloc(2, shape, storage, fd.data_ptr(), hd.data_ptr(), a, fT.data_ptr(), Pr.data_ptr(),
                        R[i:].data_ptr(), st)
    torch.cuda.synchronize()
    r = R.cpu().numpy()
    print("rms in one launch", shape, storage, r[0], ref, flush=True)
    assert np.all(r == r[0])
    assert abs(r[0] - ref) <= 1e-13 * ref


def test_residual_under_capture(M):
    import torch

    a, shapes = 1.0 / 40.0, [(64, 64), (1024, 64), (16, 8)]
    data = [_device(s, "fp64", 40 + i) for i, s in enumerate(shapes)]
    ref = [_reference(M, s, "fp64", d[0], d[1], a) for s, d in zip(shapes, data)]
    R = torch.zeros(3, dtype=torch.float64, device="cuda")

    def calls():
        st = torch.cuda.current_stream().cuda_stream
        for i, (s, d) in enumerate(zip(shapes, data)):
            M.sweep_noalloc(2, s, "fp64", d[2].data_ptr(), d[3].data_ptr(), a, d[4].data_ptr(), d[5].data_ptr(),
                            R[i:].data_ptr(), st)

    calls()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        calls()
    for _ in range(4):
        R.zero_()
        g.replay()
        torch.cuda.synchronize()
        np.testing.assert_allclose(R.cpu().numpy(), ref, rtol=1e-13, atol=0)
        R.zero_()
        calls()
        torch.cuda.synchronize()
        np.testing.assert_allclose(R.cpu().numpy(), ref, rtol=1e-13, atol=0)
