"""msc_sweep_noalloc behind calls that overlapped in time (on two streams, as
live calls and as replays of captured ones): their own R is undefined, every
serialised call after them forms the right one.  Also calls of two threads in
turn.  Bar: the sums of a context's sweep in another order, 1e-13."""
import threading

import numpy as np
import pytest

from test_gpu_batches import trace
from test_gpu_noalloc_rms import _device, _reference

pytestmark = pytest.mark.gpu

A = 3.0 / 128.0
SHAPES = [(256, 64), (64, 64), (128, 256), (512, 64)]


@pytest.fixture(scope="module")
def M():
    from paper_2609_39474_amd import msc
    msc.lib()
    return msc


def _call(M, shape, d, R, stream):
    M.sweep_noalloc(2, shape, "fp64", d[2].data_ptr(), d[3].data_ptr(), A, d[4].data_ptr(), d[5].data_ptr(),
                    R.data_ptr(), stream)


def _check_serial(M, data, ref, rounds=64):
    import torch

    R = torch.zeros((rounds, len(SHAPES)), dtype=torch.float64, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    for i in range(rounds):
        for k, shape in enumerate(SHAPES):
            _call(M, shape, data[k], R[i, k:], st)
    torch.cuda.synchronize()
    np.testing.assert_allclose(R.cpu().numpy(), np.tile(ref, (rounds, 1)), rtol=1e-13, atol=0)


@pytest.fixture(scope="module")
def sets(M):
    data = [_device(s, "fp64", 60 + i) for i, s in enumerate(SHAPES)]
    ref = np.array([_reference(M, s, "fp64", d[0], d[1], A) for s, d in zip(SHAPES, data)])
    return data, ref


def test_after_overlapping_calls(M, sets):
    import torch

    data, ref = sets
    streams = [torch.cuda.Stream() for _ in SHAPES]
    R = torch.zeros(len(SHAPES), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    for i in range(100):
        for k, shape in enumerate(SHAPES):
            _call(M, shape, data[k], R[k:], streams[k].cuda_stream)
    torch.cuda.synchronize()
    print("overlapping calls: R off by", (R.cpu().numpy() / ref - 1.0).tolist(), flush=True)
    _check_serial(M, data, ref)


def test_after_overlapping_replays(M, sets):
    """A graph of two branches of captured calls, each pair 256 calls apart."""
    import torch

    data, ref = sets
    shape, pairs = (512, 256), 8
    d = [_device(shape, "fp64", 70 + k) for k in range(2)]
    want = np.array([_reference(M, shape, "fp64", x[0], x[1], A) for x in d])
    R = torch.zeros(3, dtype=torch.float64, device="cuda")
    live, branch = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        main = torch.cuda.current_stream()
        branch.wait_stream(main)
        for _ in range(pairs):
            for k, s in enumerate((main, branch)):
                _call(M, shape, d[k], R[k:], s.cuda_stream)
                for _ in range(255):
                    _call(M, SHAPES[0], data[0], R[2:], live.cuda_stream)
        main.wait_stream(branch)
    torch.cuda.synchronize()
    for _ in range(50):
        g.replay()
    torch.cuda.synchronize()
    print("overlapping replays: R off by", (R.cpu().numpy()[:2] / want - 1.0).tolist(), flush=True)
    _check_serial(M, data, ref)


def test_threads_in_turn(M, sets):
    """Two threads on one stream, each call awaited before the other's."""
    import torch

    data, ref = sets
    st = torch.cuda.current_stream().cuda_stream
    lock, bad = threading.Lock(), []

    def work(k):
        R = torch.zeros(1, dtype=torch.float64, device="cuda")
        for _ in range(50):
            with lock:
                _call(M, SHAPES[k], data[k], R, st)
                torch.cuda.synchronize()
                if abs(R.item() - ref[k]) > 1e-13 * ref[k]:
                    bad.append((k, R.item()))

    th = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not bad, bad[:4]


@pytest.mark.parametrize("shape,one", [((4, 4), True), ((128, 16), True), ((256, 64), True), ((256, 256), True),
                                       ((512, 16), False), ((512, 256), False)])
def test_few_blocks_form_the_residual_themselves(M, shape, one):
    import torch

    d = _device(shape, "fp64", 80)
    want = _reference(M, shape, "fp64", d[0], d[1], A)
    R = torch.zeros(1, dtype=torch.float64, device="cuda")
    ev = trace(lambda: _call(M, shape, d, R, torch.cuda.current_stream().cuda_stream))
    n = sum("k_noalloc_rms" in e.name for e in ev)
    print("residual", shape, "launches of its own", n, flush=True)
    assert (n == 0) == one
    np.testing.assert_allclose(R.item(), want, rtol=1e-13, atol=0)
