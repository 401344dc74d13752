"""Slab launches of several batches, each on its own thread and stream and each
with more workgroups than half the GPU holds: all of them must end, with the
results of the same batch alone."""
import threading

import numpy as np
import pytest

from paper_0907_1720_amd import lbm
from paper_0907_1720_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    lbm.library()
    yield


@pytest.mark.parametrize("kind,n,count", [("kdv", 9001, 90), ("kdv", 200003, 1), ("kdv", 5000, 1), ("power", 9001, 60)])
def test_concurrent_slab_batches_end(kind, n, count):
    import torch

    print("case slab threads", kind, n, count, flush=True)
    if kind == "kdv":
        probs = [W.kdv(0.5 + 0.001 * i, n, 0.1, 1e-4, 2.0, 0.0) for i in range(count)]
    else:
        probs = [W.power_kdv(0.5, 0.01, n, 0.1, 1e-3, 2.0, 0.0) for i in range(count)]
    phis = [0.6 + 0.3 * np.sin(2 * np.pi * np.arange(n) / n + i) for i in range(count)]
    streams = [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()

    def run(stream):
        b = lbm.Batch(probs, stream=stream.cuda_stream)
        b.load_phi(phis)
        for _ in range(6):
            b.advance(150)
        out = [b.read_phi(i) for i in range(0, count, 16)]
        b.close()
        return out

    want = run(streams[0])
    got = [None] * len(streams)

    def work(k):
        got[k] = run(streams[k])

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(streams))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for out in got:
        assert out is not None
        for (a, sa), (c, sc) in zip(out, want):
            assert sa == sc == lbm.OK and np.array_equal(a, c)
