"""A batch of power sums whose largest grid takes far more than an even share of
the CUs goes in slabs, except its smallest grids; every result must equal the
streaming kernel's bit for bit (the same arithmetic in the same order)."""
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


@pytest.mark.parametrize("prec,hi", [(W.F64, 4000), (W.F32_DEV, 8000)])
def test_uneven_power_batch_equals_stream(prec, hi):
    count = 260
    print("case uneven", prec, flush=True)
    ns = [int(round(200 * (hi / 200) ** ((0.5 + 0.6180339887498949 * i) % 1.0))) for i in range(count)]
    ps = [W.power_kdv(0.5 if i % 2 else 1.5, 0.01, n, 0.1, 1e-3, 2.0, 0.0, prec=prec) for i, n in enumerate(ns)]
    phis = [0.6 + 0.2 * np.sin(2 * np.pi * np.arange(n) / n + i) for i, n in enumerate(ns)]
    b = lbm.Batch(ps)
    b.load_phi(phis)
    b.advance(41)
    b.advance([20 + i % 3 for i in range(count)])
    for i in sorted({int(np.argmax(ns)), int(np.argmin(ns))} | set(range(0, count, 13))):
        got, st = b.read_phi(i)
        assert st == lbm.OK, i
        s = lbm.Solver(ps[i])
        s.set_path(lbm.PATH_STREAM)
        s.load_phi(phis[i])
        s.advance(41)
        s.advance(20 + i % 3)
        want = s.read_phi()
        s.close()
        assert np.array_equal(got, want), (i, ns[i])
    b.close()
