"""Arrays that a caller names as device memory: torch tensors on the GPU, and host
tensors, which go by copies."""
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


@pytest.mark.parametrize("prec", [W.F64, W.F32_DEV])
@pytest.mark.parametrize("n", [257, 20011])
def test_read_phi_into_tensors_on_the_gpu_and_on_the_host(n, prec):
    import torch

    print("case arrays", n, prec, flush=True)
    x = np.arange(n) * (2 * np.pi / n)
    s = lbm.Solver(W.kdv(0.5, n, 0.1, 1e-4, 2.0, 0.0, prec=prec))
    s.load_phi(torch.tensor(0.4 + 0.3 * np.sin(x), device="cuda"))
    s.advance(5)
    want = s.read_phi()
    for out in (torch.zeros(n, dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.float64),
                torch.zeros(n, dtype=torch.float64, pin_memory=True)):
        s.read_phi(out)
        assert np.array_equal(out.cpu().numpy(), want), out.device
    s.close()
