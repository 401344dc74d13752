"""The read-out at the edges of its workgroups, on an idle stream and behind an
advance that is still running, against the sums of the saved populations."""
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
def test_read_phi_at_workgroup_edges_and_behind_an_advance(prec):
    import torch

    ns = [7, 255, 256, 257, 1024, 1025, 5000]
    print("case readout", prec, flush=True)
    x = [np.arange(n) * (2 * np.pi / n) for n in ns]
    phis = [0.4 + 0.3 * np.sin(v) for v in x]
    b = lbm.Batch([W.kdv(0.5, n, 0.1, 1e-4, 2.0, 0.0, prec=prec) for n in ns])
    b.load_phi(phis)
    # at rest: the sum of the equilibrium populations is phi0 to rounding (five
    # terms below 1 each; FP32 storage holds them to 2^-24 of their size)
    tol = 5 * 2.0 ** (-24 if prec else -52)
    for i, p0 in enumerate(phis):
        got, st = b.read_phi(i)
        assert st == lbm.OK and np.max(np.abs(got - p0)) <= tol, ns[i]
    for steps in (3, 20000):   # ends before, and long after, the read-out is asked for
        b.advance(steps)
        behind = [b.read_phi(i) for i in range(len(ns))]
        torch.cuda.synchronize()
        idle = [b.read_phi(i) for i in range(len(ns))]
        for n, (a, sa), (c, sc) in zip(ns, behind, idle):
            assert sa == sc == lbm.OK and np.array_equal(a, c), (n, steps)
    b.close()


@pytest.mark.parametrize("n", [64, 257, 3000])
def test_noalloc_refuses_a_non_finite_state_and_leaves_phi(n):
    import torch

    print("case noalloc refusal", n, flush=True)
    p = W.kdv(0.5, n, 0.1, 1e-4, 2.0, 0.0)
    phi0 = torch.full((n,), 0.25, dtype=torch.float64, device="cuda")
    phi0[n - 1] = float("inf")
    out = torch.full_like(phi0, 7.0)
    with pytest.raises(lbm.LBMError) as e:
        lbm.advance_noalloc(p, phi0, 5, out)
    assert e.value.status == lbm.INVALID_ARG
    assert bool((out == 7.0).all())
