"""Slab groups whose steps go in chunks, one launch after another: every result
must equal the streaming kernel's bit for bit (the same arithmetic in the same
order, so there is no tolerance)."""
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


def _problem(kind, n, prec):
    if kind == "power":
        return W.power_kdv(0.5, 0.01, n, 0.1, 1e-3, 2.0, 0.0, prec=prec)
    return (W.kdv if kind == "kdv" else W.mkdv)(0.5, n, 0.1, 1e-4, 2.0, 0.0, prec=prec)


def _check(name, problems, steps, sample):
    """The batch against the streaming path; of equal problems with equal steps, one."""
    print("case chunks", name, flush=True)
    phis = {p.n: 0.6 + 0.2 * np.sin(2 * np.pi * np.arange(p.n) / p.n) for p in problems}
    b = lbm.Batch(problems)
    b.load_phi([phis[p.n] for p in problems])
    b.advance(steps)
    want = {}
    for i in sample:
        p, key = problems[i], (problems[i].name, problems[i].n, steps[i])
        if key not in want:
            s = lbm.Solver(p)
            s.set_path(lbm.PATH_STREAM)
            s.load_phi(phis[p.n])
            s.advance(steps[i])
            want[key] = s.read_phi()
            s.close()
        got, st = b.read_phi(i)
        assert st == lbm.OK, i
        assert np.array_equal(got, want[key]), (i, p.n, steps[i])
    b.close()


def test_groups_on_their_shares_of_the_gpu_equal_stream():
    ps = [_problem("kdv", 4324, W.F32_DEV)] * 3 + [_problem("mkdv", 41530, W.F32_DEV)] * 20
    _check("shares", ps, [4000, 600, 600] + [1000] * 20, range(23))


@pytest.mark.parametrize("kind,n,few,many,steps", [("power", 4096, 511, 1, 5000), ("kdv", 20000, 30, 30, 4000)])
def test_instances_of_fewer_steps_than_chunks_equal_stream(kind, n, few, many, steps):
    ps = [_problem(kind, n, W.F64)] * (few + many)
    _check(f"few steps {kind}", ps, [1] * few + [steps] * many, [0, few - 1] + list(range(few, few + many)))
