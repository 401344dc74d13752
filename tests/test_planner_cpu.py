"""What a batch advance launches, and in which order, seen from the host runtime
alone (host_runtime.py): every step of every instance is done once, one after
another, whatever the mix of sizes, types and step counts."""
import numpy as np
import pytest

import host_runtime as H
from paper_0907_1720_amd import lbm
from paper_0907_1720_amd import workloads as W


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    path = str(tmp_path_factory.mktemp("host") / "libhost.so")
    H.compile_to(path)
    h = H.HostRuntime(path)
    yield h
    h.close()


def problem(kind, n, prec=W.F64):
    if kind == "kdv":
        return W.kdv(0.5, n, 0.1, 1e-4, 2.0, 0.0, prec=prec)
    if kind == "mkdv":
        return W.mkdv(0.7, n, 0.1, 1e-4, 2.0, 0.0, prec=prec)
    if kind == "kawahara":
        return W.kawahara(n, 0.1, 2e-5, 3.0, 0.0, prec=prec)
    return W.power_kdv(0.5, 0.01, n, 0.1, 1e-3, 2.0, 0.0, prec=prec)


def advance(host, problems, steps, path=0):
    """Launches of one advance; asserts that it did `steps` to every instance, in order."""
    b = lbm.Batch(problems, stream=0)
    b.set_path(path)
    b.load_phi([np.full(p.n, 0.5) for p in problems])
    host.reset()
    b.advance(steps)
    launches = host.launches()
    n, text = host.faults()
    got = [b.read_phi(i)[0][0] for i in range(len(problems))]
    b.close()
    assert n == 0, text
    assert got == [float(s) for s in steps]
    return launches


def test_step_chunks_of_a_group_on_its_share_of_the_gpu_stay_in_order(host):
    """Several slab groups, each on its share of the CUs, which one of them exceeds."""
    P = problem
    advance(host, [P("kdv", 4324, W.F32_DEV)] * 3 + [P("mkdv", 41530, W.F32_DEV)] * 20, [4000, 600, 600] + [1000] * 20)
    advance(host, [P("kdv", 229000)] * 2 + [P("kdv", 20000, W.F32_DEV)] * 4 + [P("kdv", 1024)] * 2650, [4000] * 2656)
