"""The register-resident kernels at the edges of their lanes, waves and jobs.

A wave holds 64 R nodes, R per lane; an instance takes as many waves as its
nodes need beside the halos, exchanges every few steps, and a grid shorter than
a wave's core is held as several periods of itself.  Every result must equal
the streaming kernel's bit for bit (the same per-node arithmetic in the same
order), so the comparison has no tolerance.
"""
import dataclasses

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


def say(*a):
    print(*a, flush=True)


def _problem(kind, n, prec):
    x = np.arange(n) * (2 * np.pi / n)
    phi0 = 0.4 + 0.3 * np.sin(x + 0.1 * n) + 0.05 * np.cos(3 * x)
    if kind == "kdv":
        p = W.kdv(0.5, n, 0.1, 1e-4, 2.0, 0.0, prec=prec)
    elif kind == "mkdv":
        p = W.mkdv(0.7, n, 0.1, 1e-4, 2.0, 0.0, prec=prec)
    elif kind == "kawahara":
        p = W.kawahara(n, 0.1, 2e-5, 3.0, 0.0, prec=prec)
    elif kind == "m6":
        p = dataclasses.replace(W.random_m6_problem(W.rng(5, 1), n), prec=prec, tau=3.0)
    else:
        p = W.even_lattice_instance(0, 4 if kind == "d1q4" else 6, prec=prec).problem
        p = dataclasses.replace(p, n=n)
    return p, phi0


def _run(p, phi0, steps, path):
    s = lbm.Solver(p)
    s.set_path(path)
    s.load_phi(phi0)
    for k in steps:
        s.advance(k)
    out = s.read_phi()
    s.close()
    return out


# 7..60: several periods in one wave; 112/113, 174/175, 300/301, 360/361: one wave full, two begun;
# 1054/1055 and 2464/2465: the same for wider lanes; 2925, 4096: the largest grids of one LDS in FP64
@pytest.mark.parametrize("n", [7, 20, 60, 112, 113, 174, 175, 300, 301, 360, 361, 1054, 1055, 2464, 2465, 2925, 4096])
@pytest.mark.parametrize("kind", ["kdv", "mkdv", "d1q4", "d1q6", "kawahara", "m6"])
@pytest.mark.parametrize("prec", [W.F64, W.F32_DEV, W.F32_DEV_ARITH32])
def test_resident_equals_stream_at_lane_and_wave_edges(kind, n, prec):
    if kind in ("d1q6", "kawahara", "m6") and prec == W.F64 and n > 2925:
        pytest.skip("beyond one LDS")
    p, phi0 = _problem(kind, n, prec)
    steps = (1, 2, 5, 34)   # fewer than an exchange, odd, and several exchanges
    say("case registers", kind, n, prec)
    assert np.array_equal(_run(p, phi0, steps, lbm.PATH_RESIDENT), _run(p, phi0, steps, lbm.PATH_STREAM))


@pytest.mark.parametrize("prec", [W.F64, W.F32_DEV])
@pytest.mark.parametrize("lo,hi,count", [(100, 420, 1500), (300, 4000, 700)])
def test_split_jobs_equal_solo(prec, lo, hi, count):
    """Batches whose jobs outnumber the CUs: jobs of several instances, some split
    in two between workgroups, with several step counts."""
    ns = [int(round(lo * (hi / lo) ** ((0.5 + 0.6180339887498949 * i) % 1.0))) for i in range(count)]
    ps, phis = zip(*[_problem("kdv" if i % 3 else "mkdv", n, prec) for i, n in enumerate(ns)])
    steps = [201 + 50 * (i % 2) for i in range(count)]
    say("case split jobs", prec, lo, hi, count)
    b = lbm.Batch(list(ps))
    b.load_phi(list(phis))
    b.advance(steps)
    b.advance([k // 2 for k in steps])
    sample = sorted({0, 1, 2, 3, count - 1, int(np.argmax(ns)), int(np.argmin(ns))} | set(range(5, count, count // 12)))
    for k in range(count):
        got, st = b.read_phi(k)
        assert st == lbm.OK, k
        if k in sample:
            want = _run(ps[k], phis[k], (steps[k], steps[k] // 2), lbm.PATH_STREAM)
            assert np.array_equal(got, want), (k, ns[k])
    b.close()


# Slabs (one per workgroup) and tiles of instances beyond one workgroup, at the planner's own choice and
# with it forced narrow and wide: 1031..9973: node counts that leave a part of the last lane; steps: fewer
# than an exchange, odd, several exchanges (an odd number of tile launches), a call that ends on one.
@pytest.mark.parametrize("n", [1031, 4099, 9973])
@pytest.mark.parametrize("kind", ["kdv", "mkdv", "d1q4", "d1q6", "kawahara", "m6"])
@pytest.mark.parametrize("prec", [W.F64, W.F32_DEV, W.F32_DEV_ARITH32])
def test_slabs_and_tiles_equal_stream(kind, n, prec):
    p, phi0 = _problem(kind, n, prec)
    steps = (1, 2, 83, 64)
    say("case segments", kind, n, prec)
    want = _run(p, phi0, steps, lbm.PATH_STREAM)
    for path in (lbm.PATH_SLAB, lbm.PATH_TILED):
        for tiling in ((0, 0), (6, 1), (24, 8), (3, 2), (4096, 8)):
            s = lbm.Solver(p)
            s.set_path(path)
            s.set_tiling(*tiling)
            s.load_phi(phi0)
            for k in steps:
                s.advance(k)
            got = s.read_phi()
            s.close()
            assert np.array_equal(got, want), (path, tiling)


def test_mixed_batch_of_slabs_tiles_and_rings_equals_solo():
    """Groups of several variants and precisions that need more workgroups than
    the GPU has CUs: their slab launches run one after another, in step chunks."""
    kinds = [("kdv", 20011, W.F64), ("mkdv", 9001, W.F32_DEV), ("kawahara", 12007, W.F64), ("kdv", 301, W.F64)]
    ps, phis = zip(*[_problem(*kinds[i % 4][:2], kinds[i % 4][2]) for i in range(240)])
    steps = [600 + i % 3 for i in range(240)]
    say("case mixed segments")
    b = lbm.Batch(list(ps))
    b.load_phi(list(phis))
    b.advance(steps)
    b.advance([37] * 240)
    for k in range(240):
        got, st = b.read_phi(k)
        assert st == lbm.OK, k
        if k < 12 or k > 235:
            assert np.array_equal(got, _run(ps[k], phis[k], (steps[k], 37), lbm.PATH_STREAM)), k
    b.close()


# bounded instances: one wave (in LDS) and the fewest nodes of two, odd and even places of the interior
# node, the most nodes of 16 waves and one more (in LDS again); 6 layers are the most computed on D1Q5
@pytest.mark.parametrize("n", [63, 112, 113, 114, 801, 1791, 1792, 1793])
@pytest.mark.parametrize("kind", ["kdv", "mkdv", "d1q4"])
@pytest.mark.parametrize("prec", [W.F64, W.F32_DEV, W.F32_DEV_ARITH32])
def test_bounded_resident_equals_stream_at_wave_edges(kind, n, prec):
    p, phi0 = _problem(kind, n, prec)
    for bc, layers in ((1, p.lattice() // 2), (2, p.lattice() // 2), (2, 6), (2, 7)):
        p = dataclasses.replace(p, bc=bc)
        say("case bounded registers", kind, n, prec, bc, layers)
        outs = []
        for path in (lbm.PATH_STREAM, lbm.PATH_RESIDENT):
            s = lbm.Solver(p)
            s.set_path(path)
            s.load_phi(phi0)
            for steps in (1, 2, 3, 4, 5, 34):
                rows = np.random.default_rng(steps).uniform(0.35, 0.45, (steps, 2 * layers))
                s.advance_bounded(rows)
            outs.append(s.read_phi())
            s.close()
        assert np.array_equal(outs[0], outs[1]), (bc, layers)
