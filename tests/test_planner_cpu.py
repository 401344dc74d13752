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


@pytest.mark.parametrize("kind,prec,n,few,many", [("power", W.F64, 4096, [1] * 511, [5000]),
                                                  ("kdv", W.F64, 20000, [1] * 30, [4000] * 30),
                                                  ("kdv", W.F64, 50000, [1] * 20, [4000] * 20)])
def test_a_launch_holds_one_step_chunk_of_an_instance(host, kind, prec, n, few, many):
    """Instances of fewer steps than chunks drop out of the later chunks."""
    steps = few + many
    launches = advance(host, [problem(kind, n, prec)] * len(steps), steps)
    assert sum(r[0] in (H.SLABS, H.LDS_SLABS) for r in launches) > 1


@pytest.mark.parametrize("seed", range(40))
def test_random_mixed_batches_do_every_step_in_order(host, seed):
    rng = np.random.default_rng([20261205, seed])
    count = int(np.exp(rng.uniform(np.log(4), np.log(300))))
    top = rng.choice([4000, 16384, 60000])
    kinds = ["kdv", "mkdv", "kawahara", "power"][: int(rng.integers(1, 5))]
    ps, steps = [], []
    for _ in range(count):
        n = int(np.exp(rng.uniform(np.log(128), np.log(top))))
        kind = kinds[int(rng.integers(len(kinds)))]
        ps.append(problem(kind, n, int(rng.integers(2))))
        steps.append(int(np.exp(rng.uniform(0, np.log(8000)))) if seed % 2 else [1000, 4000, 1][int(rng.integers(3))])
    for path in (0, 3, 4):
        advance(host, ps, steps, path)


def kawahara_k22(prec):
    return [W.config4_instance(i, prec=prec).problem for i in range(512)]


@pytest.mark.parametrize("prec", [W.F64, W.F32_DEV])
def test_slab_launches_are_counted_as_they_are_filled(host, prec):
    """Whole instances fill the launches: none is a short tail, and a group takes at most
    an eighth more launch time than its workgroups would take on all CUs."""
    launches = [r for r in advance(host, kawahara_k22(prec), [5000] * 512) if r[0] == H.SLABS]
    for width in {r[6] for r in launches}:
        groups = [r[2] for r in launches if r[6] == width]
        assert 2 * min(groups) >= max(groups), groups
        work = sum(r[2] * r[3] for r in launches if r[6] == width)
        assert sum(r[3] for r in launches if r[6] == width) <= max(5000, 1.125 * work / 256), launches


@pytest.mark.parametrize("prec", [W.F64, W.F32_DEV])
def test_whole_instances_have_the_gpu_where_slabs_follow_them(host, prec):
    launches = advance(host, kawahara_k22(prec), [5000] * 512)
    assert max(r[2] for r in launches if r[0] == H.SLABS) >= 240
    assert sum(r[2] for r in launches if r[0] == H.REG) >= 240


@pytest.mark.parametrize("kind,prec,n,count,widest", [("kdv", W.F64, 16384, 128, 14), ("mkdv", W.F64, 16384, 128, 14),
                                                      ("kawahara", W.F32_DEV, 20000, 128, 10)])
def test_slabs_are_not_planned_with_lanes_wider_than_their_registers(host, kind, prec, n, count, widest):
    """The slab kernels of these tables spill the widest lanes' nodes (2 to 3 times the step)."""
    for steps in (300, 5000):
        launches = [r for r in advance(host, [problem(kind, n, prec)] * count, [steps] * count) if r[0] == H.SLABS]
        assert launches and max(r[6] for r in launches) <= widest


@pytest.mark.parametrize("prec", [W.F64, W.F32_DEV])
def test_few_steps_are_planned_without_step_chunks(host, prec):
    """400 steps cannot be cut into chunks, so that a plan of a little more than one
    launch would take two launches' time."""
    launches = [r for r in advance(host, [problem("kawahara", 30000, prec)] * 20, [400] * 20) if r[0] == H.SLABS]
    assert sum(r[3] for r in launches) == 400, launches


@pytest.mark.parametrize("count", [257, 280, 300, 400, 514, 600, 1000, 1026])
def test_jobs_end_with_the_even_share(host, count):
    """Equal jobs laid end to end over the workgroups."""
    r, = [r for r in advance(host, [problem("kdv", 4096)] * count, [2000] * count) if r[0] == H.REG]
    assert r[3] <= 2000 * max(1.0, r[7] / r[2] + 0.06), r


@pytest.mark.parametrize("kind,prec,n,count", [("kdv", W.F32_DEV_ARITH32, 1000, 512), ("kdv", W.F32_DEV, 1000, 512),
                                               ("mkdv", W.F32_DEV_ARITH32, 1400, 512), ("kawahara", W.F64, 700, 700)])
def test_jobs_are_planned_as_whole_instances_fill_them(host, kind, prec, n, count):
    """Several instances to each CU: jobs that leave no quarter of a CU's waves idle,
    or one to each CU (nine waves of sixteen, one job to a CU and two rounds, before)."""
    r, = [r for r in advance(host, [problem(kind, n, prec)] * count, [600] * count) if r[0] == H.REG]
    assert r[7] <= 256 or r[4] >= 75, r


@pytest.mark.parametrize("where", ["host", "another GPU", "this GPU"])
@pytest.mark.parametrize("prec", [W.F64, W.F32_DEV])
def test_device_arrays_that_kernels_cannot_reach_go_by_copies(host, where, prec):
    """A caller's "device" array may be host memory or another GPU's: a copy takes
    either, a kernel that is given it faults."""
    import ctypes

    n = 300
    keep = np.full(n, 0.5)
    ptr = keep.ctypes.data if where == "host" else getattr(host.lib, "stub_foreign" if where == "another GPU" else "stub_device")(8 * n)
    a = np.ctypeslib.as_array(ctypes.cast(ptr, ctypes.POINTER(ctypes.c_double)), (n,))
    a[:] = 0.5
    s = lbm.Solver(problem("kdv", n, prec), stream=0)
    host.reset()
    assert host.lib.lbm_load_phi(s._h, ptr, 1) == lbm.OK
    s.advance(7)
    assert host.lib.lbm_read_phi(s._h, ptr, 1) == lbm.OK
    s.close()
    assert host.faults()[0] == 0, host.faults()[1]
    assert np.all(a == 7.0)


@pytest.mark.parametrize("kind,sizes", [("power", [256 + 15 * i for i in range(256)]), ("kdv", [900] * 16)])
def test_instances_that_fit_stay_whole_without_memory_for_a_second_state(host, kind, sizes):
    ps = [problem(kind, n) for n in sizes]
    assert any(r[0] in (H.SLABS, H.LDS_SLABS) for r in advance(host, ps, [500] * len(ps)))
    b = lbm.Batch(ps, stream=0)
    b.load_phi([np.full(n, 0.5) for n in sizes])
    host.reset()
    host.limit(64 << 10)
    try:
        b.advance(500)
    finally:
        host.limit()
    assert [b.read_phi(i)[0][0] for i in range(len(ps))] == [500.0] * len(ps)
    assert not any(r[0] in (H.SLABS, H.LDS_SLABS) for r in host.launches())
    b.close()


def test_tags_of_a_pass_do_not_wrap(host):
    """Strips are cleared to tag 0 and hold the tags of earlier passes: a block's tag
    must be above both, also in a long pass of many launches."""
    ps = [problem(kind, 9000, prec) for kind in ("kdv", "mkdv", "kawahara") for prec in range(3)]
    b = lbm.Batch(ps, stream=0)
    b.set_tiling(2, 0)
    b.load_phi([np.full(p.n, 0.5) for p in ps])
    last = 0
    for steps in (100, 1 << 30, 1 << 30, 100):
        host.reset()
        b.advance(steps)
        slabs = host.launches(H.SLABS)
        assert len(slabs) == len(ps)
        low, high = min(r[4] for r in slabs), max(r[4] + r[5] for r in slabs)
        assert 1 <= low and high < 1 << 32
        assert low > last or low == 1   # (1: after a clear)
        last = high - 1
    b.close()


def test_a_solver_pins_host_memory_twice(host):
    """Each allocation of pinned memory takes about 40 us of a solver's 700."""
    before = host.lib.stub_pinned()
    s = lbm.Solver(problem("kdv", 800), stream=0)
    assert host.lib.stub_pinned() - before <= 2
    s.close()
    assert host.lib.stub_pinned() == before


@pytest.mark.parametrize("sizes", [[300], [20000], [300, 5000, 9000, 16000] * 16])
def test_a_pass_uploads_its_tables_in_one_copy(host, sizes):
    """Each copy or clear on the stream adds some 4 us to a short advance."""
    b = lbm.Batch([problem("kdv", n) for n in sizes], stream=0)
    b.load_phi([np.full(n, 0.5) for n in sizes])
    b.advance(2)
    host.reset()
    b.advance(2)
    assert host.lib.stub_copies() == 1
    b.close()


def test_slab_launches_of_two_batches_wait_for_each_other(host):
    """Together they would hold more workgroups than there are CUs (on two streams)."""
    sizes = [[200003], [9001] * 90, [5000]]
    streams = [0x10, 0x20, 0x30]
    batches = []
    for ns, s in zip(sizes, streams):
        b = lbm.Batch([problem("kdv", n) for n in ns], stream=s)
        b.load_phi([np.full(n, 0.5) for n in ns])
        batches.append(b)
    host.reset()
    for steps in (100, 7, 100, 300):
        for b in batches:
            b.advance(steps)
    assert host.faults()[0] == 0, host.faults()[1]
    assert all(b.read_phi(0)[0][0] == 507.0 for b in batches)
    batches[1].close()
    for b in batches[::2]:
        b.advance(5)
        b.close()
    assert host.faults()[0] == 0, host.faults()[1]


def test_slab_launches_side_by_side_have_a_cu_for_every_workgroup_of_an_xcd(host):
    """Counted over the whole GPU, launches of 108 and 148 workgroups leave no room for one of them on
    three of the XCDs, and each may wait there for a place that the other holds."""
    P = problem
    for few in range(1, 7):
        for many in (20, 24, 27, 30):
            advance(host, [P("kdv", 20000)] * few + [P("mkdv", 9000 + 100 * few)] * many + [P("kawahara", 5000)] * 3,
                    [300] * (few + many + 3))
    streams, batches = [0x10, 0x20], []
    for ns, s in zip(([6001], [9001] * 2), streams):   # 94 and 162 workgroups
        b = lbm.Batch([P("kdv", n) for n in ns], stream=s)
        b.load_phi([np.full(n, 0.5) for n in ns])
        batches.append(b)
    host.reset()
    for b in batches:
        b.advance(100)
    assert host.faults()[0] == 0, host.faults()[1]
    for b in batches:
        b.close()


@pytest.mark.parametrize("groups", [[("kdv", 774, W.F32_DEV, 415), ("mkdv", 758, W.F32_DEV_ARITH32, 267)],
                                    [("kdv", 1204, W.F32_DEV_ARITH32, 303), ("kawahara", 900, W.F32_DEV, 263)],
                                    [("kdv", 2000, W.F64, 150), ("mkdv", 2100, W.F32_DEV, 130), ("kawahara", 700, W.F64, 250)]])
def test_launches_side_by_side_have_cus_of_their_own(host, groups):
    """Whole CUs of every XCD each, and no other workgroup fits beside one."""
    problems = [problem(kind, n, prec) for kind, n, prec, count in groups for _ in range(count)]
    launches = [l for l in advance(host, problems, [400] * len(problems)) if l[0] == H.REG]
    assert len(launches) == len(groups)
    assert sum((wgs + 7) // 8 for _, _, wgs, *_ in launches) <= 32
    assert all(wgs % 8 == 0 or wgs == jobs for _, _, wgs, _, _, _, _, jobs in launches)
    assert all(lds > 163840 // 2 for _, _, _, _, _, lds, _, _ in launches)


@pytest.mark.parametrize("kinds,n,large", [(("kdv", "kawahara"), 2048, 16384), (("power", "power"), 800, 30000)])
def test_slabs_wait_as_long_as_whole_instances_may_keep_their_cus(host, kinds, n, large):
    """Part of a slab launch may have its places while the rest waits for launches beside it to end."""
    steps = 10 ** 7
    problems = [problem(k, n) for k in kinds for _ in range(128)] + [problem(k, large) for k in kinds for _ in range(64)]
    launches = advance(host, problems, [steps] * len(problems))
    assert {H.REG, H.LDS} & {l[0] for l in launches} and {H.SLABS, H.LDS_SLABS} & {l[0] for l in launches}
    us = host.lib.stub_slab_wait() / 100.0   # (ticks of a 100 MHz clock)
    assert us >= 10 ** 7 + 20.0 * steps


def test_slabs_wait_as_long_as_another_batch_may_keep_their_cus(host):
    """Whole instances of another batch, ten million steps on another stream."""
    many = lbm.Batch([problem("kdv", 1000)] * 300, stream=0x10)
    many.load_phi([np.full(1000, 0.5)] * 300)
    lone = lbm.Batch([problem("kdv", 15001)], stream=0x20)
    lone.load_phi([np.full(15001, 0.5)])
    us = []
    for _ in range(2):
        many.advance(10 ** 7)
        lone.advance(100)
        us.append(host.lib.stub_slab_wait() / 100.0)
        many.last_advance_ms()
        lone.advance(100)
        us.append(host.lib.stub_slab_wait() / 100.0)
    assert all(u >= 10 ** 7 + 20.0 * 10 ** 7 for u in us[::2])
    assert all(u < 1.01 * 10 ** 7 for u in us[1::2])   # over, and not counted any more
    for b in (many, lone):
        b.close()
