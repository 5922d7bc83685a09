"""The launches that run where sweeps do not (memory short, a plane too large, or
FDTD_OPT_SWEEPS = 0, which is how they are reached here): the plain scheme's two
launches per step, direct and as replayed graphs, the fused step's one launch
per step, the persistent systolic launch, and the adjoint's one-step kernels."""
import numpy as np
import pytest

import oracle
from paper_2502_20610_amd import fdtd
from paper_2502_20610_amd import workloads as wl
from tests.test_gpu_fused import CASES
from tests.test_gpu_graphs import CALLS
from tests.test_gpu_parity import assert_bitwise

pytestmark = pytest.mark.gpu
PEC, PER = 0, 1


def _sim(w, scheme, opts=(), sigma=None, storage="fp32"):
    sim = fdtd.Simulation(w.shape, w.dt, w.dx, w.bc, scheme=scheme, storage=storage)
    sim.set_option(fdtd.OPT_SWEEPS, 0)
    for k, v in opts:
        sim.set_option(k, v)
    sim.set_materials(w.eps, sigma=sigma)
    sim.set_fields(w.fields)
    for s in w.sources:
        sim.add_source(s["comp"], s["i"], s["j"], s["k"], s["waveform"], s.get("first_step", 0))
    return sim


def _sigma(w, seed):
    return [np.random.default_rng(seed).uniform(0.0, 0.2, w.shape).astype(np.float32)] * 3


@pytest.mark.parametrize("lossy", [False, True])
@pytest.mark.parametrize("with_sources", [True, False])
def test_two_launches_direct_and_replayed(lossy, with_sources):
    """Graphs on and off over calls with remainders, a source added and the fields
    reset between replays."""
    bc = (PEC, PER, PEC)
    w = wl.small_case((33, 29, 40), bc, seed=62, nsteps=120, dipoles=[(16, 14, 20), (9, 20, 31)] if with_sources else [])
    sigma = _sigma(w, 4) if lossy else None
    sims = [_sim(w, "plain", [(fdtd.OPT_GRAPHS, g)], sigma) for g in (1, 0)]
    late = wl.dipole(wl.EY, 10, 9, 8, wl.gaussian_sine(200, 0.5), first_step=60)
    state, sources, step = w.fields, list(w.sources), 0
    try:
        for q, n in enumerate(CALLS + [48, 16]):
            if q == 3:
                sources.append(late)
                for sim in sims:
                    sim.add_source(late["comp"], late["i"], late["j"], late["k"], late["waveform"], 60)
            if q == 5:
                state = w.fields
                for sim in sims:
                    sim.set_fields(state)
            state = oracle.run(state, w.eps3(), bc, w.dt, w.dx, n, sources=sources, dtype=np.float32, step0=step, sigma=sigma)
            step += n
            for g, sim in zip((1, 0), sims):
                sim.step(n)
                assert_bitwise(sim.read_fields(), state, "graphs %d lossy %s after %d steps" % (g, lossy, step))
        sims[1].set_option(fdtd.OPT_PROFILE, 1)
        sims[1].step(5)
        assert sims[1].kernel_stats(fdtd.KERNEL_PLAIN_E)[0] == 5
    finally:
        for sim in sims:
            sim.close()


@pytest.mark.parametrize("lossy", [False, True])
@pytest.mark.parametrize("shape,bc,n,dip", CASES)
def test_fused_step_one_launch_per_step(shape, bc, n, dip, lossy):
    w = wl.small_case(shape, bc, seed=sum(shape), nsteps=n, dipoles=dip)
    sigma = _sigma(w, n) if lossy else None
    sim = _sim(w, "plain_fused", [(fdtd.OPT_PROFILE, 1)], sigma)
    try:
        sim.step(n)
        assert sim.kernel_stats(fdtd.KERNEL_PLAIN_FUSED)[0] == n
        ref = oracle.run(w.fields, w.eps3(), bc, w.dt, w.dx, n, sources=w.sources, dtype=np.float32, sigma=sigma)
        assert_bitwise(sim.read_fields(), ref, "fused step %s %s" % (shape, bc))
    finally:
        sim.close()


@pytest.mark.parametrize("storage,sigma", [("fp32", False), ("fp32", True), ("fp16", False)])
def test_persistent_launch_and_the_same_bits_as_sweeps(storage, sigma):
    w = wl.small_case((50, 45, 41), (PEC, PER, PEC), seed=4, nsteps=70, dipoles=[(25, 20, 20)])
    outs = []
    for sweeps in (0, 1):
        sim = _sim(w, "systolic", [(fdtd.OPT_SWEEPS, sweeps)], _sigma(w, 9) if sigma else None, storage)
        try:
            sim.step(23)
            sim.step(47)
            assert (sim.info(fdtd.INFO_RING_SLOTS) > 0) == (sweeps == 0)
            outs.append(sim.read_fields())
        finally:
            sim.close()
    assert_bitwise(outs[0], outs[1], "persistent and swept, %s" % storage)


@pytest.mark.parametrize("lossy", [False, True])
@pytest.mark.parametrize("every", [0, 7, 1])
def test_adjoint_one_step_kernels(every, lossy):
    """Same objective, gradient and final state, bit for bit, as the swept run."""
    w = wl.small_case((34, 25, 38), (PEC, PEC, PER), seed=12, nsteps=30, dipoles=[(8, 12, 18)])
    outs = []
    for sweeps in (0, 1):
        sim = _sim(w, "plain", [(fdtd.OPT_SWEEPS, sweeps)], _sigma(w, 2) if lossy else None)
        try:
            J, g = sim.adjoint(29, 2, (24, 3, 2), (26, 20, 33), 0.4, (12, 5, 6), (19, 17, 30), checkpoint_every=every)
            sim.step(4)
            outs.append((np.float64(J), g, sim.read_fields()))
        finally:
            sim.close()
    assert outs[0][0] == outs[1][0]
    assert np.array_equal(outs[0][1].view(np.uint32), outs[1][1].view(np.uint32)) and np.any(outs[0][1])
    assert_bitwise(outs[0][2], outs[1][2], "state after the adjoint")


@pytest.mark.parametrize("storage,bytes_per_cell", [("fp32", 24), ("fp16", 48)])
def test_sweeps_off_gives_the_second_sets_back(storage, bytes_per_cell):
    import torch
    shape = (256, 256, 200)
    cells = shape[0] * shape[1] * shape[2]
    sim = fdtd.Simulation(shape, 0.5, 1.0, (PEC, PEC, PEC), scheme="systolic", storage=storage)
    try:
        before = torch.cuda.mem_get_info()[0]
        sim.step(4)
        sim.synchronize()
        swept = torch.cuda.mem_get_info()[0]
        sim.set_option(fdtd.OPT_SWEEPS, 0)
        after = torch.cuda.mem_get_info()[0]
        # (the runtime may serve a few MiB from blocks that it already held)
        room = bytes_per_cell * cells - (16 << 20)
        assert before - swept >= room and after - swept >= room
        sim.set_option(fdtd.OPT_SWEEPS, 1)
        sim.step(4)
        sim.synchronize()
        with pytest.raises(fdtd.FdtdError):
            sim.set_option(fdtd.OPT_SWEEPS, 2)
    finally:
        sim.close()


def test_half_storage_takes_little_memory_for_sweeps():
    """FP16 storage takes its FP32 sets from a sixteenth of the free memory; a grid
    past that keeps the persistent launch and its own memory."""
    import torch
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    for share, swept in ((1.0 / 12, False), (1.0 / 40, True)):
        plane = 512 * 512
        shape = (int(share * free / 48 / plane), 512, 512)
        sim = fdtd.Simulation(shape, 0.5, 1.0, (PEC, PEC, PEC), scheme="systolic", storage="fp16")
        try:
            before = torch.cuda.mem_get_info()[0]
            sim.step(8)
            sim.synchronize()
            taken = before - torch.cuda.mem_get_info()[0]
            assert (sim.info(fdtd.INFO_RING_SLOTS) == 0) == swept
            assert (taken > 24 * plane * shape[0]) == swept
        finally:
            sim.close()


def test_adjoint_forward_run_is_timed():
    """Per-kernel timing counts the forward run's launches, swept or single."""
    w = wl.small_case((40, 36, 44), (PEC, PEC, PEC), seed=5, nsteps=30, dipoles=[(8, 12, 18)])
    for sweeps in (0, 1):
        sim = _sim(w, "plain", [(fdtd.OPT_SWEEPS, sweeps), (fdtd.OPT_PROFILE, 1)])
        try:
            sim.adjoint(24, 2, (30, 3, 2), (31, 30, 40), 0.4, (12, 5, 6), (19, 17, 30))
            single, swept = sim.kernel_stats(fdtd.KERNEL_PLAIN_E), sim.kernel_stats(fdtd.KERNEL_PLAIN_FUSED)
            assert single[0] == (0 if sweeps else 24)
            assert (6 <= swept[0] <= 24 and swept[1] > 0.0) if sweeps else swept[0] == 0
        finally:
            sim.close()


@pytest.mark.parametrize("shape,n", [((20, 24, 30), 1), ((20, 24, 30), 2), ((45, 40, 41), 3), ((45, 40, 41), 4),
                                     ((70, 61, 67), 15), ((70, 61, 67), 16)])
@pytest.mark.parametrize("boxes", ["small", "design whole", "both whole"])
def test_adjoint_at_the_lines_between_the_two_ways(shape, n, boxes):
    w = wl.small_case(shape, (PEC, PEC, PEC), seed=15, nsteps=n, dipoles=[(8, 12, 18)])
    mon = ((0, 0, 0), shape) if boxes == "both whole" else ((14, 0, 0), (15, 24, 30))
    des = ((6, 5, 6), (9, 9, 9)) if boxes == "small" else ((0, 0, 0), shape)
    outs = []
    for sweeps in (0, 1):
        sim = _sim(w, "plain", [(fdtd.OPT_SWEEPS, sweeps)])
        try:
            J, g = sim.adjoint(n, 2, *mon, 0.4, *des)
            outs.append((J, g, sim.read_fields()))
        finally:
            sim.close()
    assert outs[0][0] == outs[1][0] and np.array_equal(outs[0][1].view(np.uint32), outs[1][1].view(np.uint32))
    assert_bitwise(outs[0][2], outs[1][2], "state after the adjoint")
