"""Sweeps of grids past 1 GiB of state, whose blocks are kept in step by progress
marks: changes of the coefficients between calls (table, arrays, conductive,
material indices off), bit for bit against single steps of the plain scheme,
which update in place."""
import pytest

from paper_2502_20610_amd import fdtd
from tests.test_gpu_sweep import PEC, PER

pytestmark = pytest.mark.gpu


def _materials(kind, shape, gen):
    import torch
    few = torch.randint(0, 5, shape, device="cuda", generator=gen)
    if "arrays" in kind:
        eps = 1.0 + torch.rand(shape, device="cuda", generator=gen)
    else:
        eps = torch.tensor([1.0, 2.08, 3.5, 7.0, 12.25], device="cuda")[few]
    sigma = None
    if "lossy" in kind:
        sigma = torch.tensor([0.0, 0.01, 0.1, 0.3, 0.4], device="cuda")[few].contiguous()
    return eps.contiguous(), sigma


@pytest.mark.parametrize("bc", [(PEC, PEC, PEC), (PER, PEC, PER)])
def test_materials_change_between_sweeps(bc):
    import torch
    shape = (361, 360, 352)
    assert 24 * shape[0] * shape[1] * shape[2] > 2 ** 30
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    fields = [torch.rand(shape, device="cuda", generator=gen) - 0.5 for _ in range(6)]
    sims = [fdtd.Simulation(shape, 0.5, 1.0, bc, scheme="plain") for _ in range(2)]
    try:
        for sim in sims:
            sim.set_fields(fields)
            sim.synchronize()
        swept, stepped = sims
        for kind in ("table", "lossy arrays", "lossy table", "arrays", "table"):
            eps, sigma = _materials(kind, shape, gen)
            torch.cuda.synchronize()
            for sim in sims:
                sim.set_materials(eps, sigma=sigma)
            for ids in (1, 0):
                swept.set_option(fdtd.OPT_MATERIAL_IDS, ids)
                swept.step(9)
                for _ in range(9):
                    stepped.step(1)
                got, want = torch.empty(shape, device="cuda"), torch.empty(shape, device="cuda")
                torch.cuda.synchronize()
                for c in range(6):
                    swept.read_fields(mask=1 << c, out=[got] * 6)
                    stepped.read_fields(mask=1 << c, out=[want] * 6)
                    swept.synchronize()
                    stepped.synchronize()
                    assert torch.equal(got.view(torch.int32), want.view(torch.int32)), (kind, ids, c)
    finally:
        for sim in sims:
            sim.close()


def test_half_storage_rounds_where_the_rings_allow():
    """FP16 storage on the largest grid, 64 steps with the automatic band: the face
    rings of a 64-step band would pass 32-bit offsets, so the fields are rounded
    after a shorter one, as with that band asked for."""
    import torch
    shape = (1024, 1024, 1024)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    field = torch.rand(shape, device="cuda", generator=gen) - 0.5
    torch.cuda.synchronize()
    sims, band = [], 0
    try:
        for _ in range(2):
            sim = fdtd.Simulation(shape, 0.5, 1.0, (PEC, PEC, PEC), scheme="systolic", storage="fp16")
            sims.append(sim)
            if band:
                sim.set_option(fdtd.OPT_BAND_STEPS, band)
            sim.set_fields([field] * 6)
            sim.step(64)
            assert band in (0, sim.info(fdtd.INFO_SYSTOLIC_BAND))
            band = sim.info(fdtd.INFO_SYSTOLIC_BAND)
            assert band < 64
        want = torch.empty(shape, device="cuda")
        torch.cuda.synchronize()
        for c in range(6):
            sims[0].read_fields(mask=1 << c, out=[field] * 6)
            sims[1].read_fields(mask=1 << c, out=[want] * 6)
            for sim in sims:
                sim.synchronize()
            assert torch.equal(field.view(torch.int32), want.view(torch.int32)), c
    finally:
        for sim in sims:
            sim.close()


@pytest.mark.parametrize("shape,bc", [((30, 40, 70), (PER, PER, PEC)), ((70, 37, 33), (PEC, PER, PER)), ((3, 50, 64), (PER, PER, PER))])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_a_plane_of_sources(shape, bc, axis):
    """A source on every cell of a plane (two on some, starting at different
    steps, added in no order of planes), as one scheme after another takes them:
    more than a block keeps at hand, against the FP32 oracle."""
    import numpy as np

    import oracle
    from paper_2502_20610_amd import workloads as wl
    from tests.test_gpu_parity import assert_bitwise
    rng = np.random.default_rng(sum(shape) + axis)
    eps = rng.choice(np.float32([1.0, 2.08, 7.0]), shape)
    zero = [np.zeros(shape, np.float32) for _ in range(6)]
    cells = np.argwhere(np.ones([1 if a == axis else n for a, n in enumerate(shape)]))
    cells[:, axis] = shape[axis] // 2
    cells = cells[[all(bc[a] == PER or p[a] > 0 for a in range(3)) for p in cells]]
    cells = cells[rng.permutation(len(cells))][:600]
    cells = np.concatenate([cells, cells[:40]])
    sources = [wl.dipole(int(rng.integers(0, 3)), *(int(v) for v in p), rng.uniform(-1, 1, 9).astype(np.float32),
                         first_step=int(rng.integers(0, 4))) for p in cells]
    assert len(sources) > 64
    for scheme in ("plain", "plain_fused"):
        sim = fdtd.Simulation(shape, 0.5, 1.0, bc, scheme=scheme)
        try:
            sim.set_materials(eps)
            for s in sources:
                sim.add_source(s["comp"], s["i"], s["j"], s["k"], s["waveform"], s["first_step"])
            for n in (1, 6, 8):
                sim.step(n)
            got = sim.read_fields()
        finally:
            sim.close()
        ref = oracle.run(zero, [eps] * 3, bc, 0.5, 1.0, 15, sources=sources, dtype=np.float32)
        assert_bitwise(got, ref, "%s %s axis %d" % (scheme, shape, axis))


@pytest.mark.parametrize("shape,bc,lossy", [((250, 240, 256), (PEC, PEC, PEC), False), ((97, 130, 129), (PER, PEC, PER), True)])
def test_single_fused_steps(shape, bc, lossy):
    """Calls of one step on the fused scheme (one launch of its own on these
    grids), bit for bit as steps of the plain scheme in place."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    eps, sigma = _materials("lossy arrays" if lossy else "arrays", shape, gen)
    fields = [torch.rand(shape, device="cuda", generator=gen) - 0.5 for _ in range(6)]
    torch.cuda.synchronize()
    sims = [fdtd.Simulation(shape, 0.5, 1.0, bc, scheme=s) for s in ("plain_fused", "plain")]
    try:
        for sim in sims:
            sim.set_materials(eps, sigma=sigma)
            sim.set_fields(fields)
            sim.add_source(2, *(n // 2 for n in shape), [0.5, -1.0, 2.0], 1)
            for _ in range(5):
                sim.step(1)
            sim.synchronize()
        got, want = torch.empty(shape, device="cuda"), torch.empty(shape, device="cuda")
        torch.cuda.synchronize()
        for c in range(6):
            sims[0].read_fields(mask=1 << c, out=[got] * 6)
            sims[1].read_fields(mask=1 << c, out=[want] * 6)
            for sim in sims:
                sim.synchronize()
            assert torch.equal(got.view(torch.int32), want.view(torch.int32)), c
    finally:
        for sim in sims:
            sim.close()


@pytest.mark.parametrize("scheme,shape,bc,calls,swept", [
    ("plain", (700, 1, 600), (PEC, PER, PEC), (2, 5, 20), None), ("plain", (60, 70, 64), (PEC, PEC, PEC), (2, 3, 6), None),
    ("systolic", (520, 510, 8), (PEC, PEC, PEC), (12, 64), False), ("systolic", (520, 510, 24), (PEC, PEC, PEC), (12, 30), True),
    ("systolic", (512, 512, 3), (PEC, PER, PEC), (5, 3), False), ("systolic", (512, 512, 3), (PEC, PER, PEC), (20,), True)])
def test_thin_grids_and_short_calls_give_the_same_bits(scheme, shape, bc, calls, swept):
    """Both sides of the lines at which a call leaves sweeps for a scheme's own
    launches, against those launches."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    eps, _ = _materials("table", shape, gen)
    fields = [torch.rand(shape, device="cuda", generator=gen) - 0.5 for _ in range(6)]
    torch.cuda.synchronize()
    sims = [fdtd.Simulation(shape, 0.5, 1.0, bc, scheme=scheme) for _ in range(2)]
    try:
        sims[1].set_option(fdtd.OPT_SWEEPS, 0)
        for sim in sims:
            sim.set_materials(eps)
            sim.set_fields(fields)
            sim.synchronize()
        got, want = torch.empty(shape, device="cuda"), torch.empty(shape, device="cuda")
        torch.cuda.synchronize()
        for n in calls:
            for sim in sims:
                sim.step(n)
            if swept is not None and n * shape[0] * shape[1] >= 10 ** 7 or n < 12 and bc[1] == PER:
                assert (sims[0].info(fdtd.INFO_RING_SLOTS) == 0) == (swept or scheme == "plain")
            for c in range(6):
                sims[0].read_fields(mask=1 << c, out=[got] * 6)
                sims[1].read_fields(mask=1 << c, out=[want] * 6)
                for sim in sims:
                    sim.synchronize()
                assert torch.equal(got.view(torch.int32), want.view(torch.int32)), (n, c)
    finally:
        for sim in sims:
            sim.close()


@pytest.mark.parametrize("lossy", [False, True])
@pytest.mark.parametrize("count", [17, 255, 256, 700])
def test_tables_of_many_materials(count, lossy):
    """More distinct cells in a wavefront than it reports in a round, up to the
    largest table, one more, and many more (the arrays serve), against the
    oracle."""
    import numpy as np

    import oracle
    from tests.test_gpu_parity import assert_bitwise
    shape, bc = (30, 22, 61), (PER, PER, PER)
    rng = np.random.default_rng(count)
    which = rng.integers(0, count, shape)
    which.reshape(-1)[:count] = np.arange(count)
    eps = (1.0 + which / np.float32(32)).astype(np.float32)
    sigma = (which / np.float32(4096)).astype(np.float32) if lossy else None
    fields = [rng.uniform(-1, 1, shape).astype(np.float32) for _ in range(6)]
    sim = fdtd.Simulation(shape, 0.5, 1.0, bc, scheme="plain")
    try:
        for _ in range(2):
            sim.set_materials(eps, sigma=sigma)
            assert sim.info(fdtd.INFO_MATERIALS) == (count + 1 if count < 256 and not lossy else 0)
        sim.set_fields(fields)
        sim.step(7)
        ref = oracle.run(fields, [eps] * 3, bc, 0.5, 1.0, 7, dtype=np.float32, sigma=[sigma] * 3 if lossy else None)
        assert_bitwise(sim.read_fields(), ref, "%d materials, lossy %s" % (count, lossy))
    finally:
        sim.close()
