"""The tiles of sweeps at grid sizes that reach them: each shape of the plain
sweeps with several rows per lane, the whole-axis tile, the batch's and the
adjoint's, in every coefficient mode, bit for bit against each scheme's own
launches (which the small-grid tests hold to the oracle)."""
import numpy as np
import pytest

from paper_2502_20610_amd import fdtd
from tests.test_gpu_sweep import PEC, PER
from tests.test_gpu_sweep_large import _materials

pytestmark = pytest.mark.gpu

KINDS = ["table", "arrays", "lossy table", "lossy arrays"]


def _make(shape, bc, scheme, kind, seed, sweeps=1):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    eps, sigma = _materials(kind, shape, gen)
    fields = [torch.rand(shape, device="cuda", generator=gen) - 0.5 for _ in range(6)]
    torch.cuda.synchronize()
    sim = fdtd.Simulation(shape, 0.5, 1.0, bc, scheme=scheme)
    sim.set_option(fdtd.OPT_SWEEPS, sweeps)
    sim.set_materials(eps, sigma=sigma)
    sim.set_fields(fields)
    rng = np.random.default_rng(seed)
    for c in range(3):
        sim.add_source(c, *(int(rng.integers(1, n)) for n in shape), rng.uniform(-1, 1, 40).astype(np.float32))
    sim.synchronize()
    return sim


def _assert_same(a, b, what):
    import torch
    got, want = torch.empty(a.shape, device="cuda"), torch.empty(a.shape, device="cuda")
    torch.cuda.synchronize()
    for c in range(6):
        a.read_fields(mask=1 << c, out=[got] * 6)
        b.read_fields(mask=1 << c, out=[want] * 6)
        a.synchronize()
        b.synchronize()
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), (what, c)
    assert bool(torch.isfinite(want).all()) and bool((want != 0).any())


# (shape, {(kind, steps): (steps of the longest pass, tiles)}): on 256 CUs the
# plan takes 36 rows (3 x 12) with T = 5 and 4, 32 (2 x 16 and 4 x 8), 24 (3 x 8)
# and the 64-lane axis; (361, 360, 352) keeps its blocks in step
REACHED = [
    ((64, 64, 64), {("arrays", 7): (4, 176), ("lossy arrays", 7): (4, 176), ("lossy table", 7): (4, 176), ("table", 5): (3, 154)}),
    ((96, 96, 96), {("arrays", 7): (4, 192), ("table", 7): (4, 256), ("lossy table", 7): (4, 256)}),
    ((128, 128, 128), {("table", 9): (5, 240), ("lossy table", 9): (5, 234), ("table", 7): (4, 240), ("lossy table", 7): (4, 240),
                       ("arrays", 5): (3, 240)}),
    ((160, 150, 140), {("table", 5): (3, 240), ("lossy table", 5): (3, 240)}),
    ((200, 180, 190), {("lossy arrays", 5): (3, 240), ("lossy arrays", 3): (2, 252)}),
    ((250, 256, 256), {("arrays", 3): (2, 250), ("lossy arrays", 3): (2, 250)}),
    ((361, 360, 352), {("table", 3): (2, 234), ("lossy table", 3): (2, 234)}),
]


@pytest.mark.parametrize("bc", [(PEC, PEC, PEC), (PEC, PER, PEC)])
@pytest.mark.parametrize("shape,reached", REACHED)
def test_update_tiles(shape, reached, bc):
    import torch
    for kind in KINDS:
        sims = [_make(shape, bc, "systolic", kind, sum(shape)), _make(shape, bc, "plain", kind, sum(shape), 0)]
        try:
            for n in (7, 9, 5, 3, 10):
                for sim in sims:
                    sim.step(n)
                if torch.cuda.get_device_properties(0).multi_processor_count == 256 and (kind, n) in reached:
                    assert (sims[0].info(fdtd.INFO_SYSTOLIC_BAND), sims[0].info(fdtd.INFO_SYSTOLIC_TICKETS)) == reached[kind, n]
            _assert_same(*sims, (shape, kind, bc))
        finally:
            for sim in sims:
                sim.close()


@pytest.mark.parametrize("kinds", [("table",) * 3, ("arrays", "table", "arrays"), ("lossy table",) * 3, ("lossy arrays",) * 3])
def test_batch_tiles(kinds):
    shapes = [((130, 140, 120), (PEC, PEC, PEC)), ((90, 200, 101), (PER, PEC, PER)), ((64, 64, 64), (PEC, PER, PEC))]
    swept = [_make(s, bc, "systolic", k, q) for q, ((s, bc), k) in enumerate(zip(shapes, kinds))]
    own = [_make(s, bc, "plain", k, q, 0) for q, ((s, bc), k) in enumerate(zip(shapes, kinds))]
    try:
        for n in (8, 11, 2, 5):
            fdtd.step_batch(swept, n)
            assert all(sim.info(fdtd.INFO_RING_SLOTS) == 0 for sim in swept)
            for sim in own:
                sim.step(n)
        for q in range(3):
            _assert_same(swept[q], own[q], (shapes[q], kinds))
    finally:
        for sim in swept + own:
            sim.close()


# T = 3 at 4 x 8 and 3 x 8, T = 2 at 4 x 8, T = 4 and 3 at 1 x 16
@pytest.mark.parametrize("shape,lossy,n", [((200, 200, 64), False, 17), ((200, 180, 190), True, 16), ((250, 256, 256), False, 20),
                                           ((40, 64, 64), False, 19), ((64, 60, 70), True, 18)])
@pytest.mark.parametrize("bc", [(PEC, PEC, PEC), (PER, PEC, PER)])
def test_adjoint_tiles(shape, lossy, n, bc):
    """Boxes that cross tile seams and touch the last cells; several segments."""
    outs = []
    for sweeps in (1, 0):
        sim = _make(shape, bc, "plain", "lossy table" if lossy else "table", 9, sweeps)
        try:
            lo, hi = [s // 3 for s in shape], [s // 3 + max(2, s // 4) for s in shape]
            # the monitor passes through the box's last planes, up to the last cells of y and z
            J, g = sim.adjoint(n, 2, (hi[0] - 2, 3, shape[2] // 4), (hi[0] + 1, shape[1], shape[2]), 0.3, lo, hi, checkpoint_every=7)
            outs.append((J, g, sim))
        except Exception:
            sim.close()
            raise
    try:
        assert outs[0][0] == outs[1][0]
        same, some = np.array_equal(outs[0][1].view(np.uint32), outs[1][1].view(np.uint32)), bool(np.any(outs[0][1]))
        assert same and some
        _assert_same(outs[0][2], outs[1][2], (shape, lossy, bc))
    finally:
        for _, _, sim in outs:
            sim.close()
