"""Read-outs to device arrays that share memory: written in component order, so
the last one stays whole, as with one copy after another."""
import numpy as np
import pytest

from paper_2502_20610_amd import fdtd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(5, 7, 9), (96, 96, 96)])
def test_overlapping_destinations_in_component_order(shape):
    import torch
    n = shape[0] * shape[1] * shape[2]
    rng = np.random.default_rng(n)
    sim = fdtd.Simulation(shape, 0.5, 1.0, (1, 1, 1), scheme="plain")
    try:
        sim.set_fields([rng.uniform(-1, 1, shape).astype(np.float32) for _ in range(6)])
        want = [f.ravel() for f in sim.read_fields()]
        for step, mask in ((0, 0x3F), (0, 0x15), (n // 2, 0x3F), (n - 1, 0x3F), (n, 0x3F)):
            buf = torch.full((5 * step + n,), 7.0, device="cuda")
            ref = np.full(5 * step + n, 7.0, np.float32)
            out = [buf[c * step:c * step + n].view(shape) for c in range(6)]
            torch.cuda.synchronize()
            sim.read_fields(mask=mask, out=out)
            sim.synchronize()
            for c in range(6):
                if mask >> c & 1:
                    ref[c * step:c * step + n] = want[c]
            assert np.array_equal(buf.cpu().numpy().view(np.uint32), ref.view(np.uint32)), (step, mask)
    finally:
        sim.close()
