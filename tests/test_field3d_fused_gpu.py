"""3-D lowest-order passes fuse two steps with a vector potential too: the bits
of single steps for a static field and for a pulse whose ramp the steps cross,
on boxes at the edges of the 60 x 8 tiles, with both walls and state types,
with and without a potential, far angles included."""
import numpy as np
import pytest

from paper_1107_4650_amd import libdirac as L
from paper_1107_4650_amd.inputs import C_LIGHT, random_spinor
from tests.gpu_util import announce, same_bits

pytestmark = pytest.mark.gpu

C = C_LIGHT
DX = 0.01


@pytest.mark.parametrize("shape,bc", [((2, 3, 5), "periodic"), ((61, 8, 4), "zero"),
                                      ((60, 9, 3), "periodic"), ((130, 17, 70), "zero")])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_two_step_field_passes_keep_single_step_bits(shape, bc, dtype):
    import torch
    announce(f"field 3-D two steps {shape} {bc} {dtype}")
    ts = tuple(reversed(shape))
    tdt = torch.complex64 if dtype == "c64" else torch.complex128
    rng = np.random.default_rng(sum(shape))
    V = rng.uniform(-3, 3, ts) * C * C
    V.flat[1] = 1e12
    A = rng.uniform(-0.7, 0.7, (3,) + ts)
    A[0].flat[2] = 1e8
    psi = random_spinor(ts, seed=5)
    tV, tA = torch.from_numpy(V).to("cuda"), torch.from_numpy(A).to("cuda")
    tP = tA * (C / DX)
    dt = DX / C
    pulse = dict(omega=0.9 / dt, phase=0.3, t_on=2.5 * dt, t_flat=1.2 * dt, t_off=2.0 * dt)

    def run(depth, n, v, pulsed):
        t = torch.from_numpy(psi).to("cuda").to(tdt).contiguous()
        with L.Plan(shape, DX, dt, C, 1.0, dtype=dtype, bc=bc) as p:
            assert p.info()["field_depth"] == 2
            p.set_depth(depth)
            if pulsed:
                p.step_pulse(t, v, tP, pulse, -0.4 * dt, n)
            else:
                p.step_field(t, v, tA, n)
            torch.cuda.synchronize()
        return t.cpu().numpy()

    for n in (2, 7):
        for v in (tV, None):
            for pulsed in (False, True):
                assert same_bits(run(5, n, v, pulsed), run(1, n, v, pulsed)), (n, v is None, pulsed)
