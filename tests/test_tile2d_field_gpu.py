"""Register-tile passes of small 2-D planes with a vector potential: the bits of
single marching steps for a static field and for a pulse, at the edges of the
tiles, with both walls, every axis pair, both schemes and state types, far
angles included."""
import numpy as np
import pytest

from paper_1107_4650_amd import libdirac as L
from paper_1107_4650_amd.inputs import C_LIGHT, random_spinor
from tests.gpu_util import announce, same_bits

pytestmark = pytest.mark.gpu

C = C_LIGHT
DX = 0.01


@pytest.mark.parametrize("scheme", ["lie", "strang"])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("shape,axes,bc", [((2, 3), (0, 1), "periodic"), ((55, 7), (0, 2), "zero"),
                                           ((129, 33), (1, 2), "periodic"), ((9, 200), (0, 1), "zero"),
                                           ((500, 420), (0, 2), "zero")])  # the larger tiles
def test_field_tiles_keep_single_step_bits(shape, axes, bc, dtype, scheme):
    import torch
    announce(f"field tile {shape} {axes} {bc} {dtype} {scheme}")
    ts = tuple(reversed(shape))
    tdt = torch.complex64 if dtype == "c64" else torch.complex128
    rng = np.random.default_rng(shape[0])
    V = rng.uniform(-3, 3, ts) * C * C
    A = rng.uniform(-0.7, 0.7, (3,) + ts)
    A[1].flat[0] = 40.0  # beyond the series' range
    far = A.copy()
    far[0].flat[1] = 1e9  # beyond the fast reduction range
    psi = random_spinor(ts, seed=5)
    dt = (1 if scheme == "lie" else 2) * DX / C
    pulse = dict(omega=0.9 / dt, phase=0.3, t_on=2.5 * dt, t_flat=3.2 * dt, t_off=2.0 * dt)

    def run(depth, n, v, a, pulsed):
        t = torch.from_numpy(psi).to("cuda").to(tdt).contiguous()
        tV = None if v is None else torch.from_numpy(v).to("cuda")
        tA = torch.from_numpy(a * (C / DX if pulsed else 1.0)).to("cuda")
        with L.Plan(shape, DX, dt, C, 1.0, dtype=dtype, bc=bc, axes=axes, scheme=scheme) as p:
            if depth:
                p.set_depth(depth)
            if pulsed:
                p.step_pulse(t, tV, tA, pulse, -0.4 * dt, n)
            else:
                p.step_field(t, tV, tA, n)
            torch.cuda.synchronize()
        return t.cpu().numpy()

    for n, v, a in ((1, V, A), (7, V, far), (16, None, A)):
        for pulsed in (False, True):
            assert same_bits(run(0, n, v, a, pulsed), run(1, n, v, a, pulsed)), (n, pulsed)
