"""2-D reverse steps run in register tiles (64 columns by 16 or 24 rows, both
fields and the dL/dV accumulators in registers): the bits of single marching
reverse steps for psi, lambda and Q, at the edges of tiles, on planes smaller
than a tile, with both walls, every axis pair, both state types and phase
modes 0 to 2."""
import numpy as np
import pytest

from paper_1107_4650_amd import libdirac as L
from paper_1107_4650_amd.inputs import C_LIGHT, random_spinor
from tests.gpu_util import announce, same_bits

pytestmark = pytest.mark.gpu

C = C_LIGHT
DX = 0.01


def _reverse(shape, axes, bc, dtype, m, V, nsteps, depth):
    import torch
    tdt = torch.complex64 if dtype == "c64" else torch.complex128
    ts = tuple(reversed(shape))
    psi = torch.from_numpy(random_spinor(ts, seed=1)).to("cuda").to(tdt).contiguous()
    lam = torch.from_numpy(random_spinor(ts, seed=2)).to("cuda").to(tdt).contiguous()
    Q = torch.from_numpy(np.random.default_rng(3).standard_normal(ts)).to("cuda")
    tV = None if V is None else torch.from_numpy(V).to("cuda")
    with L.Plan(shape, DX, DX / C, C, m, dtype=dtype, bc=bc, axes=axes) as p:
        if depth:
            p.set_depth(depth)
        p.grad_step(psi, lam, tV, Q, nsteps)
        torch.cuda.synchronize()
    return psi.cpu().numpy(), lam.cpu().numpy(), Q.cpu().numpy()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("shape,axes,bc", [((2, 3), (0, 1), "periodic"), ((3, 2), (0, 2), "zero"),
                                           ((55, 7), (1, 2), "zero"), ((129, 33), (0, 1), "periodic"),
                                           ((400, 5), (0, 2), "zero"), ((6, 300), (1, 2), "periodic"),
                                           # large enough for the larger tiles
                                           ((520, 530), (0, 1), "zero")])
def test_register_tiles_keep_reverse_step_bits(shape, axes, bc, dtype):
    announce(f"reverse tile {shape} {axes} {bc} {dtype}")
    V = np.random.default_rng(shape[0]).uniform(-3, 3, size=tuple(reversed(shape))) * C * C
    V.flat[0] = 1e12  # an angle beyond the fast reduction range
    for m, Vm, nsteps in ((1.0, V, 1), (1.0, V, 7), (1.0, V, 22), (1.0, None, 9), (0.0, None, 8)):
        one = _reverse(shape, axes, bc, dtype, m, Vm, nsteps, 1)
        got = _reverse(shape, axes, bc, dtype, m, Vm, nsteps, 0)
        assert same_bits(got[0], one[0]) and same_bits(got[1], one[1]), (m, nsteps)
        assert np.array_equal(got[2], one[2]), (m, nsteps)
