"""Reverse steps of a plane run in register tiles only where those are the faster:
planes a few rows thin march; psi, lambda and Q carry the bits of single reverse steps
either way."""
import numpy as np
import pytest

from paper_1107_4650_amd import libdirac as L
from paper_1107_4650_amd.inputs import random_spinor
from tests.gpu_util import announce, same_bits

pytestmark = pytest.mark.gpu

C = 137.036
DX = 0.01


def reverse(shape, dtype, bc, nsteps, chunks, depth=None):
    import torch
    tdt = torch.complex64 if dtype == "c64" else torch.complex128
    psi = torch.from_numpy(random_spinor(shape[::-1], seed=1)).to("cuda").to(tdt)
    lam = torch.from_numpy(random_spinor(shape[::-1], seed=2)).to("cuda").to(tdt)
    V = torch.from_numpy(np.random.default_rng(3).uniform(-3, 3, shape[::-1]) * C * C).to("cuda")
    Q = torch.zeros(shape[::-1], dtype=torch.float64, device="cuda")
    with L.Plan(shape, DX, DX / C, C, 1.0, dtype=dtype, bc=bc) as p:
        if depth:
            p.set_depth(depth)
        for n in chunks or [nsteps]:
            p.grad_step(psi, lam, V, Q, n)
        torch.cuda.synchronize()
        i = p.info()
    return [t.cpu().numpy() for t in (psi, lam, Q)], i


# measured, us, one pass of one reverse step of 2^20 x 2, tiles / marching: FP32 152 / 75, FP64
# 362 / 172
@pytest.mark.parametrize("shape,dtype,nsteps,tiles", [
    ((1 << 20, 2), "c64", 1, False), ((1 << 20, 2), "c128", 1, False),
    ((1 << 20, 2), "c128", 4, False), ((300000, 3), "c128", 4, False),
    ((256, 256), "c64", 12, True), ((256, 256), "c128", 12, True),
    ((3000, 60), "c64", 12, True)])
def test_route_of_reverse_calls(shape, dtype, nsteps, tiles):
    announce(f"reverse route {shape} {dtype} n={nsteps}")
    _, i = reverse(shape, dtype, "zero", nsteps, None)
    assert (i["ran_tiles"] > 0, i["ran_marching"] > 0) == (tiles, not tiles), i


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("shape,bc", [((40000, 3), "zero"), ((40000, 5), "periodic"),
                                      ((30000, 8), "periodic")])
def test_thin_planes_keep_single_reverse_step_bits(shape, bc, dtype):
    announce(f"reverse thin {shape} {bc} {dtype}")
    for n in (1, 3, 7):
        got, _ = reverse(shape, dtype, bc, n, None)
        ref, _ = reverse(shape, dtype, bc, n, [1] * n, depth=1)
        assert all(same_bits(a, b) for a, b in zip(got, ref)), n
