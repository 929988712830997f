"""The deepest marching passes (five lowest-order or three second-order steps, two or
three with a vector potential), which a cap of 5 leaves to the register tiles: a march
segment length makes a plane march, and every axis pair, wall, state type and phase mode
gives the bits of single steps."""
import numpy as np
import pytest

from paper_1107_4650_amd import libdirac as L
from paper_1107_4650_amd.inputs import C_LIGHT, random_spinor
from tests.gpu_util import announce, same_bits

pytestmark = pytest.mark.gpu

C = C_LIGHT
DX = 0.01


def advance(shape, psi, V, A, nsteps, m, axes, bc, dtype, scheme, seg, depth=None):
    import torch
    t = torch.from_numpy(psi).to("cuda").to(torch.complex64 if dtype == "c64" else
                                            torch.complex128).contiguous()
    tV = None if V is None else torch.from_numpy(V).to("cuda")
    tA = None if A is None else torch.from_numpy(A).to("cuda")
    with L.Plan(shape, DX, (1 if scheme == "lie" else 2) * DX / C, C, m, dtype=dtype, bc=bc,
                axes=axes, scheme=scheme) as p:
        if depth:
            p.set_depth(depth)
        p.set_tiling(seg_len=seg)
        i = p.info()
        assert i["tile_2d_depth"] == 0 and i["tile_field_depth"] == 0
        d = depth or i["field_depth" if A is not None else "depth"]
        p.step_field(t, tV, tA, nsteps)
        torch.cuda.synchronize()
        i = p.info()
        left, passes = nsteps, 0
        for k in range(d, 0, -1):
            passes += left // k
            left %= k
        assert (i["ran_marching"], i["ran_tiles"]) == (passes, 0)
    return t.cpu().numpy(), d


@pytest.mark.parametrize("scheme", ["lie", "strang"])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("shape,axes,bc,seg", [((300, 140), (0, 1), "periodic", 24),
                                               ((130, 85), (0, 2), "zero", 11),
                                               ((129, 64), (0, 2), "periodic", 16),
                                               ((63, 90), (1, 2), "zero", 9),
                                               ((200, 61), (1, 2), "periodic", 61)])
def test_deepest_marching_passes_keep_single_step_bits(shape, axes, bc, seg, dtype, scheme):
    announce(f"marching {shape} {axes} {bc} {dtype} {scheme}")
    psi = random_spinor(shape[::-1], seed=shape[0])
    rng = np.random.default_rng(shape[1])
    V = rng.uniform(-3, 3, size=shape[::-1]) * C * C
    V.flat[0] = 1e12  # an angle beyond the fast reduction range
    A = rng.uniform(-2, 2, size=(3,) + shape[::-1])
    A.flat[1] = 40.0  # ... and one beyond the series of the FP32 field step
    for m, Vm, Am, deepest in ((1.0, V, None, 5 if scheme == "lie" else 3),
                               (1.0, None, None, 5 if scheme == "lie" else 3),
                               (0.0, None, None, 5 if scheme == "lie" else 3),
                               (1.0, V, A, 3 if scheme == "lie" else 1)):
        args = (m, axes, bc, dtype, scheme, seg)
        for nsteps in (deepest, 2 * deepest + 1):
            got, d = advance(shape, psi, Vm, Am, nsteps, *args)
            assert d == deepest
            ref, _ = advance(shape, psi, Vm, Am, nsteps, *args, depth=1)
            assert same_bits(got, ref), (m, nsteps)
