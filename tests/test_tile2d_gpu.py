"""2-D planes run register-tile passes (a workgroup holds 64 columns by 32 or
48 rows and advances them several steps): the same bits as single marching
steps at the edges of tiles, on planes smaller than a tile, with both walls,
every axis pair, both schemes and state types and phase modes 0 to 2."""
import numpy as np
import pytest

from paper_1107_4650_amd import libdirac as L
from paper_1107_4650_amd.inputs import C_LIGHT, random_spinor
from tests.gpu_util import announce, gpu_step, same_bits

pytestmark = pytest.mark.gpu

C = C_LIGHT
DX = 0.01


@pytest.mark.parametrize("scheme", ["lie", "strang"])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("shape,axes,bc", [((2, 3), (0, 1), "periodic"), ((3, 2), (0, 2), "zero"),
                                           ((40, 8), (0, 1), "zero"), ((41, 9), (1, 2), "periodic"),
                                           ((64, 33), (0, 2), "zero"), ((129, 70), (1, 2), "zero"),
                                           ((500, 7), (0, 1), "periodic"), ((9, 400), (0, 1), "zero"),
                                           # large enough for the larger tiles
                                           ((701, 640), (0, 1), "zero"),
                                           ((768, 769), (0, 2), "periodic")])
def test_register_tiles_keep_single_step_bits(shape, axes, bc, dtype, scheme):
    announce(f"tile 2-D {shape} {axes} {bc} {dtype} {scheme}")
    dt = (1 if scheme == "lie" else 2) * DX / C
    psi = random_spinor(tuple(reversed(shape)), seed=shape[0])
    V = np.random.default_rng(shape[1]).uniform(-3, 3, size=tuple(reversed(shape))) * C * C
    V.flat[0] = 1e12  # an angle beyond the fast reduction range
    kw = dict(dx=DX, dt=dt, c=C, axes=axes, bc=bc, dtype=dtype, scheme=scheme)
    with L.Plan(shape, DX, dt, C, 1.0, dtype=dtype, bc=bc, axes=axes, scheme=scheme) as p:
        assert p.info()["tile_2d_depth"] > 1
    small = max(shape) < 600
    for nsteps in (1, 5, 12, 31) if small else (17,):
        single = gpu_step(psi, V, m=1.0, nsteps=nsteps, depth=1, **kw)
        assert same_bits(gpu_step(psi, V, m=1.0, nsteps=nsteps, **kw), single), nsteps
    for m in (1.0, 0.0):  # constant mass phase; pure streaming
        single = gpu_step(psi, None, m=m, nsteps=13, depth=1, **kw)
        assert same_bits(gpu_step(psi, None, m=m, nsteps=13, **kw), single), m


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_register_tiles_in_graph_replays(dtype):
    announce(f"tile 2-D graph {dtype}")
    psi = random_spinor((90, 110), seed=5)
    V = np.random.default_rng(6).uniform(-3, 3, size=(90, 110)) * C * C
    kw = dict(dx=DX, dt=DX / C, c=C, m=1.0, dtype=dtype)
    single = gpu_step(psi, V, nsteps=200, depth=1, **kw)
    assert same_bits(gpu_step(psi, V, nsteps=200, graph=True, **kw), single)


def test_tiles_give_way_to_caps_and_retiling():
    with L.Plan((300, 300), DX, DX / C, C, 1.0, dry=True) as p:
        assert p.info()["tile_2d_depth"] > 5
        p.set_depth(4)
        assert p.info()["tile_2d_depth"] == 0
        p.set_depth(5)
        p.set_tiling(seg_len=16)
        assert p.info()["tile_2d_depth"] == 0
    with L.Plan((2048, 2048), DX, DX / C, C, 1.0, dtype="c128", dry=True) as p:
        assert p.info()["tile_2d_depth"] == 0
