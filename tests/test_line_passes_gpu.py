"""Lines run register passes of up to 96 transports (workgroups of 208 or 784
cells, on short lines one for each of the two uncoupled pairs of a spinor): the
same bits as single marching steps from two cells on, with both walls, every
axis, both schemes, state types and stored widths and phase modes 0 to 2."""
import numpy as np
import pytest

from paper_1107_4650_amd import libdirac as L
from paper_1107_4650_amd.inputs import C_LIGHT, random_spinor
from tests.gpu_util import announce, same_bits

pytestmark = pytest.mark.gpu

C = C_LIGHT
DX = 0.01


def advance(psi, V, m, nsteps, single, n, axis, bc, dtype, scheme, pair, graph=False):
    import torch
    t = torch.from_numpy(psi).to("cuda").to(torch.complex64 if dtype == "c64" else torch.complex128)
    t = t.contiguous()
    tV = None if V is None else torch.from_numpy(V).to("cuda")
    dt = (1 if scheme == "lie" else 2) * DX / C
    with L.Plan((n,), DX, dt, C, m, dtype=dtype, bc=bc, axes=(axis,), scheme=scheme,
                bispinor=pair, graph=graph) as p:
        if single:
            p.set_depth(1)
            p.set_tiling(allow_resident=False)
        assert (p.info()["line_1d_depth"] == 0) == single
        p.step(t, tV, nsteps)
        torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("pair", [False, True])
@pytest.mark.parametrize("scheme", ["lie", "strang"])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,axis,bc", [(2, 0, "periodic"), (3, 2, "zero"), (17, 1, "zero"),
                                       (111, 0, "periodic"), (208, 2, "zero"), (209, 1, "periodic"),
                                       (4097, 0, "zero"), (30011, 2, "periodic"),
                                       (70001, 1, "zero"), (300007, 0, "periodic"),
                                       (300007, 2, "zero")])
def test_line_passes_keep_single_step_bits(n, axis, bc, dtype, scheme, pair):
    announce(f"line passes n={n} axis={axis} {bc} {dtype} {scheme} pair={pair}")
    psi = random_spinor((n,), seed=n)
    if pair:
        psi = np.ascontiguousarray(psi[:, [0, 2 if axis == 2 else 3]])
    V = np.random.default_rng(n).uniform(-3, 3, size=(n,)) * C * C
    V[n // 2] = 1e12  # an angle beyond the fast reduction range
    args = (n, axis, bc, dtype, scheme, pair)
    for nsteps in (1, 9, 10, 203) if n < 60000 else (101,):
        assert same_bits(advance(psi, V, 1.0, nsteps, False, *args),
                         advance(psi, V, 1.0, nsteps, True, *args)), nsteps
    for m in (1.0, 0.0):  # constant mass phase; pure streaming
        assert same_bits(advance(psi, None, m, 41, False, *args),
                         advance(psi, None, m, 41, True, *args)), m


@pytest.mark.parametrize("pair", [False, True])
def test_line_passes_in_graph_replays(pair):
    announce(f"line passes graph pair={pair}")
    n = 1000
    psi = random_spinor((n,), seed=8)
    if pair:
        psi = np.ascontiguousarray(psi[:, [0, 3]])
    V = np.random.default_rng(9).uniform(-3, 3, size=(n,)) * C * C
    args = (n, 0, "periodic", "c128", "lie", pair)
    assert same_bits(advance(psi, V, 1.0, 300, False, *args, graph=True),
                     advance(psi, V, 1.0, 300, True, *args))
