"""Calls of a few lowest-order steps on lines of at most 1024 cells run in place in
one workgroup, one cell per thread: the same bits as single marching steps on
ragged and full lines, with both walls, every axis, both state types and stored
widths and phase modes 0 to 2, and around the largest step count and length."""
import numpy as np
import pytest

from paper_1107_4650_amd.inputs import C_LIGHT, random_spinor
from tests.gpu_util import announce, same_bits
from tests.test_line_passes_gpu import advance

pytestmark = pytest.mark.gpu

C = C_LIGHT


@pytest.mark.parametrize("pair", [False, True])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,axis,bc", [(2, 0, "periodic"), (63, 1, "zero"), (65, 2, "periodic"),
                                       (1000, 0, "periodic"), (1001, 2, "zero"),
                                       (1024, 1, "periodic"), (1025, 0, "periodic")])
def test_short_calls_keep_single_step_bits(n, axis, bc, dtype, pair):
    announce(f"short line n={n} axis={axis} {bc} {dtype} pair={pair}")
    psi = random_spinor((n,), seed=n)
    if pair:
        psi = np.ascontiguousarray(psi[:, [0, 2 if axis == 2 else 3]])
    V = np.random.default_rng(n).uniform(-3, 3, size=(n,)) * C * C
    V[n // 2] = 1e12  # an angle beyond the fast reduction range
    args = (n, axis, bc, dtype, "lie", pair)
    for m, Vm, counts in ((1.0, V, (1, 4, 5, 6, 10, 11)), (1.0, None, (5,)), (0.0, None, (5,))):
        for nsteps in counts:
            assert same_bits(advance(psi, Vm, m, nsteps, False, *args),
                             advance(psi, Vm, m, nsteps, True, *args)), (m, nsteps)
