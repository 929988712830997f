"""Short calls on long lines march where two marching passes are the faster (FP64 lines
of 200 thousand cells and more, FP32 two-component lines of 2^20 and more at twice the
marching depth), others run register passes, all with the bits of single steps; the
deepest marching pass of a line is among them."""
import numpy as np
import pytest

from paper_1107_4650_amd import libdirac as L
from paper_1107_4650_amd.inputs import C_LIGHT, random_spinor
from tests.gpu_util import announce, same_bits

pytestmark = pytest.mark.gpu

C = C_LIGHT
DX = 0.01


def advance(start, V, nsteps, dtype, bc, scheme, pair, depth=None):
    import torch
    n = start.shape[0]
    t = torch.from_numpy(start).to("cuda").to(torch.complex64 if dtype == "c64" else
                                              torch.complex128).contiguous()
    tV = None if V is None else torch.from_numpy(V).to("cuda")
    with L.Plan((n,), DX, (1 if scheme == "lie" else 2) * DX / C, C, 1.0, dtype=dtype, bc=bc,
                scheme=scheme, bispinor=pair) as p:
        if depth:
            p.set_depth(depth)
            p.set_tiling(allow_resident=False)
        p.step(t, tV, nsteps)
        torch.cuda.synchronize()
        i = p.info()
    return t.cpu().numpy(), (i["ran_marching"], i["ran_lines"])


# marching passes of a call (0: register passes)
CASES = [(300007, "c128", False, "lie", {1: 1, 4: 1, 5: 1, 9: 2, 10: 2, 11: 0}),
         (300007, "c128", True, "lie", {5: 1, 10: 2, 11: 0}),
         (300007, "c128", False, "strang", {2: 1, 3: 1, 5: 2, 6: 2, 7: 0}),
         (300007, "c64", False, "lie", {1: 0, 10: 0}),
         (1 << 20, "c64", True, "lie", {5: 0, 8: 0, 10: 2, 11: 0}),
         (1 << 20, "c64", True, "strang", {6: 2, 7: 0}), (100003, "c128", False, "lie", {10: 0})]


@pytest.mark.parametrize("bc", ["zero", "periodic"])
@pytest.mark.parametrize("n,dtype,pair,scheme,marching", CASES)
def test_short_calls_on_long_lines(n, dtype, pair, scheme, marching, bc):
    announce(f"line route n={n} {dtype} pair={pair} {scheme} {bc}")
    start = random_spinor((n,), seed=5)
    if pair:
        start = np.ascontiguousarray(start[:, [0, 3]])
    V = np.random.default_rng(6).uniform(-3, 3, n) * C * C
    V[n // 2] = 1e12  # an angle beyond the fast reduction range
    for nsteps, m in marching.items():
        for Vm in (V, None) if nsteps == max(marching) else (V,):
            got, ran = advance(start, Vm, nsteps, dtype, bc, scheme, pair)
            assert ran[0] == m and (ran[1] > 0) == (m == 0), (nsteps, ran)
            ref, one = advance(start, Vm, nsteps, dtype, bc, scheme, pair, depth=1)
            assert one[0] == nsteps and same_bits(got, ref), nsteps
