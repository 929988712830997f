"""A captured short call on a line takes the path with the less device time (two
register passes for 10 steps on 1000 cells, in place for few steps or cells), while an
eager one runs in place; replays with eager work between them keep the eager bits."""
import numpy as np
import pytest

from paper_1107_4650_amd import libdirac as L
from paper_1107_4650_amd.inputs import C_LIGHT, random_spinor
from tests.gpu_util import announce, same_bits

pytestmark = pytest.mark.gpu

C = C_LIGHT
DX = 0.01


# measured on the device, us, in place / two passes, with a potential: FP32 1000 cells 10
# steps 6.7 / 5.9 (two components 6.5 / 5.4), 4 steps 4.2 / 5.2, 64 cells 10 steps 4.5 / 5.2;
# FP64 1000 cells 4 steps 7.8 / 5.9, 64 cells 5 steps 3.6 / 5.2
@pytest.mark.parametrize("n,nsteps,dtype,pair,whole", [
    (1000, 10, "c64", False, False), (1000, 10, "c64", True, False), (1000, 4, "c64", False, True),
    (64, 10, "c64", False, True), (1000, 4, "c128", False, False), (64, 5, "c128", False, True)])
def test_captured_short_calls(n, nsteps, dtype, pair, whole):
    import torch
    announce(f"captured short line n={n} steps={nsteps} {dtype} pair={pair}")
    tdt = torch.complex64 if dtype == "c64" else torch.complex128
    start = random_spinor((n,), seed=n)
    if pair:
        start = np.ascontiguousarray(start[:, [0, 3]])
    psi = torch.from_numpy(start).to("cuda").to(tdt).contiguous()
    ref = psi.clone()
    V = torch.from_numpy(np.random.default_rng(n).uniform(-3, 3, n) * C * C).to("cuda")
    with L.Plan((n,), DX, DX / C, C, 1.0, dtype=dtype, bc="periodic", bispinor=pair) as p:
        p.step(ref, V, nsteps)
        i = p.info()
        assert (i["ran_whole"], i["ran_lines"], i["ran_marching"]) == (1, 0, 0)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            p.step(psi, V, nsteps)
        i = p.info()
        assert (i["ran_whole"] == 1) == whole and (i["ran_lines"] == 2) == (not whole)
        for k in range(4):
            g.replay()
            torch.cuda.synchronize()
            assert same_bits(psi.cpu().numpy(), ref.cpu().numpy()), k
            p.step(ref, V, nsteps)  # eager, in place
            torch.cuda.synchronize()
