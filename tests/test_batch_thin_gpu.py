"""Batches mostly of planes a few rows thin march: every instance ends with the bits of
its own dl_step, with and without graphs, both walls and state types, mixed with squares
and lines, and over calls that follow each other."""
import numpy as np
import pytest

from paper_1107_4650_amd import libdirac as L
from paper_1107_4650_amd.inputs import random_spinor
from tests.gpu_util import announce, same_bits

pytestmark = pytest.mark.gpu

C = 137.036
DX = 0.01


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("dtype,bc", [("c64", "zero"), ("c64", "periodic"), ("c128", "zero")])
def test_thin_batches_keep_single_plan_bits(dtype, bc, graph):
    import torch
    announce(f"thin batch {dtype} {bc} graph={graph}")
    tdt = torch.complex64 if dtype == "c64" else torch.complex128
    shapes = [(20000, 4)] * 30 + [(9000, 4), (130, 70), (700,), (20011, 5)]
    psis = [torch.from_numpy(random_spinor(s[::-1], seed=k)).to("cuda").to(tdt)
            for k, s in enumerate(shapes)]
    Vs = [torch.from_numpy(np.random.default_rng(k).uniform(-2, 2, s[::-1]) * C * C).to("cuda")
          for k, s in enumerate(shapes)]
    alone = [t.clone() for t in psis]
    nsteps = [7, 10, 0, 1, 13] * 6 + [10, 12, 9, 5]
    with L.Batch(shapes, DX, DX / C, C, 1.0, dtype=dtype, bc=bc, graph=graph) as b:
        assert b.info()["tile_depth"] == 0
        for _ in range(2):
            b.step(psis, Vs, nsteps)
        torch.cuda.synchronize()
    for k, s in enumerate(shapes):
        with L.Plan(s, DX, DX / C, C, 1.0, dtype=dtype, bc=bc) as p:
            p.step(alone[k], Vs[k], 2 * nsteps[k])
            torch.cuda.synchronize()
        assert same_bits(psis[k].cpu().numpy(), alone[k].cpu().numpy()), (k, s)
