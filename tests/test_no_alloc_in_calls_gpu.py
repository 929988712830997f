"""Step calls of an odd number of register passes allocate nothing: the free device
memory after the first call of a fresh plan is what it was before, and so after calls of
other step counts; the plan's own memory goes with it."""
import pytest

from paper_1107_4650_amd import libdirac as L
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

C = 137.036
DX = 0.01


@pytest.mark.parametrize("shape,dtype,call,nsteps", [
    ((2048, 2048), "c64", "step", 100), ((2048, 2048), "c64", "step", 20),
    ((512, 512), "c64", "step_observables", 20), ((700, 640), "c128", "step", 20),
    ((1000000,), "c64", "step", 200)])
def test_first_call_of_a_plan_allocates_nothing(shape, dtype, call, nsteps):
    import torch
    announce(f"no allocation in {call} {shape} {dtype} n={nsteps}")
    tdt = torch.complex64 if dtype == "c64" else torch.complex128
    psi = torch.ones(shape[::-1] + (4,), dtype=tdt, device="cuda")
    V = torch.zeros(shape[::-1], dtype=torch.float64, device="cuda")
    def plan():
        return L.Plan(shape, DX, DX / C, C, 1.0, dtype=dtype)
    def calls(p, check):
        p.step_observables(psi, V, 1)  # grows the partials of a fused observables pass
        torch.cuda.synchronize()
        held = torch.cuda.mem_get_info()[0]
        for n in (nsteps, nsteps + 7, 3):
            getattr(p, call)(psi, V, n)
            torch.cuda.synchronize()
            assert not check or torch.cuda.mem_get_info()[0] == held, n
    with plan() as p:  # loads the kernels' code
        calls(p, False)
    before = torch.cuda.mem_get_info()[0]
    with plan() as p:
        calls(p, True)
    assert torch.cuda.mem_get_info()[0] == before
