"""The batch tuner says whether register tiles or the marching passes it tuned run
afterwards, the batch runs what it says, and its cache file repeats it: tiles for small
planes, marching passes for planes a few rows thin."""
import numpy as np
import pytest

from paper_1107_4650_amd import libdirac as L
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

C = 137.036
DX = 0.01


# measured, 100 steps, tiles / marching, us: 190 / 1908 and 4820 / 2245
@pytest.mark.parametrize("shapes,tiles", [([(100, 100)] * 16, True), ([(20000, 4)] * 30, False)])
def test_tuner_reports_what_runs(shapes, tiles, tmp_path, monkeypatch):
    import torch
    announce(f"batch tuner {shapes[0]} x {len(shapes)}")
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("LIBDIRAC_TUNE_CACHE", str(cache))
    psis = [torch.ones(s[::-1] + (4,), dtype=torch.complex64, device="cuda") for s in shapes]
    Vs = [torch.zeros(s[::-1], dtype=torch.float64, device="cuda") for s in shapes]
    args = (shapes, DX, DX / C, C, 1.0)
    with L.Batch(*args) as b:
        ch = b.autotune(psis, Vs, trials=3)
        assert (ch["tile_depth"] > 0) == tiles and ch["tile_depth"] == b.info()["tile_depth"]
        assert ch["depth"] == b.depth()  # the marching passes it tuned
        assert f"dirac-batch c64 2d-march {2 if tiles else 1}" in cache.read_text().split("\n")
        b.set(seg_len=ch["seg_len"], depth=ch["depth"])  # marching passes by request
        assert b.info()["tile_depth"] == 0
        assert b.autotune(psis, Vs, trials=3)["tile_depth"] == ch["tile_depth"]  # and back
    with L.Batch(*args) as b:
        assert (b.info()["tile_depth"] > 0) == tiles
    assert all(np.all(t.cpu().numpy() == 1) for t in psis)
