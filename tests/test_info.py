"""dl_plan_info says which passes a plan takes: the register tiles of a plane and
their kind, those with a vector potential and of the reverse steps, a batch's
tiles; the entries are 0 where marching passes run."""
import pytest

from paper_1107_4650_amd import libdirac as L

C = 137.036
DX = 0.01


def info(shape, **kw):
    strang = kw.get("scheme") == "strang"
    with L.Plan(shape, DX, (2 if strang else 1) * DX / C, C, 1.0, dry=True, **kw) as p:
        return p.info()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("scheme", ["lie", "strang"])
def test_register_tiles_are_named(dtype, scheme):
    kw = dict(dtype=dtype, scheme=scheme)
    small = info((256, 256), **kw)
    assert small["tile_2d_kind"] in (3, 4) and small["tile_2d_depth"] > 1  # pairs apart
    assert info((256, 256), axes=(0, 2), **kw)["tile_2d_kind"] in (1, 2)  # one workgroup a tile
    assert small["tile_field_depth"] > 1
    assert (small["tile_reverse_depth"] > 1) == (scheme == "lie")  # second order has no adjoint
    line = info((777,), **kw)
    assert line["line_1d_depth"] > 1
    for k in ("tile_2d_kind", "tile_2d_depth", "tile_field_depth", "tile_reverse_depth"):
        assert line[k] == 0, k


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("scheme", ["lie", "strang"])
@pytest.mark.parametrize("shape,kind", [
    ((2, 2), 3), ((7, 3), 3), ((41, 9), 3), ((130, 127), 3), ((256, 257), 3), ((21, 1000), 3),
    ((400, 390), 4), ((511, 513), 4)])
def test_pairs_apart_on_both_tiles(shape, kind, scheme, dtype):
    # both tiles of the pairs, at sizes that the comparisons with single steps run
    assert info(shape, scheme=scheme, dtype=dtype)["tile_2d_kind"] == kind


def test_caps_leave_marching_passes():
    with L.Plan((256, 256), DX, DX / C, C, 1.0, dry=True) as p:
        p.set_depth(2)
        i = p.info()
        assert i["tile_2d_kind"] == i["tile_field_depth"] == i["tile_reverse_depth"] == 0
        assert i["depth"] == i["reverse_depth"] == 2
        assert i["ran_marching"] == i["ran_tiles"] == i["ran_lines"] == i["ran_whole"] == 0


def test_thin_batches_march():
    # measured, 100 steps, tiles / marching, us: 30 of 20000 x 4 4820 / 2245 (FP64 7473 /
    # 5086), 300 of 2000 x 4 5005 / 2713, 20 of 20000 x 4 with 8 of 512^2 3857 / 2350; 30 of
    # 20000 x 32 7466 / 7836, 100 of 256^2 3094 / 3130
    def tiles(shapes, dtype="c64", bc="zero"):
        with L.Batch(shapes, DX, DX / C, C, 1.0, dtype=dtype, bc=bc, dry=True) as b:
            return b.info()["tile_depth"] > 0
    for dtype in ("c64", "c128"):
        assert not tiles([(20000, 4)] * 30, dtype) and not tiles([(2000, 4)] * 300, dtype)
        assert tiles([(300, 300)] * 4, dtype) and tiles([(100, 100)] * 16, dtype)
        assert tiles([(256, 256)] * 100, dtype) and tiles([(20000, 32)] * 30, dtype)
        assert tiles([(100000,)] * 20, dtype) and tiles([(64,)], dtype)
    assert not tiles([(20000, 4)] * 30, bc="periodic")
    assert not tiles([(20000, 4)] * 20 + [(512, 512)] * 8)


def test_batch_names_its_tiles():
    with L.Batch([(64,), (96, 80)], DX, DX / C, C, 1.0, dry=True) as b:
        assert b.info()["tile_depth"] > 1
        b.set(seg_len=16, depth=3)
        assert b.info()["tile_depth"] == 0 and b.depth() == 3
