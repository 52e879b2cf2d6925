"""Tiles at walls (their code path: walls and periodic sides, cut tiles among
them) at the edges of the tile shapes, one step against the oracle.

Tolerance: that of the other one-step checks, 2e-13 of the largest population
in FP64; FP32 storage keeps 24 bits of populations of unit size and a few
dozen operations on them, 1e-5.
"""
import numpy as np
import pytest

import oracle
from paper_2306_11320_amd import workloads as wl
from tests.conftest import announce

pytestmark = pytest.mark.gpu

lbm = pytest.importorskip("paper_2306_11320_amd.lbm")

P, T, A, I, O = wl.PERIODIC, wl.WALL_T, wl.WALL_ADIABATIC, wl.INLET, wl.OUTLET


@pytest.mark.parametrize("bcs", [(T, A, A, T), (A, T, P, P), (P, P, A, T), (T, T, T, T), (T, T, I, O), (I, O, T, A)],
                         ids=lambda b: "bc" + "".join(map(str, b)))
@pytest.mark.parametrize("shape", [(3, 3), (64, 4), (65, 5), (63, 8), (129, 9), (32, 17), (256, 3)],
                         ids=lambda s: f"{s[0]}x{s[1]}")
@pytest.mark.parametrize("trt,potential", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_wall_tiles_one_step(bcs, shape, trt, potential):
    nx, ny = shape
    announce("wall_tiles", bcs, shape, trt, potential)
    cfg, f0 = wl.tiny(nx, ny, bc=bcs, seed=nx + ny)
    cfg["collision"], cfg["force_form"] = trt, potential
    o = oracle.Oracle(cfg, f0)
    st = o.get_state()
    d = wl.perturbation(nx, ny, seed=5)
    st = {k: st[k] + d[k] for k in ("f", "g", "h", "jprev")}
    o.set_state(**st, step=0)
    o.step(1)
    ref = o.get_state()
    for prec, tol in ((lbm.FP64, 2e-13), (lbm.FP32_DEV, 1e-5)):
        lat = lbm.Lattice(cfg, f0, prec)
        first = None
        for tile in range(6):
            lat.set_tile(tile)
            lat.set_state(0, **st, step=0)
            lat.step(1)
            got = lat.get_state()
            for q in ("f", "g", "h", "jprev"):
                if first is None:
                    assert np.abs(got[q] - ref[q]).max() <= tol * np.abs(ref[q]).max(), (q, prec)
                else:
                    assert np.array_equal(got[q], first[q]), (q, prec, tile)
            first = first or got
        lat.close()


def test_default_tiles():
    announce("default_tiles")
    wide = [wl.sweep_instance(256, 1024, 30.0, 1.0, 1.0) for _ in range(6)]
    for items, prec, tile in ((wide, lbm.FP32_DEV, 6), (wide, lbm.FP64, 7), (wide[:2], lbm.FP32_DEV, 0), (wide[:1], lbm.FP32_DEV, 3),
                              ([wl.sweep_instance(160, 320, 20.0, 1.0, 1.0)], lbm.FP64, 2),
                              ([wl.sweep_instance(200, 320, 20.0, 1.0, 1.0)], lbm.FP64, 2),
                              ([wl.sweep_instance(200, 320, 20.0, 1.0, 1.0)], lbm.FP32_DEV, 3),
                              ([wl.sweep_instance(128, 512, 20.0, 1.0, 1.0)], lbm.FP32_DEV, 0),
                              ([wl.sweep_instance(128, 520, 20.0, 1.0, 1.0)], lbm.FP32_DEV, 3),
                              ([wl.sweep_instance(192, 320, 20.0, 1.0, 1.0)], lbm.FP64, 0)):
        lat = lbm.Lattice.batch(items, prec)
        assert lat.tile() == tile and lat.grid() == 0, (len(items), prec, lat.tile(), lat.grid())
        lat.close()


@pytest.mark.parametrize("bcs,nx,ny", [((P, P, T, A), 70, 1540), ((P, P, P, P), 64, 3075), ((T, T, P, P), 129, 1027),
                                       ((P, P, I, O), 130, 1100)])
def test_cut_tiles_beyond_one_round(bcs, nx, ny):
    """More 64 x 4 tiles than the chip holds at once, some cut by a periodic end
    (columns, rows) or at walls: the FP64 BGK kernel for such tables."""
    announce("cut_tiles_many", bcs, nx, ny)
    cfg, f0 = wl.tiny(nx, ny, bc=bcs, seed=nx)
    o = oracle.Oracle(cfg, f0)
    st = o.get_state()
    d = wl.perturbation(nx, ny, seed=6)
    st = {k: st[k] + d[k] for k in ("f", "g", "h", "jprev")}
    o.set_state(**st, step=0)
    o.step(1)
    ref = o.get_state()
    lat = lbm.Lattice(cfg, f0, lbm.FP64)
    got = []
    for tile in (0, 2):
        lat.set_tile(tile)
        lat.set_state(0, **st, step=0)
        lat.step(1)
        got.append(lat.get_state())
    for q in ("f", "g", "h", "jprev"):
        assert np.abs(got[0][q] - ref[q]).max() <= 2e-13 * np.abs(ref[q]).max(), q
        assert np.array_equal(got[0][q], got[1][q]), q
    lat.close()


@pytest.mark.parametrize("nx,ny", [(140, 560), (130, 260), (270, 700), (185, 600), (112, 256), (221, 884), (240, 600),
                                   (140, 280), (40, 40)])
def test_default_tile_potential_fp32(nx, ny):
    """128 x 4 tiles are the default only where they are no more per CU than 64 x 8
    ones, their last column holds more than 8 nodes, and rows that start on
    whole lines have more than one workgroup per CU."""
    announce("default_tile_potential", nx, ny)
    cfg, f0 = wl.sweep_instance(nx, ny, 12.0, 1.0, 1.0)
    cfg["force_form"] = 1
    lat = lbm.Lattice(cfg, f0, lbm.FP32_DEV)
    tile = lat.tile()
    lat.close()

    def per_cu(tx, ty):
        return -(-(-(-nx // tx) * -(-ny // ty)) // 256)
    wide = nx % 32 != 0 and not 1 <= nx % 128 <= 8 and (nx % 16 != 0 or per_cu(64, 8) > 1)
    assert tile == (5 if wide and per_cu(128, 4) <= per_cu(64, 8) else 3)


@pytest.mark.parametrize("nx,ny", [(36, 64), (100, 100), (100, 400), (162, 256), (104, 256), (250, 500), (440, 96),
                                   (480, 96), (390, 96), (352, 96), (130, 260), (200, 256), (70, 128), (64, 32),
                                   (260, 700), (200, 800), (280, 1100), (200, 900), (390, 600), (333, 555)])
@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_DEV])
@pytest.mark.parametrize("potential", [0, 1])
def test_default_tile_columns(nx, ny, prec, potential):
    """32 x 8 tiles are the default where they leave less of a row idle: in FP32
    whole ones, up to six columns of 64 unless the form has a second ring; in FP64
    with that form down to a last column of five nodes; in FP64 without it if
    they are fewer per CU than 64 x 4 ones and at most four, and up to six columns
    also if they are at most two or if the last column of those has 5 to 8 nodes.
    64 x 4 tiles in FP32, at most one per CU, have no last column of 16 nodes or
    fewer."""
    announce("default_tile_columns", nx, ny, prec, potential)
    cfg, f0 = wl.sweep_instance(nx, ny, 10.0, 1.0, 1.0)
    cfg["force_form"] = potential
    lat = lbm.Lattice(cfg, f0, prec)
    tile = lat.tile()
    lat.close()
    r, six = nx % 64, nx <= 384

    def per_cu(tx, ty, slack=0):
        return -((slack - -(-nx // tx) * -(-ny // ty)) // 256)
    if prec == lbm.FP64 and potential:
        assert tile == (2 if 1 <= r <= 32 or (r > 36 and six) else 0)
    elif prec == lbm.FP64:
        fewer = per_cu(32, 8, 16) < min(per_cu(64, 4), 5) or (six and (5 <= r <= 8 or per_cu(32, 8) <= 2))
        assert tile == (2 if 1 <= r <= 32 and fewer else 0)
    elif r == 32 and (potential or six):
        assert tile == 2
    elif not potential:
        assert tile in (0, 3) and not (tile == 0 and per_cu(64, 4) == 1 and 1 <= r <= 16)


@pytest.mark.parametrize("nx,ny,potential", [(65, 1575, 0), (129, 1037, 1), (33, 9, 1), (64, 4100, 1)])
def test_fields_tiles_agree(nx, ny, potential):
    """The fields of an FP32 lattice alone (in 64 x 8 tiles, unless it is too large)
    and in a batch with the other force form (the same kernel, other tiles or
    none), bit by bit, against the oracle."""
    announce("fields_tiles", nx, ny, potential)
    cfg, f0 = wl.tiny(nx, ny, bc=(P, P, T, A), seed=ny)
    cfg["force_form"] = potential
    o = oracle.Oracle(cfg, f0)
    ref = o.fields()
    lat = lbm.Lattice(cfg, f0, lbm.FP32_DEV)
    got = lat.fields()
    for q in ("phi", "ux", "uy", "T", "p"):
        assert np.abs(got[q] - ref[q]).max() <= 1e-5 * max(np.abs(ref[q]).max(), 1e-2), q
    lat.close()
    other = dict(cfg, force_form=1 - potential)
    both = lbm.Lattice.batch([(cfg, f0), (other, f0)], lbm.FP32_DEV)
    for q, v in both.fields(0).items():
        assert np.array_equal(v, got[q]), q
    both.close()
