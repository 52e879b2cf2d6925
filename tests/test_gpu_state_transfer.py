"""State transfer on both sides of the size from which the device converts:
exact, with the arrays given in part and over a change of parity.

The library keeps f and h less the rest state's shares w_i phi0 and w_i T0 in the
storage precision, so a population read back is fl(x - s) + s, and (phi u) is
fl(x): both computed here in the same arithmetic."""
import numpy as np
import pytest

from paper_2306_11320_amd import workloads as wl
from tests.conftest import announce

pytestmark = pytest.mark.gpu

lbm = pytest.importorskip("paper_2306_11320_amd.lbm")

W = np.array([4 / 9] + 4 * [1 / 9] + 4 * [1 / 36])[:, None, None]


@pytest.mark.parametrize("nx,ny", [(3, 3), (63, 65), (64, 64), (241, 17), (1365, 3), (129, 40)])
@pytest.mark.parametrize("prec", [lbm.FP64, lbm.FP32_DEV])
def test_state_round_trip(nx, ny, prec):
    announce("state_round_trip", nx, ny, prec)
    cfg, f0 = wl.tiny(nx, ny, seed=nx)
    cfg["phi0_dev"], cfg["T0_dev"] = 0.75, 1.25
    real = np.float64 if prec == lbm.FP64 else np.float32
    rng = np.random.default_rng(ny)
    lat = lbm.Lattice(cfg, f0, prec)
    lat.step(3)
    want = lat.get_state()
    for step, given in ((4, ("f", "g", "h", "jprev")), (5, ("g",)), (7, ("f", "jprev")), (8, ("h",)), (9, ("jprev",)), (10, ())):
        new = {k: rng.standard_normal((2 if k == "jprev" else 9, ny, nx)) for k in given}
        lat.set_state(0, **new, step=step)
        for k, a in new.items():
            sh = W * {"f": 0.75, "h": 1.25}.get(k, 0.0) if k != "jprev" else 0.0
            want[k] = (a - sh).astype(real).astype(np.float64) + sh
        got = lat.get_state()
        assert got["step"] == step
        for k in ("f", "g", "h", "jprev"):
            assert np.array_equal(got[k], want[k]), (k, step)
    lat.step(2)
    lat.close()
