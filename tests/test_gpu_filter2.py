"""The 2D current filter and Ampere in one launch against the FP64 oracle, at every reach it takes.

One step from random fields and random electrons, then E, B and the filtered current are compared
cell by cell: on boxes with absorbing faces, periodic boxes and mixed ones, on a box whose x axis is
too short for the larger reaches (those keep the line filter), with strides (always the line
filter), and on a grid large enough for the large tile.  Tolerances as in the 3D filter's tests
(FP64 1e-11, FP32 2e-6 of the field scale).
"""
import numpy as np
import pytest

import pic_inputs as pi
from oracle import Oracle

gpu = pytest.mark.gpu
NAMES = ["Ex", "Ey", "Ez", "Bx", "By", "Bz", "Jx", "Jy", "Jz"]

GEOMETRIES = {
    # (nx, nz), pml cells, periodic x, z
    "pml": ((37, 53), 4, (0, 0)),
    "periodic": ((33, 41), 0, (1, 1)),
    "periodic x": ((7, 30), 4, (1, 0)),
    "short": ((2, 24), 4, (0, 1)),       # 11 stored x cells: reaches 5 and 6 by the line filter
    "tiny periodic": ((3, 5), 0, (1, 1)),
    "large": ((310, 1480), 5, (0, 0)),
}
MARGIN = {"pml": 1.5, "periodic": 0.0, "periodic x": 0.0, "short": 0.3, "tiny periodic": 0.0, "large": 2.0}


def _check(geom, npass, comp, real, strides=1):
    (nx, nz), pml, per = GEOMETRIES[geom]
    cfg = pi.make_config(nx, nz, 0.1, 0.09, pml_cells=pml, periodic_x=per[0], periodic_z=per[1], ck="ck2",
                         theta=0.2, filter_npass=npass, filter_compensate=comp, real=real, seed=21,
                         filter_strides=strides)
    from paper_1009_2727_amd import Sim
    n = 20000 if geom == "large" else 1500
    sim = Sim(cfg, capacity=n + 1000)
    ref = Oracle(cfg)
    for k, name in enumerate(["Ex", "Ey", "Ez", "Bx", "By", "Bz", "Exo", "Eyo", "Ezo", "Exb", "Eyb", "Ezb"]):
        f = pi.random_field(ref.shape, seed=700 + k, amp=0.4)
        ref.set_field(name, f)
        sim.set_field(name, f)
    p = pi.random_electrons(n, nx, nz, 0.1, 0.09, seed=23, umax=3.0, margin=MARGIN[geom])
    ref.set_electrons(p)
    sim.load_electrons(p)
    ref.step(1)
    sim.step(1)
    assert sim.sync_status() == 0
    tol = 1e-11 if real == "f64" else 2e-6
    for name in NAMES:
        a, b = sim.field(name), ref.field(name)
        assert np.abs(a - b).max() <= tol * max(np.abs(b).max(), 1.0), (name, float(np.abs(a - b).max()))


@gpu
@pytest.mark.parametrize("geom", list(GEOMETRIES))
@pytest.mark.parametrize("npass,comp", [(0, 0), (1, 0), (2, 0), (2, 1), (4, 0), (4, 1), (6, 0), (6, 1)])
def test_2d_filter_reaches_match_oracle(geom, npass, comp):
    _check(geom, npass, comp, "f64")


@gpu
@pytest.mark.parametrize("geom", ["pml", "periodic", "large"])
@pytest.mark.parametrize("strides", [0b1, 0b11])
def test_2d_filter_fp32_matches_oracle(geom, strides):
    _check(geom, 4, 1, "f32", strides)
