"""The 3D current filter on either side of the size where it changes its split of the work.

Small grids are filtered in cubes of 8 cells staged whole, larger ones plane by plane; the line lies
at 2300 cubes of the three components in FP64 and 3500 in FP32.  One step from random fields and
random electrons against the FP64 oracle, one layer of cubes below and above the line, with PML on
every face and periodic, the last cubes partly outside the grid.  Tolerances as in the other 3D
parity tests (FP64 1e-11, FP32 2e-6 of the field scale).
"""
import numpy as np
import pytest

import pic_inputs as pi
from oracle.pic3 import Oracle3

gpu = pytest.mark.gpu
NAMES = ["Ex", "Ey", "Ez", "Bx", "By", "Bz", "Jx", "Jy", "Jz"]


@gpu
@pytest.mark.parametrize("above", [0, 1])
@pytest.mark.parametrize("geom", ["pml", "periodic"])
@pytest.mark.parametrize("real", ["f64", "f32"])
def test_3d_filter_around_the_size_line_matches_oracle(real, geom, above):
    cubes = 2300 if real == "f64" else 3500
    layers = cubes // (3 * 20) + above             # 5 x 4 cubes across
    pml = 4 if geom == "pml" else 0
    grow = 2 * pml + 1 if pml else 0               # stored cells beyond the interior
    nx, ny, nz = 35 - grow, 29 - grow, 8 * layers - 3 - grow
    d = (0.1, 0.12, 0.09)
    per = 0 if pml else 1
    cfg = pi.make_config3(nx, ny, nz, *d, pml_cells=pml, periodic_x=per, periodic_y=per, periodic_z=per,
                          ck="ck2", theta=0.2, filter_npass=4, filter_compensate=1, real=real, seed=21)
    from paper_1009_2727_amd import Sim
    sim = Sim(cfg, capacity=6000)
    ref = Oracle3(cfg)
    for k, name in enumerate(["Ex", "Ey", "Ez", "Bx", "By", "Bz", "Exo", "Eyo", "Ezo", "Exb", "Eyb", "Ezb"]):
        f = pi.random_field(ref.shape, seed=700 + k, amp=0.4)
        ref.set_field(name, f)
        sim.set_field(name, f)
    p = pi.random_electrons3(4000, nx, ny, nz, d, seed=23, umax=3.0, margin=1.5 if pml else 0.0)
    ref.set_electrons(p)
    sim.load_electrons(p)
    ref.step(1)
    sim.step(1)
    assert sim.sync_status() == 0
    tol = 1e-11 if real == "f64" else 2e-6
    for n in NAMES:
        a, b = sim.field(n), ref.field(n)
        assert np.abs(a - b).max() <= tol * max(np.abs(b).max(), 1.0), (n, float(np.abs(a - b).max()))


# the line for each other reach
LINES = {"f32": {1: 2450, 2: 3200, 3: 2900, 4: 3100, 6: 2800}, "f64": {1: 2300, 2: 2300, 3: 2000, 4: 1650, 6: 1100}}


@gpu
@pytest.mark.parametrize("above", [0, 1])
@pytest.mark.parametrize("reach", [1, 2, 3, 4, 6])
@pytest.mark.parametrize("real", ["f64", "f32"])
def test_3d_filter_around_the_size_line_of_its_reach_matches_oracle(real, reach, above):
    layers = LINES[real][reach] // (3 * 20) + above
    comp = int(reach > 2)
    nx, ny, nz = 35 - 9, 29 - 9, 8 * layers - 3 - 9
    d = (0.1, 0.12, 0.09)
    cfg = pi.make_config3(nx, ny, nz, *d, pml_cells=4, ck="ck2", theta=0.2, filter_npass=reach - comp,
                          filter_compensate=comp, real=real, seed=21)
    from paper_1009_2727_amd import Sim
    sim = Sim(cfg, capacity=6000)
    ref = Oracle3(cfg)
    for k, name in enumerate(["Ex", "Ey", "Ez", "Bx", "By", "Bz"]):
        f = pi.random_field(ref.shape, seed=700 + k, amp=0.4)
        ref.set_field(name, f)
        sim.set_field(name, f)
    p = pi.random_electrons3(4000, nx, ny, nz, d, seed=23, umax=3.0, margin=1.5)
    ref.set_electrons(p)
    sim.load_electrons(p)
    ref.step(1)
    sim.step(1)
    assert sim.sync_status() == 0
    tol = 1e-11 if real == "f64" else 2e-6
    for n in NAMES:
        a, b = sim.field(n), ref.field(n)
        assert np.abs(a - b).max() <= tol * max(np.abs(b).max(), 1.0), (n, float(np.abs(a - b).max()))
