"""Strided current filters against the FP64 oracle where the line filter changes its form.

Away from the ends of an axis the passes are applied as one stencil, at the ends of a non-periodic
axis pass by pass, and short axes are not split.  One step from random fields and random electrons,
then E, B and the filtered current are compared cell by cell: several segments along z, with PML and
periodic; periodic axes shorter than the stencil, which keep the passes; a z axis one cell below and at the length from which it is split; the largest stride, where
only z takes the stencil; and the same along the three axes of a 3D box.  Tolerances as in the other
filter tests (FP64 1e-11, FP32 2e-6 of the field scale).
"""
import numpy as np
import pytest

import pic_inputs as pi
from oracle import Oracle
from oracle.pic3 import Oracle3

gpu = pytest.mark.gpu
SEEDED = ["Ex", "Ey", "Ez", "Bx", "By", "Bz", "Exo", "Eyo", "Ezo", "Exb", "Eyb", "Ezb"]
NAMES = SEEDED[:6] + ["Jx", "Jy", "Jz"]


def _step_and_compare(cfg, ref, p, real):
    from paper_1009_2727_amd import Sim
    sim = Sim(cfg, capacity=4000)
    for k, name in enumerate(SEEDED):
        f = pi.random_field(ref.shape, seed=700 + k, amp=0.4)
        ref.set_field(name, f)
        sim.set_field(name, f)
    ref.set_electrons(p)
    sim.load_electrons(p)
    ref.step(1)
    sim.step(1)
    assert sim.sync_status() == 0
    tol = 1e-11 if real == "f64" else 2e-6
    for n in NAMES:
        a, b = sim.field(n), ref.field(n)
        assert np.abs(a - b).max() <= tol * max(np.abs(b).max(), 1.0), (n, float(np.abs(a - b).max()))


@gpu
@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("npass,comp,mask", [(4, 1, 0b11), (2, 1, 0b1000), (1, 1, 0b10000), (1, 0, 1 << 15)])
@pytest.mark.parametrize("geom", ["pml", "periodic", "narrow", "below", "at"])
def test_2d_strided_filter_matches_oracle(geom, npass, comp, mask, real):
    per = int(geom in ("periodic", "narrow"))
    pml = 0 if per else 4
    reach = (npass + comp) * sum(k + 1 for k in range(16) if mask >> k & 1)
    nz = {"pml": 411, "periodic": 333, "narrow": 30}.get(geom, 2 * (reach + 1) + 16 - (2 * pml + 1) - (geom == "below"))
    nx = 7 if geom == "narrow" else 45
    cfg = pi.make_config(nx, nz, 0.1, 0.09, pml_cells=pml, periodic_x=per, periodic_z=per, ck="ck2", theta=0.2,
                         filter_npass=npass, filter_compensate=comp, real=real, seed=21, filter_strides=mask)
    _step_and_compare(cfg, Oracle(cfg), pi.random_electrons(3000, nx, nz, 0.1, 0.09, seed=23, umax=3.0,
                                                            margin=0.0 if per else 1.5), real)


@gpu
@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("per", [0, 1])
def test_3d_strided_filter_matches_oracle(per, real):
    n, d = (41, 60, 83), (0.1, 0.12, 0.09)
    cfg = pi.make_config3(*n, *d, pml_cells=0 if per else 4, periodic_x=per, periodic_y=per, periodic_z=per,
                          ck="ck2", theta=0.2, filter_npass=2, filter_compensate=1, real=real, seed=21,
                          filter_strides=0b11)
    _step_and_compare(cfg, Oracle3(cfg), pi.random_electrons3(3000, *n, d, seed=23, umax=3.0,
                                                              margin=0.0 if per else 1.5), real)


# Reaches whose end segments would not fit the LDS in FP64 (10 passes and compensation of strides 1
# to 4: 110; 7 and compensation of stride 16: 128), on axes long enough for end segments.  The filtered
# current is hundreds of times smaller than the raw one here, so its tolerance is of the raw scale: the
# passes in FP32 err by 4e-8 of it.  The residual div E - F[rho] is filtered in FP64 in both types and
# carries the tolerance of E over up to six differences.
LONG = [(10, 1, 0b1111, 110), (7, 1, 1 << 15, 128)]


def _long_reach(cfg, ref, p, real, dmin):
    from paper_1009_2727_amd import Sim
    sim = Sim(cfg, capacity=4000)
    for k, name in enumerate(SEEDED):
        f = pi.random_field(ref.shape, seed=700 + k, amp=0.4)
        ref.set_field(name, f)
        sim.set_field(name, f)
    ref.set_electrons(p)
    sim.load_electrons(p)
    ref.step(1)
    sim.step(1)
    assert sim.sync_status() == 0
    tol = 1e-11 if real == "f64" else 2e-6
    for n in NAMES[:6]:
        a, b = sim.field(n), ref.field(n)
        assert np.abs(a - b).max() <= tol * max(np.abs(b).max(), 1.0), (n, float(np.abs(a - b).max()))
    tol_j = 1e-11 if real == "f64" else 5e-7
    raw = max(np.abs(sim.field(n + "r")).max() for n in NAMES[6:])
    for n in NAMES[6:]:
        d = float(np.abs(sim.field(n) - ref.field(n)).max())
        assert d <= tol_j * raw, (n, d, float(raw))
    inner = (slice(1, -1),) * len(ref.shape)
    d = float(np.abs(sim.gauss_residual() - ref.gauss_residual())[inner].max())
    assert d <= 6 * tol / dmin, d


@gpu
@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("npass,comp,mask,reach", LONG)
def test_2d_long_reach_matches_oracle(npass, comp, mask, reach, real):
    nx, nz = 31, 2 * (reach + 1) + 70
    cfg = pi.make_config(nx, nz, 0.1, 0.09, pml_cells=4, ck="ck2", theta=0.2, filter_npass=npass,
                         filter_compensate=comp, real=real, seed=21, filter_strides=mask)
    _long_reach(cfg, Oracle(cfg), pi.random_electrons(3000, nx, nz, 0.1, 0.09, seed=23, umax=3.0, margin=1.5), real,
                0.09)


@gpu
@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("axis", [1, 2])
@pytest.mark.parametrize("npass,comp,mask,reach", LONG)
def test_3d_long_reach_matches_oracle(npass, comp, mask, reach, axis, real):
    n, d = [9, 9, 9], (0.1, 0.12, 0.09)
    n[axis] = 2 * (reach + 1) + 20
    cfg = pi.make_config3(*n, *d, pml_cells=4, ck="ck2", theta=0.2, filter_npass=npass, filter_compensate=comp,
                          real=real, seed=21, filter_strides=mask)
    p = pi.random_electrons3(3000, *n, d, seed=23, umax=3.0, margin=1.5)
    p["w"] *= 1e-3                       # a charge density of order one
    _long_reach(cfg, Oracle3(cfg), p, real, 0.09)


# Sizes on either side of the lengths from which an axis that is not periodic takes the stencil (8
# cells of it a cell of reach; y in FP64 with eight passes or more)
@gpu
@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("npass,comp,mask", [(4, 1, 0b11), (1, 0, 0b11), (10, 1, 0b1111)])
@pytest.mark.parametrize("above", [0, 1])
def test_2d_stencil_from_its_length_matches_oracle(above, npass, comp, mask, real):
    reach = (npass + comp) * sum(k + 1 for k in range(16) if mask >> k & 1)
    n = 8 * reach - 1 + above                      # stored cells, layers of 4 on both sides
    for nx, nz in ((n - 9, 40), (9, n - 9)):
        cfg = pi.make_config(nx, nz, 0.1, 0.09, pml_cells=4, ck="ck2", theta=0.2, filter_npass=npass,
                             filter_compensate=comp, real=real, seed=21, filter_strides=mask)
        _long_reach(cfg, Oracle(cfg), pi.random_electrons(3000, nx, nz, 0.1, 0.09, seed=23, umax=3.0, margin=1.5),
                    real, 0.09)


@gpu
@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("npass,comp,mask", [(4, 1, 0b11), (2, 1, 0b11), (1, 0, 0b11)])
@pytest.mark.parametrize("above", [0, 1])
def test_3d_stencil_from_its_length_matches_oracle(above, npass, comp, mask, real):
    d = (0.1, 0.12, 0.09)
    n = max(8 * 3 * (npass + comp) - 1 + above - 9, 6)
    for box in ((9, n, 10), (9, 10, n)):
        cfg = pi.make_config3(*box, *d, pml_cells=4, ck="ck2", theta=0.2, filter_npass=npass, filter_compensate=comp,
                              real=real, seed=21, filter_strides=mask)
        _step_and_compare(cfg, Oracle3(cfg), pi.random_electrons3(3000, *box, d, seed=23, umax=3.0, margin=1.5), real)
