"""Particle tiles beside the default ones against the FP64 oracle: the sizes where the staged tile is
just long enough or not, for drifting ions and for electrons, and the largest.  A boosted run with
laser, window and rigid ions, the tiles sorted and stepped until the particles have drifted by
several cells.  Tolerances as in the parity tests (FP64 1e-10, FP32 1e-5 of the field scales).
"""
import pytest

import pic_inputs as pi
from oracle import Oracle
from oracle.pic3 import Oracle3

gpu = pytest.mark.gpu


@gpu
@pytest.mark.parametrize("real,tol", [("f64", 1e-10), ("f32", 1e-5)])
@pytest.mark.parametrize("tile", [(26, 15), (26, 20), (26, 21), (16, 24), (26, 25), (26, 26), (26, 64), (64, 25)])
def test_2d_tile_sizes_match_oracle(tile, real, tol):
    from paper_1009_2727_amd import Sim
    from test_gpu_parity import compare_fields, compare_particles
    w = pi.small_boosted(real=real, nx=40, nz=160, ppc=3)
    sim, ref = Sim.from_workload(w, tile=tile, sort_every=6), Oracle.from_workload(w)
    sim.step(10)
    ref.step(10)
    assert sim.sync_status() == 0
    compare_fields(sim, ref, tol, tag=f"tile {tile} {real}")
    if real == "f64":
        compare_particles(sim, ref, 1e-9, 1e-9)
        compare_particles(sim, ref, 1e-9, 1e-9, species=1)


@gpu
def test_batch_of_unlike_tiles_matches_oracle():
    # one launch for runs whose tiles ask for different rows
    from paper_1009_2727_amd import Batch, Sim
    from test_gpu_parity import compare_fields
    w = [pi.small_boosted(real="f32", nx=40, nz=n, ppc=3, seed=70 + n) for n in (120, 160)]
    sims = [Sim.from_workload(v, tile=t, sort_every=6) for v, t in zip(w, ((26, 8), (16, 24)))]
    batch = Batch(sims)
    batch.step(10)
    for v, s in zip(w, sims):
        ref = Oracle.from_workload(v)
        ref.step(10)
        assert s.sync_status() == 0
        compare_fields(s, ref, 1e-5, tag="batch of unlike tiles")


@gpu
@pytest.mark.parametrize("real,tol", [("f64", 1e-10), ("f32", 1e-5)])
@pytest.mark.parametrize("tile_z", [3, 7, 8, 9, 14, 15, 24])
def test_3d_tile_sizes_match_oracle(tile_z, real, tol):
    from paper_1009_2727_amd import Sim
    from test_gpu_parity3 import compare_fields3, compare_particles3
    w = pi.small_boosted3(real=real, nx=10, ny=8, nz=52, ppc=2)
    sim, ref = Sim.from_workload(w, tile=(0, tile_z), sort_every=6), Oracle3.from_workload(w)
    sim.step(10)
    ref.step(10)
    assert sim.sync_status() == 0
    compare_fields3(sim, ref, tol)
    if real == "f64":
        compare_particles3(sim, ref, 1e-9, 1e-9)


@gpu
@pytest.mark.parametrize("real,tol", [("f64", 1e-10), ("f32", 1e-5)])
@pytest.mark.parametrize("tile,gather", [((64, 64), 0), ((64, 64), 1), ((13, 64), 0), ((64, 8), 1)])
def test_tiles_of_several_windows_match_oracle(tile, gather, real, tol):
    # more particles beside the first window than the list may keep, in up to three windows an axis
    from paper_1009_2727_amd import Batch, Sim
    from test_gpu_parity import compare_fields, compare_particles
    w = pi.small_boosted(real=real, nx=72, nz=160, ppc=6)
    w["config"]["gather_kind"] = gather
    sim, ref = Sim.from_workload(w, tile=tile, sort_every=6), Oracle.from_workload(w)
    sim.step(10)
    ref.step(10)
    assert sim.sync_status() == 0
    compare_fields(sim, ref, tol, tag=f"windows of tile {tile} {real}")
    if real == "f64":
        compare_particles(sim, ref, 1e-9, 1e-9)
    elif gather == 0:
        one = Sim.from_workload(w, tile=tile, sort_every=6)
        Batch([one]).step(10)
        assert one.sync_status() == 0
        compare_fields(one, ref, tol, tag=f"windows of tile {tile} in a batch")


@gpu
@pytest.mark.parametrize("tile,nz", [((4, 2), 160), ((27, 1), 400)])
@pytest.mark.parametrize("gather", [0, 1])
def test_many_fp64_segments_match_oracle(tile, nz, gather):
    # more than three segments a CU, in tiles that fit the staged one and that do not
    from paper_1009_2727_amd import Sim
    from test_gpu_parity import compare_fields, compare_particles
    w = pi.small_boosted(real="f64", nx=40, nz=nz, ppc=3)
    w["config"]["gather_kind"] = gather
    sim, ref = Sim.from_workload(w, tile=tile, sort_every=6), Oracle.from_workload(w)
    sim.step(10)
    ref.step(10)
    assert sim.sync_status() == 0
    compare_fields(sim, ref, 1e-10, tag=f"many segments of tile {tile}")
    compare_particles(sim, ref, 1e-9, 1e-9)
    compare_particles(sim, ref, 1e-9, 1e-9, species=1)


@gpu
@pytest.mark.parametrize("real,tol,xtol,utol", [("f64", 1e-11, 1e-9, 1e-9), ("f32", 1e-5, 2e-5, 1e-4)])
@pytest.mark.parametrize("umax", [0.3, 6.0])
def test_spread_electrons_in_default_tiles_match_oracle(umax, real, tol, xtol, utol):
    # stepped with no sort until a segment's electrons lie in many windows: a few beside the first one
    # (the list as it is) and most of them (window after window, across a periodic edge too)
    from paper_1009_2727_amd import Sim
    from test_gpu_parity import compare_fields, compare_particles
    nx, nz = 60, 53
    cfg = pi.make_config(nx, nz, 0.1, 0.13, periodic_x=1, periodic_z=1, pml_cells=0, ck="ck2",
                         theta=0.3, filter_npass=2, filter_compensate=1, real=real, seed=6)
    sim, ref = Sim(cfg, capacity=30000, sort_every=1000), Oracle(cfg)
    for k, name in enumerate(["Ex", "Ey", "Ez", "Bx", "By", "Bz", "Exo", "Eyo", "Ezo", "Exb", "Eyb", "Ezb"]):
        f = pi.random_field(ref.shape, seed=300 + k, amp=0.2)
        ref.set_field(name, f)
        sim.set_field(name, f)
    p = pi.random_electrons(20000, nx, nz, 0.1, 0.13, seed=12, umax=umax, margin=0.0)
    ref.set_electrons(p)
    sim.load_electrons(p)
    ref.step(12)
    sim.step(12)
    assert sim.sync_status() == 0
    compare_fields(sim, ref, tol, tag=f"spread over windows {umax} {real}")
    compare_particles(sim, ref, xtol, utol)
