"""Phase timers: every phase of a 2D and of a 3D step is bracketed once a step.

On the HIP runtime without a device (tests/host_hip.c), whose events are a millisecond apart.
"""
import pytest

from test_launch_limits import CHILD, ROOT, _child, fake  # noqa: F401

TIMERS = CHILD + r"""
real, dim = sys.argv[3], int(sys.argv[4])
w = (pi.small_boosted3(real=real, nx=10, ny=8, nz=40, ppc=1) if dim == 3 else
     pi.small_boosted(real=real, nx=24, nz=40, ppc=1))
make = P.make_config
P.make_config = lambda cfg, cap: make(cfg, 200000, timers=True)
r = Run(w["config"])
P.make_config = make
assert P.lib().bf_init_plasma(r.h, C.byref(P.bf_plasma(**w["plasma"]))) == 0
assert P.lib().bf_init_laser(r.h, C.byref(P.bf_laser(**w["laser"]))) == 0
for _ in range(3):
    assert r.step() == 0
t = np.zeros((len(P.PHASES), 2))
assert P.lib().bf_diagnose(r.h, P.DIAG_TIMERS, 1, t.ctypes.data_as(C.c_void_p), t.nbytes) == 0
for name, (ms, n) in zip(P.PHASES, t):
    want = {"sort": (0, 3), "beam": (0,)}.get(name, (3,))
    assert n in want and ms == n, (name, ms, n)
print("ok")
"""


@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("dim", [2, 3])
def test_every_phase_has_its_own_row(fake, dim, real):  # noqa: F811
    assert "ok" in _child(TIMERS, fake, ROOT, real, str(dim))
