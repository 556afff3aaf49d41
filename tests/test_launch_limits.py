"""Launches within the limits of a CU, over the filters that a configuration may ask for.

The library runs on a HIP runtime without a device (tests/host_hip.c) that records what each launch
asks for.  Every reach of the strided current filter up to its limit of 128 cells, along each axis,
in both precisions and at the lengths where the line filter changes its segments, has to fit the
160 KB of LDS, in the step and in the Gauss diagnostic, which filters in FP64.
"""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

CHILD = r"""
import ctypes as C, itertools, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
fake.host_hip_max_lds.restype = C.c_size_t
fake.host_hip_launches.restype = C.c_long
sys.path.insert(0, sys.argv[2])
import numpy as np
import paper_1009_2727_amd as P
import pic_inputs as pi

class Run:
    def __init__(self, cfg):
        c = P.make_config(cfg, 64)
        self.keep, bind = [], []
        for name, n, align in P.bf_query_buffers(c):
            b = np.zeros(n + align, dtype=np.uint8)
            self.keep.append(b)
            bind.append((name, -(-b.ctypes.data // align) * align, n))
        self.h = P.bf_create(c, bind, 0)
        i = P.bf_info()
        assert self.diagnose(P.DIAG_INFO, C.byref(i), C.sizeof(i)) == 0
        self.cells = i.stored_x * i.stored_z * max(i.stored_y, 1)
    def diagnose(self, kind, p, n):
        return P.lib().bf_diagnose(self.h, kind, 0, p, n)
    def step(self):
        return P.lib().bf_step(self.h, 1)
    def gauss(self):
        out = np.empty(self.cells)
        return self.diagnose(P.DIAG_GAUSS, out.ctypes.data_as(C.c_void_p), out.nbytes)
    def close(self):
        P.lib().bf_destroy(self.h)
"""

REACHES = CHILD + r"""
def filters(reach):
    # (passes, compensation, strides) of that reach: the largest strides once each, and the most passes
    # of the smallest strides that make it up
    once, left = 0, reach
    for s in range(16, 0, -1):
        if s <= left:
            once |= 1 << (s - 1)
            left -= s
    out = [(1, 0, once)]
    for k in range(11, 1, -1):
        total, m = reach // k, 0
        while (m + 1) * (m + 2) // 2 <= total:
            m += 1
        last = total - m * (m - 1) // 2
        if reach % k == 0 and last <= 16 and k * m <= 48:
            return out + [(k - 1, 1, (1 << (m - 1)) - 1 | 1 << (last - 1))]
    return out

real, axis = sys.argv[3], sys.argv[4]
P4 = 9                                   # stored cells beyond the interior with layers of 4
runs = 0
for reach in range(1, 129):
    edge = reach + 1
    for stored, (npass, comp, mask) in itertools.product((2 * edge + 15, 2 * edge + 16, 8 * reach + 8, 1200),
                                                         filters(reach)):
        n = stored - P4
        kw = dict(pml_cells=4, ck="yee", filter_npass=npass, filter_compensate=comp, real=real, filter_strides=mask)
        small = 5
        if axis in ("x2", "z2"):
            cfg = pi.make_config(n if axis == "x2" else small, n if axis == "z2" else small, 0.1, 0.1, **kw)
        else:
            dims = {a: (n if a == axis else small) for a in "xyz"}
            cfg = pi.make_config3(dims["x"], dims["y"], dims["z"], 0.1, 0.1, 0.1, **kw)
        r = Run(cfg)
        fake.host_hip_reset()
        assert r.step() == 0, (reach, stored, fake.host_hip_max_lds())
        assert r.gauss() == 0, (reach, stored, fake.host_hip_max_lds())
        assert 0 < fake.host_hip_max_lds() <= 160 * 1024, (reach, stored, fake.host_hip_max_lds())
        r.close()
        runs += 1
print("runs", runs)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    import paper_1009_2727_amd as P
    if not os.path.exists(P.LIB_PATH):
        pytest.skip("libbfpic.so not built")
    so = tmp_path_factory.mktemp("hip") / "host_hip.so"
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", str(so), os.path.join(HERE, "host_hip.c")])
    return str(so)


def _child(script, *args):
    r = subprocess.run([sys.executable, "-c", script, *args], capture_output=True, text=True, timeout=900)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout


@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("axis", ["x2", "z2", "x", "y", "z"])
def test_line_filter_fits_the_lds_at_every_reach(fake, axis, real):
    runs = int(_child(REACHES, fake, ROOT, real, axis).split()[-1])
    assert runs >= 4 * 128


FAILED = CHILD + r"""
for cfg in (pi.make_config3(8, 8, 8, 0.1, 0.1, 0.1, pml_cells=4, filter_npass=1, real=sys.argv[3]),
            pi.make_config(8, 8, 0.1, 0.1, pml_cells=4, filter_npass=1, real=sys.argv[3])):
    r = Run(cfg)
    assert r.gauss() == 0
    fake.host_hip_fail(1)
    assert r.gauss() == -5, "a launch failed and the residual was returned"
    fake.host_hip_fail(0)
    assert fake.hipGetLastError() == 0, "the error was left for a later call"
    r.close()
print("ok")
"""


@pytest.mark.parametrize("real", ["f64", "f32"])
def test_gauss_residual_reports_a_failed_launch(fake, real):
    assert "ok" in _child(FAILED, fake, ROOT, real)
