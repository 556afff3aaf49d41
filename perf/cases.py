"""Performance cases: what a user of the library has it do, through its public entry points.

A case is a dict of plain values.  "kind" is one of

* "run": `steps` PIC steps of one simulation (Sim.step).  A boosted run (gamma > 1) is a stage
  under way: the moving window is filled with plasma streaming through it and the laser pulse is
  being emitted inside it; a lab-frame run (gamma = 1) is a pulse entering plasma at rest.
  The tile sort runs at its default cadence, once every 20 steps, so 20 steps hold one.
  Single-precision runs are periodic across the box, double-precision ones have absorbing
  layers on every face: where plasma at rest touches an absorbing face, the particles within a
  rounding error of it are lost or kept by chance, and each one lost leaves its ion behind.
* "scan": the same for several independent boosted runs stepped together (Batch.step).
* "apply" and "train": the learned current filter on a stack of images (LearnedFilter).

A run returns the updated fields E and B where they lie, in the library's storage order (the z
rows are a ring that moves with the window).  The particles have no order that could be compared:
they are kept in tiles, in the order the sort's atomics left them; every one of them is in the
fields through its current.

exact() follows the method in FP64 with plain torch operations on whole arrays, from the same
seed, with no tiles, no sort and no reduced precision.
"""
import math

import numpy as np
import torch

import paper_1009_2727_amd as pic

CK = {"yee": (1.0, 0.0, 0.0), "ck": (7 / 12, 1 / 12, 1 / 48), "ck2": (19 / 24, 1 / 24, 1 / 96)}
LAMBDA_UM = 0.8
C_UM_FS = 0.299792458
LAB_CELL_UM = 0.05
WARM_STEPS = 20          # steps a run has behind it when it is handed over


def _run(dim, nx, nz, ppc, *, ny=1, gamma=13.0, real="f32", steps=20, passes=4, compensate=1, strides=1,
         learned=False, solver="ck2", theta=0.1, momentum_conserving=False, vay=False, periodic=None, **more):
    periodic = real == "f32" if periodic is None else periodic
    return dict(kind="run", dim=dim, nx=nx, ny=ny, nz=nz, ppc=ppc, gamma=gamma, real=real, steps=steps,
                passes=passes, compensate=compensate, strides=strides, learned=learned, solver=solver, theta=theta,
                momentum_conserving=momentum_conserving, vay=vay, periodic=periodic, **more)


def _lab(nx, nz, ppc, **more):
    return _run(2, nx, nz, ppc, gamma=1.0, solver="yee", theta=0.0, periodic=True, **more)


def listed():
    return [
        # the smallest run: a check of a set-up, stepped a little at a time in double precision
        dict(_run(2, 32, 96, 2, real="f64", steps=2), name="2D tiny f64"),
        # the lab-frame stage the double-precision checks are made on
        dict(_lab(64, 512, 4, real="f64", passes=1, compensate=0), name="2D lab stage f64"),
        # the scaled stage of the beam studies: one particle a cell, hundreds to tens of thousands of steps
        dict(_run(2, 75, 1691, 1, gamma=5.0, solver="yee", theta=0.0), name="2D scaled stage f32"),
        # the time-step scans of the instability: momentum-conserving gather, Vay's pusher, a wideband filter
        dict(_run(2, 187, 1531, 5, gamma=30.0, solver="ck", theta=0.0, strides=3, momentum_conserving=True, vay=True),
             name="2D nodal gather, Vay, S(1:2)"),
        # a production 2D run (the 2D throughput workload)
        dict(_run(2, 256, 4096, 16), name="2D boosted stage f32"),
        # a mid-size 2D run with the learned filter in place of the bilinear one
        dict(_run(2, 128, 2048, 4, learned=True), name="2D learned filter run"),
        # a scan over boost, density and grid
        dict(kind="scan", runs=16, nx=192, nz=2560, ppc=10, steps=20, name="scan of 16 runs"),
        # a small 3D check in double precision
        dict(_run(3, 12, 48, 2, ny=10, gamma=30.0, real="f64", steps=2), name="3D tiny f64"),
        # a 3D run of ordinary size on ragged extents with the momentum-conserving gather
        dict(_run(3, 61, 203, 4, ny=45, gamma=30.0, momentum_conserving=True), name="3D ragged, nodal gather"),
        # a production 3D run (the 3D throughput workload)
        dict(_run(3, 128, 1024, 8, ny=128, gamma=30.0), name="3D boosted stage f32"),
        # the trained filter on the three currents of a large 2D grid
        dict(kind="apply", images=3, ny=4117, nx=277, periodic=False, name="learned filter"),
        # a step of the filter's training on a batch of patches
        dict(kind="train", images=128, ny=32, nx=32, margin=6, name="learned filter training"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_run(rng, dim):
    real = "f64" if rng.random() < 0.3 else "f32"
    budget = (60e6 if dim == 3 else 17e6) / (4 if real == "f64" else 1)    # electrons
    while True:
        if dim == 2:
            nx, ny, nz, ppc = _log(rng, 24, 256), 1, _log(rng, 90, 4096), _log(rng, 1, 16)
        else:
            nx, ny, nz, ppc = _log(rng, 10, 128), _log(rng, 10, 128), _log(rng, 40, 1024), _log(rng, 1, 8)
        if nx * ny * nz * ppc <= budget:
            break
    kw = dict(real=real, steps=20 if rng.random() < 0.8 else 2)
    kw["passes"], kw["compensate"] = rng.choice([(4, 1), (4, 1), (4, 1), (1, 0), (2, 1), (0, 0)])
    if kw["passes"] == 4 and rng.random() < 0.25:
        kw["strides"] = rng.choice([0b11, 0b111, 0b1011])
    kw["momentum_conserving"] = rng.random() < 0.2
    kw["vay"] = rng.random() < 0.2
    if dim == 2 and rng.random() < 0.25:
        return _lab(nx, nz, ppc, **kw)
    kw["gamma"] = math.exp(rng.uniform(math.log(5.0), math.log(60.0)))
    kw["solver"] = rng.choice(["ck2", "ck2", "ck", "yee"])
    kw["theta"] = rng.choice([0.1, 0.1, 0.0])
    if real == "f64":
        kw["periodic"] = rng.random() < 0.25
    if dim == 2 and real == "f32" and rng.random() < 0.2:
        kw["learned"], kw["strides"] = True, 1
    return _run(dim, nx, nz, ppc, ny=ny, **kw)


def draw(rng):
    u = rng.random()
    if u < 0.45:
        return _draw_run(rng, 2)
    if u < 0.70:
        return _draw_run(rng, 3)
    if u < 0.80:
        return dict(kind="scan", runs=rng.randint(2, 16), nx=_log(rng, 64, 192), nz=_log(rng, 512, 2560),
                    ppc=rng.randint(4, 12), steps=20)
    if u < 0.92:
        return dict(kind="apply", images=rng.randint(1, 6), ny=_log(rng, 64, 4117), nx=_log(rng, 32, 300),
                    periodic=rng.random() < 0.5)
    return dict(kind="train", images=_log(rng, 16, 512), ny=rng.randint(24, 48), nx=rng.randint(24, 48), margin=6)


# ---- the workloads -----------------------------------------------------------------------------


def _workload(c, seed):
    """(config, plasma, laser) of a "run" case, as the library's set-up calls take them."""
    g = c["gamma"]
    beta = math.sqrt(1.0 - 1.0 / (g * g))
    lab = g == 1.0
    # the cell is a fixed fraction of the Doppler-stretched wavelength
    d = LAB_CELL_UM if lab else (1.0 + beta) * g * LAMBDA_UM / (16.0 if c["dim"] == 3 else 32.0)
    a, b, cc = CK[c["solver"]]
    config = dict(dim=c["dim"], nx=c["nx"], nz=c["nz"], dx_um=d, dz_um=d, pml_cells=10,
                  periodic_x=int(c["periodic"]), periodic_z=0, ck_alpha=a, ck_beta=b, ck_gamma=cc,
                  theta=c["theta"], cfl_fraction=0.95, filter_npass=c["passes"], filter_compensate=c["compensate"],
                  filter_strides=c["strides"], gamma_boost=g, moving_window=0 if lab else 1, seed=seed,
                  real=c["real"], gather_kind=int(c["momentum_conserving"]), pusher=int(c["vay"]),
                  filter_kind=pic.FILTER_LEARNED if c["learned"] else pic.FILTER_BILINEAR)
    if c["dim"] == 3:
        config.update(ny=c["ny"], dy_um=d, periodic_y=int(c["periodic"]))
    # the faster the frame, the thinner the plasma of the stages it is used for
    n0 = 1e19 if lab else c.get("density", 1.0) * 1e18 * (13.0 / g) ** 2
    z_ant = 0.5 if lab else g * 0.6 * c["nz"] * d
    plasma = dict(n0_cm3=n0, ramp_um=0.0, start_um=1.0 if lab else -1e30, ppc=c["ppc"], ion_mode=0 if lab else 1)
    # the pulse is at its peak: the emission starts one optical period before it
    laser = dict(lambda_um=LAMBDA_UM, a0=1.0 if lab else 2.0, waist_um=0.3 * c["nx"] * d, fwhm_fs=10.0 if lab else 50.0,
                 z_antenna_um=z_ant, t_peak_fs=LAMBDA_UM / C_UM_FS, pol=0)
    return config, plasma, laser


def _scan_runs(c, seed):
    """The runs of a "scan" case: grid, boost, density and particles vary from run to run."""
    r = np.random.default_rng(1000 + c["runs"])      # the same scan for every seed; the plasma differs
    out = []
    for q in range(c["runs"]):
        nx, nz = int(c["nx"] * r.uniform(0.5, 1.0)), int(c["nz"] * r.uniform(0.25, 1.0))
        gamma = float(np.exp(r.uniform(np.log(5.0), np.log(50.0))))
        out.append((_run(2, nx, nz, max(1, int(c["ppc"] * r.uniform(0.4, 1.6))), gamma=gamma,
                         density=float(r.uniform(0.3, 1.0))), seed + 7919 * q))
    return out


def _start(c, seed):
    config, plasma, laser = _workload(c, seed)
    # room for the rows that enter between two sorts (less than two a step) beside the filled window
    capacity = c["nx"] * c["ny"] * (c["nz"] + 2 * WARM_STEPS + 8) * c["ppc"] + 4096
    sim = pic.Sim(config, capacity=capacity, ppc=c["ppc"])
    sim.init_plasma(plasma)
    sim.init_laser(laser)
    if c["learned"]:
        sim.set_learned_filter(_filter_weights(seed))
    return sim


def _filter_weights(seed):
    """Weights of a trained filter, layout W1[25][16], W2[25][16][16], W3[25][16]: a smoothing
    path (binomial taps through channel 0) plus the small weights of the other channels."""
    r = np.random.default_rng(seed)
    w1 = 0.02 * r.standard_normal((25, 16))
    w2 = 0.005 * r.standard_normal((25, 16, 16))
    w3 = 0.02 * r.standard_normal((25, 16))
    t = np.array([0.0, 0.25, 0.5, 0.25, 0.0])
    taps = np.outer(t, t).ravel()
    w1[:, 0] += taps
    w2[:, 0, 0] += taps
    w3[:, 0] += taps
    return np.concatenate([w1.ravel(), w2.ravel(), w3.ravel()]).astype(np.float32)


def _images(c, seed, device):
    g = torch.Generator(device=device).manual_seed(seed)
    return torch.randn((c["images"], c["ny"], c["nx"]), generator=g, device=device, dtype=torch.float32)


def _adam_moments(seed):
    """Moments of a training that has run for a while."""
    r = np.random.default_rng(seed + 1)
    m = 1e-3 * r.standard_normal(pic.LF_PARAMS)
    return m.astype(np.float32), (1e-6 * (0.5 + r.random(pic.LF_PARAMS))).astype(np.float32)


ADAM_STEP, ADAM_LR = 40, 2e-4


def prepare(case, seed):
    if case["kind"] == "run":
        sim = _start(case, seed)
        sim.step(WARM_STEPS)
        return dict(case=case, sim=sim, views=_field_views(sim))
    if case["kind"] == "scan":
        sims = [_start(c, s) for c, s in _scan_runs(case, seed)]
        batch = pic.Batch(sims)
        batch.step(WARM_STEPS)
        return dict(case=case, batch=batch, views=[_field_views(s) for s in sims])
    device = torch.device("cuda", torch.cuda.current_device())
    lf = pic.LearnedFilter(_filter_weights(seed))
    state = dict(case=case, filter=lf, images=_images(case, seed, device))
    if case["kind"] == "train":
        state["targets"] = torch.nn.functional.avg_pool2d(state["images"], 3, 1, 1).contiguous()
        m, v = _adam_moments(seed)
        lf.m.copy_(torch.from_numpy(m))
        lf.v.copy_(torch.from_numpy(v))
        lf.t = ADAM_STEP - 1
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "run":
        state["sim"].step(case["steps"])
        return state["views"]
    if case["kind"] == "scan":
        state["batch"].step(case["steps"])
        return state["views"]
    lf = state["filter"]
    if case["kind"] == "apply":
        return lf.apply(state["images"], periodic=(case["periodic"], case["periodic"]))
    loss, grad = lf.train_step(state["images"], state["targets"], case["margin"], ADAM_LR, want_grad=True)
    return dict(loss=loss, grad=grad, params=lf.params, m=lf.m, v=lf.v)


def _field_views(sim):
    """The current E and B of a run with an even number of steps behind it: [component][z][y][x] in
    storage order, without the row padding.  Every row is padded to 256 bytes."""
    real = int(sim.cfg.real_bytes)
    sz, sy, sx = sim.shape if sim.dim == 3 else (sim.shape[0], 1, sim.shape[1])
    pitch = -(-sx * real // 256) * 256 // real
    n = sz * sy * pitch
    f = sim.buffers["fields"].view(torch.float32 if real == 4 else torch.float64)

    def vector(first):
        a = f[first * n:(first + 3) * n].view(3, sz, sy, pitch)[..., :sx]
        return a if sim.dim == 3 else a[:, :, 0]

    return dict(E=vector(0), B=vector(9 if sim.dim == 3 else 12))


def work(case):
    """Bytes: the particle state read and written, the field and current words of the cells, per
    step; the images read and written.  Operations: the interpolation, push and deposit of each
    electron, the deposit of each ion and the stencils of each cell; the filter's products."""
    if case["kind"] == "scan":
        parts = [work(c) for c, _ in _scan_runs(case, 0)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    if case["kind"] == "run":
        r, dim = (8 if case["real"] == "f64" else 4), case["dim"]
        cells = case["nx"] * case["ny"] * case["nz"]
        n = cells * case["ppc"]
        ions = 0 if case["gamma"] == 1.0 else n
        by = n * (2 * 8 * dim + 7 * r) + ions * (8 * dim + r) + cells * 51 * r
        fl = n * (3000 if dim == 3 else 700) + ions * (300 if dim == 3 else 100) + cells * (400 if dim == 3 else 150)
        if case["learned"]:
            fl += 3 * 14400 * cells
        return {"bytes": case["steps"] * by, "flops": case["steps"] * fl}
    px = case["images"] * case["ny"] * case["nx"]
    k = 3 if case["kind"] == "train" else 1      # forward, and back through inputs and weights
    return {"bytes": 8 * px + 4 * pic.LF_PARAMS * (1 if k == 1 else 7), "flops": k * 14400 * px}


# ---- the method in FP64 --------------------------------------------------------------------------

MOST_PARTICLE_TAPS = 1.5e10     # about 20 seconds of exact()


def exact(case, seed):
    device = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    if case["kind"] == "apply":
        w = _unpack(_filter_weights(seed), device)
        return _net(_images(case, seed, device).double(), w, case["periodic"])
    if case["kind"] == "train":
        return _exact_train(case, seed, device)
    runs = [(case, seed)] if case["kind"] == "run" else _scan_runs(case, seed)
    steps = WARM_STEPS + case["steps"]
    taps = sum(c["nx"] * c["ny"] * c["nz"] * c["ppc"] * (64 if c["dim"] == 3 else 16) for c, _ in runs) * steps
    if taps > MOST_PARTICLE_TAPS:
        return None
    out = []
    for c, s in runs:
        m = _Method(c, s, device)
        for _ in range(steps):
            m.step()
        out.append(m.outputs())
        del m
    return out[0] if case["kind"] == "run" else out


def _unpack(params, device):
    """The weights as the layers use them (BF16) as convolution kernels [out][in][5][5]."""
    p = torch.from_numpy(params).to(device).bfloat16().double()
    return _kernels(p)


def _kernels(p):
    w1 = p[:400].view(5, 5, 1, 16).permute(3, 2, 0, 1)
    w2 = p[400:6800].view(5, 5, 16, 16).permute(3, 2, 0, 1)
    w3 = p[6800:].view(5, 5, 16, 1).permute(3, 2, 0, 1)
    return [w1, w2, w3]


def _net(x, ws, periodic):
    """Three 5 x 5 convolutions of [n][y][x] images, zeros (or the other side) beyond the edges,
    as sums of shifted products: no library convolution chooses another algorithm here."""
    h = x[:, None]
    per = periodic if isinstance(periodic, tuple) else (periodic, periodic)
    for w in ws:
        ny, nx = h.shape[2:]
        for axis, p in ((2, per[0]), (3, per[1])):
            n = h.shape[axis]
            if p:
                h = h.index_select(axis, torch.arange(-2, n + 2, device=h.device) % n)
            else:
                h = torch.nn.functional.pad(h, (2, 2, 0, 0) if axis == 3 else (0, 0, 2, 2))
        out = 0.0
        for dy in range(5):
            for dx in range(5):
                win = h[:, :, dy:dy + ny, dx:dx + nx].permute(0, 2, 3, 1)
                out = out + win @ w[:, :, dy, dx].t().contiguous()
        h = out.permute(0, 3, 1, 2)
    return h[:, 0]


def _exact_train(case, seed, device):
    x = _images(case, seed, device)
    target = torch.nn.functional.avg_pool2d(x, 3, 1, 1).double()
    p32 = torch.from_numpy(_filter_weights(seed)).to(device)
    p = p32.bfloat16().double().requires_grad_(True)
    mg = case["margin"]
    d = (_net(x.double(), _kernels(p), False) - target)[:, mg:case["ny"] - mg, mg:case["nx"] - mg]
    loss = d.square().mean()
    grad, = torch.autograd.grad(loss, p)
    m, v = (torch.from_numpy(a).to(device).double() for a in _adam_moments(seed))
    m = 0.9 * m + 0.1 * grad
    v = 0.999 * v + 0.001 * grad * grad
    step = (m / (1 - 0.9 ** ADAM_STEP)) / ((v / (1 - 0.999 ** ADAM_STEP)).sqrt() + 1e-8)
    return dict(loss=loss.detach().reshape(1), grad=grad, params=p32.double() - ADAM_LR * step, m=m, v=v)


def _u01(seed, k):
    """SplitMix64: output number k of the generator started at seed, as a double in [0, 1)."""
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + k * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    return (z >> np.uint64(11)).astype(np.float64) / 9007199254740992.0


def _weights(f):
    """Cubic B-spline weights of the nodes j - 1 .. j + 2 at the fraction f of cell j."""
    g = 1.0 - f
    return [g * g * g / 6.0, (3.0 * f * f * f - 6.0 * f * f + 4.0) / 6.0,
            (3.0 * g * g * g - 6.0 * g * g + 4.0) / 6.0, f * f * f / 6.0]


class _Method:
    """One run in FP64.  The fields are [z][y][x]; a 2D run has one periodic y plane, which
    turns every 3D field operator into the 2D one."""

    E_STAGGER = ((1, 0, 0), (0, 1, 0), (0, 0, 1))      # (x, y, z) half-cell offsets of E and J
    B_STAGGER = ((0, 1, 1), (1, 0, 1), (1, 1, 0))

    def __init__(self, c, seed, device):
        config, plasma, laser = _workload(c, seed)
        self.c, self.cfg, self.pl, self.las, self.seed, self.dev = c, config, plasma, laser, seed, device
        two = c["dim"] == 2
        self.axes = (0, 2) if two else (0, 1, 2)
        self.N = [c["nx"], c["ny"], c["nz"]]
        self.d = [config["dx_um"], 1.0 if two else config["dy_um"], config["dz_um"]]
        self.per = [bool(c["periodic"]), two or bool(c["periodic"]), False]
        self.P = [0 if p else config["pml_cells"] for p in self.per]
        self.S = [n if p else n + 2 * q + 1 for n, p, q in zip(self.N, self.per, self.P)]
        self.gamma = c["gamma"]
        self.beta = math.sqrt(1.0 - 1.0 / (self.gamma * self.gamma))
        self.theta = c["theta"]
        self.dt = config["cfl_fraction"] * self._courant()
        z = lambda: [torch.zeros(tuple(reversed(self.S)), dtype=torch.float64, device=device) for _ in range(3)]  # noqa: E731
        self.E, self.Eo, self.Eb, self.B, self.Bo, self.SE, self.SB = (z() for _ in range(7))
        self._layer()
        self.t, self.n, self.shift, self.next_row = 0.0, 0, 0, 0
        unit = 8.8541878128e-12 * 9.1093837015e-31 * 299792458.0 ** 2 / (1.602176634e-19 ** 2 * 1e-12)
        self.n0 = plasma["n0_cm3"] * 1e6 / unit
        self.omega = 2.0 * math.pi / laser["lambda_um"]
        self.e0 = laser["a0"] * self.omega
        self.sig_t = laser["fwhm_fs"] * C_UM_FS / (2.0 * math.sqrt(math.log(2.0)))
        self.t0 = laser["t_peak_fs"] * C_UM_FS
        area = self.d[0] if two else self.d[0] * self.d[1]
        self.aw = (2.0 * self.e0 / self.gamma) * area / 0.01
        self.vw = 0.0
        if config["moving_window"]:
            bw = 1.0 / math.sqrt(1.0 + self.n0 / self.omega ** 2)
            self.vw = (bw - self.beta) / (1.0 - bw * self.beta)
        home = [torch.arange(self.N[a], device=device, dtype=torch.float64) + 0.5 for a in (0, 1)]
        self.home = [h.reshape(-1).contiguous() for h in torch.meshgrid(home[1], home[0], indexing="ij")][::-1]
        if two:
            self.home[1] = torch.zeros_like(self.home[0])
        self.moving = self.home[0].clone()
        none = torch.zeros(0, dtype=torch.float64, device=device)
        self.e = {k: none for k in ("x", "y", "z", "ux", "uy", "uz", "w")}
        self.ion = {k: none for k in ("x", "y", "z", "w")}
        self._inject()

    # -- set-up --
    def _courant(self):
        """The largest stable step: the maximum of the dispersion relation over the corners of the zone."""
        a, b, g = (self.cfg[k] for k in ("ck_alpha", "ck_beta", "ck_gamma"))
        best = 0.0
        for corner in range(1, 8):
            s = [float(corner >> k & 1) for k in range(3)]
            if 1 not in self.axes and s[1]:
                continue
            co = [1.0 - 2.0 * v for v in s]
            rhs = 0.0
            for k in range(3):
                p, q = co[(k + 1) % 3], co[(k + 2) % 3]
                rhs += (a + 2.0 * b * (p + q) + 4.0 * g * p * q) * s[k] / self.d[k] ** 2
            best = max(best, rhs)
        return math.sqrt((2.0 + self.theta) / (2.0 + 3.0 * self.theta)) / math.sqrt(best)

    def _along(self, a, v):
        return v.view([-1 if 2 - a == k else 1 for k in range(3)])

    def _layer(self):
        """Damping factor, curl coefficient and extent of the absorbing layer on each axis and stagger."""
        self.xi, self.co, self.on = {}, {}, {}
        for a in range(3):
            for h in (0, 1):
                p = torch.arange(self.S[a], device=self.dev, dtype=torch.float64) - self.P[a] + 0.5 * h
                depth = torch.clamp(torch.maximum(-p, p - self.N[a]), min=0.0)
                if self.per[a]:
                    depth = torch.zeros_like(depth)
                sig = (4.0 / self.d[a]) * (depth / 5.0) ** 2
                xi = torch.exp(-sig * self.dt)
                co = torch.where(sig > 0, (1.0 - xi) / torch.where(sig > 0, sig, torch.ones_like(sig)),
                                 torch.full_like(sig, self.dt))
                self.xi[a, h], self.co[a, h], self.on[a, h] = (self._along(a, v) for v in (xi, co, sig > 0))

    # -- fields --
    def _shift(self, F, a, o):
        """F at the neighbour o cells along axis a; zero beyond an edge."""
        G = torch.roll(F, -o, dims=2 - a)
        if not self.per[a] and o:
            G.narrow(2 - a, self.S[a] - o if o > 0 else 0, abs(o)).zero_()
        return G

    def _diff(self, F, a, half):
        return (self._shift(F, a, half) - self._shift(F, a, half - 1)) / self.d[a]

    def _wide_diff(self, F, a, half):
        """The tunable solver's difference: alpha at the point, beta and gamma across it."""
        al, be, ga = (self.cfg[k] for k in ("ck_alpha", "ck_beta", "ck_gamma"))
        D = self._diff(F, a, half)
        if be == 0.0 and ga == 0.0:
            return al * D
        p, q = (a + 1) % 3, (a + 2) % 3
        out = al * D
        for s in (-1, 1):
            Ds = self._shift(D, p, s)
            out = out + be * (Ds + self._shift(D, q, s))
            if ga != 0.0:
                out = out + ga * (self._shift(Ds, q, -1) + self._shift(Ds, q, 1))
        return out

    def _split(self, F, part, terms, axes, h, inside):
        """The field's two curl terms, each damped along its own axis inside the layer; `part` is the first."""
        (t1, t2), (a1, a2) = terms, axes
        layer = self.on[a1, h[a1]] | self.on[a2, h[a2]]
        p1 = self.xi[a1, h[a1]] * part + self.co[a1, h[a1]] * t1
        p2 = self.xi[a2, h[a2]] * (F - part) + self.co[a2, h[a2]] * t2
        new = torch.where(layer, p1 + p2, F + self.dt * (t1 + t2))
        return torch.where(inside, new, F), torch.where(inside & layer, p1, part)

    def _inside(self, h, electric):
        m = torch.ones((1, 1, 1), dtype=torch.bool, device=self.dev)
        for a in range(3):
            i = torch.arange(self.S[a], device=self.dev)
            if self.per[a]:
                ok = i >= 0
            elif electric:
                ok = (i >= (0 if h[a] else 1)) & (i <= self.S[a] - 2)
            else:
                ok = i <= self.S[a] - 1 - h[a]
            m = m & self._along(a, ok)
        return m

    def _split_axes(self, c):
        """The axes of the two curl terms, the first being the one whose part is stored."""
        if 1 not in self.axes and c == 1:
            return 0, 2
        return (c + 1) % 3, (c + 2) % 3

    def _faraday(self):
        th = self.theta
        if th > 0.0:
            self.Eb = [(1 - 0.5 * th) * o + 0.5 * th * b for o, b in zip(self.Eo, self.Eb)]
            F = [(1 + 0.25 * th) * e - 0.5 * o + (0.5 - 0.25 * th) * b for e, o, b in zip(self.E, self.Eo, self.Eb)]
        else:
            F = self.E
        new = []
        for c in range(3):
            p, q = (c + 1) % 3, (c + 2) % 3
            h = self.B_STAGGER[c]
            term = {p: -self._wide_diff(F[q], p, h[p]), q: self._wide_diff(F[p], q, h[q])}
            ax = self._split_axes(c)
            b, self.SB[c] = self._split(self.B[c], self.SB[c], [term[a] for a in ax], ax, h, self._inside(h, False))
            new.append(b)
        self.Bo, self.B = self.B, new

    def _ampere(self, J):
        new = []
        for c in range(3):
            p, q = (c + 1) % 3, (c + 2) % 3
            h = self.E_STAGGER[c]
            term = {p: self._diff(self.B[q], p, h[p]), q: -self._diff(self.B[p], q, h[q])}
            ax = self._split_axes(c)
            carrier = 2 if (1 not in self.axes and c == 0) else ax[0]     # the term the current enters
            term[carrier] = term[carrier] - J[c]
            e, self.SE[c] = self._split(self.E[c], self.SE[c], [term[a] for a in ax], ax, h, self._inside(h, True))
            new.append(e)
        self.Eo, self.E = self.E, new

    def _filter_axis(self, F, a, h):
        F = F.clone()
        n = self.S[a] if self.per[a] else self.S[a] - h
        body = F.narrow(2 - a, 0, n)

        def neighbours(v, st):
            if self.per[a]:
                return torch.roll(v, st, dims=2 - a) + torch.roll(v, -st, dims=2 - a)
            out = torch.zeros_like(v)
            if st < n:
                out.narrow(2 - a, st, n - st).add_(v.narrow(2 - a, 0, n - st))
                out.narrow(2 - a, 0, n - st).add_(v.narrow(2 - a, st, n - st))
            return out

        v = body.clone()
        passes = self.cfg["filter_npass"]
        for st in range(1, 17):
            if passes and (self.cfg["filter_strides"] or 1) >> (st - 1) & 1:
                for al in [0.5] * passes + [0.5 * passes + 1.0] * self.cfg["filter_compensate"]:
                    v = al * v + 0.5 * (1.0 - al) * neighbours(v, st)
        body.copy_(v)
        return F

    def _filter(self, J):
        if self.c["learned"]:
            ws = _unpack(_filter_weights(self.seed), self.dev)
            out = []
            for c in range(3):
                n = [self.S[a] if self.per[a] else self.S[a] - self.E_STAGGER[c][a] for a in (0, 2)]
                F = torch.zeros_like(J[c])
                F[:n[1], 0, :n[0]] = _net(J[c][:n[1], 0, :n[0]][None], ws, (False, self.per[0]))[0]
                out.append(F)
            return out
        for a in self.axes:
            J = [self._filter_axis(J[c], a, self.E_STAGGER[c][a]) for c in range(3)]
        return J

    # -- particles --
    def _index(self, a, j):
        return j % self.N[a] if self.per[a] else j + self.P[a]

    def _nodal(self, F, h):
        for a in self.axes:
            if h[a]:
                F = 0.5 * (F + self._shift(F, a, -1))
        return F

    def _gather(self, F, h, r):
        idx, w = [], []
        for a in self.axes:
            s = r[a] - 0.5 * h[a]
            j = torch.floor(s)
            w.append(_weights(s - j))
            stride = (1, self.S[0], self.S[0] * self.S[1])[a]
            idx.append([self._index(a, j.long() - 1 + m) * stride for m in range(4)])
        flat = F.reshape(-1)

        def level(k, base):
            out = 0.0
            for m in range(4):
                at = base + idx[k][m]
                out = out + w[k][m] * (flat[at] if k == 0 else level(k - 1, at))
            return out

        return level(len(self.axes) - 1, 0)

    def _push(self, E, B, ux, uy, uz):
        h = -0.5 * self.dt
        if self.cfg["pusher"]:
            g = torch.sqrt(1 + ux * ux + uy * uy + uz * uz)
            v = (ux / g, uy / g, uz / g)
            tau = [h * b for b in B]
            up = [u + 2 * h * E[k] + v[(k + 1) % 3] * tau[(k + 2) % 3] - v[(k + 2) % 3] * tau[(k + 1) % 3]
                  for k, u in enumerate((ux, uy, uz))]
            tau2 = sum(t * t for t in tau)
            us = sum(a * b for a, b in zip(up, tau))
            sig = 1 + sum(a * a for a in up) - tau2
            gn = torch.sqrt(0.5 * (sig + torch.sqrt(sig * sig + 4 * (tau2 + us * us))))
            t = [a / gn for a in tau]
            s = 1 / (1 + sum(a * a for a in t))
            ut = sum(a * b for a, b in zip(up, t))
            return [s * (up[k] + ut * t[k] + up[(k + 1) % 3] * t[(k + 2) % 3] - up[(k + 2) % 3] * t[(k + 1) % 3])
                    for k in range(3)]
        um = [u + h * e for u, e in zip((ux, uy, uz), E)]
        g = torch.sqrt(1 + sum(a * a for a in um))
        t = [h * b / g for b in B]
        s = [2 * a / (1 + sum(x * x for x in t)) for a in t]
        cross = lambda a, b, k: a[(k + 1) % 3] * b[(k + 2) % 3] - a[(k + 2) % 3] * b[(k + 1) % 3]  # noqa: E731
        up = [um[k] + cross(um, t, k) for k in range(3)]
        return [um[k] + cross(up, s, k) + h * E[k] for k in range(3)]

    def _window(self, x0, x1):
        """First node and the shape factors before and after a move, on the five nodes it can touch."""
        i0, i1 = torch.floor(x0), torch.floor(x1)
        base = torch.minimum(i0, i1) - 1
        out = []
        for x, i in ((x0, i0), (x1, i1)):
            w = _weights(x - i)
            up = i > base + 1
            zero = torch.zeros_like(x)
            out.append([torch.where(up, w[m - 1] if m else zero, w[m] if m < 4 else zero) for m in range(5)])
        return base.long(), out[0], [b - a for a, b in zip(*out)]

    def _deposit(self, J, r0, r1, q, vy=None):
        """Esirkepov's current of charges q moving r0 -> r1 (cells); vy: the velocity out of the 2D plane."""
        base, S, D, at = {}, {}, {}, {}
        for a in self.axes:
            base[a], S[a], D[a] = self._window(r0[a], r1[a])
            stride = (1, self.S[0], self.S[0] * self.S[1])[a]
            at[a] = [self._index(a, base[a] + m) * stride for m in range(5)]
        vol = math.prod(self.d[a] for a in self.axes)
        for c in self.axes:
            others = [a for a in self.axes if a != c]
            k = -q * self.d[c] / (vol * self.dt)
            flat = J[c].view(-1)
            run = 0.0
            for m in range(4):
                run = run + k * D[c][m]
                for m1 in range(5):
                    if len(others) == 1:
                        o, = others
                        flat.index_add_(0, at[c][m] + at[o][m1], run * (S[o][m1] + 0.5 * D[o][m1]))
                        continue
                    o, p = others
                    for m2 in range(5):
                        T = (S[o][m1] * S[p][m2] + 0.5 * (D[o][m1] * S[p][m2] + S[o][m1] * D[p][m2])
                             + D[o][m1] * D[p][m2] / 3.0)
                        flat.index_add_(0, at[c][m] + at[o][m1] + at[p][m2], run * T)
        if vy is not None:
            k = q * vy / vol
            flat = J[1].view(-1)
            for m in range(5):
                for n in range(5):
                    W = (S[0][m] * S[2][n] + 0.5 * (D[0][m] * S[2][n] + S[0][m] * D[2][n]) + D[0][m] * D[2][n] / 3.0)
                    flat.index_add_(0, at[0][m] + at[2][n], k * W)

    def _deposit_z(self, J, x, y, z0, z1, q):
        r, w, at = {0: x, 1: y}, {}, {}
        for a in self.axes[:-1]:
            j = torch.floor(r[a])
            w[a] = _weights(r[a] - j)
            at[a] = [self._index(a, j.long() - 1 + m) * (1, self.S[0])[a] for m in range(4)]
        base, S, D = self._window(z0, z1)
        vol = math.prod(self.d[a] for a in self.axes)
        run = 0.0
        for m in range(4):
            run = run - q * self.d[2] / (vol * self.dt) * D[m]
            iz = self._index(2, base + m) * self.S[0] * self.S[1]
            for m1 in range(4):
                if 1 not in self.axes:
                    J[2].view(-1).index_add_(0, iz + at[0][m1], run * w[0][m1])
                    continue
                for m2 in range(4):
                    J[2].view(-1).index_add_(0, iz + at[0][m1] + at[1][m2], run * w[0][m1] * w[1][m2])

    def _electrons(self, J):
        e = self.e
        if not len(e["x"]):
            return
        r0 = {a: e["xyz"[a]] for a in self.axes}
        Bn = [0.5 * (a + b) for a, b in zip(self.Bo, self.B)]
        stag = list(self.E_STAGGER) + list(self.B_STAGGER)
        F = self.E + Bn
        if self.cfg["gather_kind"]:
            F = [self._nodal(f, h) for f, h in zip(F, stag)]
            stag = [(0, 0, 0)] * 6
        v = [self._gather(f, h, r0) for f, h in zip(F, stag)]
        u = self._push(v[:3], v[3:], e["ux"], e["uy"], e["uz"])
        g = torch.sqrt(1 + sum(a * a for a in u))
        r1 = {a: r0[a] + self.dt / self.d[a] * u[a] / g for a in self.axes}
        self._deposit(J, r0, r1, -e["w"], None if 1 in self.axes else u[1] / g)
        keep = torch.ones_like(e["x"], dtype=torch.bool)
        for a in self.axes:
            if self.per[a]:
                r1[a] = r1[a] % self.N[a]
            else:
                keep &= (r1[a] >= 0) & (r1[a] < self.N[a])
        for a in self.axes:
            e["xyz"[a]] = r1[a]
        e["ux"], e["uy"], e["uz"] = u
        if not bool(keep.all()):
            for k in e:
                if len(e[k]):
                    e[k] = e[k][keep]

    def _ions(self, J, t1):
        i = self.ion
        if not len(i["x"]):
            return
        za = i["z"] - (self.beta * self.t / self.d[2] + self.shift)
        zb = i["z"] - (self.beta * t1 / self.d[2] + self.shift)
        self._deposit_z(J, i["x"], i["y"], za, zb, i["w"])
        keep = (zb >= 0) & (zb < self.N[2])
        if not bool(keep.all()):
            for k in i:
                if len(i[k]):
                    i[k] = i[k][keep]

    def _antenna(self, J, t1):
        za, zb = ((self.las["z_antenna_um"] / self.gamma - self.beta * t) / self.d[2] - self.shift for t in (self.t, t1))
        if not 0.0 <= za < self.N[2]:
            return
        two = 1 not in self.axes
        tau = (self.t + 0.5 * self.dt) / self.gamma - self.t0
        r2 = ((self.home[0] - 0.5 * self.N[0]) * self.d[0]) ** 2
        if not two:
            r2 = r2 + ((self.home[1] - 0.5 * self.N[1]) * self.d[1]) ** 2
        field = (self.e0 / self.gamma) * torch.exp(-r2 / self.las["waist_um"] ** 2) * (
            math.exp(-tau * tau / (2.0 * self.sig_t ** 2)) * math.sin(self.omega * tau))
        v = 2.0 * field * (self.d[0] if two else self.d[0] * self.d[1]) / self.aw
        to = self.moving + v * self.dt / self.d[0]
        a, b = torch.full_like(to, za), torch.full_like(to, zb)
        w = torch.full_like(to, self.aw)
        y = self.home[1]
        self._deposit(J, {0: self.moving, 1: y, 2: a}, {0: to, 1: y, 2: b}, -w)
        self._deposit(J, {0: self.home[0], 1: y, 2: a}, {0: self.home[0], 1: y, 2: b}, w)
        self.moving = to

    def _inject(self):
        """Creates the lattice rows (planes) of the lab-fixed plasma whose front edge is inside the window."""
        rows = 0
        while self.next_row + rows + 1 - self.beta * self.t / self.d[2] - self.shift <= self.N[2]:
            rows += 1
        if not rows:
            return
        per_row = self.N[0] * self.N[1] * self.pl["ppc"]
        k = np.arange(rows * per_row, dtype=np.uint64) + np.uint64(self.next_row * per_row)
        dims = len(self.axes)
        rnd = [_u01(self.seed, k * np.uint64(dims) + np.uint64(1 + m)) for m in range(dims)]
        cell = k // np.uint64(self.pl["ppc"])
        row = (cell // np.uint64(self.N[0] * self.N[1])).astype(np.float64)
        x = (cell % np.uint64(self.N[0])).astype(np.float64) + rnd[0]
        y = (cell // np.uint64(self.N[0]) % np.uint64(self.N[1])).astype(np.float64) + rnd[1]
        z = row + rnd[-1]
        z_lab = self.gamma * z * self.d[2]
        dens = np.where(z_lab < self.pl["start_um"], 0.0, self.n0)
        if self.pl["ramp_um"] > 0.0:
            dens = dens * np.clip((z_lab - self.pl["start_um"]) / self.pl["ramp_um"], 0.0, 1.0)
        w = self.gamma * dens * math.prod(self.d[a] for a in self.axes) / self.pl["ppc"]
        on = w != 0.0
        T = lambda a: torch.from_numpy(np.ascontiguousarray(a[on])).to(self.dev)  # noqa: E731
        x, y, z, w = T(x), T(y), T(z), T(w)
        zero = torch.zeros_like(x)
        new = dict(x=x, y=y, z=z - self.beta * self.t / self.d[2] - self.shift, ux=zero, uy=zero,
                   uz=zero - self.gamma * self.beta, w=w)
        self.e = {n: torch.cat([self.e[n], new[n]]) for n in new}
        if self.pl["ion_mode"]:
            self.ion = {n: torch.cat([self.ion[n], v]) for n, v in dict(x=x, y=y, z=z, w=w).items()}
        self.next_row += rows

    # -- one step --
    def step(self):
        self._faraday()
        t1 = (self.n + 1) * self.dt
        to = int(self.vw * t1 / self.d[2]) if self.cfg["moving_window"] else 0
        move = to - self.shift
        J = [torch.zeros_like(f) for f in self.E]
        self._electrons(J)
        self._ions(J, t1)
        self._antenna(J, t1)
        self._ampere(self._filter(J))
        self.n, self.t = self.n + 1, t1
        if move:
            self._advance(move)
        self.shift = to
        self._inject()

    def _advance(self, move):
        self.e["z"] = self.e["z"] - move
        for name in ("E", "Eo", "Eb", "B", "Bo", "SE", "SB"):
            rows = [torch.roll(f, -move, dims=0) for f in getattr(self, name)]
            for f in rows:
                f.narrow(0, self.S[2] - move if move > 0 else 0, abs(move)).zero_()
            setattr(self, name, rows)
        for parts, staggers in ((self.SE, self.E_STAGGER), (self.SB, self.B_STAGGER)):
            for c in range(2):         # the stored parts of rows that came out of the layer are dropped
                h = staggers[c]
                on = self.on[2, h[2]].view(-1)
                k = torch.arange(self.S[2], device=self.dev)
                was = (k + move - self.P[2] + 0.5 * h[2] < 0) | (k + move - self.P[2] + 0.5 * h[2] > self.N[2])
                came = self._along(2, ~on & was)
                drop = came & ~self.on[0, h[0]] & ~self.on[1, h[1]]
                parts[c] = torch.where(drop, torch.zeros_like(parts[c]), parts[c])
        for name in ("E", "Eo", "Eb"):
            for c in range(2):
                f = getattr(self, name)[c]
                f[0].zero_()
                f[-1].zero_()

    def outputs(self):
        """The fields in the library's storage order: stored row = (row + shift) mod rows."""
        def stored(F):
            F = torch.roll(F, self.shift % self.S[2], dims=0)
            return F[:, 0] if 1 not in self.axes else F
        return dict(E=torch.stack([stored(f) for f in self.E]), B=torch.stack([stored(f) for f in self.B]))
