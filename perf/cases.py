"""Performance cases of the library: what its users have it do, through the public entry points.

``listed()`` names the cases, ``draw(rng)`` gives further ones of the same ranges,
``prepare(case, seed)`` makes what a program has in hand before the call (inputs, problem
descriptions, workspace), ``run(state)`` is one pass, ``exact(case, seed)`` its outputs in
64-bit torch without the library, and ``work(case)`` the bytes and operations a pass cannot
do without.

Every kind of call has its own range:

* ``solve``: Algorithm S1 on a batch (one projection, a scan's projections, regions of
  interest of several sizes), with a fixed iteration count or the stopping correlation;
* ``joint``: the solve that refines the shared diffuser;
* ``steps``: the caller's own loop over ``step``;
* ``train``: the differentiable loss, forward and backward;
* ``forward``: the forward model or the RMSE image of retrieved fields;
* ``tomogram``: filtered back-projection of retrieved projections and the removal of the
  quadratic background;
* ``shells``: Fourier shell / ring correlation of two reconstructions;
* ``calibrate``: coherence lengths and diffuser from a reference speckle.

Inputs follow the repository's generators (smooth random phase objects with 5% absorption,
smoothed random-phase diffusers, 1e4 photons per pixel of Poisson noise, the same geometry),
drawn on the GPU.  The schedules are the library's built-in ones: timing the candidates on
each machine would make the outputs of two runs differ in rounding.
"""

from __future__ import annotations

import math

import torch

import paper_2503_20146_amd as pwf

PIXEL_M = 1.0e-6
WAVELENGTH_M = 0.05e-9
Z1_M = 5.0e-3
Z2_M = 200.0e-3
PHOTONS = 1.0e4
STOP_CORR = 10.0 ** -0.00001
SIDES = (128, 256, 512, 1024, 2048)
ETA_T = 0.5
WIENER_EPS = 1e-3


# --------------------------------------------------------------------------- the cases

def listed():
    return [
        # one small projection to convergence: what a user tries first, and the smallest launches
        {"name": "solve_128_one", "kind": "solve", "shapes": "128x128*1", "iters": 100, "sigma": 1.0, "stop": False},
        # one projection of the usual detector size (live reconstruction during a scan)
        {"name": "solve_1024_one", "kind": "solve", "shapes": "1024x1024*1", "iters": 100, "sigma": 1.5,
         "stop": False},
        # the projections of a half-turn scan in one batch (the repository's headline workload)
        {"name": "solve_1024_scan", "kind": "solve", "shapes": "1024x1024*180", "iters": 10, "sigma": 1.5,
         "stop": False},
        # a share of a fine scan at the largest grid
        {"name": "solve_2048_scan", "kind": "solve", "shapes": "2048x2048*36", "iters": 10, "sigma": 1.5,
         "stop": False},
        # regions of interest of three sizes, each with its own diffuser and source
        {"name": "solve_rois", "kind": "solve", "shapes": "512x512*24+1024x1024*32+2048x2048*8", "iters": 10,
         "sigma": 1.0, "stop": False},
        # wide detector, an odd number of projections, run to the stopping correlation
        {"name": "solve_wide_stop", "kind": "solve", "shapes": "1024x512*9", "iters": 60, "sigma": 1.5, "stop": True},
        # projections and the diffuser they share, refined together
        {"name": "joint_1024", "kind": "joint", "shapes": "1024x1024*40", "iters": 10, "sigma": 1.5},
        # the differentiable loss of a batch inside a caller's optimiser
        {"name": "train_512", "kind": "train", "shapes": "512x512*12", "sigma": 1.0},
        # forward model of one region: the smallest single call
        {"name": "forward_256", "kind": "forward", "shapes": "256x256*1", "sigma": 1.0, "rmse": False},
        # a slab of a tomogram from a half-turn scan, background removed
        {"name": "tomogram_1024", "kind": "tomogram", "nx": 1024, "ny": 128, "n_proj": 180, "n_out": 1024},
        # resolution of a tomogram against a second reconstruction
        {"name": "shells_512", "kind": "shells", "n": 512, "dims": 3, "part": 1},
        # source and diffuser from one reference speckle, before a scan
        {"name": "calibrate_1024", "kind": "calibrate", "nx": 1024, "ny": 1024, "sigma": 1.5},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("solve", "solve", "solve", "joint", "steps", "train", "forward", "tomogram", "shells",
                       "calibrate"))
    sigma = round(rng.uniform(0.8, 2.0), 3)
    if kind == "tomogram":
        n_out = 16 * _log_int(rng, 4, 64)
        ny = 32 * _log_int(rng, 1, 4)
        return {"kind": kind, "nx": _log_int(rng, 64, 1024), "ny": ny, "n_proj": _log_int(rng, 11, 180),
                "n_out": n_out}
    if kind == "shells":
        dims = rng.choice((2, 3))
        return {"kind": kind, "n": rng.choice(SIDES if dims == 2 else SIDES[:3]), "dims": dims,
                "part": rng.choice((0, 1)), "gain": round(10.0 ** rng.uniform(-2.0, 2.0), 4)}
    if kind == "calibrate":
        return {"kind": kind, "nx": rng.choice(SIDES), "ny": rng.choice(SIDES), "sigma": max(sigma, 1.2)}
    if kind == "solve" and rng.random() < 0.3:   # two or three sizes
        sides = sorted(rng.sample(SIDES, rng.choice((2, 3))))
        shapes = "+".join("%dx%d*%d" % (s, s, _log_int(rng, 1, max(2, 8 * 1024 * 1024 // (s * s)))) for s in sides)
        return {"kind": kind, "shapes": shapes, "iters": rng.randint(5, 20), "sigma": sigma, "stop": False}
    nx = rng.choice(SIDES)
    ny = nx if rng.random() < 0.6 else rng.choice(SIDES)
    most = {"solve": 160, "joint": 40, "steps": 12, "train": 24, "forward": 24}[kind]   # megapixels
    count = _log_int(rng, 1, max(1, min(60, most * 1024 * 1024 // (nx * ny))))
    case = {"kind": kind, "shapes": "%dx%d*%d" % (nx, ny, count), "sigma": sigma}
    if kind == "solve":
        mpx = nx * ny * count / 1048576.0
        case["iters"] = _log_int(rng, 5, max(6, min(100, int(1600 / mpx))))
        case["stop"] = rng.random() < 0.25
    elif kind == "joint":
        case["iters"] = rng.randint(3, 10)
    elif kind == "steps":
        case["iters"] = rng.randint(2, 10)
    elif kind == "forward":
        case["rmse"] = rng.random() < 0.5
    return case


def _classes(case):
    """[(nx, ny, count)] of a batch written nxXny*count+..."""
    out = []
    for part in case["shapes"].split("+"):
        dims, count = part.split("*")
        nx, ny = dims.split("x")
        out.append((int(nx), int(ny), int(count)))
    return out


# --------------------------------------------------------------------------- inputs

def _gen(seed, *key):
    g = torch.Generator(device="cuda")
    s = int(seed)
    for k in key:
        s = (s * 1000003 + int(k) + 12345) % (2 ** 62)
    g.manual_seed(s)
    return g


def _freqs(n):
    return torch.fft.fftfreq(n, dtype=torch.float64, device="cuda")


def _lowpass(a, sigma_px):
    ny, nx = a.shape[-2:]
    fy, fx = _freqs(ny)[:, None], _freqs(nx)[None, :]
    w = torch.exp(-2.0 * math.pi ** 2 * sigma_px ** 2 * (fx * fx + fy * fy)).to(torch.float32)
    return torch.fft.ifft2(torch.fft.fft2(a) * w).real


def _phase_objects(gen, n, ny, nx):
    """Smooth random samples -mu + i phi, phi in [0, 2] or [0, 4] rad, mu = 0.05 phi (complex64)."""
    side = max(nx, ny)
    smooth, top = (16.0, 4.0) if side >= 1024 else (4.0, 2.0)
    out = torch.empty((n, ny, nx), dtype=torch.complex64, device="cuda")
    for i in range(n):
        s = _lowpass(torch.randn((ny, nx), generator=gen, device="cuda"), smooth)
        lo, hi = s.min(), s.max()
        phi = top * (s - lo) / (hi - lo)
        out[i] = torch.complex(-0.05 * phi, phi)
    return out


def _diffusers(gen, n, ny, nx):
    out = torch.empty((n, ny, nx), dtype=torch.complex64, device="cuda")
    for i in range(n):
        theta = _lowpass(math.pi * torch.rand((ny, nx), generator=gen, device="cuda"), 1.0)
        out[i] = torch.polar(0.9 + 0.1 * torch.rand((ny, nx), generator=gen, device="cuda"), theta)
    return out


def _noisy(gen, f):
    return (torch.poisson(f.clamp_min(0.0).to(torch.float32) * PHOTONS, generator=gen) / PHOTONS).contiguous()


def _scene(case, seed):
    """Per size class: diffusers, sigmas, samples and measured speckles."""
    out = []
    rois = len(_classes(case)) > 1
    for c, (nx, ny, n) in enumerate(_classes(case)):
        gen = _gen(seed, c, nx, ny)
        nt = n if rois else 1
        t = _diffusers(gen, nt, ny, nx)
        base = case["sigma"]
        sig = [base if not rois else 0.5 + (base + 0.37 * i) % 1.5 for i in range(n)]
        psi = _phase_objects(gen, n, ny, nx)
        y = torch.empty((n, ny, nx), dtype=torch.float32, device="cuda")
        for i in range(n):
            m = _Model(t[i if nt > 1 else 0], sig[i])
            y[i] = _noisy(gen, m.forward(psi[i].to(torch.complex128))[0])
        if case["kind"] == "joint":   # the diffuser a joint solve starts from: 5% off in amplitude
            t = t * (1.0 + 0.05 * torch.randn((nt, ny, nx), generator=gen, device="cuda"))
        out.append({"nx": nx, "ny": ny, "n": n, "t": t, "sigma": sig, "psi": psi, "y": y})
    return out


def _problems(scene):
    probs = []
    for s in scene:
        for i in range(s["n"]):
            t = s["t"][i if s["t"].shape[0] > 1 else 0]
            probs.append(pwf.Problem(nx=s["nx"], ny=s["ny"], pixel_m=PIXEL_M, wavelength_m=WAVELENGTH_M, z1_m=Z1_M,
                                     z2_m=Z2_M, sigma_x_px=s["sigma"][i], sigma_y_px=s["sigma"][i], diffuser=t))
    return probs


def _views(stacks):
    return [a[i] for a in stacks for i in range(a.shape[0])]


def _volumes(case, seed):
    """Two reconstructions of one object: its smooth part, and noise of their own."""
    n, dims = case["n"], case["dims"]
    gen = _gen(seed, n, dims)
    shape = (n,) * dims
    f = [_freqs(n).to(torch.float32).reshape([-1 if a == d else 1 for a in range(dims)]) for d in range(dims)]
    w = torch.exp(-2.0 * math.pi ** 2 * 4.0 * sum(x * x for x in f))

    def field():
        a = torch.complex(torch.randn(shape, generator=gen, device="cuda"),
                          torch.randn(shape, generator=gen, device="cuda"))
        return a

    obj = torch.fft.ifftn(torch.fft.fftn(field()) * w)
    obj *= 1.0 / obj.abs().square().mean().sqrt()
    g1 = obj + 0.3 * field()
    g2 = case.get("gain", 1.0) * (obj + 0.3 * field())
    return g1.contiguous(), g2.contiguous()


def _sinogram(case, seed):
    gen = _gen(seed, case["nx"], case["ny"], case["n_proj"])
    nx, ny, p = case["nx"], case["ny"], case["n_proj"]
    ang = [math.pi * j / p for j in range(p)]
    # projections of Gaussian blobs: smooth in the detector, consistent over the angles
    blobs = 24
    r = torch.rand((blobs, 5), generator=gen, device="cuda", dtype=torch.float64)
    x = (r[:, 0] - 0.5) * 0.6 * nx
    z = (r[:, 1] - 0.5) * 0.6 * nx
    s = (0.01 + 0.05 * r[:, 2]) * nx
    cy = r[:, 3] * ny
    amp = 1.0 + r[:, 4]
    u = (torch.arange(nx, device="cuda", dtype=torch.float64) + 0.5 - 0.5 * nx)[None, :]
    v = (torch.arange(ny, device="cuda", dtype=torch.float64) + 0.5)[:, None]
    along = amp[:, None, None] * torch.exp(-0.5 * ((v[None] - cy[:, None, None]) / (0.2 * ny)) ** 2)   # [b, ny, 1]
    out = torch.empty((p, ny, nx), dtype=torch.complex64, device="cuda")
    for j, th in enumerate(ang):
        uc = x * math.cos(th) - z * math.sin(th)
        prof = torch.exp(-0.5 * ((u - uc[:, None]) / s[:, None]) ** 2)   # [b, nx]
        phi = (along[:, :, 0].T @ prof) + 0.01 * torch.randn((ny, nx), generator=gen, device="cuda")
        out[j] = torch.complex(-0.05 * phi, phi).to(torch.complex64)
    return out, ang


def _reference(case, seed):
    nx, ny = case["nx"], case["ny"]
    gen = _gen(seed, nx, ny)
    t = _diffusers(gen, 1, ny, nx)[0]
    m = _Model(t, case["sigma"])
    f = m.forward(torch.zeros((ny, nx), dtype=torch.complex128, device="cuda"))[0]
    return t, _noisy(gen, f)


# --------------------------------------------------------------------------- prepare and run

def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "tomogram":
        s["psi"], s["angles"] = _sinogram(case, seed)
        s["vol"] = torch.empty((case["ny"], case["n_out"], case["n_out"]), dtype=torch.complex64, device="cuda")
        return s
    if kind == "shells":
        s["g1"], s["g2"] = _volumes(case, seed)
        return s
    if kind == "calibrate":
        t, s["ref"] = _reference(case, seed)
        s["problem"] = pwf.Problem(nx=case["nx"], ny=case["ny"], pixel_m=PIXEL_M, wavelength_m=WAVELENGTH_M,
                                   z1_m=Z1_M, z2_m=Z2_M, sigma_x_px=case["sigma"], sigma_y_px=case["sigma"],
                                   diffuser=t)
        return s
    scene = _scene(case, seed)
    s["batch"] = pwf.PWF(_problems(scene))
    s["y"] = _views([c["y"] for c in scene])
    if kind in ("solve", "joint"):
        s["out"] = [torch.empty_like(c["psi"]) for c in scene]
        s["views"] = _views(s["out"])
    if kind == "joint":
        s["t"], s["t0"] = scene[0]["t"], scene[0]["t"].clone()
    elif kind == "train":
        s["psi"] = (0.5 * scene[0]["psi"]).requires_grad_(True)
    elif kind == "forward":
        s["psi"] = _views([0.5 * c["psi"] for c in scene])
        s["means"] = [1.0] * len(s["psi"])
    return s


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        # (psi is what the program goes on with; it does not ask for the loss history)
        if case["stop"]:
            _, _, done = state["batch"].solve(state["y"], case["iters"], psi_out=state["views"], loss_hist=False,
                                              corr_tol=STOP_CORR, return_iters=True)
            return {"psi": state["out"], "iterations": torch.tensor(done)}
        state["batch"].solve(state["y"], case["iters"], psi_out=state["views"], loss_hist=False)
        return {"psi": state["out"]}
    if kind == "joint":
        state["t"].copy_(state["t0"])   # the diffuser is refined in place: every run starts from the estimate
        state["batch"].solve_joint(state["y"], case["iters"], eta_t=ETA_T, psi_out=state["views"], loss_hist=False)
        return {"psi": state["out"], "t": state["t"]}
    if kind == "steps":
        states = state["batch"].init_states(state["y"])
        for _ in range(case["iters"]):
            state["batch"].step(states)
        return {"psi": [st["psi"] for st in states]}
    if kind == "train":
        loss = pwf.pwf_loss(state["psi"], state["batch"], state["y"])
        (grad,) = torch.autograd.grad(loss.sum(), state["psi"])
        return {"grad": grad, "loss": loss.tolist()}   # the training log's numbers
    if kind == "forward":
        if case["rmse"]:
            return {"rmse": state["batch"].rmse_image(state["psi"], state["y"], state["means"])}
        return {"f": state["batch"].forward(state["psi"])}
    if kind == "tomogram":
        scale = WAVELENGTH_M / (2.0 * math.pi * PIXEL_M)
        vol = pwf.fbp(list(state["psi"]), state["angles"], n_out=case["n_out"], scale=scale, out=state["vol"])
        return {"vol": pwf.background_quadratic(vol, 0.46 * case["n_out"])}
    if kind == "shells":
        return {"fsc": torch.tensor(pwf.shell_correlation(state["g1"], state["g2"], part=case["part"]))}
    if kind == "calibrate":
        src = pwf.calibrate_source(state["ref"], PIXEL_M)
        t = pwf.diffuser_from_reference(state["problem"], state["ref"], eps=WIENER_EPS)
        return {"x_coh_m": src["x_coh_m"], "y_coh_m": src["y_coh_m"], "g2x": torch.tensor(src["g2x"]),
                "g2y": torch.tensor(src["g2y"]), "t": t}
    raise ValueError(kind)


# --------------------------------------------------------------------------- floors

def _fft2_flops(nx, ny):
    return 5.0 * nx * ny * math.log2(nx * ny)


def work(case):
    """Inputs read once and outputs written once, and per iteration the state that the
    algorithm carries from one to the next (psi, z and y read, psi and z written); operations
    of the Fourier transforms (5 n log2 n each) and interpolations."""
    kind = case["kind"]
    if kind == "tomogram":
        p, nx, ny, n = case["n_proj"], case["nx"], case["ny"], case["n_out"]
        pad = 64
        while pad < 2 * nx:
            pad *= 2
        return {"bytes": 8.0 * p * nx * ny + 8.0 * ny * n * n,
                "flops": 13.0 * p * ny * n * n + 10.0 * p * ny * pad * math.log2(pad)}
    if kind == "shells":
        m = float(case["n"]) ** case["dims"]
        return {"bytes": 16.0 * m, "flops": 5.0 * m * math.log2(m) + 10.0 * m}
    if kind == "calibrate":
        m = float(case["nx"]) * case["ny"]
        return {"bytes": 12.0 * m, "flops": 4 * _fft2_flops(case["nx"], case["ny"]) + 132.0 * m}
    total = {"bytes": 0.0, "flops": 0.0}
    for nx, ny, n in _classes(case):
        m = float(nx) * ny * n
        f2 = _fft2_flops(nx, ny) * n
        # a forward pass is 5 complex 2-D transforms of propagation and 1 (two real ones) of the blur;
        # the gradient as much again, direction and update 4 more
        if kind == "forward":
            total["bytes"] += 16.0 * m
            total["flops"] += 5 * f2
        elif kind == "train":
            total["bytes"] += 20.0 * m
            total["flops"] += 15 * f2
        else:
            iters = case["iters"]
            per = (8 + 8 + 4 + 8 + 8) * m + (8.0 * nx * ny if kind == "joint" else 0.0)
            total["bytes"] += (per if not case.get("stop") else 0.5 * per) * iters
            total["flops"] += 12 * f2 * (iters if not case.get("stop") else 0.5 * iters)
    return total


# --------------------------------------------------------------------------- 64-bit values

class _Model:
    """The forward model, gradient and update of one instance in complex128 (natural layout)."""

    def __init__(self, t, sigma):
        self.t = t.to(torch.complex128)
        ny, nx = t.shape
        fx, fy = _freqs(nx)[None, :], _freqs(ny)[:, None]
        rho2 = fx * fx + fy * fy
        lp2 = (WAVELENGTH_M / PIXEL_M) ** 2
        root = torch.sqrt(1.0 - lp2 * rho2)

        def q(z):
            th = -2.0 * math.pi * (z * WAVELENGTH_M / PIXEL_M ** 2) * rho2 / (1.0 + root)
            return torch.polar(torch.ones_like(th), th)

        self.q1, self.q2 = q(Z1_M), q(Z2_M)
        coh2 = (2.0 * math.sqrt(math.pi) * sigma) ** 2
        self.iotf = torch.exp(-0.5 * math.pi * coh2 * rho2)
        self.gamma2 = -torch.expm1(-math.pi * pwf.DEFAULT_GAMMA * coh2 * rho2)
        self.pinv = torch.where(rho2 > 0, pwf.DEFAULT_PRECOND_SCALE / rho2.clamp_min(1e-30),
                                torch.zeros_like(rho2))
        self.maxt2 = self.t.abs().square().max()

    @staticmethod
    def filt(a, w):
        return torch.fft.ifft2(torch.fft.fft2(a) * w)

    def forward(self, psi):
        x = torch.exp(psi)
        u1 = self.filt(x, self.q1)
        v = self.filt(self.t * u1, self.q2)
        f = self.filt(v.abs().square().to(torch.complex128), self.iotf).real
        return f, x, u1, v

    def backward(self, f, x, v, y):
        """Loss, the field back-propagated to the diffuser, and conj(x) times it at the sample."""
        e = y.to(torch.float64) - f
        a2 = self.filt(v * self.filt((-e).to(torch.complex128), self.iotf).real, self.q2.conj())
        return e.square().sum(), a2, x.conj() * self.filt(self.t.conj() * a2, self.q1.conj())

    def direction(self, psi, g):
        d = torch.complex(g.real, self.filt(g.imag.to(torch.complex128), self.pinv).real)
        r = self.filt(psi, self.gamma2)
        al = pwf.DEFAULT_ALPHA
        return d + torch.complex(al.real * r.real, al.imag * r.imag)


def _next_tau(tau):
    return 0.5 * (1.0 + math.sqrt(1.0 + 4.0 * tau * tau))


def _solve64(model, y, iters, stop):
    psi = torch.zeros(y.shape, dtype=torch.complex128, device="cuda")
    z, tau, done = psi, 1.0, 0
    for _ in range(iters):
        f, x, _, v = model.forward(psi)
        _, _, g = model.backward(f, x, v, y)
        zn = psi - pwf.DEFAULT_ETA * model.direction(psi, g / model.maxt2)
        nt = _next_tau(tau)
        new = zn + ((tau - 1.0) / nt) * (zn - z)
        z, tau, done = zn, nt, done + 1
        if stop:
            xn = torch.exp(new)
            c = (xn.conj() * x).sum().abs() / (xn.abs().square().sum() * x.abs().square().sum()).sqrt()
            psi = new
            if c > STOP_CORR:
                break
        psi = new
    return psi, done


def _joint64(scene, iters):
    s = scene[0]
    t = s["t"][0].to(torch.complex128)
    n = s["n"]
    model = _Model(t, s["sigma"][0])
    psi = [torch.zeros((s["ny"], s["nx"]), dtype=torch.complex128, device="cuda") for _ in range(n)]
    z, tau = list(psi), 1.0
    for _ in range(iters):
        nt = _next_tau(tau)
        gt, norm = torch.zeros_like(t), 0.0
        for i in range(n):
            f, x, u1, v = model.forward(psi[i])
            _, a2, g = model.backward(f, x, v, s["y"][i])
            zn = psi[i] - pwf.DEFAULT_ETA * model.direction(psi[i], g / model.maxt2)
            psi[i], z[i] = zn + ((tau - 1.0) / nt) * (zn - z[i]), zn
            gt += u1.conj() * a2
            norm = norm + u1.abs().square().max()
        tau = nt
        model.t = model.t - ETA_T * gt / norm
        model.maxt2 = model.t.abs().square().max()
    return torch.stack(psi), model.t[None]


def _tomogram64(case, psi, angles):
    p, ny, nx = psi.shape
    n = case["n_out"]
    pad = 64
    while pad < 2 * nx:
        pad *= 2
    k = torch.arange(pad, device="cuda")
    k = torch.where(k <= pad // 2, k, k - pad).to(torch.float64)
    h = torch.where(k.remainder(2) == 1, -1.0 / (math.pi ** 2 * k.square().clamp_min(1.0)), torch.zeros_like(k))
    h[0] = 0.25
    ramp = torch.fft.fft(h).real
    q = torch.fft.ifft(torch.fft.fft(psi.to(torch.complex128), n=pad, dim=-1) * ramp, dim=-1)[..., :nx]
    q = torch.nn.functional.pad(torch.view_as_real(q), (0, 0, 1, 1))   # a zero sample on each side
    c = torch.arange(n, device="cuda", dtype=torch.float64) + 0.5 - 0.5 * n
    vol = torch.zeros((ny, n, n, 2), dtype=torch.float64, device="cuda")
    for j, th in enumerate(angles):
        u = c[None, :] * math.cos(th) - c[:, None] * math.sin(th) + 0.5 * nx - 0.5
        i0 = torch.floor(u)
        w = (u - i0)[..., None]
        lo = (i0.to(torch.int64) + 1).clamp(0, nx + 1)
        hi = (i0.to(torch.int64) + 2).clamp(0, nx + 1)
        for y in range(ny):
            row = q[j, y]
            vol[y] += torch.lerp(row[lo], row[hi], w)
    vol *= (math.pi / p) * WAVELENGTH_M / (2.0 * math.pi * PIXEL_M)
    x = (c / (0.5 * n))[None, :].expand(n, n)
    zz = (c / (0.5 * n))[:, None].expand(n, n)
    basis = torch.stack([torch.ones_like(x), x, zz, x * x, x * zz, zz * zz]).reshape(6, -1)
    keep = (c[None, :].square() + c[:, None].square() >= (0.46 * n) ** 2).reshape(-1)
    a = basis[:, keep].T.contiguous().cpu()
    pinv = torch.linalg.inv(a.T @ a).to("cuda")
    a = a.to("cuda")
    for y in range(ny):
        sl = vol[y].reshape(-1, 2)
        coef = pinv @ (a.T @ sl[keep])
        vol[y] -= (basis.T @ coef).reshape(n, n, 2)
    return torch.view_as_complex(vol)


def _shells64(case, g1, g2):
    n, dims = case["n"], case["dims"]
    pick = (lambda g: g.imag) if case["part"] else (lambda g: g.real)
    G1 = torch.fft.fftn(pick(g1).to(torch.complex128))
    G2 = torch.fft.fftn(pick(g2).to(torch.complex128))
    k = _freqs(n) * n
    r2 = sum((k * k).reshape([-1 if a == d else 1 for a in range(dims)]) for d in range(dims))
    shell = torch.round(torch.sqrt(r2)).to(torch.int64).reshape(-1)
    nsh = n // 2 + 1
    shell.clamp_max_(nsh)

    def sums(v):
        return torch.bincount(shell, weights=v.reshape(-1), minlength=nsh + 1)[:nsh]

    num = sums((G1.conj() * G2).real)
    return num / torch.sqrt(sums(G1.abs().square()) * sums(G2.abs().square()))


def _calibrate64(case, t, ref):
    a = ref.to(torch.float64)
    m2 = a.mean().square()
    g = {ax: torch.stack([(a * torch.roll(a, -d, dims=ax)).mean() / m2 for d in range(33)]) for ax in (0, 1)}
    coh = {}
    for ax in (0, 1):
        s = (g[ax] - 1.0).cpu()
        k = 1
        while k + 1 < len(s) and s[k + 1] >= 0.02 * s[1]:
            k += 1
        d = torch.arange(1, k + 1, dtype=torch.float64)
        x, v = (d * PIXEL_M).square(), torch.log(s[1:k + 1])
        slope = ((x - x.mean()) * (v - v.mean())).sum() / (x - x.mean()).square().sum()
        coh[ax] = math.sqrt(-math.pi / float(slope))
    m = _Model(t, case["sigma"])
    w = m.filt(a.to(torch.complex128), m.iotf / (m.iotf.square() + WIENER_EPS)).real
    return {"x_coh_m": coh[1], "y_coh_m": coh[0], "g2x": g[1], "g2y": g[0],
            "t": m.filt(w.clamp_min(0.0).sqrt().to(torch.complex128), m.q2.conj())}


def exact(case, seed):
    kind = case["kind"]
    if kind == "tomogram":
        return {"vol": _tomogram64(case, *_sinogram(case, seed))}
    if kind == "shells":
        return {"fsc": _shells64(case, *_volumes(case, seed))}
    if kind == "calibrate":
        return _calibrate64(case, *_reference(case, seed))
    scene = _scene(case, seed)
    if kind == "joint":
        psi, t = _joint64(scene, case["iters"])
        return {"psi": [psi], "t": t}
    out = []
    for s in scene:
        res = []
        for i in range(s["n"]):
            m = _Model(s["t"][i if s["t"].shape[0] > 1 else 0], s["sigma"][i])
            y, psi = s["y"][i], s["psi"][i]
            if kind in ("solve", "steps"):
                res.append(_solve64(m, y, case["iters"], case.get("stop", False)))
                continue
            f, x, _, v = m.forward((0.5 * psi).to(torch.complex128))
            if kind == "forward":
                res.append(100.0 * (y.to(torch.float64) - f).abs() if case["rmse"] else f)
            else:
                loss, _, g = m.backward(f, x, v, y)
                res.append((4.0 * g, float(loss)))
        out.append(res)
    if kind == "solve":
        psi = [torch.stack([r[0] for r in res]) for res in out]
        if case["stop"]:
            return {"psi": psi, "iterations": torch.tensor([r[1] for res in out for r in res])}
        return {"psi": psi}
    if kind == "steps":
        return {"psi": [r[0] for r in out[0]]}
    if kind == "train":
        return {"grad": torch.stack([r[0] for r in out[0]]), "loss": [r[1] for r in out[0]]}
    return {"rmse" if case["rmse"] else "f": list(out[0])}
