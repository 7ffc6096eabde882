"""Timed cases of the channel library's public entry points.

A case is one piece of work that a program built on the package does again and
again: time steps of a channel (Channel.step, with or without the statistics
being read), adjoint steps of a sweep (Channel.adjoint_step), a whole training
step through the torch.autograd function (plane_statistics), or the inlet plane
at one time (Channel.stg_fill, Channel.stg_fill_noalloc).

listed() names the cases, draw() gives more of the same ranges, prepare() makes
what the program has in hand before the call, run() is one pass, work() the
bytes and operations a pass cannot do without, and exact() the same results in
64 bits from plain torch, with none of the package's code.
"""
import math

import numpy as np
import torch
import torch.utils.checkpoint

# Friction velocities whose Reichardt centreline speed is 0.1 at each Re_tau, lattice units.
U_TAU = {1000: 0.004448498381757104, 2000: 0.004137851781451391, 5200: 0.0037741807439038936}
KAPPA, B_REICH, U_CONV, CS, SPONGE_NU = 0.41, 7.8, 0.1, 0.1, 0.1
RATES = (1.0, 1.19, 1.6, 1.0, 1.2, 1.0, 1.2, 1.0, 1.2, 1.0, 1.6, 1.0, 1.6, 1.0, 1.0, 1.0, 1.98, 1.98, 1.98)

_STEP = dict(kind="step", storage="f32", ywall="slip", xbc="inflow", wall_model=True, wall_avg="local",
             wall_law="reichardt", outlet="convective", sponge=0, spectrum=False, modes=200, re=1000, force=0.0,
             planes=0, read=False, steps=1)
_ADJ = dict(kind="adjoint", storage="f32", ywall="slip", xbc="inflow", wall_model=True, wall_avg="local",
            wall_law="reichardt", outlet="convective", sponge=0, spectrum=False, modes=200, re=1000, force=0.0,
            planes=1, steps=3)


def listed():
    return [
        # a program that looks at the flow after every step: the smallest lattice, one step a call
        dict(_STEP, name="one step 64x32x32", nx=64, ny=32, nz=32, ywall="bounceback", wall_model=False, modes=100,
             re=0, steps=1),
        # the inflow-recovery run at its coarsest: 20 cells across, the outlet sponge, long runs of small steps
        dict(_STEP, name="recovery 200x20x16", nx=200, ny=20, nz=16, sponge=10, steps=100),
        # the same at 40 cells in FP16, per-row spectra, its statistics sampled on twelve planes and read
        dict(_STEP, name="recovery 400x40x32 f16", nx=400, ny=40, nz=32, sponge=20, storage="f16ref", spectrum=True,
             re=5200, planes=12, read=True, steps=50),
        # a body-forced periodic channel of odd sizes with resting walls
        dict(_STEP, name="ragged 150x45x101", nx=150, ny=45, nz=101, ywall="bounceback", xbc="periodic",
             wall_model=False, re=0, force=1e-6, steps=9),
        # the Re_tau = 1000 channel while its statistics are sampled, in both storages of record
        dict(_STEP, name="re1000 768x64x192", nx=768, ny=64, nz=192, planes=4, steps=7),
        dict(_STEP, name="re1000 768x64x192 f16", nx=768, ny=64, nz=192, storage="f16ref", planes=4, steps=10),
        # the Re_tau = 5200 channel: the largest runs
        dict(_STEP, name="re5200 1536x128x384", nx=1536, ny=128, nz=384, modes=300, re=5200, planes=4, steps=4),
        dict(_STEP, name="re5200 1536x128x384 f16", nx=1536, ny=128, nz=384, storage="f16dev", modes=300, re=5200,
             steps=4),
        # adjoint steps in the middle of a sweep, the states and inlet planes kept by the recompute
        dict(_ADJ, name="adjoint 256x64x64", nx=256, ny=64, nz=64),
        dict(_ADJ, name="adjoint 512x64x128 f16", nx=512, ny=64, nz=128, storage="f16ref", modes=300),
        # a training step: forward statistics with checkpoints, loss, recompute and adjoint sweep
        dict(_ADJ, name="gradient 256x64x64", kind="gradient", nx=256, ny=64, nz=64, steps=30),
        # the inlet plane alone, as a program that couples or inspects the inflow takes it
        dict(_STEP, name="inlet 128x384", kind="inlet", nx=8, ny=128, nz=384, modes=300, re=5200, noalloc=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step",) * 5 + ("adjoint", "adjoint", "gradient", "inlet", "inlet"))
    base = _ADJ if kind in ("adjoint", "gradient") else _STEP
    big = kind == "step"
    while True:
        nx, ny, nz = _log_int(rng, 16, 1536 if big else 512), _log_int(rng, 8, 160), _log_int(rng, 8, 384)
        if nx * ny * nz <= (40_000_000 if big else 4_200_000):
            break
    if rng.random() < 0.5:  # multiples of eight are as common as odd sizes
        nx, ny, nz = (max(8, 8 * round(v / 8)) for v in (nx, ny, nz))
    ywall = rng.choice(("slip", "slip", "slip", "bounceback", "periodic"))
    wall_model = ywall != "periodic" and rng.random() < 0.7
    xbc = "inflow" if kind in ("inlet", "gradient") or rng.random() < 0.75 else "periodic"
    real = ywall == "slip" and wall_model
    c = dict(base, kind=kind, nx=nx, ny=ny, nz=nz, ywall=ywall, wall_model=wall_model, xbc=xbc,
             storage=rng.choice(("f32", "f32", "f16ref", "f16dev")), re=rng.choice((1000, 2000, 5200)) if real else 0,
             wall_avg="line" if wall_model and rng.random() < 0.15 else "local",
             wall_law="musker" if wall_model and rng.random() < 0.2 else "reichardt",
             outlet=rng.choice(("convective", "convective", "zero-gradient")),
             sponge=min(nx // 3, ny // 2) if xbc == "inflow" and rng.random() < 0.4 else 0,
             spectrum=ywall != "periodic" and xbc == "inflow" and rng.random() < 0.3, modes=_log_int(rng, 30, 400),
             force=0.0 if xbc == "inflow" else 1e-6)
    if kind == "step":
        c["steps"] = max(1, min(100, _log_int(rng, 1, 100), 250_000_000 // (nx * ny * nz)))
        c["planes"] = rng.choice((0, 0, 1, 4, 12)) if nx >= 24 else 0
        c["read"] = c["planes"] > 0 and rng.random() < 0.5
    elif kind == "adjoint":
        c["steps"], c["planes"] = rng.randint(1, 4), 1
    elif kind == "gradient":
        c["steps"] = max(3, min(_log_int(rng, 4, 40), 30_000_000 // (nx * ny * nz)))
    else:
        c["nx"], c["noalloc"] = 8, rng.random() < 0.5
        c["sponge"] = min(c["sponge"], 4)
        while c["noalloc"] and 8 * c["modes"] * nz + (4 * ny * c["modes"] if c["spectrum"] else 0) > 3_500_000:
            c["modes"] //= 2  # the tables have to fit in the library's scratch
    return c


def work(case):
    """The state read and written once (19 populations a node), the inlet planes' mode sums, and a node's collision
    (about 330 operations: two moment transforms, the relaxation and the equilibrium; its adjoint three times that)."""
    n, face = case["nx"] * case["ny"] * case["nz"], case["ny"] * case["nz"]
    pop = 19 * (4 if case["storage"] == "f32" else 2)
    stg = 8.0 * case["modes"] * face if case["xbc"] == "inflow" else 0.0
    k = case["steps"]
    if case["kind"] == "inlet":
        return {"bytes": 12.0 * face, "flops": stg}
    if case["kind"] == "step":
        return {"bytes": 2.0 * pop * n, "flops": k * (330.0 * n + stg)}
    if case["kind"] == "adjoint":
        return {"bytes": k * float(pop) * n + 2 * 76.0 * n, "flops": k * 1000.0 * n}
    return {"bytes": 2.0 * pop * n, "flops": k * (2 * 330.0 * n + 1000.0 * n + stg)}


# ---------------------------------------------------------------- inputs, shared by prepare() and exact()

def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _physics(case):
    """tau0, u_tau and the mean inflow U(y): the Reichardt law of the case's Re_tau, or a mild one at tau0 = 0.52."""
    ny = case["ny"]
    delta = ny / 2.0
    u_tau = U_TAU[case["re"]] if case["re"] else 0.008
    nu0 = u_tau * delta / case["re"] if case["re"] else 0.02 / 3
    d = np.minimum(np.arange(ny) + 0.5, ny - np.arange(ny) - 0.5)
    yp = d * u_tau / nu0
    U = u_tau * (np.log1p(KAPPA * yp) / KAPPA - B_REICH * (np.expm1(-yp / 11) + yp / 11 * np.exp(-yp / 3)))
    return 0.5 + 3 * nu0, u_tau, np.minimum(U, 0.11)


def _stg_inputs(case, seed):
    """Random Fourier modes, mean inflow, Reynolds stresses, amplitude bins and (optional) RANS k, omega."""
    _, u_tau, U = _physics(case)
    g = np.random.Generator(np.random.PCG64(seed))
    n, ny = case["modes"], case["ny"]
    delta = ny / 2.0
    ct, az = g.uniform(-1, 1, n), g.uniform(0, 2 * np.pi, n)
    st = np.sqrt(1 - ct * ct)
    d = np.stack([st * np.cos(az), st * np.sin(az), ct])
    ref = np.where(np.abs(d[0]) < 0.9, [[1.0], [0.0], [0.0]], [[0.0], [1.0], [0.0]])
    e1 = np.cross(d.T, ref.T).T
    e1 /= np.linalg.norm(e1, axis=0)
    ang = g.uniform(0, 2 * np.pi, n)
    sigma = np.cos(ang) * e1 + np.sin(ang) * np.cross(d.T, e1.T).T
    kmag = np.geomspace(np.pi / (2 * delta) if case["spectrum"] else 2 * np.pi / delta, 1.5 * np.pi, n)
    r = kmag * delta / (4 * np.pi)
    q = r ** 4 / (1 + 2.4 * r * r) ** (17 / 6) * np.exp(-(12 * kmag / (4 * np.pi)) ** 2) * np.gradient(kmag)
    modes = dict(q=q / q.sum(), sigma=sigma, kmag=kmag, d=d, phi=g.uniform(0, 2 * np.pi, n),
                 omega=g.normal(0, 2 * np.pi, n) * 0.1 / delta)
    eta = (np.arange(ny) + 0.5) / delta - 1
    R = np.zeros((6, ny))
    R[0], R[1], R[2], R[5] = 1 + 3 * eta ** 2, eta, 0.5 + 0.5 * eta ** 2, 0.7 + 0.8 * eta ** 2
    R *= u_tau ** 2
    k = om = None
    if case["spectrum"]:
        k = 0.5 * (R[0] + R[2] + R[5])
        dw = np.minimum(np.arange(ny) + 0.5, ny - np.arange(ny) - 0.5)
        om = np.sqrt(k) / (0.09 ** 0.25 * np.minimum(0.41 * dw, 0.09 * delta))
    amp = 1 + 0.1 * g.uniform(-1, 1, ny)
    return dict(modes=modes, U=np.stack([U, 0 * U, 0 * U]), R=R, amp=amp, bins=np.arange(ny, dtype=np.int32), k=k, om=om)


def _c():
    """Velocity set, lexicographic in (c_z, c_y, c_x): c [19, 3] and weights."""
    c = [(x, y, z) for z in (-1, 0, 1) for y in (-1, 0, 1) for x in (-1, 0, 1) if abs(x) + abs(y) + abs(z) < 3]
    return c, [{0: 1 / 3, 1: 1 / 18, 2: 1 / 36}[abs(x) + abs(y) + abs(z)] for x, y, z in c]


def _populations(case, seed, k=0):
    """A developed-looking state: the mean inflow with large-scale and grid-scale fluctuations and a small
    non-equilibrium part, float32 [19, nx, ny, nz]."""
    dev, (nx, ny, nz) = _device(), (case["nx"], case["ny"], case["nz"])
    g = torch.Generator(device=dev)
    g.manual_seed(1000003 * seed + k)
    U = torch.as_tensor(_physics(case)[2], device=dev)[:, None]
    x, y, z = (torch.arange(n, device=dev, dtype=torch.float64) for n in (nx, ny, nz))
    u = []
    for a in range(3):
        ph = 6.2831853 * torch.rand(3, generator=g, device=dev, dtype=torch.float64)
        wave = torch.sin(12.566371 * x / nx + ph[0])[:, None, None] * torch.sin(6.2831853 * y / ny + ph[1])[:, None] * \
            torch.sin(12.566371 * z / nz + ph[2])
        u.append(4e-3 * wave + 1e-3 * (2 * torch.rand((nx, ny, nz), generator=g, device=dev) - 1) + (U if a == 0 else 0))
    rho = 1 + 1e-3 * (2 * torch.rand((nx, ny, nz), generator=g, device=dev) - 1)
    uu = 1.5 * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2])
    f = torch.empty((19, nx, ny, nz), dtype=torch.float32, device=dev)
    for i, (ci, w) in enumerate(zip(*_c())):
        cu = ci[0] * u[0] + ci[1] * u[1] + ci[2] * u[2]
        noise = 2 * torch.rand((nx, ny, nz), generator=g, device=dev) - 1
        f[i] = w * (rho * (1 + 3 * cu + 4.5 * cu * cu - uu) + 1e-3 * noise)
    return f


_OUT5 = [1, 5, 8, 11, 15]  # the directions of the outlet history: c_x = -1


def _planes(case):
    p = case["planes"]
    if case["kind"] == "gradient":  # near enough to the inlet for its waves to arrive within the run
        return [min(case["nx"] - 2, max(1, case["steps"] // 3))]
    return [] if not p else sorted({min(case["nx"] - 2, max(1, (j + 1) * case["nx"] // (p + 1))) for j in range(p)})


def _normal(shape, seed, scale=1.0):
    g = torch.Generator(device=_device())
    g.manual_seed(seed)
    return scale * torch.randn(shape, generator=g, device=_device(), dtype=torch.float32)


def _coef(case, seed):
    """dL/d(sums over z) of a statistics loss on the sampled planes."""
    return _normal((len(_planes(case)), case["ny"], 9), 7 * seed + 1, 1e-3)


# ---------------------------------------------------------------- the package's side

def _channel(case, seed):
    from paper_2304_04214_amd.channel import Channel
    tau0, _, U = _physics(case)
    ch = Channel(case["nx"], case["ny"], case["nz"], tau0=tau0, ywall=case["ywall"], xbc=case["xbc"],
                 storage="f32" if case["storage"] == "f32" else "f16dev", wall_model=case["wall_model"],
                 cs_smag=CS, u_conv=U_CONV, g=(case["force"], 0.0, 0.0), sponge_cells=case["sponge"],
                 sponge_nu=SPONGE_NU if case["sponge"] else 0.0, outlet=case["outlet"], wall_law=case["wall_law"],
                 wall_avg=case["wall_avg"])
    for b in ch.f:
        b.zero_()
    if case["storage"] == "f16ref":
        ch.set_reference(U)
    if case["xbc"] == "inflow":
        s = _stg_inputs(case, seed)
        ch.set_stg(s["modes"], s["U"], s["R"], s["amp"], s["bins"], want_fluct=case["kind"] == "inlet",
                   k_rans=s["k"], omega_rans=s["om"])
    return ch


def _load(case, ch, f):
    ch.load_populations(f)
    if case["xbc"] == "inflow":
        ch.state()[1].copy_(f[_OUT5, case["nx"] - 1])


def prepare(case, seed):
    ch = _channel(case, seed)
    s = dict(case=case, ch=ch)
    if case["kind"] == "inlet":
        s["t"] = 1 + seed % 1000
        return s
    if case["kind"] == "step":
        _load(case, ch, _populations(case, seed))
        if case["planes"]:
            ch.stats_attach(_planes(case))
        return s
    if case["kind"] == "gradient":
        from paper_2304_04214_amd.adjoint import StatsGradient
        _load(case, ch, _populations(case, seed))
        s["run"] = StatsGradient(ch, _planes(case), case["steps"])
        st = _stg_inputs(case, seed)
        s["amp"] = torch.tensor(st["amp"], dtype=torch.float32, requires_grad=True)
        s["cs"] = torch.tensor(CS, dtype=torch.float32, requires_grad=True)
        s["target"] = torch.as_tensor(st["U"][0] * 1.05), torch.as_tensor(st["R"][1])
        return s
    ch.stats_attach(_planes(case))
    ch.stats_detach()
    s["states"], s["inlets"] = [], []
    for j in range(case["steps"]):
        _load(case, ch, _populations(case, seed, j))
        s["states"].append(tuple(t.clone() for t in ch.state()))
        if case["xbc"] == "inflow":
            s["inlets"].append(tuple(t.float().contiguous() for t in _inlet(case, seed, j + 1.0)))
    s["lam0"] = ch.field_import(_normal((19, case["nx"], case["ny"], case["nz"]), 7 * seed + 2))
    s["eta0"] = _normal((5, case["ny"], case["nz"]), 7 * seed + 3)
    s["lam"], s["eta"] = [ch.new_field(), ch.new_field()], [torch.zeros_like(s["eta0"]) for _ in range(2)]
    s["coef"], s["g_uin"] = _coef(case, seed), torch.zeros((3, case["ny"], case["nz"]), device=s["eta0"].device)
    return s


def run(s):
    case, ch = s["case"], s["ch"]
    if case["kind"] == "inlet":
        s["t"] += 1
        u = (ch.stg_fill_noalloc if case["noalloc"] else ch.stg_fill)(s["t"])
        return {"u": u, "fluct": ch.fluct}
    if case["kind"] == "step":
        ch.step(case["steps"])
        f, hist = ch.state()
        out = {"f": f}
        if case["xbc"] == "inflow":
            out["hist"] = hist
        if case["read"]:  # the means go on as a float32 tensor
            out["means"] = torch.as_tensor(ch.stats_read()[0], dtype=torch.float32)
        return out
    if case["kind"] == "gradient":
        from paper_2304_04214_amd.adjoint import mean_profile_loss, plane_statistics
        amp, cs = s["amp"], s["cs"]
        amp.grad = cs.grad = None
        m = plane_statistics(s["run"], amp, cs)
        loss = mean_profile_loss(m[0], *s["target"])
        loss.backward()
        return {"loss": loss.detach().float(), "amp": amp.grad, "cs": cs.grad}
    inflow = case["xbc"] == "inflow"
    lam, eta = s["lam0"], s["eta0"] if inflow else None
    for j in reversed(range(case["steps"])):
        to, eto = s["lam"][j % 2], s["eta"][j % 2] if inflow else None
        u, fl = s["inlets"][j] if inflow else (None, None)
        ch.adjoint_step(*s["states"][j], j + 1.0, lam, to, eta, eto, coef=s["coef"],
                        g_uin=s["g_uin"] if inflow else None, u_in=u, fluct=fl)
        lam, eta = to, eto
    return {"lam": lam, "eta": eta, "g_uin": s["g_uin"]} if inflow else {"lam": lam}


# ---------------------------------------------------------------- the same in 64 bits

def _basis():
    """The moment matrix M [19, 19] of the D3Q19 MRT scheme (orthogonal rows)."""
    c = np.array(_c()[0], dtype=np.float64)
    x, y, z = c.T
    n = (c * c).sum(1)
    a, b, s = 3 * x * x - n, y * y - z * z, 3 * n - 5
    return np.stack([n ** 0, 19 * n - 30, (21 * n * n - 53 * n + 24) / 2, x, (5 * n - 9) * x, y, (5 * n - 9) * y, z,
                     (5 * n - 9) * z, a, s * a, b, s * b, x * y, y * z, x * z, b * x, (z * z - x * x) * y,
                     (x * x - y * y) * z])


def _t(x):
    return torch.as_tensor(x, dtype=torch.float64, device=_device())


def _weights(case, s):
    """Mode amplitudes sqrt(6 q) of each row, [ny or 1, N]."""
    m = s["modes"]
    if s["k"] is None:
        return _t(np.sqrt(6 * m["q"]))[None]
    nu = (_physics(case)[0] - 0.5) / 3
    ny, kn = case["ny"], m["kmag"]
    dw = np.minimum(np.arange(ny) + 0.5, ny - np.arange(ny) - 0.5)
    ke = (2 * np.pi / np.minimum(2 * dw, 3 * np.sqrt(s["k"]) / (0.09 * s["om"])))[:, None]
    keta = (2 * np.pi / (nu ** 3 / (0.09 * s["k"] * s["om"])) ** 0.25)[:, None]
    r = kn / ke
    e = r ** 4 / (1 + 2.4 * r * r) ** (17 / 6) * np.exp(-(12 * kn / keta) ** 2) * \
        np.exp(-(4 * np.maximum(kn - 0.9 * np.pi, 0) / np.pi) ** 3) * np.gradient(kn)
    return _t(np.sqrt(6 * e / e.sum(1, keepdims=True)))


def _mm(a, x):
    """a @ x for a [19, 19] and x [19, nodes], over ranges of nodes that 32-bit offsets reach."""
    return torch.cat([a @ v.contiguous() for v in x.split(1 << 22, 1)], 1)


def _inlet(case, seed, t):
    """u_in and a v' at time t: float64 [3, ny, nz] each."""
    s = _stg_inputs(case, seed)
    m, ny, nz = s["modes"], case["ny"], case["nz"]
    amp, sig = _weights(case, s), _t(m["sigma"])
    rows = _t(m["kmag"] * m["d"][1])[None] * (torch.arange(ny, device=_device())[:, None] + 0.5) + \
        _t(m["omega"] * t + m["phi"])[None]
    cols = _t(m["kmag"] * m["d"][2])[:, None] * torch.arange(nz, device=_device())
    a, b = torch.cos(rows) * amp, torch.sin(rows) * amp
    v = [(a * sig[k]) @ torch.cos(cols) - (b * sig[k]) @ torch.sin(cols) for k in range(3)]
    R = s["R"]
    a11 = np.sqrt(R[0])
    a21, a31 = R[1] / a11, R[3] / a11
    a22 = np.sqrt(R[2] - a21 ** 2)
    a32 = (R[4] - a21 * a31) / a22
    a33 = np.sqrt(R[5] - a31 ** 2 - a32 ** 2)
    a11, a21, a22, a31, a32, a33 = (_t(w)[:, None] for w in (a11, a21, a22, a31, a32, a33))
    fl = torch.stack([a11 * v[0], a21 * v[0] + a22 * v[1], a31 * v[0] + a32 * v[1] + a33 * v[2]])
    return _t(s["U"])[:, :, None] + _t(s["amp"])[:, None] * fl, fl


def _law(case, yp):
    """u+ and its derivative."""
    if case["wall_law"] == "musker":
        t, t0 = (2 * yp - 8.15) / 16.7, -8.15 / 16.7
        up = 5.424 * torch.atan2(2 * yp / 16.7, 1 + t0 * t) + \
            (9.6 * torch.log1p(yp / 10.6) - 2 * torch.log1p(yp * (yp - 8.15) / 86)) / math.log(10)
        q = yp * yp - 8.15 * yp + 86
        return up, 5.424 * (2 / 16.7) / (1 + t * t) + (9.6 / (yp + 10.6) - 2 * (2 * yp - 8.15) / q) / math.log(10)
    e11, e3 = torch.exp(-yp / 11), torch.exp(-yp / 3)
    up = torch.log1p(KAPPA * yp) / KAPPA - B_REICH * (torch.expm1(-yp / 11) + yp / 11 * e3)
    return up, 1 / (1 + KAPPA * yp) + B_REICH * ((e11 - e3) / 11 + yp / 33 * e3)


def _u_tau(case, ua, nu0):
    """The root of u_tau u+(u_tau / 2 nu0) = ua with its derivative: Newton, the last step differentiable."""
    with torch.no_grad():
        ut = torch.sqrt(nu0 * ua / 0.5)
        for _ in range(12):
            up, dup = _law(case, 0.5 * ut / nu0)
            ut = ut - (ut * up - ua) / (up + 0.5 * ut / nu0 * dup)
    up, dup = _law(case, 0.5 * ut / nu0)
    return ut - (ut * up - ua) / (up + 0.5 * ut / nu0 * dup)


def _wall_force(case, nu0, rho, uw, u2):
    """(F_x, F_z) of a first off-wall row from its own and the next row's velocities (x, z), each [nx, 1, nz]."""
    tn = torch.sqrt(u2[0] ** 2 + u2[1] ** 2)
    ex, ez = u2[0] / tn, u2[1] / tn
    uh = uw[0] * ex + uw[1] * ez
    if case["wall_avg"] == "line":
        uh = uh.mean(2, keepdim=True)
    ut = _u_tau(case, uh.abs(), nu0)
    tw = -torch.sign(uh) * rho * ut * ut
    return tw * ex, tw * ez


def _step64(case, f, hist, uin, cs):
    """One time step on post-collision populations f [19, nx, ny, nz]: (f, outlet history, velocity)."""
    c, w = _c()
    idx = {v: i for i, v in enumerate(c)}
    nx, ny = case["nx"], case["ny"]
    tau0 = _physics(case)[0]
    nu0 = (tau0 - 0.5) / 3
    p = []
    for i, (cx, cy, cz) in enumerate(c):
        v = torch.roll(f[i], (cx, cy, cz), (0, 1, 2))
        if cy and case["ywall"] != "periodic":
            row = 0 if cy > 0 else ny - 1
            if case["ywall"] == "slip":
                e = torch.roll(f[idx[cx, -cy, cz], :, row], (cx, cz), (0, 1))
            else:
                e = f[idx[-cx, -cy, -cz], :, row]
            v = torch.cat([e[:, None], v[:, 1:]] if cy > 0 else [v[:, :-1], e[:, None]], 1)
        p.append(v)
    if case["xbc"] == "inflow":
        wh, wu = (1 / (1 + U_CONV), U_CONV / (1 + U_CONV)) if case["outlet"] == "convective" else (0.0, 1.0)
        hist = torch.stack([wh * hist[k] + wu * p[i][nx - 2] for k, i in enumerate(_OUT5)])
        for k, i in enumerate(_OUT5):
            p[i] = torch.cat([p[i][:-1], hist[k][None]])
        m0 = sum(p[i][0] for i in range(19) if c[i][0] == 0)
        mm = sum(p[i][0] for i in range(19) if c[i][0] < 0)
        rin = (m0 + 2 * mm) / (1 - uin[0])
        uu = uin[0] ** 2 + uin[1] ** 2 + uin[2] ** 2
        feq, pi = [], [[0.0] * 3 for _ in range(3)]
        for i in range(19):
            cu = c[i][0] * uin[0] + c[i][1] * uin[1] + c[i][2] * uin[2]
            feq.append(w[i] * rin * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * uu))
        for i in range(19):
            j = i if c[i][0] <= 0 else 18 - i
            fn = p[j][0] - feq[j]
            for a in range(3):
                for b in range(3):
                    pi[a][b] = pi[a][b] + (c[i][a] * c[i][b] - (a == b) / 3) * fn
        for i in range(19):
            qp = sum((c[i][a] * c[i][b] - (a == b) / 3) * pi[a][b] for a in range(3) for b in range(3))
            p[i] = torch.cat([(feq[i] + 4.5 * w[i] * qp)[None], p[i][1:]])
    shape = f.shape[1:]
    M = _basis()
    p = torch.stack(p).reshape(19, -1)
    m = _mm(_t(M), p)
    rho, j = m[0].reshape(shape), [m[k].reshape(shape) for k in (3, 5, 7)]
    F = [rho * case["force"], None, None]
    if case["wall_model"]:
        u = [j[0] / rho, j[2] / rho]
        r = lambda t, y: t[:, y:y + 1]  # noqa: E731
        bx, bz = _wall_force(case, nu0, r(rho, 0), [r(t, 0) for t in u], [r(t, 1) for t in u])
        tx, tz = _wall_force(case, nu0, r(rho, ny - 1), [r(t, ny - 1) for t in u], [r(t, ny - 2) for t in u])
        mid = torch.zeros_like(rho[:, 2:])
        F[0] = F[0] + torch.cat([bx, mid, tx], 1)
        F[2] = torch.cat([bz, mid, tz], 1)
    zero = torch.zeros((), dtype=f.dtype, device=f.device)
    F = [(zero if t is None else t.reshape(-1)) for t in F]
    rho = m[0]
    q = [m[k] + 0.5 * F[a] for a, k in enumerate((3, 5, 7))]
    ux, uy, uz = (t / rho for t in q)
    uu = ux * ux + uy * uy + uz * uz
    q9, q11 = rho * (2 * ux * ux - uy * uy - uz * uz), rho * (uy * uy - uz * uz)
    eq = {0: rho, 1: rho * (19 * uu - 11), 2: rho * (3 - 5.5 * uu), 3: q[0], 4: -2 / 3 * q[0], 5: q[1],
          6: -2 / 3 * q[1], 7: q[2], 8: -2 / 3 * q[2], 9: q9, 10: -0.5 * q9, 11: q11, 12: -0.5 * q11,
          13: rho * ux * uy, 14: rho * uy * uz, 15: rho * ux * uz}
    uF = ux * F[0] + uy * F[1] + uz * F[2]
    F9, F11 = 2 * (2 * ux * F[0] - uy * F[1] - uz * F[2]), 2 * (uy * F[1] - uz * F[2])
    Fm = {1: 38 * uF, 2: -11 * uF, 3: F[0], 4: -2 / 3 * F[0], 5: F[1], 6: -2 / 3 * F[1], 7: F[2], 8: -2 / 3 * F[2],
          9: F9, 10: -0.5 * F9, 11: F11, 12: -0.5 * F11, 13: ux * F[1] + uy * F[0], 14: uy * F[2] + uz * F[1],
          15: ux * F[2] + uz * F[0]}
    e = {k: m[k] - eq[k] for k in (1, 9, 11, 13, 14, 15)}
    dc2 = e[1] / 19
    pxx = (e[9] + dc2) / 3
    pyy, pzz = 0.5 * (dc2 - pxx + e[11]), 0.5 * (dc2 - pxx - e[11])
    qh = torch.sqrt(pxx ** 2 + pyy ** 2 + pzz ** 2 + 2 * (e[13] ** 2 + e[14] ** 2 + e[15] ** 2))
    t0 = torch.full((nx, 1, 1), tau0, dtype=f.dtype, device=f.device)
    if case["sponge"]:
        L = case["sponge"]
        r = (torch.arange(nx - L, nx, device=f.device) - (nx - L) + 1) / L
        t0[nx - L:, 0, 0] = 0.5 + 3 * (nu0 + (SPONGE_NU - nu0) * r.double() ** 2)
    t0 = t0.expand(shape).reshape(-1)
    sv = 1 / (0.5 * t0 + 0.5 * torch.sqrt(t0 * t0 + 18 * math.sqrt(2.0) * cs * cs * qh / rho))
    delta = []
    for k in range(19):
        s = sv if k in (9, 11, 13, 14, 15) else RATES[k]
        if k in (0, 3, 5, 7):  # conserved: the force alone
            delta.append(torch.zeros_like(rho) if k == 0 else Fm[k] + torch.zeros_like(rho))
        else:
            delta.append(-s * (m[k] - eq.get(k, 0.0)) + (1 - 0.5 * s) * Fm.get(k, 0.0))
    out = p + _mm(_t(M.T / (M * M).sum(1)), torch.stack(delta))
    return out.reshape(f.shape), hist, torch.stack([t.reshape(shape) for t in (ux, uy, uz)])


def _reference(case):
    """Offsets of the stored populations, [19, 1, ny, 1]: the weights, with f16ref the equilibrium at U(y)."""
    c, w = _c()
    U = _physics(case)[2]
    r = np.zeros((19, case["ny"]))
    if case["storage"] == "f16ref":
        for i in range(19):
            cu = c[i][0] * U
            r[i] = (w[i] * (3.0 * cu + 4.5 * cu * cu - 1.5 * (U * U))).astype(np.float32)
    return np.array(w)[:, None], r


def _stored(case, f):
    """What the library's import keeps of float32 populations, as float64."""
    if case["storage"] == "f32":
        return f.double()
    w, r = _reference(case)
    out = torch.empty(f.shape, dtype=torch.float64, device=f.device)
    for i in range(19):
        ri = torch.as_tensor(r[i], dtype=torch.float32, device=f.device)[:, None]
        out[i] = ((f[i] - np.float32(w[i, 0])) - ri).half().double() + ri.double() + w[i, 0]
    return out


def _bricks(f):
    """[19, nx, ny, nz] as the library's 64-node bricks (nx, zc, ny, 19, 64), zeros in the padding."""
    _, nx, ny, nz = f.shape
    zc = (nz + 63) // 64
    b = torch.zeros((nx, zc, ny, 19, 64), dtype=f.dtype, device=f.device)
    for z in range(zc):
        n = min(64, nz - 64 * z)
        b[:, z, :, :, :n] = f[..., 64 * z:64 * z + n].permute(1, 2, 0, 3)
    return b


def _sums(u, planes):
    """Sums over z of u v w uu vv ww uv uw vw at the planes: [planes, ny, 9]."""
    v = u[:, planes]
    return torch.stack([t.sum(-1) for t in (v[0], v[1], v[2], v[0] ** 2, v[1] ** 2, v[2] ** 2, v[0] * v[1],
                                            v[0] * v[2], v[1] * v[2])], -1)


def exact(case, seed):
    inflow = case["xbc"] == "inflow"
    if case["kind"] == "inlet":
        u, fl = _inlet(case, seed, 2.0 + seed % 1000)
        return {"u": u, "fluct": fl}
    hist0 = lambda f: f[_OUT5, case["nx"] - 1].double() if inflow else None  # noqa: E731
    if case["kind"] == "step":
        with torch.no_grad():
            f = _populations(case, seed)
            hist, f = hist0(f), _stored(case, f)
            planes, acc = _planes(case), 0.0
            for n in range(case["steps"]):
                f, hist, u = _step64(case, f, hist, _inlet(case, seed, n + 1.0)[0] if inflow else None, CS)
                if case["read"]:
                    acc = acc + _sums(u, planes)
                del u
            if case["storage"] != "f32":
                w, r = _reference(case)
                for i in range(19):
                    f[i] -= w[i, 0] + _t(r[i])[:, None]
            out = {"f": _bricks(f)}
            if inflow:
                out["hist"] = hist
            if case["read"]:
                out["means"] = acc / (case["nz"] * case["steps"])
            return out
    if case["kind"] == "gradient":
        s = _stg_inputs(case, seed)
        amp = _t(s["amp"]).float().double().requires_grad_()
        cs = _t(CS).float().double().requires_grad_()
        f = _populations(case, seed)
        hist, f = hist0(f), _stored(case, f)
        U, acc = _t(s["U"])[:, :, None], 0.0

        def one(f, hist, amp, cs, fl):
            f, hist, u = _step64(case, f, hist, U + amp[:, None] * fl, cs)
            return f, hist, _sums(u, _planes(case))

        for n in range(case["steps"]):
            f, hist, t = torch.utils.checkpoint.checkpoint(one, f, hist, amp, cs, _inlet(case, seed, n + 1.0)[1],
                                                           use_reentrant=False)
            acc = acc + t
        m = acc[0] / (case["nz"] * case["steps"])
        ut, r12 = U[0, :, 0] * 1.05, _t(s["R"][1])
        loss = ((m[:, 0] - ut) ** 2).sum() / (ut ** 2).sum() + \
            ((m[:, 6] - m[:, 0] * m[:, 1] - r12) ** 2).sum() / (r12 ** 2).sum()
        loss.backward()
        return {"loss": loss.detach(), "amp": amp.grad, "cs": cs.grad}
    lam = _normal((19, case["nx"], case["ny"], case["nz"]), 7 * seed + 2).double()
    eta = _normal((5, case["ny"], case["nz"]), 7 * seed + 3).double()
    coef, g_uin = _coef(case, seed).double(), None
    for j in reversed(range(case["steps"])):
        f = _populations(case, seed, j)
        hist, f = hist0(f), _stored(case, f).requires_grad_()
        uin = None
        if inflow:
            hist.requires_grad_()
            uin = _inlet(case, seed, j + 1.0)[0].float().double().requires_grad_()
        f1, h1, u = _step64(case, f, hist, uin, CS)
        loss = (f1 * lam).sum() + (_sums(u, _planes(case)) * coef).sum()
        if inflow:
            loss = loss + (h1 * eta).sum()
        got = torch.autograd.grad(loss, [f] + ([hist, uin] if inflow else []))
        lam = got[0]
        if inflow:
            eta, g_uin = got[1], got[2]
        del f1, h1, u, loss, f
    return {"lam": _bricks(lam), "eta": eta, "g_uin": g_uin} if inflow else {"lam": _bricks(lam)}
