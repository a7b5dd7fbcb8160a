"""The work that programs have this framework do, as timed cases.

Every case is one program's inner loop through the public entry points: a
lattice advanced some steps and its fields read, a batch of channels driven to
its next convergence check, a coupled step of the droplet or of the
magnetohydrodynamic runs, one convolution layer's training passes, and the
warm-start network's inference.  `exact` gives the same results in plain FP64
torch, straight from the method's equations.
"""
import math

import numpy as np
import torch

from paper_1905_10182_amd import Lattice, cmnn, warmstart
from paper_1905_10182_amd.cmlbm2d import Lattice2D
from paper_1905_10182_amd.mhd import CoupledMHD
from paper_1905_10182_amd.unet import UNet3D

DEV = "cuda:0"
F64 = torch.float64


def listed():
    return [
        # the smallest lattice in use: the Poiseuille start-up channel, FP64, walls in y, a few
        # hundred wavefronts a step, so launches and latency are all there is
        dict(name="channel_fp64", kind="box", storage="fp64", nx=32, ny=16, nz=16, steps=100, tau=0.8,
             force="uniform", walls=True),
        # the headline run: a periodic Taylor-Green vortex in FP32, fields read every 20 steps
        dict(name="vortex_fp32", kind="box", storage="fp32", nx=256, ny=256, nz=256, steps=20, tau=0.5038,
             force="none", walls=False),
        # a double-precision run on an odd-sized box with a force field of its own in every cell
        dict(name="ragged_fp64", kind="box", storage="fp64", nx=250, ny=191, nz=130, steps=10, tau=0.55,
             force="field", walls=False),
        # the sinusoidally forced box of the precision study in 16-bit storage with stochastic rounding
        dict(name="kolmogorov_fp16sr", kind="box", storage="fp16sr", nx=384, ny=384, nz=384, steps=10, tau=0.5005,
             force="profile_y", walls=False),
        # the largest vortex, in moment storage
        dict(name="vortex_mom32", kind="box", storage="mom32", nx=512, ny=512, nz=512, steps=10, tau=0.5076,
             force="none", walls=False),
        # warm-start data generation and solving: 64 channels with sphere obstacles, one convergence check
        dict(name="spheres_fp64", kind="channels", nb=64, check=100),
        # the Shan-Chen droplet: density, force and step in turn
        dict(name="droplet_fp32", kind="droplet", n=200, storage="fp32", steps=4),
        # the three-dimensional Orszag-Tang vortex: fluid and magnetic lattice in turn
        dict(name="orszag_tang_fp64", kind="mhd", n=128, storage="fp64", current="stencil", steps=4),
        # a rung of the four-rolls convergence study: a small plane advanced very many steps
        dict(name="rolls_fp64", kind="rolls", n=64, storage="fp64", steps=200),
        # the largest four-rolls plane
        dict(name="rolls_fp32", kind="rolls", n=8192, storage="fp32", steps=10),
        # the layer that most of the network's training time goes to: forward, data gradient with the
        # activation gradient of the layer below, weight gradient
        dict(name="conv_train", kind="conv", batch=16, d=32, h=32, w=64, cin=32, cout=32),
        # warm-start inference: the whole network on 16 channels
        dict(name="unet_infer", kind="unet", batch=16, d=32, h=32, w=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["box", "box", "box", "box", "channels", "droplet", "mhd", "rolls", "rolls", "conv", "conv", "unet"])
    if kind == "box":
        storage = rng.choice(["fp32", "fp32", "fp64", "fp64", "mom32", "fp16", "fp16sr", "bf16", "bf16sr"])
        nx, ny, nz = _log(rng, 16, 512), _log(rng, 8, 320), _log(rng, 8, 320)
        while nx * ny * nz > 1 << 24:
            ny, nz = max(8, ny // 2), max(8, nz // 2)
        steps = _log(rng, 1, 100)
        steps = max(1, min(steps, (1 << 29) // (nx * ny * nz)))
        walls = storage != "mom32" and rng.random() < 0.35
        monitor = storage in ("fp64", "fp32") and rng.random() < 0.25
        return dict(kind="box", storage=storage, nx=nx, ny=ny, nz=nz, steps=min(steps, 8) if monitor else steps,
                    tau=round(rng.uniform(0.55, 1.0), 4), force=rng.choice(["none", "uniform", "profile_y", "field"]),
                    walls=walls, monitor=monitor)
    if kind == "channels":
        return dict(kind="channels", nb=_log(rng, 4, 64), check=rng.choice([50, 100]))
    if kind == "droplet":
        return dict(kind="droplet", n=_log(rng, 40, 200), storage=rng.choice(["fp32", "fp64"]), steps=rng.randint(1, 4))
    if kind == "mhd":
        return dict(kind="mhd", n=_log(rng, 32, 128), storage=rng.choice(["fp64", "fp32"]),
                    current=rng.choice(["stencil", "populations"]), steps=rng.randint(1, 6))
    if kind == "rolls":
        n = _log(rng, 8, 4096)
        return dict(kind="rolls", n=n, storage=rng.choice(["fp64", "fp64", "fp32", "fp16"]),
                    steps=max(1, min(_log(rng, 4, 400), (1 << 27) // (n * n))))
    if kind == "conv":
        lv = rng.randint(0, 2)
        return dict(kind="conv", batch=_log(rng, 1, 16), d=4 * rng.randint(2, 8 >> lv), h=4 * rng.randint(2, 8 >> lv),
                    w=16 * rng.randint(1, 4 >> lv), cin=32 * rng.randint(1, 3 + 2 * (lv == 1)),
                    cout=32 * rng.randint(1, 3))
    return dict(kind="unet", batch=_log(rng, 1, 16), d=32, h=32, w=64)


# ---------------------------------------------------------------------------
# inputs, made from the seed alone

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) + 12345)
    return g


def _noise(g, shape, amp):
    return (torch.rand(shape, generator=g, device=DEV, dtype=F64) * 2 - 1) * amp


def _axes(nz, ny, nx, g):
    """2 pi x / n along each axis, shifted by a random phase, shaped to broadcast."""
    ph = torch.rand(3, generator=g, device=DEV, dtype=F64) * 2 * math.pi
    ax = [torch.arange(n, device=DEV, dtype=F64) * (2 * math.pi / n) + ph[i] for i, n in enumerate((nz, ny, nx))]
    return ax[0][:, None, None], ax[1][None, :, None], ax[2][None, None, :]


def _box_fields(case, seed):
    """(rho, u, force values or field) of a box: a Taylor-Green vortex of random phase with noise."""
    g = _gen(seed)
    nz, ny, nx = case["nz"], case["ny"], case["nx"]
    shape = (1, nz, ny, nx)
    z, y, x = _axes(nz, ny, nx, g)
    u = torch.zeros((3,) + shape, dtype=F64, device=DEV)
    rho = torch.ones(shape, dtype=F64, device=DEV) + _noise(g, shape, 1e-6)
    if not case["walls"]:
        u0 = 0.05
        u[0, 0] = u0 * torch.sin(x) * torch.cos(y) * torch.cos(z)
        u[1, 0] = -u0 * torch.cos(x) * torch.sin(y) * torch.cos(z)
        rho[0] += 3 * u0 * u0 / 16 * (torch.cos(2 * x) + torch.cos(2 * y)) * (torch.cos(2 * z) + 2)
    for a in range(3):
        u[a] += _noise(g, shape, 1e-4)
    fmode = case["force"]
    if fmode == "uniform":
        force = 1e-6 * (1 + 9 * torch.rand(1, generator=g, device=DEV, dtype=F64)) * torch.tensor([1.0, 0.0, 0.2], device=DEV, dtype=F64)
    elif fmode == "profile_y":
        force = torch.zeros((ny, 3), dtype=F64, device=DEV)
        force[:, 0] = 1e-5 * torch.sin(4 * y.reshape(-1))
    elif fmode == "field":
        force = 1e-5 * torch.stack([torch.sin(y) * torch.cos(z) + 0 * x, torch.cos(x) * torch.sin(z) + 0 * y,
                                    torch.sin(x) * torch.cos(y) + 0 * z])[:, None].contiguous()
    else:
        force = None
    return rho, u, force


def _channel_fields(case, seed):
    """(solid, force, rho, u) of channels with one to four spheres each; the flow starts as a laminar profile."""
    g = _gen(seed)
    nb, (nz, ny, nx) = case["nb"], (warmstart.NZ, warmstart.NY, warmstart.NX)
    r = torch.rand((nb, 4, 4), generator=g, device=DEV, dtype=F64)
    count = torch.randint(1, 5, (nb,), generator=g, device=DEV)
    z = torch.arange(nz, device=DEV, dtype=F64)[:, None, None]
    y = torch.arange(ny, device=DEV, dtype=F64)[None, :, None]
    x = torch.arange(nx, device=DEV, dtype=F64)[None, None, :]
    solid = torch.zeros((nb, nz, ny, nx), dtype=torch.bool, device=DEV)
    for k in range(4):
        rad = (3 + 5 * r[:, k, 0])[:, None, None, None]
        cx, cz = nx * r[:, k, 1][:, None, None, None], nz * r[:, k, 2][:, None, None, None]
        cy = rad + (ny - 1 - 2 * rad) * r[:, k, 3][:, None, None, None]
        dx, dz = (x - cx).abs(), (z - cz).abs()
        dx, dz = torch.minimum(dx, nx - dx), torch.minimum(dz, nz - dz)
        solid |= (dx * dx + (y - cy) ** 2 + dz * dz <= rad * rad) & (k < count)[:, None, None, None]
    fx = 1e-6 + 9e-6 * torch.rand(nb, generator=g, device=DEV, dtype=F64)
    force = torch.zeros((nb, 3), dtype=F64, device=DEV)
    force[:, 0] = fx
    u = torch.zeros((3, nb, nz, ny, nx), dtype=F64, device=DEV)
    yp = y + 0.5
    u[0] = fx[:, None, None, None] * (yp * (ny - yp) / (2 * warmstart.NU)) * (~solid)
    return solid, force, torch.ones((nb, nz, ny, nx), dtype=F64, device=DEV), u


def _droplet_fields(case, seed):
    g = _gen(seed)
    n = case["n"]
    c = (torch.arange(n, device=DEV, dtype=F64) - (n - 1) / 2) ** 2
    r = torch.sqrt(c[:, None, None] + c[None, :, None] + c[None, None, :])
    rho = 0.5625 - 0.4375 * torch.tanh(0.25 * (r - n / 5))
    rho = (rho + _noise(g, (n, n, n), 1e-4))[None].contiguous()
    return rho, torch.zeros((3, 1, n, n, n), dtype=F64, device=DEV)


MHD_U0, MHD_RE = 0.0203, 100.0


def _mhd_fields(case, seed):
    n = case["n"]
    z, y, x = _axes(n, n, n, _gen(seed))
    o = torch.zeros((n, n, n), dtype=F64, device=DEV)
    u = MHD_U0 * torch.stack([-2 * torch.sin(y) + o, 2 * torch.sin(x) + o, o])
    b = 0.8 * MHD_U0 * torch.stack([-2 * torch.sin(2 * y) + torch.sin(z) + o, 2 * torch.sin(x) + torch.sin(z) + o,
                                    torch.sin(x) + torch.sin(y) + o])
    return u, b


def _mhd_taus(case):
    nu = MHD_U0 * case["n"] / (2 * math.pi * MHD_RE)
    return 0.5 + 3 * nu, 0.5 + 4 * nu


def _rolls_fields(case, seed):
    g = _gen(seed)
    n, u0 = case["n"], 1e-3
    nu = u0 * n / 100.0
    ph = torch.rand(2, generator=g, device=DEV, dtype=F64) * 2 * math.pi
    c = torch.arange(n, device=DEV, dtype=F64) * (2 * math.pi / n)
    x, y = (c + ph[0])[None, :], (c + ph[1])[:, None]
    u = u0 * torch.stack([torch.sin(x) * torch.sin(y), torch.cos(x) * torch.cos(y)])
    force = 2 * nu * (2 * math.pi / n) ** 2 * u
    rho = torch.ones((n, n), dtype=F64, device=DEV)
    return rho, u * (0.5 + torch.rand(1, generator=g, device=DEV, dtype=F64)), force, 0.5 + 3 * nu


def _conv_tensors(case, seed):
    g = _gen(seed)
    n, d, h, w, ci, co = (case[k] for k in ("batch", "d", "h", "w", "cin", "cout"))

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)

    x = normal(n, d, h, w, ci)
    x = torch.where(x > 0, x, 0.1 * x).bfloat16()  # the output of the layer below: leaky ReLU
    return x, (normal(27, co, ci) * math.sqrt(2 / (27 * ci))), 0.1 * normal(co), (normal(n, d, h, w, co) * 0.01).bfloat16()


def _unet_input(case, seed):
    """Fluid mask and wall feature of channels with one sphere each, [2][n d h w] FP32."""
    g = _gen(seed)
    n, d, h, w = case["batch"], case["d"], case["h"], case["w"]
    c = torch.rand((n, 4), generator=g, device=DEV, dtype=F64)
    z = torch.arange(d, device=DEV, dtype=F64)[None, :, None, None] - d * c[:, 0, None, None, None]
    y = torch.arange(h, device=DEV, dtype=F64)[None, None, :, None] - h * c[:, 1, None, None, None]
    x = torch.arange(w, device=DEV, dtype=F64)[None, None, None, :] - w * c[:, 2, None, None, None]
    fluid = (x * x + y * y + z * z > ((3 + 5 * c[:, 3]) ** 2)[:, None, None, None]).to(torch.float32)
    yp = torch.arange(h, device=DEV, dtype=torch.float32) + 0.5
    return torch.stack([fluid, fluid * (4 * yp * (h - yp) / (h * h))[None, None, :, None]]).reshape(2, -1).contiguous()


# ---------------------------------------------------------------------------
# what a program has in hand, and one pass of its loop

def prepare(case, seed):
    kind = case["kind"]
    if kind == "box":
        rho, u, force = _box_fields(case, seed)
        st = case["storage"]
        lat = Lattice(case["nx"], case["ny"], case["nz"], tau=case["tau"], storage=st.replace("sr", ""),
                      wall=(0, 1, 0) if case["walls"] else (0, 0, 0), stochastic=st.endswith("sr"),
                      fused_reduce=bool(case.get("monitor")), device=DEV)
        if case["force"] == "field":
            lat.set_force("field", field=force)
        elif force is not None:
            lat.set_force(case["force"], values=force.cpu().numpy())
        lat.init(rho, u)
        return dict(case=case, lat=lat, dtype=F64 if st == "fp64" else torch.float32)
    if kind == "channels":
        solid, force, rho, u = _channel_fields(case, seed)
        lat = warmstart.new_lattice(case["nb"])
        lat.set_solid(solid)
        lat.set_force("batch", values=force.cpu().numpy())
        lat.init(rho, u)
        return dict(case=case, lat=lat)
    if kind == "droplet":
        rho, u = _droplet_fields(case, seed)
        n = case["n"]
        dt = F64 if case["storage"] == "fp64" else torch.float32
        lat = Lattice(n, n, n, tau=2.0, storage=case["storage"], device=DEV)
        field = torch.zeros((3,) + lat.shape, dtype=dt, device=DEV)
        lat.set_force("field", field=field)
        lat.init(rho, u)
        return dict(case=case, lat=lat, field=lat.force_field, rho=torch.empty(lat.shape, dtype=dt, device=DEV), dtype=dt)
    if kind == "mhd":
        u, b = _mhd_fields(case, seed)
        n = case["n"]
        tau, tau_m = _mhd_taus(case)
        S = CoupledMHD(n, n, n, tau, tau_m, storage=case["storage"], current=case["current"], device=DEV)
        S.init(np.ones((1, n, n, n)), u[:, None].cpu().numpy(), b)
        return dict(case=case, S=S)
    if kind == "rolls":
        rho, u, force, tau = _rolls_fields(case, seed)
        lat = Lattice2D(case["n"], case["n"], tau=tau, storage=case["storage"], device=DEV)
        lat.set_force("field", field=force)
        lat.init(rho, u)
        return dict(case=case, lat=lat, dtype=F64 if case["storage"] == "fp64" else torch.float32)
    if kind == "conv":
        x, w, b, dy = _conv_tensors(case, seed)
        n, d, h, wd, ci, co = (case[k] for k in ("batch", "d", "h", "w", "cin", "cout"))
        g = cmnn.geom(n, d, h, wd)
        wf = torch.empty((27, co, ci), dtype=torch.bfloat16, device=DEV)
        wt = torch.empty((27, ci, co), dtype=torch.bfloat16, device=DEV)
        cmnn.pack_weights(w, ci, co, wf, wt)
        ws = torch.empty((cmnn.conv_bwd_weight_workspace(g, ci, co) + 3) // 4, dtype=torch.float32, device=DEV)
        return dict(case=case, g=g, x=x, b=b, dy=dy, wf=wf, wt=wt, ws=ws, y=torch.empty_like(dy), dx=torch.empty_like(x),
                    dw=torch.empty_like(w), db=torch.empty_like(b))
    xs = _unet_input(case, seed)
    n, d, h, w = case["batch"], case["d"], case["h"], case["w"]
    net = UNet3D((d, h, w), in_ch=2, out_ch=4, seed=seed % 1000, device=DEV)
    x = torch.empty((n, d, h, w, net.cin0), dtype=torch.bfloat16, device=DEV)
    cmnn.pack_channels(n * d * h * w, xs, 2, x, net.cin0)
    return dict(case=case, net=net, x=x)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "box":
        lat = state["lat"]
        if case.get("monitor"):  # every step with the sums of the state it starts from
            sums = np.stack([lat.step_reduce() for _ in range(case["steps"])])
            # sums over FP32 arithmetic carry FP32's digits
            return lat.moments(dtype=state["dtype"]), sums if state["dtype"] == F64 else sums.astype(np.float32)
        lat.step(case["steps"])
        return lat.moments(dtype=state["dtype"])
    if kind == "channels":
        res, _ = warmstart.advance_check(state["lat"], case["check"])
        return state["lat"].moments(), res
    if kind == "droplet":
        lat = state["lat"]
        for _ in range(case["steps"]):
            lat.density(dtype=state["dtype"], out=state["rho"])
            lat.pseudopotential_force(-6.0, state["rho"], out=state["field"])
            lat.step(1)
        return lat.moments(dtype=state["dtype"]), state["field"]
    if kind == "mhd":
        state["S"].step(case["steps"])
        return state["S"].state()
    if kind == "rolls":
        state["lat"].step(case["steps"])
        return state["lat"].moments(dtype=state["dtype"])
    if kind == "conv":
        s, ci, co = state, case["cin"], case["cout"]
        cmnn.conv_fwd(s["g"], s["x"], ci, s["wf"], s["b"], co, cmnn.ACT_LEAKY, s["y"])
        cmnn.conv_bwd_data_act(s["g"], s["dy"], co, s["wt"], ci, s["x"], cmnn.ACT_LEAKY, s["dx"])
        cmnn.conv_bwd_weight(s["g"], s["x"], ci, s["dy"], co, s["dw"], s["db"], s["ws"])
        return s["y"], s["dx"], s["dw"], s["db"]
    return state["net"].forward(state["x"])


def work(case):
    """The state read once and written once for the whole pass, whatever its number of steps, the
    force field read once, the fields at the end written once, and the arithmetic of every step."""
    kind = case["kind"]
    if kind in ("box", "channels", "droplet"):
        if kind == "box":
            cells, st = case["nx"] * case["ny"] * case["nz"], case["storage"]
        elif kind == "channels":
            cells, st = case["nb"] * warmstart.NX * warmstart.NY * warmstart.NZ, "fp64"
        else:
            cells, st = case["n"] ** 3, case["storage"]
        size = 8 if st == "fp64" else 4 if st in ("fp32", "mom32") else 2
        io = 8 if st == "fp64" else 4
        per = 2 * (9 if st == "mom32" else 27) * size + 4 * io
        if case.get("force") == "field" or kind == "droplet":
            per += 3 * io
        return {"bytes": cells * per, "flops": cells * case.get("steps", case.get("check", 1)) * 700.0}
    if kind == "mhd":
        io = 8 if case["storage"] == "fp64" else 4
        return {"bytes": case["n"] ** 3 * io * (2 * 27 + 2 * 21 + 10), "flops": case["n"] ** 3 * case["steps"] * 950.0}
    if kind == "rolls":
        size = {"fp64": 8, "fp32": 4, "fp16": 2}[case["storage"]]
        return {"bytes": case["n"] ** 2 * (18 * size + 5 * (8 if size == 8 else 4)),
                "flops": case["n"] ** 2 * case["steps"] * 150.0}
    nv = case["batch"] * case["d"] * case["h"] * case["w"]
    if kind == "conv":
        ci, co = case["cin"], case["cout"]
        return {"bytes": nv * 2 * (2 * ci + 2 * co) + 27 * ci * co * 8, "flops": 3 * 2.0 * 27 * ci * co * nv}
    w0, w1, w2 = 32, 64, 96
    macs = 2 * w0 + w0 * w0 + (w0 * w1 + w1 * w1) / 8 + (w1 * w2 + 2 * w2 * w2) / 64 + ((w1 + w2) * w1 + w1 * w1) / 8 + \
        (w0 + w1) * w0 + w0 * w0 + 4 * w0
    return {"bytes": nv * 2 * (2 + 4), "flops": 2.0 * 27 * macs * nv}


# ---------------------------------------------------------------------------
# the same results in FP64, from the equations

Q = [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)]
W1 = {-1: 1 / 6, 0: 2 / 3, 1: 1 / 6}


def _inverse(m0, m1, m2, u):
    """(g-, g0, g+) with sum g = m0, sum g (c - u) = m1, sum g (c - u)^2 = m2."""
    odd = m1 + u * m0
    even = m2 + 2 * u * m1 + u * u * m0
    return {-1: 0.5 * (even - odd), 0: m0 - even, 1: 0.5 * (even + odd)}


def _equilibrium(rho, u):
    p = [{c: 1 + 3 * c * v + 4.5 * (c * c - 1 / 3) * v * v for c in (-1, 0, 1)} for v in u]
    return {(a, b, c): W1[a] * W1[b] * W1[c] * rho * p[0][a] * p[1][b] * p[2][c] for a, b, c in Q}


def _macro(f, F):
    rho = sum(f.values())
    u = [(sum(q[a] * f[q] for q in Q if q[a]) + 0.5 * F[a]) / rho for a in range(3)]
    return rho, u


def _collide(f, F, omega):
    """The five-step collision: relax the shear moments, take every other central moment from the printed table."""
    rho, (ux, uy, uz) = _macro(f, F)
    Fx, Fy, Fz = F

    def second(i, j):
        return sum(q[i] * q[j] * f[q] for q in Q if q[i] and q[j])

    om = 1 - omega
    pxx = second(0, 0) - rho * ux * ux + ux * Fx
    s = [om * (second(0, 1) - rho * ux * uy + 0.5 * (ux * Fy + uy * Fx)),
         om * (second(0, 2) - rho * ux * uz + 0.5 * (ux * Fz + uz * Fx)),
         om * (second(1, 2) - rho * uy * uz + 0.5 * (uy * Fz + uz * Fy)),
         om * (pxx - (second(1, 1) - rho * uy * uy + uy * Fy)), om * (pxx - (second(2, 2) - rho * uz * uz + uz * Fz))]
    zero = 0.0 * rho
    K = {(p, q, r): zero for p in range(3) for q in range(3) for r in range(3)}
    K[0, 0, 0] = rho
    K[1, 0, 0], K[0, 1, 0], K[0, 0, 1] = 0.5 * Fx + zero, 0.5 * Fy + zero, 0.5 * Fz + zero
    K[1, 1, 0], K[1, 0, 1], K[0, 1, 1] = s[0], s[1], s[2]
    K[2, 0, 0], K[0, 2, 0], K[0, 0, 2] = (rho + s[3] + s[4]) / 3, (rho - 2 * s[3] + s[4]) / 3, (rho + s[3] - 2 * s[4]) / 3
    K[1, 2, 0] = K[1, 0, 2] = Fx / 6 + zero
    K[2, 1, 0] = K[0, 1, 2] = Fy / 6 + zero
    K[2, 0, 1] = K[0, 2, 1] = Fz / 6 + zero
    K[2, 2, 0] = K[2, 0, 2] = K[0, 2, 2] = rho / 9
    K[1, 2, 2], K[2, 1, 2], K[2, 2, 1], K[2, 2, 2] = Fx / 18 + zero, Fy / 18 + zero, Fz / 18 + zero, rho / 27
    A = {(p, q): _inverse(K[p, q, 0], K[p, q, 1], K[p, q, 2], uz) for p in range(3) for q in range(3)}
    del K
    B = {(p, c): _inverse(A[p, 0][c], A[p, 1][c], A[p, 2][c], uy) for p in range(3) for c in (-1, 0, 1)}
    del A
    out = {}
    for b in (-1, 0, 1):
        for c in (-1, 0, 1):
            g = _inverse(B[0, c][b], B[1, c][b], B[2, c][b], ux)
            for a in (-1, 0, 1):
                out[a, b, c] = g[a]
    return out


def _bounces(solid, wall_y, shape):
    """Per velocity: where the population is pulled from a wall or a solid node."""
    if solid is None and not wall_y:
        return None
    found = {}
    for a, b, c in Q:
        m = torch.zeros(shape, dtype=torch.bool, device=DEV)
        if solid is not None:
            m |= torch.roll(solid, (c, b, a), (1, 2, 3))
        if wall_y and b:
            m[:, :, 0 if b > 0 else -1] = True
        found[a, b, c] = m
    return found


def _stream(f, bounces):
    g = {}
    for q in Q:
        v = torch.roll(f[q], (q[2], q[1], q[0]), (1, 2, 3))
        g[q] = v if bounces is None else torch.where(bounces[q], f[-q[0], -q[1], -q[2]], v)
    return g


def _exact_box(case, seed):
    rho, u, force = _box_fields(case, seed)
    shape = tuple(rho.shape)
    F = [0.0, 0.0, 0.0]
    if case["force"] == "uniform":
        F = list(force)
    elif case["force"] == "profile_y":
        F = [force[:, a][None, None, :, None] for a in range(3)]
    elif case["force"] == "field":
        F = [force[a] for a in range(3)]
    f = _equilibrium(rho, u)
    bounces = _bounces(None, case["walls"], shape)
    sums = []
    n = float(rho.numel())
    for _ in range(case["steps"]):
        if case.get("monitor"):
            r, v = _macro(f, F)
            v2 = sum(c * c for c in v)
            j = [r * v[a] - 0.5 * F[a] for a in range(3)]
            row = [r.sum(), *(x.sum() for x in j), (0.5 * r * v2).sum(), v2.max().sqrt(), 0.0, n, 0.0, v2.sum(), 0.0]
            sums.append([float(x) for x in row])
        f = _stream(_collide(f, F, 1 / case["tau"]), bounces)
    rho, u = _macro(f, F)
    if case.get("monitor"):
        return (rho, torch.stack(u)), _red_rows(sums)
    return rho, torch.stack(u)


def _red_rows(sums):
    """Sums in the order of the library's reduction rows."""
    from paper_1905_10182_amd.cmlbm import NRED, RED
    order = ["mass", "momx", "momy", "momz", "ke", "umax", "nonfinite", "fluid", "du2", "u2", "residual"]
    out = np.zeros((len(sums), 1, NRED))
    for k, row in enumerate(sums):
        for name, v in zip(order, row):
            out[k, 0, RED[name]] = v
    return out


def _exact_channels(case, seed):
    solid, force, rho, u = _channel_fields(case, seed)
    F = [force[:, a][:, None, None, None] for a in range(3)]
    bounces = _bounces(solid, True, tuple(rho.shape))
    f = _equilibrium(rho, u)
    fluid = (~solid).to(F64)
    before = None
    for k in range(case["check"]):
        if k == case["check"] - 2:
            before = torch.stack(_macro(f, F)[1]) * fluid
        f = _stream(_collide(f, F, 1 / warmstart.TAU), bounces)
    rho, u = _macro(f, F)
    u = torch.stack(u) * fluid
    d2, u2 = ((u - before) ** 2).sum((0, 2, 3, 4)), (u * u).sum((0, 2, 3, 4))
    return (torch.where(solid, torch.ones_like(rho), rho), u), (d2 / u2).sqrt() / 2


def _exact_droplet(case, seed):
    rho, u = _droplet_fields(case, seed)
    f = _equilibrium(rho, u)
    for _ in range(case["steps"]):
        psi = 1 - torch.exp(-sum(f.values()))
        F = [torch.zeros_like(psi) for _ in range(3)]
        for q in Q:
            p = (W1[q[0]] * W1[q[1]] * W1[q[2]]) * torch.roll(psi, (-q[2], -q[1], -q[0]), (1, 2, 3))
            for a in range(3):
                F[a] += 6.0 * q[a] * psi * p
        f = _stream(_collide(f, F, 0.5), None)
    rho, u = _macro(f, F)
    return (rho, torch.stack(u)), torch.stack(F)


def _cross(p, q):
    return [p[1] * q[2] - p[2] * q[1], p[2] * q[0] - p[0] * q[2], p[0] * q[1] - p[1] * q[0]]


def _exact_mhd(case, seed):
    u, b = _mhd_fields(case, seed)
    tau, tau_m = _mhd_taus(case)
    u, b = [v[None] for v in u], [v[None] for v in b]
    xi = [(0, 0, 0)] + [tuple(s if k == a else 0 for k in range(3)) for a in range(3) for s in (1, -1)]  # along (x, y, z)
    wm = [0.25] + [0.125] * 6

    def heq(b, u):
        return [[wm[l] * (b[a] + 4 * sum(xi[l][k] * (u[k] * b[a] - b[k] * u[a]) for k in range(3) if xi[l][k]))
                 for a in range(3)] for l in range(7)]

    def ddx(v, axis):  # axis 0, 1, 2 = x, y, z
        return 0.5 * (torch.roll(v, -1, 3 - axis) - torch.roll(v, 1, 3 - axis))

    def current(h, b, u):
        if case["current"] == "stencil":
            return [ddx(b[2], 1) - ddx(b[1], 2), ddx(b[0], 2) - ddx(b[2], 0), ddx(b[1], 0) - ddx(b[0], 1)]

        def neq(k, a):
            return sum(xi[l][k] * h[l][a] for l in range(7) if xi[l][k]) - (u[k] * b[a] - b[k] * u[a])

        s = -4 / tau_m
        return [s * (neq(1, 2) - neq(2, 1)), s * (neq(2, 0) - neq(0, 2)), s * (neq(0, 1) - neq(1, 0))]

    f = _equilibrium(torch.ones_like(u[0]), u)
    h = heq(b, u)
    F = [torch.zeros_like(u[0]) for _ in range(3)]
    for _ in range(case["steps"]):
        lag = _macro(f, F)[1]
        b = [sum(h[l][a] for l in range(7)) for a in range(3)]
        F = _cross(current(h, b, lag), b)
        u = _macro(f, F)[1]
        e = heq(b, u)
        h = [[torch.roll(h[l][a] + (e[l][a] - h[l][a]) / tau_m, (xi[l][2], xi[l][1], xi[l][0]), (1, 2, 3))
              for a in range(3)] for l in range(7)]
        f = _stream(_collide(f, F, 1 / tau), None)
    rho, u = _macro(f, F)
    b = [sum(h[l][a] for l in range(7)) for a in range(3)]
    j = current(h, b, u)
    return rho[0], torch.cat(u), torch.cat(b), torch.cat(j)


def _exact_rolls(case, seed):
    rho, u, F, tau = _rolls_fields(case, seed)
    om = 1 - 1 / tau
    Q2 = [(a, b) for a in (-1, 0, 1) for b in (-1, 0, 1)]
    p = [{c: 1 + 3 * c * v + 4.5 * (c * c - 1 / 3) * v * v for c in (-1, 0, 1)} for v in u]
    f = {(a, b): W1[a] * W1[b] * rho * p[0][a] * p[1][b] for a, b in Q2}

    def macro(f):
        r = sum(f.values())
        return r, [(sum(q[a] * f[q] for q in Q2 if q[a]) + 0.5 * F[a]) / r for a in range(2)]

    for _ in range(case["steps"]):
        r, (ux, uy) = macro(f)
        sxx, syy = sum(f[q] for q in Q2 if q[0]), sum(f[q] for q in Q2 if q[1])
        sxy = sum(q[0] * q[1] * f[q] for q in Q2 if q[0] and q[1])
        k4 = om * ((sxx - r * ux * ux + ux * F[0]) - (syy - r * uy * uy + uy * F[1]))
        k5 = om * (sxy - r * ux * uy + 0.5 * (ux * F[1] + uy * F[0]))
        K = {(0, 0): r, (1, 0): F[0] / 2, (0, 1): F[1] / 2, (2, 0): r / 3 + k4 / 2, (0, 2): r / 3 - k4 / 2, (1, 1): k5,
             (2, 1): F[1] / 6, (1, 2): F[0] / 6, (2, 2): r / 9}
        A = {m: _inverse(K[m, 0], K[m, 1], K[m, 2], uy) for m in range(3)}
        new = {}
        for b in (-1, 0, 1):
            g = _inverse(A[0][b], A[1][b], A[2][b], ux)
            for a in (-1, 0, 1):
                new[a, b] = torch.roll(g[a], (b, a), (0, 1))
        f = new
    r, u = macro(f)
    return r, torch.stack(u)


TAPS = [(dz, dy, dx) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]


def _shift(x, dz, dy, dx):
    """out[v] = x[v + (dz, dy, dx)]: periodic in z and x, zero beyond y."""
    v = torch.roll(x, (-dz, -dy, -dx), (1, 2, 3))
    if dy:
        v = v.clone()
        v[:, :, -1 if dy > 0 else 0] = 0
    return v


def _conv64(x, w, b):
    y = torch.zeros(x.shape[:4] + (w.shape[1],), dtype=F64, device=DEV)
    for t, o in enumerate(TAPS):
        y += (_shift(x, *o).reshape(-1, x.shape[4]) @ w[t].T.contiguous()).reshape(y.shape)
    return y if b is None else y + b


def _leaky(v):
    return torch.where(v > 0, v, 0.1 * v)


def _exact_conv(case, seed):
    x, w, b, dy = _conv_tensors(case, seed)
    x, w, b, dy = x.to(F64), w.bfloat16().to(F64), b.to(F64), dy.to(F64)
    y = _leaky(_conv64(x, w, b))
    # the adjoint of a shifted read is the opposite shift
    dx = _conv64(dy, torch.stack([w[26 - t].T.contiguous() for t in range(27)]), None)
    dx = dx * torch.where(x > 0, 1.0, 0.1)
    flat = dy.reshape(-1, dy.shape[4])
    dw = torch.stack([flat.T.contiguous() @ _shift(x, *o).reshape(-1, x.shape[4]) for o in TAPS])
    return y, dx, dw, flat.sum(0)


def _exact_unet(case, seed):
    xs = _unet_input(case, seed).to(F64)
    n, d, h, w = case["batch"], case["d"], case["h"], case["w"]
    net = UNet3D((d, h, w), in_ch=2, out_ch=4, seed=seed % 1000, device=DEV)
    L = {k: (v["w"].to(F64), v["b"].to(F64)) for k, v in net.layers.items()}
    x = torch.zeros((n, d, h, w, net.cin0), dtype=F64, device=DEV)
    x[..., :2] = xs.reshape(2, n, d, h, w).permute(1, 2, 3, 4, 0)

    def conv(name, v):
        y = _conv64(v, *L[name])
        return y if name == "head" else _leaky(y)

    def pool(v):
        s = v.shape
        return v.reshape(s[0], s[1] // 2, 2, s[2] // 2, 2, s[3] // 2, 2, s[4]).mean((2, 4, 6))

    def up(v):
        return v.repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)

    s0 = conv("e0b", conv("e0a", x))
    s1 = conv("e1b", conv("e1a", pool(s0)))
    m = conv("ma", pool(s1))
    m = conv("mb", torch.cat([m, m.mean((1, 2, 3), keepdim=True).expand_as(m)], 4))
    v = conv("d1b", conv("d1a", torch.cat([s1, up(m)], 4)))
    v = conv("d0b", conv("d0a", torch.cat([s0, up(v)], 4)))
    return conv("head", v)


def exact(case, seed):
    return {"box": _exact_box, "channels": _exact_channels, "droplet": _exact_droplet, "mhd": _exact_mhd,
            "rolls": _exact_rolls, "conv": _exact_conv, "unet": _exact_unet}[case["kind"]](case, seed)
