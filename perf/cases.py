"""Performance cases of the lifted-PROPELLER library: what users run, timed as they run it.

Each case is a dict of plain values; ``prepare`` builds what a program holds before the
call (inputs drawn from a seed, the plan, the session), ``run`` makes one pass through the
public entry points and returns its outputs whole, ``work`` states the bytes and operations
the pass cannot do without, and ``exact`` evaluates the same outputs in FP64 with plain torch.

Kinds of pass
  operators  one optimiser step on caller-held device arrays: residual (vp_forward), data
             gradient (vp_adjoint), regularised Adam update (vp_step)
  autograd   a torch user's gradient: Regulariser and lifted_forward, then backward
  fit        a resident fit resumed in its middle: graph-replayed steps, then the renders
  nu         the blade-aligned sampling operators, forward and adjoint
  nu_fit     the resident blade-aligned fit resumed in its middle, then its read-out
  kplanes    the resident K-Planes fit resumed in its middle, then its state
  batch      resident slices of mixed sizes stepped together, then read out
  eval       the evaluation calls: windowed baselines and PSNR

Fits start from the state a fit has in its middle (a volume near the solution, second
moments that remember the early gradients), where the optimiser's map is well conditioned;
the batch, whose calls start from zero, descends by plain gradient steps.
"""

import math

import numpy as np
import torch

from paper_2311_13177_amd import autograd as A
from paper_2311_13177_amd import binding as B

GOLDEN = 180.0 / ((1.0 + math.sqrt(5.0)) / 2.0)
RESUME_STEP = 200
TV_W, TV_EPS, LR = 1e-3, 1e-3, 1e-2


# ------------------------------------------------------------------ the cases

def _case(name, kind, n, S, T, nb, lines, f, **more):
    c = dict(name=name, kind=kind, n=n, S=S, T=T, blades=nb, lines=lines, f=float(f), steps=0, autotune=False,
             l1=0.0, feat=0, half=0, slices=0)
    c.update(more)
    return c


def listed():
    return [
        # the 64^2 workload's step driven from Python: launches and host work
        _case("op_static_64", "operators", 64, 16, 1, 5, 16, 2),
        # an odd small size (a length without a compiled DFT plan), dynamic, with L1, through autograd
        _case("autograd_150_dynamic", "autograd", 150, 12, 5, 9, 14, 2.5, l1=1e-4),
        # the 256^2 workload's step on caller-held arrays
        _case("op_static_256", "operators", 256, 32, 1, 12, 32, 4),
        # the dynamic 192^2 workload's step on caller-held arrays
        _case("op_dynamic_192", "operators", 192, 32, 16, 32, 24, 3),
        # a large served request's sizes, the largest arrays listed
        _case("op_served_384", "operators", 384, 64, 8, 24, 32, 6),
        # the three named fits, resident and graph-replayed
        _case("fit_static_64", "fit", 64, 16, 1, 5, 16, 2, steps=100),
        _case("fit_static_256", "fit", 256, 32, 1, 12, 32, 4, steps=50),
        _case("fit_dynamic_192", "fit", 192, 32, 16, 32, 24, 3, steps=40, autotune=True),
        # the fit on blade-aligned samples of the 256^2 geometry
        _case("nu_fit_256", "nu_fit", 256, 32, 1, 12, 32, 4, steps=40),
        # the K-Planes fit of the dynamic 192^2 geometry (two scales, eight features)
        _case("kplanes_192", "kplanes", 192, 32, 16, 32, 24, 3, steps=8, feat=8, half=1),
        # a batch of mixed slices (sizes of the 64-slice batch)
        _case("batch_6", "batch", 256, 32, 1, 16, 32, 4, steps=40, slices=6),
        # evaluation of a dynamic scan: five-blade baselines of every frame, PSNR of the frames
        _case("eval_dynamic_192", "eval", 192, 32, 16, 32, 24, 3),
    ]


def _smooth(m):
    for p in (2, 3, 5):
        while m % p == 0:
            m //= p
    return m == 1


# lengths with no prime factor above 5, with a compiled DFT plan or without, odd ones among them
_SIZES = [m for m in range(48, 385) if _smooth(m)]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["operators", "operators", "autograd", "fit", "fit", "nu", "nu_fit", "kplanes", "batch", "eval"])
    top = 256 if kind in ("nu", "nu_fit", "batch") else (192 if kind == "kplanes" else 384)
    want = _log_int(rng, 48, top)
    n = min((m for m in _SIZES if m <= top), key=lambda m: abs(m - want))
    S = _log_int(rng, 4, 64 if kind in ("operators", "autograd", "fit", "eval") else 32)
    T = 1 if kind == "batch" or rng.random() < 0.4 else rng.randint(2, 16)
    nb = rng.randint(4, 32)
    lines = rng.randint(8, 32)
    f = round(rng.uniform(1.5, max(2.0, n / 64.0)), 3)
    while T * S * n * n > 40e6:
        T = max(1, T // 2)
    c = _case("", kind, n, S, T, nb, lines, f, l1=rng.choice([0.0, 0.0, 1e-4]) if kind in ("operators", "autograd") else 0.0)
    del c["name"]
    if kind in ("fit", "nu_fit"):
        c["steps"] = rng.randint(10, 40)
        c["autotune"] = kind == "fit" and rng.random() < 0.3
    if kind == "kplanes":
        c["T"] = max(2, c["T"])
        c.update(steps=rng.randint(2, 6), feat=rng.choice([2, 4, 8]), half=rng.randint(0, 1))
    if kind == "batch":
        c.update(steps=rng.randint(10, 40), slices=rng.randint(2, 6))
    return c


# ------------------------------------------------------------------ geometry and inputs

def _geometry(c):
    n, S, T, nb = c["n"], c["S"], c["T"], c["blades"]
    if T == 1:
        ang = np.deg2rad(180.0 * np.arange(nb) / nb)
        tau = None
    else:
        ang = np.deg2rad(np.mod(np.arange(nb) * GOLDEN, 180.0))
        tau = np.arange(nb) / float(nb)
    shift = (np.arange(S) - S / 4.0) * 2.0 * c["f"] / S
    return dict(n=n, n_spec=S, n_time=T, angle_rad=ang, lines=np.full(nb, c["lines"], np.int32), blade_time=tau,
                spec_shift_px=shift)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _noise(g, shape):
    return torch.view_as_complex(torch.randn(*shape, 2, generator=g, device="cuda"))


def _masks(g):
    """Blade supports in unshifted order, FP64 (the library's stated rule)."""
    n = g["n"]
    j = torch.arange(n, device="cuda", dtype=torch.float64)
    k = torch.where(j <= (n - 1) // 2, j, j - n)
    ky, kx = k[:, None], k[None, :]
    out = []
    for th, L in zip(g["angle_rad"], g["lines"]):
        cs, sn = math.cos(th), math.sin(th)
        r, q = kx * cs + ky * sn, -kx * sn + ky * cs
        out.append((r >= -n / 2.0 - 1e-9) & (r < n / 2.0 - 1e-9) & (q >= -L / 2.0 - 1e-9) & (q < L / 2.0 - 1e-9))
    return torch.stack(out)


def _layers(n, f, seed, taus):
    """Fat and water frames [len(taus)][n][n] of a moving random-ellipse phantom, with a smooth phase."""
    rng = np.random.default_rng([int(seed), 77])
    m = max(3, int(round(8 + (n - 64) / 12.0)))
    ax = torch.arange(n, device="cuda", dtype=torch.float32)
    t = torch.tensor(np.asarray(taus, dtype=np.float32), device="cuda")[:, None, None]
    W = torch.zeros(len(taus), n, n, device="cuda")
    F = torch.zeros_like(W)
    for i in range(m):
        a, b = rng.uniform(0.05 * n, 0.2 * n, 2)
        rot = rng.uniform(0, math.pi)
        rad = max(1.0, n / 2.0 - max(a, b) - 2 * f - 2)
        cx, cy = rng.uniform(n / 2.0 - rad, n / 2.0 + rad, 2)
        amp, ph = rng.uniform(0, 6.0 * n / 192.0), rng.uniform(0, 2 * math.pi)
        wa, fa = rng.uniform(0.2, 1.0), rng.uniform(0.2, 0.8) * (rng.uniform() < 0.3)
        dx = ax[None, None, :] - (cx + (amp * torch.sin(2 * math.pi * t + ph) if len(taus) > 1 else 0.0))
        dy = ax[None, :, None] - cy
        u = (dx * math.cos(rot) + dy * math.sin(rot)) / a
        v = (dy * math.cos(rot) - dx * math.sin(rot)) / b
        inside = ((u * u + v * v) <= 1.0).float()
        W += wa * inside
        F += fa * inside
    phase = torch.polar(torch.ones(n, n, device="cuda"), 0.6 * torch.sin(2 * math.pi * ax / n)[:, None] + 0.4 * ax[None, :] / n)
    return W * phase, F * phase


def _taps(d, th):
    dx, dy = d * math.cos(th), d * math.sin(th)
    ox, oy = math.floor(-dx), math.floor(-dy)
    fx, fy = -dx - ox, -dy - oy
    return ox, oy, ((1 - fy) * (1 - fx), (1 - fy) * fx, fy * (1 - fx), fy * fx)


def _shifted(P, oy, ox):
    """P[..., y + oy, x + ox], zero outside."""
    n = P.shape[-1]
    out = torch.zeros_like(P)
    ys, yd, xs, xd = max(0, oy), max(0, -oy), max(0, ox), max(0, -ox)
    h, w = n - abs(oy), n - abs(ox)
    if h > 0 and w > 0:
        out[..., yd:yd + h, xd:xd + w] = P[..., ys:ys + h, xs:xs + w]
    return out


def _shear(P, d, th):
    ox, oy, w = _taps(d, th)
    return (w[0] * _shifted(P, oy, ox) + w[1] * _shifted(P, oy, ox + 1) + w[2] * _shifted(P, oy + 1, ox)
            + w[3] * _shifted(P, oy + 1, ox + 1))


def _blade_frames(c, g, seed):
    """The projection of the truth at every blade's time: water and fat on their two bins."""
    taus = [0.0] if c["T"] == 1 else list(g["blade_time"])
    W, F = _layers(c["n"], c["f"], seed, taus)
    sw, sf = g["spec_shift_px"][c["S"] // 4], g["spec_shift_px"][min(c["S"] - 1, 3 * c["S"] // 4)]
    out = []
    for b, th in enumerate(g["angle_rad"]):
        i = 0 if c["T"] == 1 else b
        out.append(_shear(W[i], sw, th) + _shear(F[i], sf, th))
    return torch.stack(out)


def _kspace(c, g, seed):
    n = c["n"]
    k = torch.fft.fft2(_blade_frames(c, g, seed), norm="ortho")
    k = k + 2e-3 * _noise(_gen(seed * 8 + 1), (c["blades"], n, n))
    return (k * _masks(g)).to(torch.complex64)


def _nu_points(c, g, b):
    n, L = c["n"], int(g["lines"][b])
    cs, sn = math.cos(g["angle_rad"][b]), math.sin(g["angle_rad"][b])
    r = torch.arange(n, device="cuda", dtype=torch.float64) - n / 2.0
    q = torch.arange(L, device="cuda", dtype=torch.float64)[:, None] - L / 2.0
    return (r * cs - q * sn).reshape(-1), (r * sn + q * cs).reshape(-1)


def _nu_waves(c, g, b):
    """exp(-2 pi i k x / n) of blade b's samples for x and for y, FP64 [L n][n] each."""
    n = c["n"]
    x = torch.arange(n, device="cuda", dtype=torch.float64)
    kx, ky = _nu_points(c, g, b)
    one = torch.ones((), device="cuda", dtype=torch.float64)
    return (torch.polar(one, -2 * math.pi / n * kx[:, None] * x[None, :]),
            torch.polar(one, -2 * math.pi / n * ky[:, None] * x[None, :]))


def _nu_forward(c, g, b, img):
    ex, ey = _nu_waves(c, g, b)
    return ((ex @ img.transpose(0, 1).contiguous()) * ey).sum(1).reshape(-1, c["n"]) / c["n"]


def _nu_adjoint(c, g, b, smp):
    ex, ey = _nu_waves(c, g, b)
    left = (ey.conj() * smp.reshape(-1)[:, None]).transpose(0, 1).contiguous()
    return left @ ex.conj().resolve_conj() / c["n"]


def _samples(c, g, seed):
    img = _blade_frames(c, g, seed).to(torch.complex128)
    y = torch.stack([_nu_forward(c, g, b, img[b]) for b in range(c["blades"])])
    return (y + 2e-3 * _noise(_gen(seed * 8 + 1), tuple(y.shape))).to(torch.complex64)


def _volume(c, seed):
    """A volume as a fit has it in its middle: the layers spread over nearby bins, and a residue."""
    n, S, T = c["n"], c["S"], c["T"]
    W, F = _layers(n, c["f"], seed, [0.0] if T == 1 else np.arange(T) / (T - 1.0))
    s = torch.arange(S, device="cuda", dtype=torch.float32)
    prof = [torch.exp(-((s - m) ** 2) / (2 * max(0.7, S / 16.0) ** 2)) for m in (S // 4, 3 * S // 4)]
    pw, pf = (p / p.sum() for p in prof)
    vol = 0.03 * _noise(_gen(seed * 8 + 2), (T, S, n, n))
    for k in range(T):
        vol[k] += pw[:, None, None] * W[k] + pf[:, None, None] * F[k]
    return vol


def _stiff(c):
    """The data term's largest curvature: every bin of every blade that sees a voxel, at the lowest frequency."""
    return c["S"] * (c["blades"] if c["T"] == 1 else 2.0 * c["blades"] / c["T"] + 1.0)


def _moments(shape, seed, scale):
    """Adam moments in the middle of a fit: the second moments remember the first steps' gradients."""
    g = _gen(seed * 8 + 3)
    m = 0.05 * scale * _noise(g, shape)
    v = torch.view_as_complex((scale * scale) * (0.2 + 0.8 * torch.rand(*shape, 2, generator=g, device="cuda")))
    return m, v


def _options(c, **more):
    return B.vp_options_default(**dict(dict(tv_weight=TV_W, tv_eps=TV_EPS, l1_weight=c["l1"], lr=LR,
                                            autotune=int(c["autotune"])), **more))


def _batch_cases(c):
    """Slices of the batch: sizes vary as in the 64-slice batch, the first the largest."""
    out = []
    for i in range(c["slices"]):
        n = c["n"] if i == 0 else max(m for m in (48, 64, 96, 128, 192, 256) if m <= max(48, c["n"] * (4 - i % 3) // 4))
        S = c["S"] if i % 2 == 0 else max(4, c["S"] // 2)
        out.append(dict(c, n=n, S=S, blades=max(4, c["blades"] - 2 * i), lines=min(n, max(8, c["lines"] - 2 * i)),
                        kind="slice"))
    return out


def _kp_model(c):
    res = (c["n"], c["n"] // 2) if c["half"] else (c["n"],)
    return res, dict(tv_weight=1e-1, smooth_weight=1e-2, sparse_weight=1e-3, eps=1e-3)


def _kp_shapes(c):
    res, _ = _kp_model(c)
    F, S, Rt = c["feat"], c["S"], c["T"]
    out = []
    for R in res:
        out += [(R, R, F), (S, R, F), (S, R, F), (Rt, R, F), (Rt, R, F), (Rt, S, F)]
    return out + [(F,)]


def _kp_params(c, seed):
    g = _gen(seed * 8 + 4)
    parts = []
    for i, shp in enumerate(_kp_shapes(c)):
        z = _noise(g, shp)
        if len(shp) == 1:
            parts.append(0.3 * z)                        # decoder weights
        elif i % 6 >= 3:
            parts.append((1.0 + 0.05 * z).reshape(-1))   # time grids, near one
        else:
            u = torch.rand(*shp, generator=g, device="cuda")
            parts.append((0.1 + 0.4 * u + 0.05 * z).reshape(-1))
    return torch.cat([p.reshape(-1) for p in parts]).to(torch.complex64)


def _inputs(c, seed):
    """The pass's arrays on the GPU, from the seed alone."""
    g = _geometry(c)
    kind = c["kind"]
    d = dict(g=g)
    if kind in ("operators", "autograd", "fit", "nu", "nu_fit"):
        d["vol"] = _volume(c, seed)
        d["y"] = _samples(c, g, seed) if kind.startswith("nu") else _kspace(c, g, seed)
        if kind in ("operators", "fit", "nu_fit"):
            d["m"], d["v"] = _moments(tuple(d["vol"].shape), seed, max(0.3, LR * _stiff(c) / 5.0))
    elif kind == "slice":
        d["y"] = _kspace(c, g, seed)
    elif kind == "kplanes":
        d["y"] = _kspace(c, g, seed)
        d["p"] = _kp_params(c, seed)
        d["m"], d["v"] = _moments(tuple(d["p"].shape), seed, 100.0)
    elif kind == "eval":
        d["y"] = _kspace(c, g, seed)
        W, F = _layers(c["n"], c["f"], seed, [0.0] if c["T"] == 1 else np.arange(c["T"]) / (c["T"] - 1.0))
        d["truth"] = (W + F).contiguous()
        d["frames"] = d["truth"] + 0.03 * _noise(_gen(seed * 8 + 5), tuple(d["truth"].shape))
    return d


def _host(t):
    return t.cpu().numpy()


# ------------------------------------------------------------------ a program's state, and one pass

def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "batch":
        cs = _batch_cases(c)
        ins = [_inputs(s, seed + 100 * i) for i, s in enumerate(cs)]
        plans = [B.Plan.from_geometry(d["g"]) for d in ins]
        opts = [_options(s, n_steps=1 << 30, optimizer=B.VP_OPT_GD, lr=1.0 / _stiff(s)) for s in cs]
        return dict(c=c, batch=B.Batch(plans, [_host(d["y"]) for d in ins], opts))
    d = _inputs(c, seed)
    plan = B.Plan.from_geometry(d["g"])
    s = dict(c=c, plan=plan)
    if kind == "operators":
        s.update(vol=d["vol"], y=d["y"], m=d["m"], v=d["v"], opts=_options(c), t=RESUME_STEP)
    elif kind == "autograd":
        s.update(vol=d["vol"].requires_grad_(True), y=d["y"])
    elif kind == "nu":
        s.update(vol=d["vol"], y=d["y"])
    elif kind == "eval":
        s.update(y=d["y"], truth=d["truth"], frames=d["frames"])
    elif kind in ("fit", "nu_fit"):
        S = B.Session if kind == "fit" else B.NuSession
        s["sess"] = S(plan, _host(d["y"]), _options(c))
        s["sess"].set_state(dict(vol=_host(d["vol"]), m=_host(d["m"]), v=_host(d["v"]), step=RESUME_STEP))
    else:
        res, w = _kp_model(c)
        model = B.vp_kplanes.make(c["feat"], c["T"], res, **w)
        p = _host(d["p"])
        s["sess"] = B.KPlanesSession(plan, model, _host(d["y"]), p, _options(c))
        s["sess"].set_state(dict(params=p, m=_host(d["m"]), v=_host(d["v"]), step=RESUME_STEP))
    return s


def run(state):
    c = state["c"]
    kind = c["kind"]
    if kind == "operators":
        plan, vol = state["plan"], state["vol"]
        res = B.vp_forward(plan, vol, state["y"])
        grad = B.vp_adjoint(plan, res)
        new = B.vp_step(plan, state["opts"], vol, grad, state["m"], state["v"], state["t"] + 1)
        return dict(res=res, grad=grad, vol=new, m=state["m"], v=state["v"])
    if kind == "autograd":
        vol = state["vol"]
        vol.grad = None
        res = A.lifted_forward(A.Regulariser.apply(vol, state["plan"], TV_W, c["l1"], TV_EPS), state["plan"], state["y"])
        res.backward(res.detach())  # the gradient of 0.5 |res|^2
        return dict(res=res, grad=vol.grad)
    if kind == "nu":
        res = B.vp_nu_forward(state["plan"], state["vol"], state["y"])
        return dict(res=res, grad=B.vp_nu_adjoint(state["plan"], res))
    if kind == "fit":
        state["sess"].step(c["steps"])
        r = state["sess"].read(volume=False)
        return {k: r[k] for k in ("proj", "water", "fat")}
    if kind == "nu_fit":
        state["sess"].step(c["steps"])
        r = state["sess"].read()
        return {k: r[k] for k in ("vol", "proj", "water", "fat")}
    if kind == "kplanes":
        state["sess"].step(c["steps"])
        r = state["sess"].get_state()
        return {k: r[k] for k in ("params", "m", "v")}
    if kind == "batch":
        b = state["batch"]
        b.step(c["steps"])
        return [{k: r[k] for k in ("vol", "proj", "water", "fat")} for r in (b.read(i) for i in range(c["slices"]))]
    frames = B.vp_baseline(state["plan"], state["y"], window=5, first_frame=0, n_frames=c["blades"])
    psnr, mse, peak = B.vp_psnr(state["frames"], state["truth"])
    return dict(baseline=frames, psnr=psnr, mse=mse, peak=peak)


# ------------------------------------------------------------------ what a pass cannot do without

def _parts(c):
    if c["T"] == 1:
        return c["blades"]
    u = np.arange(c["blades"]) / float(c["blades"]) * (c["T"] - 1)
    a = u - np.minimum(np.floor(u), c["T"] - 2)
    return int(np.sum(a != 1.0) + np.sum(a != 0.0))


def work(case):
    c, kind = case, case["kind"]
    if kind == "batch":
        parts = [work(dict(s, kind="gd")) for s in _batch_cases(c)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    n, nb = c["n"], c["blades"]
    vox, px, nn = c["T"] * c["S"] * n * n, nb * n * n, n * n
    smp = nb * c["lines"] * n
    project = 16 * c["S"] * nn * _parts(c)
    dft = 5 * px * 2 * math.log2(n)
    if kind == "operators":
        return dict(bytes=56 * vox + 17 * px, flops=2 * project + 2 * dft + 60 * vox)
    if kind == "autograd":
        return dict(bytes=16 * vox + 17 * px, flops=2 * project + 2 * dft + 45 * vox)
    if kind == "nu":
        return dict(bytes=16 * vox + 16 * smp, flops=2 * project + 8 * dft + 2 * 4 * 36 * smp)
    k = c["steps"]
    out = 24 * c["T"] * nn
    if kind == "fit":
        return dict(bytes=k * (48 * vox + 9 * px) + out, flops=k * (2 * project + 2 * dft + 60 * vox))
    if kind == "nu_fit":
        return dict(bytes=k * (48 * vox + 8 * smp) + 8 * vox + out,
                    flops=k * (2 * project + 8 * dft + 2 * 4 * 36 * smp + 60 * vox))
    if kind == "gd":
        return dict(bytes=k * (16 * vox + 9 * px) + 8 * vox + out, flops=k * (2 * project + 2 * dft + 50 * vox))
    if kind == "kplanes":
        np_ = sum(int(np.prod(s)) for s in _kp_shapes(c))
        bvox = c["S"] * px
        scales = 1 + c["half"]
        # decode and three factor gradients, one complex product and one multiply-add each
        return dict(bytes=k * (48 * np_ + 9 * px) + 24 * np_,
                    flops=k * (4 * 14 * c["feat"] * scales * bvox + 2 * 16 * bvox + 2 * dft))
    frames = c["T"] * nn
    return dict(bytes=9 * px + 8 * px + 16 * frames, flops=5 * px * 2 * math.log2(n) + 10 * px + 12 * frames)


# ------------------------------------------------------------------ the same outputs in FP64

class _Model:
    """The lifted operator of a geometry in FP64: bins with the same integer offsets go together."""

    def __init__(self, c, g):
        self.c, self.g, self.n, self.T = c, g, c["n"], c["T"]
        self.mask = _masks(g).to(torch.float64)
        self.groups = []
        for th in g["angle_rad"]:
            runs = []
            for s, d in enumerate(g["spec_shift_px"]):
                ox, oy, w = _taps(float(d), float(th))
                if runs and runs[-1][:2] == [oy, ox]:
                    runs[-1][3] = s + 1
                    runs[-1][4].append(w)
                else:
                    runs.append([oy, ox, s, s + 1, [w]])
            self.groups.append([(oy, ox, s0, s1, torch.tensor(w, dtype=torch.complex128, device="cuda"))
                                for oy, ox, s0, s1, w in runs])

    def knots(self, b):
        if self.T == 1:
            return [(0, 1.0)]
        u = float(self.g["blade_time"][b]) * (self.T - 1)
        k = min(int(math.floor(u)), self.T - 2)
        return [(k, 1.0 - (u - k)), (k + 1, u - k)]

    def project(self, b, P):
        """Blade image of a bin stack P [S][n][n]."""
        n = self.n
        out = torch.zeros(n, n, dtype=torch.complex128, device="cuda")
        for oy, ox, s0, s1, w in self.groups[b]:
            planes = P[s0:s1].reshape(s1 - s0, n * n)
            taps = (w.transpose(0, 1).contiguous() @ planes).reshape(4, n, n)
            out += (_shifted(taps[0], oy, ox) + _shifted(taps[1], oy, ox + 1) + _shifted(taps[2], oy + 1, ox)
                    + _shifted(taps[3], oy + 1, ox + 1))
        return out

    def back(self, b, img, G):
        """G [S][n][n] += the transpose of project applied to img."""
        n = self.n
        for oy, ox, s0, s1, w in self.groups[b]:
            taps = torch.stack([_shifted(img, -oy, -ox), _shifted(img, -oy, -ox - 1), _shifted(img, -oy - 1, -ox),
                                _shifted(img, -oy - 1, -ox - 1)]).reshape(4, n * n)
            G[s0:s1] += (w @ taps).reshape(s1 - s0, n, n)

    def image(self, b, vol):
        (k0, w0), *rest = self.knots(b)
        P = w0 * vol[k0]
        for k, w in rest:
            if w != 0.0:
                P = P + w * vol[k]
        return self.project(b, P)

    def spread(self, b, img, grad):
        for k, w in self.knots(b):
            if w != 0.0:
                self.back(b, w * img, grad[k])

    def residual(self, b, vol, y):
        return self.mask[b] * (torch.fft.fft2(self.image(b, vol), norm="ortho") - y[b])

    def adjoint(self, b, r, grad):
        self.spread(b, torch.fft.ifft2(self.mask[b] * r, norm="ortho"), grad)

    def data_gradient(self, vol, y, nu=False):
        grad, res = torch.zeros_like(vol), []
        for b in range(self.c["blades"]):
            if nu:
                r = _nu_forward(self.c, self.g, b, self.image(b, vol)) - y[b]
                self.spread(b, _nu_adjoint(self.c, self.g, b, r), grad)
            else:
                r = self.residual(b, vol, y)
                self.adjoint(b, r, grad)
            res.append(r)
        return torch.stack(res), grad


def _charb(d, eps):
    return d / torch.sqrt(d.real ** 2 + d.imag ** 2 + eps * eps)


def _reg_gradient(vol, l1):
    g = torch.zeros_like(vol)
    for ax in range(4):
        m = vol.shape[ax]
        if m > 1:
            w = _charb(vol.narrow(ax, 1, m - 1) - vol.narrow(ax, 0, m - 1), TV_EPS)
            g.narrow(ax, 1, m - 1).add_(w)
            g.narrow(ax, 0, m - 1).sub_(w)
    g *= TV_W
    if l1:
        g += l1 * _charb(vol, TV_EPS)
    return g


def _adam(x, g, m, v, t):
    m = 0.9 * m + 0.1 * g
    v = torch.complex(0.999 * v.real + 0.001 * g.real ** 2, 0.999 * v.imag + 0.001 * g.imag ** 2)
    b1, b2 = 1 - 0.9 ** t, 1 - 0.999 ** t
    dx = torch.complex(m.real / (torch.sqrt(v.real / b2) + 1e-8), m.imag / (torch.sqrt(v.imag / b2) + 1e-8))
    return x - LR / b1 * dx, m, v


def _renders(c, vol):
    h = c["S"] // 2
    w, f = vol[:, :h].sum(1), vol[:, h:].sum(1)
    return dict(proj=w + f, water=w, fat=f)


def _kp_factors(c, parts):
    """Per scale, the separable factors at the blades' times of parameter grids [c][6]."""
    n, S, Rt = c["n"], c["S"], c["T"]
    t = torch.arange(c["blades"], device="cuda", dtype=torch.float64) / c["blades"]

    def lerp(p, u, ax):
        R = p.shape[ax]
        if R == 1:
            return p.expand(*[len(u) if i == ax else q for i, q in enumerate(p.shape)])
        i0 = torch.clamp(torch.floor(u).long(), max=R - 2)
        w = (u - i0).reshape([-1 if i == ax else 1 for i in range(p.dim())])
        return (1 - w) * p.index_select(ax, i0) + w * p.index_select(ax, i0 + 1)

    out = []
    for xy, xs, ys, xt, yt, st in parts:
        R = xy.shape[0]
        u = torch.arange(n, device="cuda", dtype=torch.float64) * ((R - 1) / (n - 1.0))
        tu = t * (Rt - 1)
        out.append((lerp(lerp(xy, u, 0), u, 1), lerp(xs, u, 1), lerp(ys, u, 1), lerp(lerp(xt, u, 1), tu, 0),
                    lerp(lerp(yt, u, 1), tu, 0), lerp(st, tu, 0)))
    return out


def _kp_reg(parts, w):
    e2 = w["eps"] ** 2

    def ch(z):
        return (torch.sqrt(z.real ** 2 + z.imag ** 2 + e2) - w["eps"]).sum()

    r = 0.0
    for grids in parts:
        for i, p in enumerate(grids):
            if i < 3:
                r = r + w["tv_weight"] * ch(p[1:] - p[:-1])
            r = r + w["tv_weight"] * ch(p[:, 1:] - p[:, :-1])
            if i >= 3:
                d2 = p[2:] - 2 * p[1:-1] + p[:-2]
                r = r + w["smooth_weight"] * (d2.real ** 2 + d2.imag ** 2).sum() + w["sparse_weight"] * ch(p - 1)
    return r


def _kp_gradient(c, M, y, flat):
    leaf = flat.detach().clone().requires_grad_(True)
    shapes = _kp_shapes(c)
    split = torch.split(leaf, [int(np.prod(s)) for s in shapes])
    grids = [p.reshape(s) for p, s in zip(split, shapes)]
    a = grids[-1]
    parts = [grids[6 * i:6 * i + 6] for i in range(1 + c["half"])]
    fac = _kp_factors(c, parts)
    held = [[x.detach().requires_grad_(True) for x in f] for f in fac]
    ah = a.detach().requires_grad_(True)
    for b in range(c["blades"]):
        V = 0
        for Z, Xs, Ys, qx, qy, qs in held:
            for f in range(c["feat"]):
                xa = ah[f] * Xs[:, :, f] * qx[b, :, f] * qs[b, :, f][:, None]
                yf = Ys[:, :, f] * qy[b, :, f]
                V = V + Z[None, :, :, f] * xa[:, None, :] * yf[:, :, None]
        with torch.no_grad():
            r = M.mask[b] * (torch.fft.fft2(M.project(b, V.detach()), norm="ortho") - y[b])
            G = torch.zeros_like(V)
            M.back(b, torch.fft.ifft2(r, norm="ortho"), G)
        V.backward(G)
    outs = [x for f in fac for x in f] + [a]
    grads = [x.grad for f in held for x in f] + [ah.grad]
    torch.autograd.backward(outs, grads, retain_graph=True)
    _kp_reg(parts, _kp_model(c)[1]).backward()
    return leaf.grad


def _wide(t):
    return t.detach().to(torch.complex128)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "batch":
        out = []
        for i, s in enumerate(_batch_cases(c)):
            d = _inputs(s, seed + 100 * i)
            M, y = _Model(s, d["g"]), _wide(d["y"])
            vol = torch.zeros(1, s["S"], s["n"], s["n"], dtype=torch.complex128, device="cuda")
            for _ in range(c["steps"]):
                vol = vol - (1.0 / _stiff(s)) * (M.data_gradient(vol, y)[1] + _reg_gradient(vol, 0.0))
            out.append(dict(_renders(s, vol), vol=vol))
        return out
    d = _inputs(c, seed)
    M, y = _Model(c, d["g"]), _wide(d["y"])
    if kind == "operators":
        vol = _wide(d["vol"])
        res, grad = M.data_gradient(vol, y)
        new, m, v = _adam(vol, grad + _reg_gradient(vol, c["l1"]), _wide(d["m"]), _wide(d["v"]), RESUME_STEP + 1)
        return dict(res=res, grad=grad, vol=new, m=m, v=v)
    if kind == "autograd":
        vol = _wide(d["vol"])
        res, grad = M.data_gradient(vol, y)
        return dict(res=res, grad=grad + _reg_gradient(vol, c["l1"]))
    if kind == "nu":
        res, grad = M.data_gradient(_wide(d["vol"]), y, nu=True)
        return dict(res=res, grad=grad)
    if kind in ("fit", "nu_fit"):
        vol, m, v = _wide(d["vol"]), _wide(d["m"]), _wide(d["v"])
        for k in range(c["steps"]):
            grad = M.data_gradient(vol, y, nu=kind == "nu_fit")[1]
            vol, m, v = _adam(vol, grad + _reg_gradient(vol, 0.0), m, v, RESUME_STEP + k + 1)
        return _renders(c, vol) if kind == "fit" else dict(_renders(c, vol), vol=vol)
    if kind == "kplanes":
        p, m, v = _wide(d["p"]), _wide(d["m"]), _wide(d["v"])
        for k in range(c["steps"]):
            p, m, v = _adam(p, _kp_gradient(c, M, y, p), m, v, RESUME_STEP + k + 1)
        return dict(params=p, m=m, v=v)
    frames = []
    for f in range(c["blades"]):
        lo = max(0, f - 4)
        mk = M.mask[lo:f + 1]
        frames.append(torch.fft.ifft2((mk * y[lo:f + 1]).sum(0) / mk.sum(0).clamp(min=1.0), norm="ortho"))
    img, truth = _wide(d["frames"]).abs(), _wide(d["truth"]).abs()
    mse = ((img - truth) ** 2).mean((1, 2))
    peak = truth.amax((1, 2))
    return dict(baseline=torch.stack(frames), psnr=10 * torch.log10(peak ** 2 / mse), mse=mse, peak=peak)
