"""Workloads of the framework, as its users run them, through the public
entry points of ``paper_1409_8336_amd`` (``pmc.Engine``, ``unet.UNet`` and
the single-layer and evaluation calls).

A case is a dict of plain values; ``kind`` names the path:

- ``spots``: one plan transported on one CT, dose and variance into device
  tensors (or host arrays), optionally with LET_d, the intranuclear cascade,
  Vavilov straggling or Moliere scattering;
- ``plans``: plans of uneven size in one persistent launch;
- ``denoise``: U-Net inference on a dose grid (padded to the network's shape
  where the grid's sides are no multiples of 8);
- ``train``: forward, loss and backward of one volume, gradients read back;
- ``conv_forward`` / ``conv_backward``: one 3x3x3 convolution layer;
- ``evaluate``: the gamma index of an evaluated dose and the denoiser's
  fallback rule.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1409_8336_amd import pmc, synth, unet

DEV = "cuda:0"
VOXEL_CM = (0.2, 0.2, 0.2)
K_GROUPS = 10

_SPOTS = dict(kind="spots", phantom="ct", layers=1, per_layer=1, e_lo=150.0, e_hi=150.0, histories=1_000_000,
              let=False, inc=False, vavilov=False, moliere=False, host=False)


def _spots(name, **kw):
    return dict(_SPOTS, name=name, **kw)


def listed():
    return [
        # the smallest run in earnest: one pencil in a water tank, where the
        # serial chain of the longest histories and the launches count
        _spots("water_pencil_1e5", phantom="water", nx=64, ny=64, nz=128, e_lo=100.0, e_hi=100.0,
               histories=100_000),
        # a single beam spot on a CT: many histories into few voxels
        _spots("ct_spot_1e6", nx=128, ny=128, nz=160),
        # a treatment field: 40 energy layers, 2000 spots, 1e7 histories
        _spots("field_1e7", nx=256, ny=256, nz=200, layers=40, per_layer=50, e_lo=70.0, e_hi=230.0,
               histories=10_000_000),
        # dose and dose-averaged LET of a small field on a CT with odd sides
        _spots("field_let_2e6", nx=171, ny=147, nz=133, layers=12, per_layer=37, e_lo=80.0, e_hi=175.0,
               histories=2_000_000, let=True),
        # the detailed non-elastic model: cascade and evaporation of every event
        _spots("field_inc_1e6", nx=145, ny=247, nz=169, layers=9, per_layer=61, e_lo=90.0, e_hi=210.0,
               histories=1_000_000, inc=True),
        # several patients' plans of uneven size in one persistent launch
        dict(name="plans_6", kind="plans", plan_seed=100, plans=6, hist_scale=0.4, max_x=224, max_y=224, max_z=200),
        # denoiser inference on one full volume
        dict(name="denoise_160x128x128", kind="denoise", d=160, h=128, w=128),
        # denoiser inference on a plan's own grid, sides no multiples of 8
        dict(name="denoise_ragged", kind="denoise", d=109, h=121, w=187),
        # the gradient of one training volume (the training loop's inner call)
        dict(name="train_volume", kind="train", d=160, h=128, w=128),
        # one decoder layer of the network by itself
        dict(name="conv_forward_level1", kind="conv_forward", n=1, d=80, h=64, w=64, cin=96, cout=32, relu=True),
        # both gradients of a layer on a batch with odd sides
        dict(name="conv_backward_odd", kind="conv_backward", n=2, d=41, h=53, w=75, cin=48, cout=32),
        # judging an evaluated dose: 3-D gamma index and the fallback rule
        dict(name="evaluate_2mm", kind="evaluate", d=160, h=128, w=128, dose_frac=0.02, dta_cm=0.2, noise=0.03),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("spots",) * 5 + ("plans",) + ("denoise",) * 2 + ("train",) * 2 +
                      ("conv_forward",) * 2 + ("conv_backward",) * 2 + ("evaluate",) * 2)
    if kind == "spots":
        water = rng.random() < 0.2
        layers = rng.choice((1, 1, rng.randint(2, 30)))
        e_lo = rng.uniform(70.0, 180.0)
        opt = rng.choice(("none", "none", "let", "inc", "vavilov", "moliere"))
        c = dict(_SPOTS, phantom="water" if water else "ct", nx=rng.randint(48, 224), ny=rng.randint(48, 224),
                 nz=rng.randint(96, 200), layers=layers, per_layer=_log_int(rng, 1, 60), e_lo=round(e_lo, 1),
                 e_hi=round(rng.uniform(e_lo + 2.0, 220.0), 1), histories=_log_int(rng, 1e4, 4e6),
                 host=rng.random() < 0.15)
        if opt != "none":
            c[opt] = True
        return c
    if kind == "plans":
        return dict(kind=kind, plan_seed=rng.randint(200, 100000), plans=rng.randint(2, 6),
                    hist_scale=round(math.exp(rng.uniform(math.log(0.02), math.log(0.35))), 4),
                    max_x=rng.randint(100, 220), max_y=rng.randint(100, 220), max_z=rng.randint(100, 200))
    if kind == "denoise":
        return dict(kind=kind, d=_log_int(rng, 24, 160), h=_log_int(rng, 24, 128), w=_log_int(rng, 24, 190))
    if kind == "train":
        return dict(kind=kind, d=8 * _log_int(rng, 3, 20), h=8 * _log_int(rng, 3, 16), w=8 * _log_int(rng, 3, 16))
    if kind == "evaluate":
        tight = rng.random() < 0.5
        return dict(kind=kind, d=rng.randint(40, 160), h=rng.randint(40, 128), w=rng.randint(40, 128),
                    dose_frac=0.01 if tight else 0.02, dta_cm=0.1 if tight else 0.2,
                    noise=round(rng.uniform(0.005, 0.05), 4))
    chans = (8, 16, 16, 24, 32, 32, 48, 64, 96, 128, 192)
    while True:
        c = dict(kind=kind, n=rng.choice((1, 1, 2, 3)), d=_log_int(rng, 5, 160), h=_log_int(rng, 5, 128),
                 w=_log_int(rng, 5, 128), cin=rng.choice(chans), cout=rng.choice(chans))
        if kind == "conv_forward":
            c["relu"] = rng.random() < 0.7
        if 1e8 <= _conv_flops(c) <= 1.2e11 and c["n"] * c["d"] * c["h"] * c["w"] * (c["cin"] + c["cout"]) <= 2.0e8:
            return c


# ------------------------------------------------------------------- inputs

_nuclear = None


def _engine(case):
    global _nuclear
    if _nuclear is None:
        _nuclear = synth.nuclear_data()
    flags = (pmc.PMC_VAVILOV if case.get("vavilov") else 0) | (pmc.PMC_MOLIERE if case.get("moliere") else 0) | \
            (pmc.PMC_INC if case.get("inc") else 0)
    eng = pmc.Engine(0, flags=flags)
    eng.load_physics(_nuclear)
    return eng


def _phantom(case, seed):
    if case["phantom"] == "water":
        return synth.water_phantom(case["nx"], case["ny"], case["nz"])
    return synth.scaled_ct_phantom(case["nx"], case["ny"], case["nz"], seed=1000 + seed)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV)


def _dose(shape, seed, noise, n_beams=12):
    """A smooth dose of a few pencils that stop at their own depths (entrance
    plateau, peak, fall-off, in units of 1e-9 Gy as one history leaves it),
    the same dose with Monte Carlo noise, and a density map."""
    d, h, w = shape
    rng = np.random.default_rng(seed)
    z = torch.arange(d, device=DEV, dtype=torch.float64)[:, None, None]
    y = torch.arange(h, device=DEV, dtype=torch.float64)[None, :, None]
    x = torch.arange(w, device=DEV, dtype=torch.float64)[None, None, :]
    dose = torch.zeros(shape, dtype=torch.float64, device=DEV)
    for _ in range(n_beams):
        cx, cy = w * rng.uniform(0.35, 0.65), h * rng.uniform(0.35, 0.65)
        depth, sig = d * rng.uniform(0.3, 0.8), rng.uniform(1.8, 3.5)
        along = (0.35 + 0.3 * z / depth + 0.9 * torch.exp(-((z - depth + 2.0) / 3.0) ** 2)) * torch.sigmoid((depth - z) / 0.8)
        dose += rng.uniform(0.5, 1.5) * along * torch.exp(-((x - cx) ** 2 + (y - cy) ** 2) / (2 * sig * sig))
    dose *= 1e-9
    dose[dose < 1e-5 * dose.max()] = 0.0
    g = _gen(seed)
    sd = noise * (dose * dose.max()).sqrt()
    noisy = (dose + sd * torch.randn(shape, generator=g, device=DEV, dtype=torch.float64)).clamp_(min=0.0)
    rho = torch.ones(shape, dtype=torch.float32, device=DEV)
    for _ in range(9):
        c = [n * rng.uniform(0.1, 0.9) for n in shape]
        r = [rng.uniform(5.0, 20.0) for _ in range(3)]
        inside = ((z - c[0]) / r[0]) ** 2 + ((y - c[1]) / r[1]) ** 2 + ((x - c[2]) / r[2]) ** 2 <= 1.0
        rho[inside] = float(rng.choice((0.25, 1.04, 1.6)))
    return dose, noisy, sd * sd, rho


_CONVS = ((8, 16), (16, 32), (32, 64), (64, 128), (192, 64), (96, 32), (48, 16))   # enc1..4, dec3..1


def _net_params(seed):
    """A network in training: He-normal convolutions (BF16-representable), small
    biases and a head whose correction is a few per cent of the dose."""
    rng = np.random.default_rng(seed)
    parts = []
    for i, (cin, cout) in enumerate(_CONVS):
        bits, val = synth.conv_weights(rng, cin, cout, sd=(2.0 / (27 * (2 if i == 0 else cin))) ** 0.5)
        w = val.copy()
        if i == 0:
            w[:, :27 * cin].reshape(cout, 27, cin)[:, :, 2:] = 0.0
        parts += [w.ravel(), rng.normal(0.0, 0.02, cout)]
    parts += [rng.normal(0.0, 0.01, 16), rng.normal(0.0, 0.001, 1)]
    return np.concatenate(parts).astype(np.float32)


def _round8(v):
    return (v + 7) // 8 * 8


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "spots":
        eng = _engine(case)
        hu = _phantom(case, seed)
        eng.load_geometry(hu, VOXEL_CM, synth.material_table())
        if case["layers"] * case["per_layer"] == 1:
            spots = synth.pencil_spot(0.1 * case["nx"], 0.1 * case["ny"], case["e_lo"])
        else:
            spots = synth.spot_field((0.1 * case["nx"], 0.1 * case["ny"]), case["layers"], case["per_layer"],
                                     case["e_lo"], case["e_hi"], seed=seed)
        s.update(eng=eng, spots=spots, seed=seed + 1)
        if not case["host"]:
            for name in ("dose", "var") + (("let",) if case["let"] else ()):
                s[name] = torch.empty(hu.shape, dtype=torch.float64, device=DEV)
    elif kind == "plans":
        eng = _engine(case)
        mt = synth.material_table()
        # the batch's grids, spot positions and history counts are the case's;
        # patients (phantoms) and spot weights the seed's
        plans = synth.plan_set(case["plans"], case["plan_seed"], case["hist_scale"],
                               (case["max_x"], case["max_y"], case["max_z"]))
        rng = np.random.default_rng(seed)
        batch = []
        for i, p in enumerate(plans):
            nz, ny, nx = p["hu"].shape
            p["hu"] = synth.scaled_ct_phantom(nx, ny, nz, seed=int(rng.integers(1 << 40)))
            p["spots"][:, 5] = rng.lognormal(0.0, 0.5, len(p["spots"]))
            if i == 0:
                eng.load_geometry(p["hu"], p["voxel_cm"], mt)
            gid = pmc.pmc_load_geometry_slot(eng.ctx, p["hu"], p["voxel_cm"], mt) if i else 0
            batch.append(dict(geometry_id=gid, spots=p["spots"], n_histories=p["n_histories"],
                              d_dose=torch.empty(p["hu"].shape, dtype=torch.float64, device=DEV),
                              d_var=torch.empty(p["hu"].shape, dtype=torch.float64, device=DEV)))
        s.update(eng=eng, plans=batch, seed=seed + 1)
    elif kind == "denoise":
        shape = (case["d"], case["h"], case["w"])
        net_shape = tuple(_round8(v) for v in shape)
        net = unet.UNet((1,) + net_shape, seed=1)
        net.set_params(_net_params(seed))
        _, noisy, _, rho = _dose(shape, seed, 0.05)
        s.update(net=net, whole=net_shape == shape, dose=noisy.float(), rho=rho,
                 out=torch.empty(shape, dtype=torch.float32, device=DEV))
    elif kind == "train":
        shape = (case["d"], case["h"], case["w"])
        net = unet.UNet((1,) + shape, seed=1)
        net.set_params(_net_params(seed))
        dose, noisy, _, rho = _dose(shape, seed, 0.05)
        s.update(net=net, dose=noisy.float(), rho=rho, target=dose.float())
    elif kind in ("conv_forward", "conv_backward"):
        g = _gen(seed)
        vox = (case["n"], case["d"], case["h"], case["w"])
        x = _normal(g, *vox, case["cin"])
        x = torch.where(x > 0, x, 0.01 * x).bfloat16()     # what a leaky ReLU leaves
        wk = torch.zeros(case["cout"], unet.kp(case["cin"]), dtype=torch.bfloat16, device=DEV)
        wk[:, :27 * case["cin"]] = (_normal(g, case["cout"], 27 * case["cin"]) * (2.0 / (27 * case["cin"])) ** 0.5).bfloat16()
        s.update(x=x, w=wk)
        if kind == "conv_forward":
            s.update(bias=0.05 * _normal(g, case["cout"]),
                     y=torch.empty(*vox, case["cout"], dtype=torch.bfloat16, device=DEV))
        else:
            s.update(dy=(0.01 * _normal(g, *vox, case["cout"])).bfloat16(), dx=torch.empty_like(x),
                     dw=torch.zeros(case["cout"], unet.kp(case["cin"]), dtype=torch.float32, device=DEV))
    elif kind == "evaluate":
        shape = (case["d"], case["h"], case["w"])
        dose, noisy, var, _ = _dose(shape, seed, case["noise"])
        s.update(ref=dose, ev=noisy, var=var, den=(0.5 * (dose + noisy)).float(),
                 gamma=torch.empty(shape, dtype=torch.float32, device=DEV))
    else:
        raise ValueError("unknown kind %r" % kind)
    return s


# --------------------------------------------------------------------- runs

_COUNTS = ("histories", "steps", "secondaries", "n_elastic", "n_nonelastic", "n_short_steps")
_ENERGIES = ("incident", "deposited", "escaped", "neutral")


def _summary(sm):
    return {**{k: int(sm[k]) for k in _COUNTS}, **{k: float(sm[k]) for k in _ENERGIES}}


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "spots":
        eng, n = s["eng"], case["histories"]
        if case["host"]:
            if case["let"]:
                dose, var, let, sm = eng.run_spots_let(s["spots"], n, s["seed"])
                return {"dose": dose, "var": var, "let": let, **_summary(sm)}
            dose, var, sm = eng.run_spots(s["spots"], n, s["seed"])
            return {"dose": dose, "var": var, **_summary(sm)}
        if case["let"]:
            sm = eng.run_spots_let_dev(s["spots"], n, s["seed"], s["dose"], s["let"], s["var"])
            return {"dose": s["dose"], "var": s["var"], "let": s["let"], **_summary(sm)}
        sm = eng.run_spots_dev(s["spots"], n, s["seed"], s["dose"], s["var"])
        return {"dose": s["dose"], "var": s["var"], **_summary(sm)}
    if kind == "plans":
        sums = pmc.pmc_run_plans(s["eng"].ctx, s["plans"], s["seed"])
        # (secondaries are counted for the whole batch where they pass
        # through the shared queues: the sum is the plan-independent number)
        return {"dose": [p["d_dose"] for p in s["plans"]], "var": [p["d_var"] for p in s["plans"]],
                "steps": np.array([m["steps"] for m in sums], np.int64),
                "energies": np.array([[m[k] for k in _ENERGIES] for m in sums])}
    if kind == "denoise":
        if s["whole"]:
            s["net"].forward(s["dose"], s["rho"], s["out"])
        else:
            s["net"].forward_region(s["dose"], s["rho"], s["out"])
        return {"out": s["out"]}
    if kind == "train":
        net = s["net"]
        net.zero_grads()
        loss = net.backward(s["dose"], s["rho"], s["target"])
        return {"loss": loss, "grad_norm": net.grad_norm(), "grads": net.grads()}
    if kind == "conv_forward":
        unet.pmc_nn_conv3d_forward(s["x"], s["w"], s["bias"], s["y"], case["relu"])
        return {"y": s["y"]}
    if kind == "conv_backward":
        s["dw"].zero_()
        unet.pmc_nn_conv3d_backward_weight(s["x"], s["dy"], s["dw"])
        unet.pmc_nn_conv3d_backward_data_noalloc(s["dy"], s["w"], s["dx"])
        return {"dx": s["dx"], "dw": s["dw"]}
    if kind == "evaluate":
        rate, n = unet.pmc_gamma_index(s["ref"], s["ev"], VOXEL_CM, case["dose_frac"], case["dta_cm"], 0.1, 0.3, 0.05,
                                       gamma=s["gamma"])
        off, n_off = unet.pmc_denoise_disagreement(s["den"], s["ev"], s["var"], 0.1, 4.0)
        return {"gamma": s["gamma"], "pass_rate": rate, "n_eval": n, "disagreement": off, "n_above": n_off}
    raise ValueError("unknown kind %r" % kind)


# --------------------------------------------------------------------- work

def _conv_flops(c):
    return 2.0 * 27 * c["cin"] * c["cout"] * c["n"] * c["d"] * c["h"] * c["w"]


def _net_flops(d, h, w):
    level = (0, 1, 2, 3, 2, 1, 0)
    return sum(54.0 * (2 if i == 0 else cin) * cout * (d * h * w / 8.0 ** level[i])
               for i, (cin, cout) in enumerate(_CONVS))


def _steps(e_lo, e_hi, n, depth_cm):
    """Proton steps of n histories: one per voxel of path, to the range in
    water (Bragg-Kleeman) or the far face."""
    e = np.linspace(e_lo, e_hi, 16)
    return n * float(np.mean(np.minimum(0.0022 * e ** 1.77, depth_cm))) / VOXEL_CM[2]


def _transport_work(nvox, steps, let):
    # voxel records read, dose and variance (and LET_d) written; of the order
    # of 300 FP32 operations per step (random numbers, range table twice,
    # straggling, scattering, rotation)
    return {"bytes": nvox * (8 + 16 + (8 if let else 0)), "flops": 300.0 * steps}


def work(case):
    kind = case["kind"]
    if kind == "spots":
        return _transport_work(case["nx"] * case["ny"] * case["nz"],
                               _steps(case["e_lo"], case["e_hi"], case["histories"], 0.2 * case["nz"]), case["let"])
    if kind == "plans":
        nvox = case["plans"] * (96 + case["max_x"]) * (96 + case["max_y"]) * (96 + case["max_z"]) / 8.0
        return _transport_work(nvox, _steps(90.0, 190.0, case["plans"] * case["hist_scale"] * 3.9e6, 29.0), False)
    if kind in ("denoise", "train", "evaluate"):
        nv = case["d"] * case["h"] * case["w"]
        if kind == "denoise":
            return {"bytes": 12.0 * nv + 2.0 * 730_481, "flops": _net_flops(case["d"], case["h"], case["w"])}
        if kind == "train":
            return {"bytes": 12.0 * nv + 6.0 * 730_481, "flops": 3.0 * _net_flops(case["d"], case["h"], case["w"])}
        # reference, evaluated dose, its variance and the denoised dose read,
        # the gamma map written
        return {"bytes": 32.0 * nv, "flops": 100.0 * nv}
    nv = case["n"] * case["d"] * case["h"] * case["w"]
    wbytes = 2.0 * 27 * case["cin"] * case["cout"]
    if kind == "conv_forward":
        return {"bytes": 2.0 * nv * (case["cin"] + case["cout"]) + wbytes, "flops": _conv_flops(case)}
    return {"bytes": 2.0 * nv * (2 * case["cin"] + case["cout"]) + 3 * wbytes, "flops": 2.0 * _conv_flops(case)}


# -------------------------------------------------------------------- exact

class _Conv(torch.autograd.Function):
    """3x3x3 convolution, zero padding 1, of x [d][h][w][cin] with weights
    [27][cin][cout], as 27 shifted matrix products."""

    @staticmethod
    def _pad(x):
        return torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))

    @staticmethod
    def _shift(xp, t, shape):
        kz, ky, kx = t // 9, t // 3 % 3, t % 3
        d, h, w = shape
        return xp[kz:kz + d, ky:ky + h, kx:kx + w].reshape(d * h * w, -1)

    @staticmethod
    def forward(ctx, x, wt):
        shape = x.shape[:3]
        xp = _Conv._pad(x)
        y = torch.zeros(x[..., 0].numel(), wt.shape[2], dtype=x.dtype, device=x.device)
        for t in range(27):
            y += _Conv._shift(xp, t, shape) @ wt[t]
        ctx.save_for_backward(x, wt)
        return y.reshape(*shape, -1)

    @staticmethod
    def backward(ctx, dy):
        x, wt = ctx.saved_tensors
        shape = x.shape[:3]
        xp, dyp = _Conv._pad(x), _Conv._pad(dy)
        dy2 = dy.reshape(-1, dy.shape[-1])
        dx = torch.zeros(x[..., 0].numel(), x.shape[3], dtype=x.dtype, device=x.device)
        dw = torch.empty_like(wt)
        for t in range(27):
            dw[t] = _Conv._shift(xp, t, shape).T.contiguous() @ dy2
            dx += _Conv._shift(dyp, 26 - t, shape) @ wt[t].T.contiguous()
        return dx.reshape(x.shape), dw


def _taps(wk, cin):
    """[cout][Kp] -> [27][cin][cout] in 64 bits."""
    return wk[:, :27 * cin].double().reshape(-1, 27, cin).permute(1, 2, 0).contiguous()


def _leaky(x):
    return torch.where(x > 0, x, 0.01 * x)


def _net(dose, rho, p):
    """The network in 64 bits: dose and density [d][h][w], p the float64
    parameter vector; returns (denoised dose, scale)."""
    off = 0
    taken = []
    for cin, cout in _CONVS:
        kp = unet.kp(cin)
        wt = p[off:off + cout * kp].reshape(cout, kp)[:, :27 * cin].reshape(cout, 27, cin).permute(1, 2, 0).contiguous()
        off += cout * kp
        taken.append((wt, p[off:off + cout]))
        off += cout

    def layer(i, x):
        return _leaky(_Conv.apply(x, taken[i][0]) + taken[i][1])

    def pool(x):
        d, h, w, c = x.shape
        return x.reshape(d // 2, 2, h // 2, 2, w // 2, 2, c).mean((1, 3, 5))

    def up(x):
        d, h, w, c = x.shape
        return x[:, None, :, None, :, None].expand(d, 2, h, 2, w, 2, c).reshape(2 * d, 2 * h, 2 * w, c)

    scale = dose.max().clamp(min=1e-30)
    x = torch.zeros(*dose.shape, 8, dtype=torch.float64, device=dose.device)
    x[..., 0] = dose / scale
    x[..., 1] = 0.5 * rho
    e1 = layer(0, x)
    e2 = layer(1, pool(e1))
    e3 = layer(2, pool(e2))
    e4 = layer(3, pool(e3))
    d3 = layer(4, torch.cat((up(e4), e3), 3))
    d2 = layer(5, torch.cat((up(d3), e2), 3))
    d1 = layer(6, torch.cat((up(d2), e1), 3))
    head = d1 @ p[off:off + 16] + p[off + 16]
    return dose + scale * head, scale


def _exact_gamma(ref, ev, case):
    """The gamma map (-1 below the cutoff) over the search sphere, in 64 bits."""
    step, search = 0.05, 0.3
    dmax = ref.max()
    zs, ys, xs = torch.nonzero(ref >= float(np.float32(0.1)) * dmax, as_tuple=True)
    r = ref[zs, ys, xs]
    crit = float(np.float32(case["dose_frac"])) * dmax
    dta = case["dta_cm"]
    best = ((ev[zs, ys, xs] - r) / crit) ** 2
    nz, ny, nx = ref.shape
    m = int(math.floor(search / step + 1e-4))
    flat = ev.reshape(-1)
    for k in range(-m, m + 1):
        for j in range(-m, m + 1):
            for i in range(-m, m + 1):
                if i * i + j * j + k * k > (search / step) ** 2 * (1 + 1e-6) or (i, j, k) == (0, 0, 0):
                    continue
                pos, ok = [], None
                for v, o, n, c in ((xs, i, nx, VOXEL_CM[0]), (ys, j, ny, VOXEL_CM[1]), (zs, k, nz, VOXEL_CM[2])):
                    f = v.double() + o * step / c
                    good = (f >= 0) & (f <= n - 1)
                    ok = good if ok is None else ok & good
                    f = f.clamp(0, n - 1)
                    i0 = f.long().clamp(max=n - 1)
                    pos.append((i0, (i0 + 1).clamp(max=n - 1), f - i0))
                (x0, x1, tx), (y0, y1, ty), (z0, z1, tz) = pos
                e = 0.0
                for za, wz in ((z0, 1 - tz), (z1, tz)):
                    for ya, wy in ((y0, 1 - ty), (y1, ty)):
                        base = (za * ny + ya) * nx
                        e = e + wz * wy * (flat[base + x0] * (1 - tx) + flat[base + x1] * tx)
                g2 = (i * i + j * j + k * k) * step * step / (dta * dta) + ((e - r) / crit) ** 2
                best = torch.where(ok & (g2 < best), g2, best)
    out = torch.full_like(ref, -1.0)
    out[zs, ys, xs] = best.sqrt()
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("spots", "plans"):
        return None        # a random realisation: the engine's own FP32 decisions define it
    s = prepare(case, seed)
    if kind == "conv_forward":
        wt = _taps(s["w"], case["cin"])
        y = torch.stack([_Conv.apply(x, wt) for x in s["x"].double()]) + s["bias"].double()
        return {"y": _leaky(y) if case["relu"] else y}
    if kind == "conv_backward":
        wt = _taps(s["w"], case["cin"]).requires_grad_()
        dxs = []
        for x, dy in zip(s["x"].double(), s["dy"].double()):
            x.requires_grad_()
            _Conv.apply(x, wt).backward(dy)
            dxs.append(x.grad)
        dw = torch.zeros(s["dw"].shape, dtype=torch.float64, device=DEV)
        dw[:, :27 * case["cin"]] = wt.grad.permute(2, 0, 1).reshape(case["cout"], -1)
        return {"dx": torch.stack(dxs), "dw": dw}
    if kind == "denoise":
        pad = [q for n in (case["w"], case["h"], case["d"]) for q in (0, _round8(n) - n)]
        p = torch.from_numpy(s["net"].params()).to(DEV).double()
        dose, rho = (torch.nn.functional.pad(s[k].double(), pad) for k in ("dose", "rho"))
        out, _ = _net(dose, rho, p)
        return {"out": out[:case["d"], :case["h"], :case["w"]].contiguous()}
    if kind == "train":
        p = torch.from_numpy(s["net"].params()).to(DEV).double().requires_grad_()
        dose = s["dose"].double()
        out, scale = _net(dose, s["rho"].double(), p)
        region = (s["dose"] >= 0.01 * s["dose"].max()).sum().clamp(min=1)
        loss = (((out - s["target"].double()) / scale) ** 2).sum() / region
        loss.backward()
        return {"loss": float(loss.detach()), "grad_norm": float(p.grad.norm()), "grads": p.grad}
    return {"gamma": _exact_gamma(s["ref"], s["ev"], case), "pass_rate": None, "n_eval": None, "disagreement": None,
            "n_above": None}
