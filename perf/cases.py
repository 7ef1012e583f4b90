"""The work that users of this package have it do, as cases that can be timed.

Each case is a dict of plain values; `prepare` makes what a program holds
before the call (media, sources, measured data, weights), `run` is one pass
through the public entry points, `work` what a pass cannot do without, and
`exact` its result in 64 bits where plain torch can give it.  The Monte Carlo
runs have no such value: their outputs are a function of the packets' random
numbers.

Kinds of case ("op"):
  forward   rmc.mc_forward: the coefficient maps of an illumination
  adjoint   rmc.mc_adjoint of a signed volumetric source
  gradient  one evaluation of the error functional and its gradients:
            forward, residual, adjoint, gradient
  autograd  autograd.absorbed_energy, error_functional and backward(), as a
            reconstruction evaluates them
  batch     rmc.mc_run_batch over problems of several grids and wavelengths
  post      residual, gradients and detector readout of given maps
  conv      one 3x3 convolution layer of the denoiser, forward and backward
  unet      denoise.denoise of coefficient maps
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1608_05238_amd import autograd as A
from paper_1608_05238_amd import denoise as D
from paper_1608_05238_amd import rmc

SIDE = 25.6   # mm, the width of the disc workloads


def listed():
    return [
        # the smallest call: a coarse grid and a few thousand packets, as a
        # test, a finite difference or an interactive preview runs it
        {"name": "preview_24", "op": "forward", "nx": 24, "nz": 24, "side": 6.0, "mua": 0.05, "mus": 6.0, "g": 0.85,
         "source": "point", "packets": 4000, "n_harm": 5},
        # pencil beam on 32 x 32 pixels of 0.5 mm, 1e5 packets, N = 8
        {"name": "pencil_32", "op": "forward", "nx": 32, "nz": 32, "side": 16.0, "mua": 0.05, "mus": 5.0, "g": 0.8,
         "source": "pencil", "packets": 100_000, "n_harm": 8},
        # the same grid at the benchmark's packet count: more packets than the
        # whole-grid transport takes
        {"name": "pencil_32_1e8", "op": "forward", "nx": 32, "nz": 32, "side": 16.0, "mua": 0.05, "mus": 5.0, "g": 0.8,
         "source": "pencil", "packets": 100_000_000, "n_harm": 8},
        # a low-count input of the denoiser: 256 x 256 discs, four line sources
        {"name": "disc_256_1e6", "op": "forward", "nx": 256, "nz": 256, "side": SIDE, "mua": 0.01, "mus": 10.0,
         "g": 0.9, "source": "lines", "packets": 1_000_000, "n_harm": 16},
        # the benchmark's forward run
        {"name": "disc_256_1e8", "op": "forward", "nx": 256, "nz": 256, "side": SIDE, "mua": 0.01, "mus": 10.0,
         "g": 0.9, "source": "lines", "packets": 100_000_000, "n_harm": 16},
        # the highest harmonic order, on a grid that is not a multiple of
        # anything
        {"name": "adjoint_n32", "op": "adjoint", "nx": 149, "nz": 101, "side": 20.0, "mua": 0.02, "mus": 8.0, "g": 0.85,
         "packets": 500_000, "n_harm": 32},
        # a gradient at the packet count that first meets the error targets
        {"name": "gradient_256", "op": "gradient", "nx": 256, "nz": 256, "side": SIDE, "mua": 0.01, "mus": 10.0,
         "g": 0.9, "source": "lines", "packets": 2_830_000, "n_harm": 16},
        # one evaluation of a small reconstruction
        {"name": "recon_48", "op": "autograd", "nx": 48, "nz": 48, "side": 12.0, "mua": 0.02, "mus": 8.0, "g": 0.85,
         "source": "lines", "packets": 200_000, "n_harm": 10},
        # wavelengths and grids of one study in one packet pool
        {"name": "batch_12", "op": "batch", "problems": 12, "grid": 192, "side": SIDE, "mua": 0.01, "mus": 10.0,
         "g": 0.9, "packets": 1_000_000, "n_harm": 16},
        # the arithmetic between the runs: residual, gradients, readout
        {"name": "post_256", "op": "post", "nx": 256, "nz": 256, "side": SIDE, "mua": 0.01, "mus": 10.0, "g": 0.9,
         "n_harm": 16},
        # a layer of the denoiser at full resolution in training
        {"name": "conv_48", "op": "conv", "n": 16, "ci": 48, "co": 48, "h": 256, "w": 256},
        # the denoiser on an input and its two halves
        {"name": "unet_256", "op": "unet", "n": 3, "h": 256, "w": 256, "n_harm": 16, "widths": "24,32,48,64,96,128"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["small", "forward", "forward", "adjoint", "gradient", "autograd", "batch", "post", "conv", "unet"])
    tissue = {"mua": round(rng.uniform(0.005, 0.05), 4), "mus": round(rng.uniform(4.0, 12.0), 2),
              "g": round(rng.uniform(0.7, 0.92), 3)}
    if op == "small":
        return {"op": "forward", "nx": rng.randint(7, 32), "nz": rng.randint(7, 32), "side": round(rng.uniform(4, 16), 2),
                **tissue, "source": rng.choice(["point", "pencil", "lines", "lambertian"]),
                "packets": _log(rng, 1000, 1_000_000), "n_harm": rng.randint(1, 8)}
    if op in ("forward", "adjoint", "gradient"):
        top = {"forward": 20_000_000, "adjoint": 5_000_000, "gradient": 3_000_000}[op]
        c = {"op": op, "nx": rng.randint(64, 300), "nz": rng.randint(64, 300), "side": round(rng.uniform(10, SIDE), 2),
             **tissue, "packets": _log(rng, 50_000, top), "n_harm": rng.choice([4, 8, 10, 16, 16, 16, 24, 32])}
        if op != "adjoint":
            c["source"] = rng.choice(["lines", "lines", "lambertian", "pencil", "point"])
        return c
    if op == "autograd":
        return {"op": op, "nx": rng.randint(28, 128), "nz": rng.randint(28, 128), "side": round(rng.uniform(6, 20), 2),
                **tissue, "source": rng.choice(["lines", "lambertian"]), "packets": _log(rng, 50_000, 1_000_000),
                "n_harm": rng.choice([4, 8, 10, 16])}
    if op == "batch":
        return {"op": op, "problems": rng.randint(3, 20), "grid": rng.randint(64, 200), "side": SIDE, **tissue,
                "packets": _log(rng, 50_000, 1_000_000), "n_harm": rng.choice([8, 16, 16])}
    if op == "post":
        return {"op": op, "nx": rng.randint(32, 512), "nz": rng.randint(32, 512), "side": SIDE, **tissue,
                "n_harm": rng.randint(0, 32)}
    if op == "conv":
        return {"op": op, "n": rng.randint(1, 16), "ci": rng.choice([17, 24, 33, 48, 64, 96, 112, 160, 224]),
                "co": rng.choice([24, 32, 48, 64, 96, 128]), "h": rng.randint(16, 256), "w": rng.randint(16, 256)}
    return {"op": "unet", "n": rng.randint(1, 16), "h": rng.randint(48, 256), "w": rng.randint(48, 256),
            "n_harm": rng.choice([8, 10, 16]), "widths": rng.choice(["48,64,96", "24,32,48,64,96,128"])}


# ---------------------------------------------------------------- inputs

def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _centres(c):
    dx = c["side"] / max(c["nx"], c["nz"])
    return (*np.meshgrid((np.arange(c["nx"]) + 0.5) * dx, (np.arange(c["nz"]) + 0.5) * dx), dx)


def _medium(c, seed):
    """Background with three to six random discs: mua x 2-10, mus x 0.5-2."""
    rng = np.random.default_rng(seed)
    X, Z, dx = _centres(c)
    mua = np.full(X.shape, c["mua"], np.float32)
    mus = np.full(X.shape, c["mus"], np.float32)
    w, h = c["nx"] * dx, c["nz"] * dx
    for _ in range(int(rng.integers(3, 7))):
        r = rng.uniform(0.04, 0.16) * min(w, h)
        inside = (X - rng.uniform(r, w - r)) ** 2 + (Z - rng.uniform(r, h - r)) ** 2 <= r * r
        mua[inside] = c["mua"] * rng.uniform(2, 10)
        mus[inside] = c["mus"] * rng.uniform(0.5, 2)
    dev = _dev()
    return rmc.Medium(torch.as_tensor(mua, device=dev), torch.as_tensor(mus, device=dev),
                      torch.full(mua.shape, c["g"], dtype=torch.float32, device=dev), dx)


def _sources(kind, med):
    w, h = med.nx * med.dx, med.nz * med.dx
    if kind == "pencil":
        return [rmc.Source("pencil", x0=w / 2, z0=0.0, dir_x=0.0, dir_z=1.0)]
    if kind == "point":
        return [rmc.Source("point", x0=0.4 * w, z0=0.45 * h)]
    lam = int(kind == "lambertian")
    return [rmc.Source("line", 0.0, 0.0, w, 0.0, 0.0, 1.0, lam, 0.25), rmc.Source("line", 0.0, h, w, h, 0.0, -1.0, lam, 0.25),
            rmc.Source("line", 0.0, 0.0, 0.0, h, 1.0, 0.0, lam, 0.25), rmc.Source("line", w, 0.0, w, h, -1.0, 0.0, lam, 0.25)]


def _blobs(c, med, seed):
    """A signed smooth map shaped like an adjoint source mua (Hmeas - H)."""
    rng = np.random.default_rng(seed)
    X, Z, dx = _centres(c)
    q = np.zeros(X.shape)
    for _ in range(6):
        s = rng.uniform(0.05, 0.2) * c["side"]
        q += rng.choice([-1.0, 1.0]) * rng.uniform(0.5, 1.5) * np.exp(
            -((X - rng.uniform(0, c["nx"] * dx)) ** 2 + (Z - rng.uniform(0, c["nz"] * dx)) ** 2) / (2 * s * s))
    mua = med.mua.double()
    return 1e-3 * torch.as_tensor(q, device=mua.device) * mua / mua.mean()


def _measured(c, src_kind, seed):
    """Absorbed energy of another phantom, as the measured data."""
    other = _medium(c, seed + 500)
    f, _ = rmc.mc_forward(other, _sources(src_kind, other), rmc.make_run(200_000, 0, seed=seed + 900), ledger=False)
    return rmc.mc_absorbed(other, f)


def _maps(c, seed, n):
    """Coefficient maps of n fields: a smooth fluence and harmonics that fall
    off with the order, with Monte Carlo noise."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dev, N, h, w = _dev(), c["n_harm"], c.get("h", c.get("nz")), c.get("w", c.get("nx"))
    order = torch.cat([torch.arange(N + 1), torch.arange(1, N + 1)]).to(dev)
    x, z = torch.linspace(0, 1, w, device=dev), torch.linspace(0, 1, h, device=dev)
    k = torch.rand(n, 2 * N + 1, 2, generator=g, device=dev) * 6
    smooth = torch.cos(k[..., :1, None] * z[:, None] + k[..., 1:, None] * x[None, :])
    smooth[:, 0] = 1.5 + 0.5 * smooth[:, 0]
    noise = torch.randn(smooth.shape, generator=g, device=dev)
    return ((smooth + 0.05 * noise) * (0.85 ** order)[None, :, None, None] * 0.05).double()


def prepare(case, seed):
    c, op = case, case["op"]
    if op == "conv":
        g = torch.Generator(device="cuda").manual_seed(seed)
        layer = D.Conv3x3(c["ci"], c["co"]).to(_dev())
        with torch.no_grad():
            layer.weight.copy_(torch.randn(layer.weight.shape, generator=g, device=_dev()) * math.sqrt(2.0 / (9 * c["ci"])))
            layer.bias.copy_(0.1 * torch.randn(layer.bias.shape, generator=g, device=_dev()))
        # activations after a ReLU, channels last as the layers hand them on
        x = torch.randn(c["n"], c["ci"], c["h"], c["w"], generator=g, device=_dev()).relu_()
        gy = torch.randn(c["n"], c["co"], c["h"], c["w"], generator=g, device=_dev())
        cl = torch.channels_last
        return {"op": op, "layer": layer, "x": x.contiguous(memory_format=cl).requires_grad_(True),
                "gy": gy.contiguous(memory_format=cl)}
    if op == "unet":
        g = torch.Generator(device="cuda").manual_seed(seed)
        model = D.UNet(2 * c["n_harm"] + 1, tuple(int(v) for v in c["widths"].split(","))).to(_dev())
        with torch.no_grad():
            for name, p in model.named_parameters():
                if p.dim() == 4:
                    p.copy_(torch.randn(p.shape, generator=g, device=_dev()) * math.sqrt(2.0 / (9 * p.shape[1])))
                else:   # biases; the output layer of a trained network corrects by a few percent
                    p.copy_(0.01 * torch.randn(p.shape, generator=g, device=_dev()))
        return {"op": op, "model": model, "maps": _maps(c, seed, c["n"])}
    if op == "batch":
        probs = []
        for i in range(c["problems"]):
            n = c["grid"] * (2, 3, 4)[i % 3] // 3
            ci = {**c, "nx": n, "nz": n, "mua": c["mua"] * (0.5, 1.0, 2.0, 4.0)[i % 4]}
            med = _medium(ci, seed * 64 + i)
            adj = i % 4 == 3
            src = [rmc.Source("map", map=_blobs(ci, med, seed + i))] if adj else _sources("lines", med)
            run_i = rmc.make_run(c["packets"] * (1 + i % 3) // 2, c["n_harm"], seed=seed + i, stream_tag=int(adj))
            probs.append(rmc.Problem(med, src, run_i, adj))
        return {"op": op, "probs": probs}
    med = _medium(c, seed)
    s = {"op": op, "case": c, "med": med}
    if op == "forward":
        return {**s, "src": _sources(c["source"], med), "run": rmc.make_run(c["packets"], c["n_harm"], seed=seed)}
    if op == "adjoint":
        return {**s, "src": [rmc.Source("map", map=_blobs(c, med, seed))],
                "run": rmc.make_run(c["packets"], c["n_harm"], seed=seed, stream_tag=1)}
    if op == "gradient":
        return {**s, "src": _sources(c["source"], med), "run": rmc.make_run(c["packets"], c["n_harm"], seed=seed),
                "run_adj": rmc.make_run(c["packets"], c["n_harm"], seed=seed, stream_tag=1),
                "hmeas": _measured(c, c["source"], seed)}
    if op == "autograd":
        return {**s, "src": _sources(c["source"], med), "cfg": A.MCConfig(c["packets"], c["n_harm"], seed=seed),
                "hmeas": _measured(c, c["source"], seed), "mua": med.mua.double().requires_grad_(True),
                "mus": med.mus.double().requires_grad_(True)}
    fwd, adj, det = _maps(c, seed, 3).unbind(0)
    return {**s, "fwd": fwd.contiguous(), "adj": 1e-4 * (adj - adj.mean()), "det": det.contiguous(),
            "hmeas": (fwd[0] * med.mua.double() * (1.0 + 0.1 * torch.sin(3.0 * adj[0]))).contiguous()}


# ---------------------------------------------------------------- one pass

def run(state):
    s, op = state, state["op"]
    if op == "forward":
        return rmc.mc_forward(s["med"], s["src"], s["run"])[0]
    if op == "adjoint":
        return rmc.mc_adjoint(s["med"], s["src"], s["run"])[0]
    if op == "gradient":
        N = s["case"]["n_harm"]
        fwd, _ = rmc.mc_forward(s["med"], s["src"], s["run"], ledger=False)
        q, eps = rmc.mc_residual(s["med"], fwd, s["hmeas"])
        adj, _ = rmc.mc_adjoint(s["med"], [rmc.Source("map", map=q)], s["run_adj"], ledger=False)
        dmua, dmus = rmc.mc_gradient(s["med"], N, fwd, adj, s["hmeas"])
        return {"fwd": fwd, "q": q, "eps": eps, "adj": adj, "dmua": dmua, "dmus": dmus}
    if op == "autograd":
        s["mua"].grad = s["mus"].grad = None
        h = A.absorbed_energy(s["mua"], s["mus"], s["med"].g, s["med"].dx, s["src"], s["cfg"])
        eps = A.error_functional(h, s["hmeas"], s["med"].dx)
        eps.backward()
        return {"h": h, "eps": eps, "dmua": s["mua"].grad, "dmus": s["mus"].grad}
    if op == "batch":
        return [out for out, _ in rmc.mc_run_batch(s["probs"])]
    if op == "post":
        N = s["case"]["n_harm"]
        q, eps = rmc.mc_residual(s["med"], s["fwd"], s["hmeas"])
        dmua, dmus = rmc.mc_gradient(s["med"], N, s["fwd"], s["adj"], s["hmeas"])
        read = rmc.mc_detect(s["med"], N, s["fwd"], s["det"])
        return {"q": q, "eps": eps, "dmua": dmua, "dmus": dmus, "read": read}
    if op == "conv":
        x, layer = s["x"], s["layer"]
        x.grad = layer.weight.grad = layer.bias.grad = None
        y = layer(x)
        y.backward(s["gy"])
        return {"y": y, "gx": x.grad, "gw": layer.weight.grad, "gb": layer.bias.grad}
    return D.denoise(s["model"], s["maps"])


# ---------------------------------------------------------------- what a pass needs

def _mc_work(c, packets, n_harm, adjoint):
    """Inputs and outputs once, and the method's arithmetic: the mean path of
    light that enters through the boundary is pi area / perimeter whatever the
    scattering, about 2.2 times that for a volumetric source; a path crosses
    4 / (pi dx) pixel faces and scatters mus times per length.  Per segment 23
    operations and a multiply-add per channel, per scatter 82 + 2 N."""
    dx = c["side"] / max(c["nx"], c["nz"])
    w, h = c["nx"] * dx, c["nz"] * dx
    path = math.pi * w * h / (2 * (w + h)) * (2.2 if adjoint else 1.0)
    K, npix = 2 * n_harm + 1, c["nx"] * c["nz"]
    scatters = path * c["mus"]
    segments = scatters + path * 4 / (math.pi * dx)
    return {"bytes": npix * (12.0 + 8 * K + (8 if adjoint else 0)),
            "flops": packets * (89.0 + segments * (23 + 2 * K) + scatters * (82 + 2 * n_harm))}


def _sum(*works):
    return {k: sum(w[k] for w in works) for k in ("bytes", "flops")}


def _unet_layers(c):
    """(pixels, ci, co) of each convolution, and the output layer's width."""
    widths, ch = [int(v) for v in c["widths"].split(",")], 2 * c["n_harm"] + 1
    size, h, w = [], c["h"], c["w"]
    for _ in widths:
        size.append(c["n"] * h * w)
        h, w = -(-h // 2), -(-w // 2)
    convs, ci = [], ch
    for s, v in zip(size, widths):
        convs += [(s, ci, v), (s, v, v)]
        ci = v
    for s, v in reversed(list(zip(size, widths))[:-1]):
        convs += [(s, ci + v, v), (s, v, v)]
        ci = v
    return convs, ci, ch


def work(case):
    c, op = case, case["op"]
    if op in ("forward", "adjoint"):
        return _mc_work(c, c["packets"], c["n_harm"], op == "adjoint")
    if op in ("gradient", "autograd"):
        npix, K = c["nx"] * c["nz"], 2 * c["n_harm"] + 1
        return _sum(_mc_work(c, c["packets"], c["n_harm"], False), _mc_work(c, c["packets"], c["n_harm"], True),
                    {"bytes": npix * (16.0 * K + 40), "flops": npix * 4.0 * K})
    if op == "batch":
        return _sum(*(_mc_work({**c, "nx": n, "nz": n}, c["packets"] * (1 + i % 3) // 2, c["n_harm"], i % 4 == 3)
                      for i in range(c["problems"]) for n in [c["grid"] * (2, 3, 4)[i % 3] // 3]))
    if op == "post":
        npix, K = c["nx"] * c["nz"], 2 * c["n_harm"] + 1
        # forward, adjoint and detector maps, mua, g, Hmeas; q*, two gradients
        return {"bytes": npix * (3 * 8.0 * K + 8 + 8 + 24), "flops": npix * 9.0 * K}
    if op == "conv":
        P = c["n"] * c["h"] * c["w"]
        # x, gy read; y, gx written, FP32; the weights and their gradient
        return {"bytes": 4.0 * P * (2 * c["ci"] + 2 * c["co"]) + 4.0 * 2 * 9 * c["ci"] * c["co"],
                "flops": 3 * 2.0 * 9 * c["ci"] * c["co"] * P}
    convs, last, ch = _unet_layers(c)
    P = c["n"] * c["h"] * c["w"]
    return {"bytes": P * ch * 12.0 + 4.0 * 9 * sum(ci * co for _, ci, co in convs),
            "flops": sum(2.0 * 9 * p * ci * co for p, ci, co in convs) + 2.0 * P * ch * last}


# ---------------------------------------------------------------- results in 64 bits

def _conv64(x, w, b):
    """3x3 convolution with zero padding 1 as nine matrix products per image."""
    n, ci, h, wd = x.shape
    co = w.shape[0]
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1))
    y = torch.empty(n, co, h, wd, dtype=torch.float64, device=x.device)
    for i in range(n):
        acc = b[:, None].expand(co, h * wd).clone()
        for ky in range(3):
            for kx in range(3):
                acc += w[:, :, ky, kx].contiguous() @ xp[i, :, ky:ky + h, kx:kx + wd].reshape(ci, h * wd)
        y[i] = acc.view(co, h, wd)
    return y


def _wgrad64(x, gy):
    n, ci, h, wd = x.shape
    co = gy.shape[1]
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1))
    gw = torch.zeros(co, ci, 3, 3, dtype=torch.float64, device=x.device)
    for i in range(n):
        g = gy[i].reshape(co, h * wd)
        for ky in range(3):
            for kx in range(3):
                gw[:, :, ky, kx] += g @ xp[i, :, ky:ky + h, kx:kx + wd].reshape(ci, h * wd).t().contiguous()
    return gw


def _unet64(model, x):
    F = torch.nn.functional
    conv = lambda m, v: F.relu(_conv64(v, m.weight.double(), m.bias.double()))
    skips, h = [], x
    for i, (c1, c2) in enumerate(model.enc):
        h = conv(c2, conv(c1, h))
        if i < len(model.enc) - 1:
            skips.append(h)
            h = F.max_pool2d(h, 2, ceil_mode=True)
    for c1, c2 in model.dec:
        s = skips.pop()
        h = F.interpolate(h, scale_factor=2, mode="nearest")[:, :, :s.shape[2], :s.shape[3]]
        h = conv(c2, conv(c1, torch.cat([h, s], 1)))
    corr = torch.stack([(model.out.double() @ v.reshape(v.shape[0], -1)).view(-1, *v.shape[1:]) for v in h])
    return x + corr + model.out_bias.double()[None, :, None, None]


@torch.no_grad()
def exact(case, seed):
    op = case["op"]
    if op not in ("post", "conv", "unet"):
        return None
    s = prepare(case, seed)
    if op == "conv":
        x, gy, w = s["x"].detach().double().contiguous(), s["gy"].double().contiguous(), s["layer"].weight.double()
        zero = torch.zeros(case["ci"], dtype=torch.float64, device=x.device)
        return {"y": _conv64(x, w, s["layer"].bias.double()), "gx": _conv64(gy, w.flip(2, 3).transpose(0, 1), zero),
                "gw": _wgrad64(x, gy), "gb": gy.sum((0, 2, 3))}
    if op == "unet":
        x = s["maps"]
        scale = x[:, 0].pow(2).mean((1, 2)).sqrt()[:, None, None, None]
        return _unet64(s["model"], x / scale) * scale
    med, fwd, adj, N = s["med"], s["fwd"], s["adj"], case["n_harm"]
    mua, g, area = med.mua.double(), med.g.double(), float(np.float32(med.dx)) ** 2
    r = s["hmeas"] - mua * fwd[0]
    n = torch.arange(1, N + 1, device=g.device)[:, None, None]
    pr = fwd[1:N + 1] * adj[1:N + 1] + fwd[N + 1:] * adj[N + 1:]
    dmua = area * (-fwd[0] * r + fwd[0] * adj[0] / (2 * math.pi) + pr.sum(0) / math.pi)
    d = s["det"]
    read = area * (fwd[0] * d[0] / (2 * math.pi) + (fwd[1:] * d[1:]).sum(0) / math.pi).sum()
    return {"q": mua * r, "eps": 0.5 * area * (r * r).sum(), "dmua": dmua,
            "dmus": area * (pr * (1 - g[None] ** n)).sum(0) / math.pi, "read": read}
