"""The workloads that performance work on this package is measured on.

Each case is one call a program makes: a two-step transport run whose images
stay on the GPU (``Context.run`` + ``images_device``), a denoiser inference,
or a denoiser gradient.  Media, cameras and networks are those of
``workloads.py`` (the flared disk, the clumped slab, the uniform and refined
spheres, the dust cylinder, tabulated grains; the default and the wide
U-Net), at the sizes the training driver, the benchmark and the tests use,
and at odd ones.
"""
import math

import numpy as np
import torch

from paper_2512_01283_amd import denoiser as DN
from paper_2512_01283_amd import polrad as P
from paper_2512_01283_amd import workloads as W


def listed():
    return [
        # a parity-sized run: latency, one camera, FP64 polarisation
        dict(name="sphere32", kind="sphere", n=32, packets=4000, views=1, npix=64, fp64=True),
        # the denoiser's training inputs: a million packets through a 256^3
        # disk seen at 8 inclinations, Rayleigh spheres ...
        dict(name="disk256_1e6", kind="disk", n=256, packets=1_000_000, views=8, npix=256),
        # ... or aligned oblate grains in a helical field
        dict(name="aligned256_1e6", kind="aligned_disk", n=256, packets=1_000_000, views=8, npix=256),
        # the benchmark's disk at its packet count
        dict(name="disk256_1e8", kind="disk", n=256, packets=100_000_000, views=8, npix=256),
        # several wavelengths with uneven packet counts in one launch, many cameras, a grid of odd size
        dict(name="batched150_8", kind="batched", n=150, n_lambda=8, packets=4_000_000, views=16, npix=150),
        # the clumped dichroic slab of the verification runs
        dict(name="slab128_3e6", kind="slab", n=128, packets=3_000_000, views=4, npix=128),
        # grains with a tabulated scattering matrix: one source per camera
        dict(name="table128_2e6", kind="table", n=128, packets=2_000_000, views=8, npix=128),
        # static mesh refinement around the star
        dict(name="mesh128_2e6", kind="mesh", rx=8, block=16, packets=2_000_000, views=2, npix=128),
        # the dust's own thermal emission, self-scattered
        dict(name="cylinder101_1e6", kind="cylinder", n=101, packets=1_000_000, views=2, npix=101),
        # one image pair denoised in passing: launches and latency, sizes that fill no tile
        dict(name="infer_2x100x172", kind="infer", batch=2, h=100, w=172, wide=False, tta=False),
        # the 8 maps of one run denoised in the configuration whose gain is quoted
        dict(name="infer_tta_8x256", kind="infer", batch=8, h=256, w=256, wide=True, tta=True),
        # the gradient of one training step on the 8 maps of one disk, augmented
        dict(name="grad_8x256", kind="grad", batch=8, h=256, w=256, wide=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sphere", "disk", "aligned_disk", "batched", "slab", "table", "mesh", "cylinder",
                       "infer", "infer", "grad"])
    if kind in ("infer", "grad"):
        # maps whose sides are multiples of 4 (three levels); square ones are augmented by quarter turns too
        h = 4 * _log(rng, 8, 64)
        w = h if rng.random() < 0.5 else 4 * _log(rng, 8, 64)
        case = dict(kind=kind, batch=rng.randint(1, 8), h=h, w=w, wide=rng.random() < 0.5)
        if kind == "infer":
            case["tta"] = rng.random() < 0.5
        return case
    case = dict(kind=kind, packets=_log(rng, 2_000, 3_000_000), views=rng.randint(1, 8), npix=_log(rng, 24, 256))
    if kind == "mesh":
        case["rx"] = rng.randint(3, 8)
        case["block"] = rng.choice([6, 8, 11, 16])
        case["packets"] = _log(rng, 2_000, 2_000_000)
    else:
        case["n"] = _log(rng, 32, {"table": 128, "slab": 128, "batched": 150}.get(kind, 256))
    if kind == "batched":
        case["n_lambda"] = rng.randint(2, 8)
    if kind in ("sphere", "disk"):
        case["fp64"] = rng.random() < 0.25
        if not case["fp64"]:
            case["packets"] = _log(rng, 2_000, 30_000_000)
    return case


# --------------------------------------------------------------------------
# media (built on the GPU: 256^3 cells per medium)
# --------------------------------------------------------------------------
def _axes(n):
    c = (torch.arange(n, dtype=torch.float64, device="cuda") + 0.5) * (2.0 / n) - 1.0
    return c[None, None, :], c[None, :, None], c[:, None, None]  # x fastest


def _host(t):
    return t.to(torch.float32).reshape(-1).cpu().numpy()


def _disk(n, h0):
    """Density and opacity of ``workloads.flared_disk``."""
    x, y, z = _axes(n)
    r = torch.sqrt(x * x + y * y)
    h = h0 * r * r ** 0.25
    rho = torch.where((r >= 0.05) & (r <= 1.0), torch.exp(-z * z / (2 * h * h)) / r, torch.zeros_like(r * z))
    column = float(rho[n // 2, n // 2, n // 2:].sum()) * 2.0 / n
    return _host(rho), 1e4 / column


def _helical(n):
    """Alignment field of ``workloads.helical_field``."""
    x, y, z = _axes(n)
    r = torch.sqrt(x * x + y * y)
    r = torch.where(r > 0, r, torch.ones_like(r))  # the axis of a grid of odd size
    one = torch.ones_like(z * x * y)
    s = math.sin(30.0 * W.DEG)
    b = torch.stack([-y / r * one, x / r * one, s / math.cos(30.0 * W.DEG) * one])
    b = b / torch.sqrt((b * b).sum(0, keepdim=True))
    return _host(b).reshape(3, -1)


def _slab(n, seed):
    """Density of ``workloads.slab_clump``: log-normal cells smoothed over
    two cells, and one opaque clump."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    g = torch.randn((n, n, n), generator=gen, device="cuda", dtype=torch.float64)
    k = torch.fft.fftfreq(n, device="cuda", dtype=torch.float64) * (2 * math.pi)
    damp = torch.exp(-2.0 * (k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2))
    g = torch.fft.ifftn(torch.fft.fftn(g) * damp).real
    g = (g - g.mean()) / g.std()
    x, y, z = _axes(n)
    tau = 0.02 * torch.exp(g) + 100.0 * torch.exp(-((x - 0.4) ** 2 + y ** 2 + z ** 2) / (2 * 0.05 ** 2))
    tau = tau.clamp(1e-3, 100.0)
    return _host(torch.where(z.abs() <= 0.25, tau * (n / 2.0), torch.zeros_like(tau)))


def _medium(case, rng, seed):
    """A workload record (see ``workloads.py``) of the case's medium."""
    kind, n, packets, npix = case["kind"], case.get("n"), case["packets"], case["npix"]
    star = dict(kind=0, pos=(0.0, 0.0, 0.0), dir=(0.0, 0.0, 1.0), lum=1.0)
    views = [W.view(math.degrees(math.acos(rng.uniform(0.0, 1.0))), rng.uniform(0.0, 360.0), npix)
             for _ in range(case["views"])]
    cfg = dict(bhat=None, source=star, views=views, packets=[packets], opts=W.default_opts(seed), precision="f32")
    if kind == "mesh":
        m = W.mesh_sphere(rx=case["rx"], block=case["block"], packets=packets, tau_radius=rng.uniform(0.5, 2.0))
        return dict(cfg, grid=m["grid"], rho=m["rho"], dust=m["dust"])
    cfg["grid"] = dict(nx=n, ny=n, nz=n, x0=-1.0, y0=-1.0, z0=-1.0, dx=2.0 / n)
    if kind == "sphere":
        x, y, z = _axes(n)
        cfg.update(rho=_host(x * x + y * y + z * z < 1.0), dust=[W.sphere_dust(rng.uniform(0.5, 2.0), 1.0)])
    elif kind == "cylinder":
        x, y, z = _axes(n)
        rho = _host(torch.exp(-(y * y + z * z) / 0.25 ** 2).expand(n, n, n))
        cfg.update(rho=rho, dust=[W.sphere_dust(rng.uniform(0.5, 2.0) / (0.25 * math.sqrt(math.pi)), 0.5)],
                   source=dict(W.THERMAL_SOURCE), emission=np.ones((1, rho.size), np.float32))
    elif kind == "slab":
        a = math.sin(45 * W.DEG)
        bhat = np.repeat(np.array([[a], [0.0], [a]], np.float32), n ** 3, axis=1)
        cfg.update(rho=_slab(n, seed), bhat=bhat, dust=[W.oblate_dust(1.0, 0.5)])
    else:
        rho, kext = _disk(n, rng.uniform(0.05, 0.15))
        cfg["rho"] = rho
        if kind == "disk":
            cfg["dust"] = [W.sphere_dust(kext, 0.5)]
        elif kind == "aligned_disk":
            cfg.update(dust=[W.oblate_dust(kext, 0.5)], bhat=_helical(n))
        elif kind == "table":
            cfg["dust"] = [W.table_dust(kext, 0.5, W.hg_table(rng.uniform(0.3, 0.7), n_theta=181))]
        else:
            nl = case["n_lambda"]
            share = W.batched_lambda_counts(nl)
            cfg.update(dust=[W.oblate_dust(kext * 10.0 ** (-1.5 * k / 31.0), 0.5) for k in range(nl)], bhat=_helical(n),
                       packets=[max(1, packets * s // sum(share)) for s in share])
    if case.get("fp64"):
        cfg["precision"] = "f64"
    return cfg


# --------------------------------------------------------------------------
# denoiser
# --------------------------------------------------------------------------
def _widths(case):
    return (64, 128, 256) if case["wide"] else DN.WIDTHS


def _denoiser_inputs(case, seed):
    b, h, w = case["batch"], case["h"], case["w"]
    params = W.denoiser_params(seed, _widths(case), bias_std=0.05, head_std=0.05)
    low = W.synthetic_stokes_maps([seed, 0], b, h, w, noise=0.3)
    high = W.synthetic_stokes_maps([seed, 0], b, h, w, noise=0.05) if case["kind"] == "grad" else None
    rng = np.random.default_rng([seed, 1])
    aug = rng.integers(0, 8, b) if h == w else 2 * rng.integers(0, 4, b)
    return params, low, high, aug


# --------------------------------------------------------------------------
# preparation, one pass, its least work
# --------------------------------------------------------------------------
def prepare(case, seed):
    if case["kind"] in ("infer", "grad"):
        params, low, high, aug = _denoiser_inputs(case, seed)
        return dict(case=case, dn=DN.Denoiser(0, widths=_widths(case), params=params), low=torch.from_numpy(low).cuda(),
                    high=None if high is None else torch.from_numpy(high).cuda(), aug=aug)
    cfg = _medium(case, np.random.default_rng(seed), seed)
    return dict(case=case, ctx=P.Context(0).load(cfg))


def run(state):
    case = state["case"]
    if case["kind"] == "infer":
        return state["dn"].infer(state["low"], tta=case["tta"])
    if case["kind"] == "grad":
        loss = state["dn"].backward(state["low"], state["high"], state["aug"])
        return loss, state["dn"].grads()
    ctx = state["ctx"]
    ctx.run()
    return ctx.images_device()


def work(case):
    kind = case["kind"]
    if kind in ("infer", "grad"):
        pix = case["batch"] * case["h"] * case["w"]
        c1 = _widths(case)[0]
        per, n = 2.0 * 2.0 * c1, 2 * c1 + 2
        level = {0: 0, 1: 0, 2: 1, 3: 1, 4: 2, 5: 2, 6: 1, 7: 1, 8: 0, 9: 0}
        for k, (ci, co) in enumerate(W.denoiser_layer_io(_widths(case))):
            per += 2.0 * 9.0 * ci * co / 4 ** level[k]
            n += (9 * ci + 1) * co
        if kind == "grad":
            return dict(bytes=8.0 * 8 * pix + 8.0 * n, flops=3.0 * pix * per)
        passes = 1 if not case["tta"] else 8 if case["h"] == case["w"] else 4
        return dict(bytes=8.0 * 8 * pix + 4.0 * n, flops=float(passes) * pix * per)
    # a packet's path crosses about as many cells as one axis has; each cell
    # it crosses costs the geometry of the step, its extinction and its share of the
    # source; the grid is read once, the source written and read once, the images written once
    n = case["rx"] * case["block"] * 2 if kind == "mesh" else case["n"]
    nl = case.get("n_lambda", 1)
    dichroic = kind in ("aligned_disk", "batched", "slab")
    cells = float(n) ** 3 * (0.3 if kind == "mesh" else 1.0)
    source = 9 if dichroic else 4 * case["views"] if kind == "table" else 6
    step = 250.0 if dichroic else 60.0 + 60.0 * case["views"] if kind == "table" else 80.0
    pixels = float(nl * case["views"] * case["npix"] ** 2)
    return dict(bytes=cells * (16.0 if dichroic else 4.0) + 16.0 * source * nl * cells + 32.0 * pixels,
                flops=step * n * case["packets"] + 60.0 * n * pixels)


# --------------------------------------------------------------------------
# 64-bit values of the denoiser's outputs, in plain torch (a Monte Carlo run
# has no such value short of following every packet on the CPU)
# --------------------------------------------------------------------------
def _conv(x, w, b):
    """3x3 convolution + relu, one matrix product per image: x [C][H][W], w [cout][3][3][C]."""
    c, h, wd = x.shape
    cols = torch.nn.functional.unfold(x[None], 3, padding=1)[0]  # [C * 9][H * W], tap fastest
    m = w.permute(0, 3, 1, 2).reshape(w.shape[0], -1)
    return torch.relu(m @ cols + b[:, None]).reshape(-1, h, wd)


def _network(flat, widths, x):
    """The corrections [2][H][W] the U-Net predicts for features x [4][H][W]."""
    at, layers = 0, []
    for ci, co in W.denoiser_layer_io(widths):
        w = flat[at:at + co * 9 * ci].reshape(co, 3, 3, ci)
        at += co * 9 * ci
        layers.append((w, flat[at:at + co]))
        at += co
    hw, hb = flat[at:at + 2 * widths[0]].reshape(2, -1), flat[at + 2 * widths[0]:]
    k, skips = 0, []
    for _ in widths[:-1]:
        x = _conv(_conv(x, *layers[k]), *layers[k + 1])
        k += 2
        skips.append(x)
        x = torch.nn.functional.avg_pool2d(x[None], 2)[0]
    x = _conv(_conv(x, *layers[k]), *layers[k + 1])
    k += 2
    for s in reversed(skips):
        x = torch.cat([x.repeat_interleave(2, 1).repeat_interleave(2, 2), s])
        x = _conv(_conv(x, *layers[k]), *layers[k + 1])
        k += 2
    return torch.einsum("oc,chw->ohw", hw, x) + hb[:, None, None]


def _turn(m, code, back=False):
    """Dihedral element r + 4 f of a Stokes map [4][H][W] (or fractions
    [2][H][W], Q and U): mirrored if f, then r quarter turns, with the signs of
    the turned basis; back undoes it."""
    r, f = int(code) & 3, int(code) >> 2
    sign = [1.0, (-1.0) ** r, (-1.0) ** (r + f), (-1.0) ** f]
    sign = torch.tensor(sign if m.shape[0] == 4 else sign[1:3], dtype=m.dtype, device=m.device)[:, None, None]
    if back:
        m = torch.rot90(m, -r, (1, 2))
        return sign * (m.flip(2) if f else m)
    return sign * torch.rot90(m.flip(2) if f else m, r, (1, 2))


def _fractions(flat, widths, m, s):
    """Predicted (Q/I, U/I) of one map with mean intensity s."""
    frac = (m[1:] / m[:1]).clamp(-1.0, 1.0)
    x = torch.cat([torch.log((m[:1] / s).clamp(min=1e-6)), frac])
    return frac[:2] + _network(flat, widths, x)


def exact(case, seed):
    if case["kind"] not in ("infer", "grad"):
        return None
    params, low, high, aug = _denoiser_inputs(case, seed)
    widths = _widths(case)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    flat = torch.from_numpy(params).to(dev, torch.float64)
    low = torch.from_numpy(low).to(dev)
    if case["kind"] == "infer":
        codes = [0] if not case["tta"] else range(0, 8, 1 if case["h"] == case["w"] else 2)
        out = low.clone()
        with torch.no_grad():
            for b, m in enumerate(low):
                acc = sum(_turn(_fractions(flat, widths, _turn(m, c), m[0].mean()), c, back=True) for c in codes)
                out[b, 1:3] = acc / len(codes) * m[0]
        return out.cpu()
    high = torch.from_numpy(high).to(dev)
    flat.requires_grad_()
    total = 0.0
    for b in range(case["batch"]):
        m, t, s = _turn(low[b], aug[b]), _turn(high[b], aug[b]), low[b, 0].mean()
        e = _fractions(flat, widths, m, s) * (m[0] / s) - t[1:3] / s
        loss = (e * e).sum() / (case["batch"] * ((m[0] / s) ** 2).sum())
        loss.backward()
        total += float(loss)
    return total, flat.grad.cpu().numpy()
