"""The cells around a point source, tallied in copies when a run has 2^15
packets or more, against the FP64 oracle: images of a box whose 8^3 cells
around the source lie inside the grid, partly outside it (a source in a
corner) and on periodic axes, for spheres, aligned grains and two wavelengths,
and through the allocation-free entry point.  Every packet follows the
oracle's path (counters), so the images differ by the order of FP64 sums
alone: a cell's ~1e5 additions keep 1e5 2^-53 ~ 1e-11 of its value."""
import numpy as np
import pytest

from paper_2512_01283_amd import workloads as W
from parity_util import gpu_run, say
from test_gpu_tally_layout import odd_box

pytestmark = pytest.mark.gpu

TOL = 1e-10


@pytest.fixture(scope="module")
def O():
    from oracle import oracle as o
    o.lib()
    return o


def case(name, packets):
    aligned = "aligned" in name
    cfg = odd_box(packets=packets, grains="aligned" if aligned else "sphere")
    cfg["rho"] = np.where(cfg["rho"] > 0, cfg["rho"], np.float32(0.3)).astype(np.float32)
    if "corner" in name:
        g = cfg["grid"]
        cfg["source"] = dict(cfg["source"], pos=(g["x0"] + 0.05, g["y0"], g["z0"] + 1.1))
    if "pencil" in name:
        cfg["source"] = dict(kind=1, pos=(0.0, 0.0, -0.2), dir=(0.3, -0.2, 0.933), lum=1.0)
    if "periodic" in name:
        cfg["grid"] = dict(cfg["grid"], boundary=3)
        cfg["source"] = dict(cfg["source"], pos=(-0.88, 0.6, 0.0))
    if "two" in name:
        cfg["dust"] = [cfg["dust"][0], (W.oblate_dust if aligned else W.sphere_dust)(0.8, 0.4)]
        cfg["packets"] = [packets // 3, packets - packets // 3]
    return cfg


@pytest.mark.parametrize("packets", [32767, 32768, 50001])
@pytest.mark.parametrize("name", ["sphere", "aligned"])
def test_around_the_threshold(O, name, packets):
    check(O, name, packets)


@pytest.mark.parametrize("name", ["corner sphere", "corner aligned", "pencil sphere", "periodic sphere", "two sphere",
                                  "two aligned corner"])
def test_boxes_and_wavelengths(O, name):
    check(O, name, 40000)


def check(O, name, packets):
    cfg = case(name, packets)
    say(f"case: {name}, {packets} packets")
    ctx = gpu_run(cfg, transport_fp64=1)
    try:
        img = ctx.images()
        st = ctx.stats()
        ref = [O.run(cfg, lam=l) for l in range(len(cfg["dust"]))]
        for k in ("cell_steps", "scatterings", "escaped", "rr_kills"):
            assert st[k] == sum(r[3][k] for r in ref), k
        for l, r in enumerate(ref):
            d = np.abs(img[l] - r[0]).max() / np.abs(r[0][:, 0]).max()
            say(f"[{name}] wavelength {l}: image max |d|/I_max = {d:.3e}")
            assert d < TOL
    finally:
        ctx.close()


def test_static_entry(O):
    import torch

    from paper_2512_01283_amd import polrad as P
    cfg = case("two aligned", 40000)
    v = cfg["views"]
    with P.Context(0) as ctx:
        ctx.load(cfg)
        out = torch.zeros((2, len(v), 4, v[0]["npy"], v[0]["npx"]), dtype=torch.float64, device="cuda")
        P.kp_run_static(ctx.h, cfg["packets"], ctx.opts(transport_fp64=1), out)
        img = out.cpu().numpy()
    for l in range(2):
        ref = O.run(cfg, lam=l)[0]
        assert np.abs(img[l] - ref).max() < TOL * np.abs(ref[:, 0]).max()
