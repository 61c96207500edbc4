"""One run whose wavelengths mix spheres and dipole grains (the general
kernels serve both): paths, counters, images and peel-off images of every
wavelength against the FP64 oracle, where a sphere extinguishes every
polarisation and direction alike.  FP64, bars as in test_gpu_tally_layout.py
and test_gpu_boundaries_peel.py."""
import numpy as np
import pytest

from paper_2512_01283_amd import workloads as W
from parity_util import gpu_run, say
from test_gpu_tally_layout import odd_box

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def O():
    from oracle import oracle as o
    o.lib()
    return o


def mixed(grains, order, packets=6000):
    cfg = odd_box(packets=packets, grains=grains)
    ball = dict(W.sphere_dust(1.2, 0.7), a_perp=0.4 + 0.3j, a_par=0.4 + 0.3j, alpha3_scale=0.7)
    oblate = W.oblate_dust(1.5, 0.6, alpha3_scale=-0.8)
    cfg["dust"] = [dict(sphere=ball, oblate=oblate)[k] for k in order]
    cfg["packets"] = [packets + 500 * l for l in range(len(order))]
    return cfg


@pytest.mark.parametrize("grains", ["aligned", "unaligned"])
@pytest.mark.parametrize("order", [("sphere", "oblate"), ("oblate", "sphere", "sphere")])
def test_images_and_counters(O, grains, order):
    cfg = mixed(grains, order)
    say(f"case: {grains}, wavelengths {order}")
    ctx = gpu_run(cfg, transport_fp64=1)
    try:
        img, st = ctx.images(), ctx.stats()
        ref = [O.run(cfg, lam=l) for l in range(len(order))]
        for k in ("cell_steps", "scatterings", "escaped", "rr_kills"):
            assert st[k] == sum(r[3][k] for r in ref), k
        for l, r in enumerate(ref):
            d = np.abs(img[l] - r[0]).max() / np.abs(r[0][:, 0]).max()
            say(f"wavelength {l} ({order[l]}): image max |d|/I_max = {d:.3e}")
            assert d < 1e-10
    finally:
        ctx.close()


def test_thermal_emission(O):
    order = ("sphere", "oblate")
    cfg = mixed("aligned", order)
    cfg["source"] = dict(W.THERMAL_SOURCE)
    cfg["emission"] = np.ones((len(order), len(cfg["rho"])), np.float32)
    ctx = gpu_run(cfg, transport_fp64=1)
    try:
        img = ctx.images()
        for l in range(len(order)):
            r = O.run(cfg, lam=l)[0]
            assert np.abs(img[l] - r).max() < 1e-10 * np.abs(r[:, 0]).max(), order[l]
    finally:
        ctx.close()


def test_peel_off(O):
    order = ("sphere", "oblate")
    cfg = mixed("aligned", order)
    ctx = gpu_run(cfg, transport_fp64=1, peel_off=1)
    try:
        peel = ctx.peel_images()
        for l in range(len(order)):
            r = O.transport_peel(cfg, lam=l)[0]
            assert np.abs(peel[l] - r).max() < 1e-10 * np.abs(r[:, 0]).max(), order[l]
    finally:
        ctx.close()


def test_fp32_paths(O):
    """FP32 polarisation changes a path only where a rejection or roulette
    draw falls within its rounding of the threshold: a few of 6000 packets
    at most."""
    cfg = mixed("aligned", ("sphere", "oblate"))
    cfg["packets"] = [6000, 0]
    ctx = gpu_run(cfg, transport_fp64=2)
    try:
        st, ref = ctx.stats(), O.run(cfg, lam=0)
        for k in ("cell_steps", "escaped"):
            assert abs(st[k] - ref[3][k]) <= 2e-3 * ref[3][k], k
        d = np.abs(ctx.images()[0] - ref[0]).sum() / np.abs(ref[0]).sum()
        assert d < 1e-3, d
    finally:
        ctx.close()
