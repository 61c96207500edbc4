"""Images of shapes that fill no wavefront or tile: single pixels, strips, odd
sides, and small maps whose wavefronts hold pixels of several cameras and
wavelengths.  Step 2 of spheres, aligned grains, a mesh, tabulated grains and a
caller's source, and thermal emission, against the FP64 oracle: images to
1e-10 of their maximum."""
import numpy as np
import pytest

from paper_2512_01283_amd import workloads as W
from parity_util import gpu_run, say
from test_gpu_tally_layout import odd_box

pytestmark = pytest.mark.gpu

# pixels of a map and, where smaller than 0.7 of its wavefronts, shared ones
SHAPES = [(1, 1), (3, 2), (5, 9), (7, 7), (9, 9), (1, 65), (130, 1), (17, 17), (20, 13), (33, 16)]


@pytest.fixture(scope="module")
def O():
    from oracle import oracle as o
    o.lib()
    return o


def case(kind, npx, npy):
    if kind == "mesh":
        cfg = W.mesh_sphere(rx=2, block=5, packets=2000, tau_radius=1.0)
    else:
        cfg = odd_box(packets=2000, grains=kind if kind in ("aligned", "table") else "sphere")
    cfg["views"] = [dict(W.view(t, p, 1, half_width=h), npx=npx, npy=npy)
                    for t, p, h in ((35.0, 70.0, 1.0), (123.0, 211.0, 0.7), (80.0, 10.0, 0.9), (0.0, 0.0, 1.1), (90.0, 0.0, 0.6))]
    if kind == "table":
        cfg["dust"] = [W.table_dust(1.5 - 0.4 * l, 0.8, W.hg_table(0.5, n_theta=181)) for l in range(2)]
    else:
        cfg["dust"] = [cfg["dust"][0], dict(cfg["dust"][0], kappa_abs=cfg["dust"][0]["kappa_abs"] + 0.3)]
    cfg["packets"] = [2000, 1500]
    if kind == "thermal":
        cfg["source"] = dict(W.THERMAL_SOURCE)
        cfg["emission"] = np.ones((2, len(cfg["rho"])), np.float32)
    return cfg


@pytest.mark.parametrize("npx,npy", SHAPES)
@pytest.mark.parametrize("kind", ["sphere", "aligned", "mesh", "table", "thermal"])
def test_run(O, kind, npx, npy):
    cfg = case(kind, npx, npy)
    ctx = gpu_run(cfg, transport_fp64=1)
    try:
        img = ctx.images()
        for l in range(2):
            r = O.run(cfg, lam=l)[0]
            assert np.abs(img[l] - r).max() < 1e-10 * np.abs(r[:, 0]).max(), l
    finally:
        ctx.close()


@pytest.mark.parametrize("npx,npy", SHAPES)
@pytest.mark.parametrize("kind", ["sphere", "aligned"])
def test_callers_source(O, kind, npx, npy):
    import torch
    from paper_2512_01283_amd import polrad as P
    cfg = case(kind, npx, npy)
    rng = np.random.default_rng(npx + 100 * npy)
    S = rng.uniform(-0.3, 0.3, (len(cfg["rho"]), 5, 4))
    S[..., 0] = 1.0
    out = torch.full((5, 4, npy, npx), float("nan"), dtype=torch.float64, device="cuda")
    with P.Context(0) as ctx:
        ctx.load(cfg)
        P.kp_image_source(ctx.h, torch.from_numpy(S).cuda(), out)
    ref = O.image(cfg, S)
    say(f"case: {kind} {npx} x {npy}")
    assert np.abs(out.cpu().numpy() - ref).max() < 1e-10 * ref[:, 0].max()
