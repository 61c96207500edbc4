"""Pencil beams, whose packets cross the same cells together: a drain adds the
entries of one cell up before they go to the tally.  Counters and images
against the FP64 oracle (images differ by the order of FP64 sums: 1e-10) for
packet counts that leave short and partial drains, spheres and aligned grains, a
mesh, two wavelengths and the allocation-free entry point; and far fewer
blocks added than cells crossed."""
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


def beam(packets, grains="sphere", two=False, mesh=False):
    cfg = odd_box(packets=packets, grains=grains)
    if mesh:
        cfg = W.mesh_sphere(rx=2, block=5, packets=packets, tau_radius=1.0)
        cfg["precision"] = "f64"
    cfg["source"] = dict(kind=1, pos=(0.0, 0.0, -0.2), dir=(0.3, -0.2, 0.933), lum=1.0)
    if two:
        cfg["dust"] = [cfg["dust"][0], dict(cfg["dust"][0], kappa_sca=0.3, kappa_abs=0.2)]
        cfg["packets"] = [packets // 3, packets - packets // 3]
    return cfg


def check(O, cfg, ctx):
    img, st = ctx.images(), ctx.stats()
    ref = [O.run(cfg, lam=l) for l in range(len(cfg["dust"]))]
    for k in ("cell_steps", "scatterings", "escaped", "rr_kills"):
        assert st[k] == sum(r[3][k] for r in ref), k
    for l, r in enumerate(ref):
        d = np.abs(img[l] - r[0]).max() / np.abs(r[0][:, 0]).max()
        say(f"wavelength {l}: image max |d|/I_max = {d:.3e}")
        assert d < 1e-10


@pytest.mark.parametrize("grains", ["sphere", "aligned"])
@pytest.mark.parametrize("packets,opts", [(1, {}), (50, dict(blocks_per_cu=1)), (65, {}), (6000, {}), (40000, {}),
                                          (3000, dict(blocks_per_cu=1, block_size=64))])
def test_beam(O, grains, packets, opts):
    say(f"case: {grains}, {packets} packets, {opts}")
    cfg = beam(packets, grains)
    ctx = gpu_run(cfg, transport_fp64=1, **opts)
    try:
        check(O, cfg, ctx)
    finally:
        ctx.close()


@pytest.mark.parametrize("kw", [dict(two=True), dict(two=True, grains="aligned"), dict(mesh=True)])
def test_wavelengths_and_mesh(O, kw):
    cfg = beam(20000, **kw)
    ctx = gpu_run(cfg, transport_fp64=1)
    try:
        check(O, cfg, ctx)
    finally:
        ctx.close()


def test_static_entry(O):
    import torch

    from paper_2512_01283_amd import polrad as P
    cfg = beam(20000, two=True)
    v = cfg["views"]
    with P.Context(0) as ctx:
        ctx.load(cfg)
        out = torch.zeros((2, len(v), 4, v[0]["npy"], v[0]["npx"]), dtype=torch.float64, device="cuda")
        P.kp_run_static(ctx.h, cfg["packets"], ctx.opts(transport_fp64=1), out)
        img = out.cpu().numpy()
    for l in range(2):
        ref = O.run(cfg, lam=l)[0]
        assert np.abs(img[l] - ref).max() < 1e-10 * np.abs(ref[:, 0]).max()


def test_blocks_added():
    """A column that scatters next to nothing: its cells' entries meet in the
    drains, at least the eight packets that a refill starts together."""
    ctx = gpu_run(W.pencil_column(packets=300000))
    try:
        st = ctx.stats()
        say(f"{st['cell_steps']} cells crossed, {st['tally_flushes']} blocks added")
        assert st["tally_flushes"] < st["cell_steps"] / 4
    finally:
        ctx.close()
