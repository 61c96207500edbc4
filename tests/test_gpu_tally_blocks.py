"""The tally blocks of aligned grains (density and grain frame beside the
coherency sums) where the cell count is no multiple of the 64 slots a wavefront
prepares: a refined mesh of 3^3-cell blocks and a 7 x 5 x 3 grid, two
wavelengths.  FP64, images and counters against the oracle (1e-10, as in
test_gpu_mesh.py)."""
import numpy as np
import pytest

from paper_2512_01283_amd import workloads as W
from parity_util import gpu_run
from test_gpu_tally_layout import odd_box

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def O():
    from oracle import oracle as o
    o.lib()
    return o


@pytest.mark.parametrize("mesh", [True, False])
def test_images(O, mesh):
    rng = np.random.default_rng(3)
    cfg = odd_box(packets=5000, grains="aligned")
    n = (6, 6, 6) if mesh else (7, 5, 3)
    cfg["grid"] = dict(nx=n[0], ny=n[1], nz=n[2], x0=-0.3, y0=-0.25, z0=-0.15, dx=0.1)
    cfg["rho"] = rng.uniform(0.5, 3.0, n[0] * n[1] * n[2]).astype(np.float32)
    b = rng.normal(size=(3, cfg["rho"].size))
    cfg["bhat"] = (b / np.linalg.norm(b, axis=0)).astype(np.float32)
    cfg["dust"] = [W.oblate_dust(1.5, 0.6), W.oblate_dust(0.7, 0.3)]
    cfg["packets"] = [2500, 2500]
    if mesh:
        cfg = W.mesh_of_uniform(cfg, block=3, max_level=1)
        assert len(cfg["rho"]) % 64 != 0
    ctx = gpu_run(cfg, transport_fp64=1)
    try:
        img, st = ctx.images(), ctx.stats()
        ref = [O.run(cfg, lam=l) for l in range(2)]
        assert st["cell_steps"] == sum(r[3]["cell_steps"] for r in ref)
        for l, r in enumerate(ref):
            assert np.abs(img[l] - r[0]).max() < 1e-10 * np.abs(r[0][:, 0]).max()
    finally:
        ctx.close()
