"""Tabulated grains at the edges of where their tables are read from: a
block's LDS (up to 459 nodes for one wavelength and three cameras, 247 for two)
or memory, the smallest table, and runs of 2^15 packets and more, whose
cells around the source are tallied in copies; uniform grid and composite
mesh.  FP64, against the oracle: counters equal, images within the 1e-10 of
test_gpu_tables.py."""
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


@pytest.mark.parametrize("n_theta,n_lambda,packets,mesh",
                         [(2, 1, 6000, False), (3, 1, 6000, False), (459, 1, 6000, False), (460, 1, 6000, False),
                          (247, 2, 6001, False), (248, 2, 6001, False), (181, 1, 32768, False), (181, 2, 40000, False),
                          (600, 2, 40000, False), (181, 1, 6000, True), (181, 2, 6001, True), (600, 1, 6000, True)])
def test_images(O, n_theta, n_lambda, packets, mesh):
    cfg = odd_box(packets=packets, grains="table")
    if mesh:
        cfg = W.mesh_of_uniform(W.table_sphere(n=8, packets=packets), block=4, max_level=2)
    cfg["dust"] = [W.table_dust(1.5 - 0.4 * l, 0.8, W.hg_table(0.5 + 0.2 * l, n_theta=n_theta))
                   for l in range(n_lambda)]
    cfg["packets"] = [packets] if n_lambda == 1 else [packets // 3, packets - packets // 3]
    say(f"case: {n_theta} nodes, {n_lambda} wavelengths, {packets} packets, mesh {mesh}")
    ctx = gpu_run(cfg, transport_fp64=1)
    try:
        img = ctx.images()
        st = ctx.stats()
        ref = [O.run(cfg, lam=l) for l in range(n_lambda)]
        for k in ("cell_steps", "scatterings", "escaped"):
            assert st[k] == sum(r[3][k] for r in ref), k
        for l, r in enumerate(ref):
            d = np.abs(img[l] - r[0]).max() / np.abs(r[0][:, 0]).max()
            say(f"wavelength {l}: image max |d|/I_max = {d:.3e}")
            assert d < 1e-10
    finally:
        ctx.close()
