"""kp_transport followed by kp_image, as opposed to both in kp_run: step 2 then
takes the grain axes from the alignment planes, which are unit vectors only to
1e-5, instead of from step 1's tally.  Aligned grains on a uniform grid and on a
mesh and two wavelengths, against the FP64 oracle (1e-10) and
against kp_run; and alignment planes that their owner changes in between,
which belong to step 2."""
import numpy as np
import pytest

from paper_2512_01283_amd import workloads as W
from test_gpu_tally_layout import odd_box

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def O():
    from oracle import oracle as o
    o.lib()
    return o


def case(mesh):
    rng = np.random.default_rng(11)
    cfg = odd_box(packets=4000, grains="aligned")
    if mesh:
        cfg["grid"] = dict(nx=6, ny=6, nz=6, x0=-0.3, y0=-0.3, z0=-0.3, dx=0.1)
        cfg["rho"] = rng.uniform(0.5, 3.0, 216).astype(np.float32)
    b = rng.normal(size=(3, len(cfg["rho"])))
    b *= (1.0 + rng.uniform(-8e-6, 8e-6, len(cfg["rho"]))) / np.linalg.norm(b, axis=0)
    cfg["bhat"] = b.astype(np.float32)
    cfg["dust"] = [W.oblate_dust(1.5, 0.6), W.oblate_dust(0.7, 0.3, alpha3_scale=-0.8)]
    cfg["packets"] = [4000, 3000]
    return W.mesh_of_uniform(cfg, block=3, max_level=1) if mesh else cfg


@pytest.mark.parametrize("mesh", [False, True])
def test_against_oracle_and_run(O, mesh):
    from paper_2512_01283_amd import polrad as P
    cfg = case(mesh)
    with P.Context(0) as ctx:
        ctx.load(cfg).run(transport_fp64=1)
        both = ctx.images()
        ctx.transport(transport_fp64=1)
        ctx.image()
        img = ctx.images()
    for l in range(2):
        ref = O.run(cfg, lam=l)[0]
        peak = np.abs(ref[:, 0]).max()
        assert np.abs(img[l] - ref).max() < 1e-10 * peak
        assert np.abs(img[l] - both[l]).max() < 1e-10 * peak


def test_planes_changed_in_between():
    """Step 2 follows the planes as they are when it runs.  In a medium of optical
    depth ~1e-9 the tally does not depend on them, so the image equals that of a
    context whose step 1 ran under the new planes already."""
    import torch

    from paper_2512_01283_amd import polrad as P
    cfg = case(False)
    cfg["dust"] = [W.oblate_dust(1e-9, 0.5), W.oblate_dust(1e-9, 0.5)]
    rho = torch.from_numpy(cfg["rho"]).cuda()
    old = torch.from_numpy(cfg["bhat"].copy()).cuda()
    new = torch.roll(old, 1, 0).contiguous()
    imgs = []
    for first, second in ((old, new), (new, new), (old, old)):
        planes = first.clone()
        with P.Context(0) as ctx:
            ctx.load(cfg)
            P.kp_set_grid_device(ctx.h, cfg["grid"], rho, planes)
            ctx.transport(transport_fp64=1)
            planes.copy_(second)
            torch.cuda.synchronize()
            ctx.image()
            imgs.append(ctx.images())
    peak = np.abs(imgs[1][:, :, 0]).max()
    assert np.abs(imgs[0] - imgs[1]).max() < 1e-7 * peak
    assert np.abs(imgs[0] - imgs[2]).max() > 1e-2 * peak
