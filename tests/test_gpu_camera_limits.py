"""Camera directions with a component so small that its reciprocal overflows
(a subnormal number), rays starting on the box's faces included: images of a
caller's source against the FP64 oracle, which divides by the component."""
import math

import numpy as np
import pytest

from paper_2512_01283_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("theta", [1e-300, 1e-310, 5e-324])
@pytest.mark.parametrize("phi", [0.0, 90.0, 180.0, 270.0])
def test_subnormal_direction_component(theta, phi):
    import torch

    from oracle import oracle as O
    from paper_2512_01283_amd import polrad as P
    n, npix = 8, 5
    cfg = W.uniform_sphere(n=n, packets=10)
    cfg["rho"] = np.ones(n ** 3, np.float32)
    # pixel centres at -1, -1/2, 0, 1/2, 1: the outermost lie on the box's faces
    cfg["views"] = [dict(W.view(0.0, 0.0, npix, half_width=1.25), theta=theta, phi=math.radians(phi))]
    S = np.zeros((n ** 3, 1, 4))
    S[..., 0] = 1.0
    S[..., 1] = 0.25
    out = torch.zeros((1, 4, npix, npix), dtype=torch.float64, device="cuda")
    with P.Context(0) as ctx:
        ctx.load(cfg)
        P.kp_image_source(ctx.h, torch.from_numpy(S).cuda(), out)
    ref = O.image(cfg, S)
    assert ref[0, 0].max() > 0.5
    assert np.abs(out.cpu().numpy() - ref).max() < 1e-12
