"""The weight gradient over its block shapes: 1, 2 and 3 groups of 16 output
channels, blocks of 64, 32 and 16 input channels (and a 64 with an empty
group), layers taken in two ranges (map below, skip), images smaller than a
tile of 8 x 32 and ones that leave remainders, one chunk and several.  Against
the exact oracle under the bars of dn_util."""
import numpy as np
import pytest

from oracle import denoiser as D
from paper_2512_01283_amd import workloads as W
from dn_util import check_gradients

pytestmark = pytest.mark.gpu

# (widths, shape): channels / 16 of the inputs are 1, 2, 3, 4, 5 (64 + 16), 6 (64 + 32) and 7 (64 + 48)
CASES = [((16, 32), (1, 6, 10)), ((16, 48), (2, 18, 70)), ((32, 64), (1, 34, 30)), ((80, 32), (1, 14, 66)),
         ((112, 64), (1, 10, 40)), ((48, 96), (2, 38, 98)), ((16, 16, 16), (1, 40, 36)), ((32, 96, 64), (1, 36, 68))]


@pytest.mark.parametrize("widths,shape", CASES)
@pytest.mark.parametrize("runs", [1, 2])
def test_gradients(widths, shape, runs):
    import torch
    from paper_2512_01283_amd import denoiser as DN
    b, h, w = shape
    cin = 4 * runs
    params = W.denoiser_params(41, widths=widths, bias_std=0.05, head_std=0.05, cin=cin)
    low = np.concatenate([W.synthetic_stokes_maps(42 + k, b, h, w, noise=0.3) for k in range(runs)], axis=1)
    high = W.synthetic_stokes_maps(42, b, h, w, noise=0.0)
    d = DN.Denoiser(0, widths=widths, params=params, runs=runs)
    d.backward(torch.from_numpy(low).cuda(), torch.from_numpy(high).cuda())
    g = D.unflatten(d.grads().astype(np.float64), widths, cin=cin)
    check_gradients(g, low, high, params, f"widths {widths} {shape} runs {runs}", widths, cin=cin)
    d.close()


def test_repeated_gradients_are_the_same():
    """The weight and bias gradients add up in a fixed order (the head's do not)."""
    import torch
    from paper_2512_01283_amd import denoiser as DN
    widths = (48, 96)
    low = torch.from_numpy(W.synthetic_stokes_maps(43, 3, 70, 90, noise=0.3)).cuda()
    high = torch.from_numpy(W.synthetic_stokes_maps(43, 3, 70, 90, noise=0.0)).cuda()
    d = DN.Denoiser(0, widths=widths, params=W.denoiser_params(44, widths=widths, bias_std=0.05, head_std=0.05))
    runs = []
    for _ in range(3):
        d.backward(low, high)
        g = D.unflatten(d.grads(), widths)
        runs.append([g[k] for k in g if not k.startswith("head")])
    d.close()
    for r in runs[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(runs[0], r))


def test_rows_further_apart_than_a_buffer_offset_reaches():
    """A map so wide that a tile's rows span more than 2^31 bytes, against the
    same periodic map cut into 36 images: equal means, equal weights in the
    loss, and gradients that differ only by the halos of the 70 cuts, about
    1e-4 of the pixels (a wrong address gives differences of order 1)."""
    import torch
    from paper_2512_01283_amd import denoiser as DN
    widths, period, images, wide = (16, 32), 64, 36, 36000
    rng = np.random.default_rng(45)
    base = rng.integers(1, 16, (1, 4, 2, period)).astype(np.float64)
    base[:, 1:] = rng.uniform(-0.3, 0.3, (1, 3, 2, period)) * base[:, :1]
    assert 10 * wide * period * 48 * 2 > 2 ** 31
    t = torch.from_numpy(base).cuda()
    target = t.clone()
    target[:, 1:] *= 0.5
    d = DN.Denoiser(0, widths=widths, params=W.denoiser_params(46, widths=widths, bias_std=0.05, head_std=0.05))

    def grads(n, reps):
        d.backward(t.repeat(n, 1, 1, reps), target.repeat(n, 1, 1, reps))
        return D.unflatten(d.grads().astype(np.float64), widths)

    cut, whole = grads(images, wide // images), grads(1, wide)
    d.close()
    for k in whole:
        e = np.linalg.norm(whole[k] - cut[k]) / np.linalg.norm(cut[k])
        assert e < 5e-3, (k, e)
