"""The tiled convolution over its tile shapes, at sizes that leave remainders.

A launch takes the tile (32, 16 or 8 rows, 1 to 4 channel groups of 16) with
the least estimated time; `tile` repeats the rule, and the networks below
reach each shape forward and for input gradients, with image sides that no
tile divides, channel counts that fill no block of 32, pooling and in-place
upsampling.  Forward and gradients are compared with the exact oracle and its
BF16 replay under the bars of dn_util.
"""
import math

import numpy as np
import pytest

from oracle import denoiser as D
from paper_2512_01283_amd import workloads as W
from dn_util import bf16_replay, check_forward, check_gradients, fractions, oracle_pass

CUS = 256


def tile(b, h, w, cin, cout):
    best, pick = 1e30, None
    for r in (32, 16, 8):
        for n in (4, 3, 2, 1):
            if cout // 16 % n:
                continue
            items = b * -(-h // r) * -(-w // 16) * (cout // 16 // n)
            res = 160 * 1024 // (2048 * (((r + 2) * 18 + 15) // 16 + 9 * n) + 2048)
            t = -(-cin // 32) * (0.45 * math.ceil(items / (CUS * res)) + math.ceil(items / CUS) * r * (0.004 + 0.0165 * n))
            if t < best:
                best, pick = t, (r, n)
    return pick


def tiles(widths, b, h, w):
    """(forward tiles, input-gradient tiles) of a network's convolutions of at least 1024 pixels."""
    fwd, bwd = set(), set()
    n = len(widths)
    levels = [l for l in range(n - 1) for _ in "ab"] + [n - 1] * 2 + [l for l in reversed(range(n - 1)) for _ in "ab"]
    for k, (l, (ci, co)) in enumerate(zip(levels, W.denoiser_layer_io(widths))):
        if (b * h * w) >> (2 * l) < 1024:
            continue
        fwd.add(tile(b, h >> l, w >> l, -(-ci // 8) * 8, co))
        if k:
            bwd.add(tile(b, h >> l, w >> l, co, ci))
    return fwd, bwd


NETS = [((16, 48), (3, 36, 44)), ((16, 32), (4, 202, 318)), ((32, 64), (3, 150, 134)), ((32, 64), (5, 166, 202)),
        ((48, 96), (2, 70, 90)), ((48, 48), (3, 86, 118)), ((48, 96), (3, 98, 130)), ((48, 48), (6, 86, 118)),
        ((48, 96), (5, 170, 170)),
        ((64, 64), (1, 46, 62)), ((64, 128), (2, 134, 102)), ((64, 128), (2, 194, 226))]


def test_networks_reach_every_tile():
    fwd, bwd = (set().union(*(tiles(w, *s)[k] for w, s in NETS)) for k in (0, 1))
    every = {(r, n) for r in (32, 16, 8) for n in (1, 2, 3, 4)}
    print("forward lacks", sorted(every - fwd), "gradients lack", sorted(every - bwd))
    assert fwd == every


@pytest.mark.gpu
@pytest.mark.parametrize("widths,shape", NETS)
def test_forward_and_gradients(widths, shape):
    import torch
    from paper_2512_01283_amd import denoiser as DN
    b, h, w = shape
    params = W.denoiser_params(31, widths=widths, bias_std=0.05, head_std=0.05)
    low = W.synthetic_stokes_maps(32, b, h, w, noise=0.3)
    high = W.synthetic_stokes_maps(32, b, h, w, noise=0.0)
    d = DN.Denoiser(0, widths=widths, params=params)
    out = d.infer(torch.from_numpy(low).cuda()).cpu().numpy()
    ref = oracle_pass(params, low, None, widths)
    rep = bf16_replay(params, low, None, widths)
    check_forward(np.moveaxis(out[:, 1:3] / out[:, :1], 1, -1) - fractions(low), ref["delta"], rep["delta"],
                  f"widths {widths} {shape}")
    if b * h * w < 20000:  # the oracle's gradient of the larger ones takes minutes
        d.backward(torch.from_numpy(low).cuda(), torch.from_numpy(high).cuda())
        g = D.unflatten(d.grads().astype(np.float64), widths)
        check_gradients(g, low, high, params, f"widths {widths} {shape}", widths)
    d.close()


@pytest.mark.gpu
def test_gradients_of_small_and_large_tiles_agree():
    """The gradient of a batch is the mean of its halves' (the loss is a mean
    over images): the two sizes take different tiles, so this ties the input
    gradients of the tall tiles to those the oracle checks above.  FP32 sums in
    different orders over up to 1e5 products: 1e-4 of a tensor's norm."""
    import torch
    from paper_2512_01283_amd import denoiser as DN
    for widths, (b, h, w) in [((48, 96), (4, 166, 170)), ((64, 128), (4, 162, 178)), ((16, 32), (4, 202, 318))]:
        assert tiles(widths, b, h, w)[1] != tiles(widths, 1, h, w)[1]
        params = W.denoiser_params(33, widths=widths, bias_std=0.05, head_std=0.05)
        low = W.synthetic_stokes_maps(34, b, h, w, noise=0.3)
        high = W.synthetic_stokes_maps(34, b, h, w, noise=0.05)
        d = DN.Denoiser(0, widths=widths, params=params)

        def grads(lo, hi):
            d.backward(torch.from_numpy(np.ascontiguousarray(lo)).cuda(), torch.from_numpy(np.ascontiguousarray(hi)).cuda())
            return d.grads().astype(np.float64)

        whole = D.unflatten(grads(low, high), widths)
        parts = D.unflatten(sum(grads(low[k:k + 1], high[k:k + 1]) for k in range(b)) / b, widths)
        d.close()
        for k in whole:
            e = np.linalg.norm(whole[k] - parts[k]) / np.linalg.norm(parts[k])
            assert e < 1e-4, (widths, k, e)


@pytest.mark.gpu
def test_rows_further_apart_than_a_buffer_offset_reaches():
    """A map so wide that a tile's rows span more than 2^31 bytes: periodic
    input whose mean is exact, so far from the ends every period must repeat
    the narrow map's values bit for bit."""
    import torch
    from paper_2512_01283_amd import denoiser as DN
    widths, period, narrow, wide = (16, 32), 64, 32, 36000
    rng = np.random.default_rng(35)
    base = rng.integers(1, 16, (1, 4, 2, period)).astype(np.float64)
    base[:, 1:] = rng.uniform(-0.3, 0.3, (1, 3, 2, period)) * base[:, :1]
    assert 10 * wide * period * 48 * 2 > 2 ** 31
    d = DN.Denoiser(0, widths=widths, params=W.denoiser_params(36, widths=widths, bias_std=0.05, head_std=0.05))
    t = torch.from_numpy(base).cuda()
    a = d.infer(t.repeat(1, 1, 1, narrow))[..., 8 * period:9 * period].clone()
    out = d.infer(t.repeat(1, 1, 1, wide))
    assert not torch.equal(a[:, 1:3], t[:, 1:3])
    mid = out[..., 8 * period:(wide - 8) * period].reshape(1, 4, 2, wide - 16, period)
    assert torch.equal(mid, a[:, :, :, None].expand_as(mid))
    d.close()
