"""GPU activation gradient of convolutions from patches of g in LDS, on shapes beyond the direct kernels: every tile (32 x 256, 64 x 128,
128 x 64, four classes), patches taken in parts, ragged channels, kernels that are not square, odd sizes with and without padding,
four to six limbs, non-finite entries.

The reference adds up the taps in double on the GPU.  Tolerance: the rounding of g to limbs changes an output by at most 9e-7 (six limbs may
not reach that: then what they leave, 2^-47 of the largest entry times the step and the sum of |w|), rounding to fp32 by 2^-24 of it."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = [(13, 14, 14, 256, 256, 3, 3, 1, 1), (11, 28, 28, 128, 128, 3, 3, 1, 1), (9, 56, 56, 64, 64, 3, 3, 1, 1),
         (13, 7, 7, 512, 512, 3, 3, 1, 1), (2, 24, 60, 256, 512, 3, 3, 1, 1),                     # in parts
         (17, 23, 31, 100, 84, 3, 3, 1, 1), (14, 20, 20, 96, 128, 5, 5, 1, 0), (21, 17, 19, 132, 36, 5, 3, 1, 2),
         (40, 29, 31, 128, 128, 3, 3, 2, 0), (41, 28, 27, 80, 132, 3, 3, 2, 1), (30, 13, 15, 200, 100, 5, 5, 2, 2),
         (60, 28, 28, 256, 256, 1, 1, 2, 0), (300, 5, 3, 256, 128, 3, 3, 1, 1)]


def _call(g, w, geom, step):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    B, H, W, C = geom[:4]
    dx = gu.empty((B, H, W, C), torch.float32)
    dx.fill_(123.0)
    ws = gu.workspace(cdl.qconv_bwd_activations_workspace_bytes(*geom))
    ws.fill_(0x77)
    for _ in range(2):
        cdl.cdl_qconv_bwd_activations(g, w, *geom, step, dx, ws)
    torch.cuda.synchronize()
    return dx


def _reference(g, w, geom, step):
    torch = gu.torch_mod()
    B, H, W, C, N, R, S, stride, pad = geom
    P, Q = g.shape[1], g.shape[2]
    out = torch.zeros((B, H + 2 * pad + R, W + 2 * pad + S, C), dtype=torch.float64, device="cuda")
    g2, w64 = g.double().reshape(-1, N), w.double()
    for r in range(R):
        for s in range(S):
            out[:, r:r + stride * P:stride, s:s + stride * Q:stride] += (g2 @ w64[:, r, s].contiguous()).reshape(B, P, Q, C)
    return step * out[:, pad:pad + H, pad:pad + W]


def _inputs(geom, scale):
    torch = gu.torch_mod()
    B, H, W, C, N, R, S, stride, pad = geom
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H * W + C)
    g = torch.randn((B, P, Q, N), device="cuda", generator=gen) * scale
    # (neighbouring images of very different size: a block's own scale)
    g *= torch.exp2(torch.randint(-6, 7, (B, 1, 1, 1), device="cuda", generator=gen).float())
    return g, torch.randint(-128, 128, (N, R, S, C), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)


@pytest.mark.parametrize("geom", CASES)
@pytest.mark.parametrize("scale", [1.0, 2.0e-6, 30.0, 3.0e4])
def test_activation_gradient(geom, scale):
    torch = gu.torch_mod()
    step = 0.0625
    g, w = _inputs(geom, scale)
    got, ref = _call(g, w, geom, step).double(), _reference(g, w, geom, step)
    six = 2.0 ** -46 * float(g.abs().max()) * step * 128.0 * w.shape[0] * w.shape[1] * w.shape[2]
    off = (got - ref).abs()
    assert bool((off <= max(9e-7, six) + 2.0 ** -23 * ref.abs()).all()), float((off - 2.0 ** -23 * ref.abs()).max())


@pytest.mark.parametrize("geom", [CASES[0], CASES[8]])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_entries_show(geom, value):
    torch = gu.torch_mod()
    g, w = _inputs(geom, 1.0)
    g[3, 5, 6, 7] = value
    got, ref = _call(g, w, geom, 0.0625), _reference(g, w, geom, 0.0625)
    assert bool(torch.isnan(got[~torch.isfinite(ref)]).all())
    rest = [b for b in range(geom[0]) if abs(b - 3) > 1 + 128 // (geom[1] * geom[2])]      # images that share no tile with it
    assert bool(torch.isfinite(got[rest]).all())


# The limb count is that of the whole tensor: one entry per image that sets the scale, meeting zeros in half of the channels, whose other contributions are
# 2^-12 of it; in the first image it is twice as large, and there the bound asks for a limb more.  Tolerance: the bound with that limb, for all images.
@pytest.mark.parametrize("geom", [CASES[0], CASES[3], CASES[9]])
def test_limb_count_of_the_whole_tensor(geom):
    torch = gu.torch_mod()
    step = 0.0625
    g, w = _inputs(geom, 1.0)
    w[5, :, :, ::2] = 0
    sums = float(w.abs().double().sum(dim=(0, 1, 2)).max()) if geom[7] == 1 else max(
        float(w[:, r::2, s::2].abs().double().sum(dim=(0, 1, 2)).max()) for r in range(2) for s in range(2))
    e = int(np.floor(np.log2(9e-7 * 2.0 ** 32 / (step * sums))))      # the largest sigma = 2^e that four limbs serve
    g = torch.randn_like(g) * 2.0 ** (e - 14)
    g[:, 1, 1, 5] = 0.9 * 2.0 ** e
    g[0, 1, 1, 5] *= 2.0
    got, ref = _call(g, w, geom, step).double()[..., ::2], _reference(g, w, geom, step)[..., ::2]
    off = (got - ref).abs()
    assert bool((off <= step * sums * 2.0 ** (e + 1 - 40) + 2.0 ** -23 * ref.abs()).all()), float(off.max())


# a prime number of 32 channels that do not fit together: parts of one k-step a tap, an odd number of steps, the weights at the end of a workspace of
# just the size asked for
@pytest.mark.parametrize("geom", [(1, 11, 11, 1280, 992, 3, 3, 1, 1), (4, 7, 7, 1408, 544, 3, 3, 1, 0), (12, 15, 14, 64, 224, 5, 5, 1, 2), (60, 13, 13, 96, 352, 3, 3, 2, 1)])
@pytest.mark.parametrize("scale", [1.0, 3.0e4])
def test_parts_of_one_step(geom, scale):
    test_activation_gradient(geom, scale)


# few pixels of g, more output channels than a block has words for: a fully connected head as a convolution
@pytest.mark.parametrize("geom", [(1, 7, 7, 512, 2048, 7, 7, 1, 0), (4, 7, 7, 512, 1280, 7, 7, 1, 0), (8, 7, 7, 512, 2048, 7, 7, 1, 0), (16, 7, 7, 512, 1056, 7, 7, 1, 0)])
@pytest.mark.parametrize("scale", [1.0, 3.0e4])
def test_few_pixels_many_channels(geom, scale):
    test_activation_gradient(geom, scale)


# four limbs put together in pairs as integers where the largest column sum of |w| leaves room, on both sides of that line: (N taps) 127 = 64770 and 65024, digits of one sign
@pytest.mark.parametrize("channels,last", [(510, 0), (512, 0), (508, 127)])
@pytest.mark.parametrize("value", [0.98046875, -0.9960784])
def test_limb_pairs(channels, last, value):
    torch = gu.torch_mod()
    geom = (90, 15, 14, 128, 512, 2, 1, 1, 0)
    g, _ = _inputs(geom, 1.0)
    g = torch.where(g.abs() < 1e30, torch.full_like(g, value), g)
    w = torch.zeros((512, 2, 1, 128), dtype=torch.int8, device="cuda")
    w[:channels, 0] = 127
    if last:
        w[channels:channels + 4, 1] = last
    step = 2.0 ** -20      # (four limbs)
    got = _call(g, w, geom, step).double()
    ref = _reference(g, w, geom, step)
    assert bool(((got - ref).abs() <= 1e-12 + 2.0 ** -23 * ref.abs()).all())
