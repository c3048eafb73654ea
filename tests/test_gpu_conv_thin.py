"""GPU activation gradient of convolutions with few channels, from digits of patches of g and on the other sides of that rule: one and two tiles of
channels, channels and output channels that fill them or not, runs that cross rows and images, wide images, entries spread over so many powers of
two that a patch takes several rounds of digits, infinities next to the image's edge; 1 x 1, stride 2 and more output channels go elsewhere.

Tolerance: sums in double, one rounding to fp32 (2^-24 relative), and 2^-45 of the sum of magnitudes for at most 2^8 terms rounded at 2^-53 (a sum of n)."""
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu

# B, H, W, C, N, R, stride
CASES = [(40, 32, 32, 16, 16, 3, 1), (700, 7, 7, 16, 4, 3, 1), (33, 32, 32, 32, 32, 3, 1), (9, 61, 62, 28, 24, 3, 1), (60, 25, 24, 24, 16, 5, 1), (700, 7, 8, 4, 28, 3, 1), (36, 31, 33, 12, 12, 3, 1), (2, 140, 131, 16, 20, 3, 1), (33, 32, 32, 32, 16, 3, 1),
         (33, 32, 33, 20, 8, 5, 1), (12, 56, 56, 16, 68, 3, 1), (130, 17, 19, 4, 16, 1, 1), (64, 28, 28, 16, 16, 3, 2), (150, 15, 17, 16, 24, 5, 2),
         (129, 16, 16, 32, 36, 3, 2), (40, 30, 31, 8, 4, 1, 2), (33, 32, 32, 16, 88, 3, 1),
         (1400, 7, 8, 4, 28, 3, 1), (80, 30, 31, 28, 28, 3, 1), (150, 30, 31, 12, 8, 3, 1), (140, 31, 33, 16, 20, 3, 1), (70, 31, 33, 8, 24, 3, 1), (70, 31, 33, 20, 12, 3, 1),
         (30, 71, 73, 12, 12, 3, 1), (70, 32, 33, 20, 8, 5, 1), (36, 31, 33, 20, 12, 5, 1)]


def _reference(G, w, H, W, C, R, stride):
    torch = gu.torch_mod()
    g = G.cpu().double().permute(0, 3, 1, 2).contiguous()
    x = torch.zeros((G.shape[0], C, H, W), dtype=torch.float64, requires_grad=True)
    y = torch.nn.functional.conv2d(x, w.cpu().double().permute(0, 3, 1, 2).contiguous(), stride=stride, padding=R // 2)
    return torch.autograd.grad(y, x, g)[0].permute(0, 2, 3, 1)


@pytest.mark.parametrize("case", CASES, ids=str)
@pytest.mark.parametrize("inf", [False, True])
def test_activation_gradient(case, inf):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    B, H, W, C, N, R, stride = case
    pad = R // 2
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    gen = torch.Generator(device="cuda").manual_seed(B + C + N)
    G = torch.randn((B, P, Q, N), device="cuda", generator=gen) * torch.exp2(8 * torch.randn((B, P, Q, 1), device="cuda", generator=gen))
    if inf:
        G[0, 0, Q - 1, 0], G[B - 1, P - 1, 0, N - 1], G[B // 2, P // 2, Q // 2, 1] = float("inf"), -float("inf"), float("nan")
    w = torch.randint(-127, 128, (N, R, R, C), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)
    geom = (B, H, W, C, N, R, R, stride, pad)
    got = gu.empty((B, H, W, C), torch.float32)
    got.fill_(5.0)
    ws = gu.workspace(cdl.qconv_bwd_activations_workspace_bytes(*geom))
    cdl.cdl_qconv_bwd_activations(G, w, *geom, 0.125, got, ws)
    ref = _reference(G, w, H, W, C, R, stride) * 0.125
    size = _reference(G.abs(), w.abs(), H, W, C, R, stride) * 0.125
    got = got.cpu().double()
    finite = torch.isfinite(ref)
    assert bool((torch.isfinite(got) == finite).all()) and (not inf or not bool(finite.all()))
    off = (got - ref).abs()[finite]
    assert bool((off <= 2.0 ** -24 * ref.abs()[finite] * 1.01 + 2.0 ** -45 * size[finite]).all()), float(off.max())
