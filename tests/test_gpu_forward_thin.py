"""GPU forward products with up to 32 output columns, on rows and on the windows of a convolution: remainders of 64 contraction entries and of 16
columns, ragged numbers of rows, taps outside the image on every side, strides, an offset, outputs that are no multiple of four wide or lie at any address.

Sums are integers below 2^24 in magnitude, and the steps powers of two: every output is exact."""
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu


def _indices(shape, seed, lo, hi):
    torch = gu.torch_mod()
    return torch.randint(lo, hi, shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed), dtype=torch.int32).to(torch.int8)


@pytest.mark.parametrize("M,N", [(70_001, 16), (40_007, 27), (33_003, 32), (33_025, 4), (90_000, 1), (40_000, 17)])
@pytest.mark.parametrize("K", [16, 17, 48, 63, 64, 65, 144, 192, 255, 1000, 1040])
@pytest.mark.parametrize("offset", [0, 128])
def test_rows(M, N, K, offset):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    a, b = _indices((M, K), M + K, -128, 128), _indices((N, K), N + K, -127, 128)
    y, acc = gu.empty((M, N), torch.float32), gu.empty((M, N), torch.int32)
    y.fill_(7.0)
    ws = gu.workspace(cdl.qgemm_fwd_offset_workspace_bytes(M, N, K))
    cdl.cdl_qgemm_fwd_offset(a, b, M, N, K, 0.25, 0.5, offset, 0, acc, y, ws)
    ref = (a.double() + offset) @ b.double().t()
    assert bool((acc.double() == ref).all()) and bool((y.double() == ref * 0.125).all())


@pytest.mark.parametrize("B,H,W,C,N,R,stride", [(20, 32, 32, 16, 16, 3, 1), (400, 7, 9, 32, 32, 3, 1), (60, 33, 35, 16, 20, 5, 2), (3, 130, 131, 16, 30, 3, 1),
                                                (90, 14, 14, 48, 4, 1, 1), (70, 31, 32, 32, 7, 3, 2), (25, 29, 28, 16, 32, 4, 1), (5, 70, 71, 64, 16, 2, 1)])
@pytest.mark.parametrize("offset", [0, 128])
@pytest.mark.parametrize("shift", [0, 1])
def test_windows(B, H, W, C, N, R, stride, offset, shift):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    pad = R // 2
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    x, w = _indices((B, H, W, C), B + C, -128 if offset else 0, 128), _indices((N, R, R, C), N + C, -127, 128)
    buf = gu.empty((B * P * Q * N + 4,), torch.float32)
    buf.fill_(7.0)
    y, acc = buf[shift:shift + B * P * Q * N].view(B, P, Q, N), gu.empty((B, P, Q, N), torch.int32)
    ws = gu.workspace(cdl.qconv_fwd_workspace_bytes(N, offset))
    cdl.cdl_qconv_fwd(x, w, B, H, W, C, N, R, R, stride, pad, 0.25, 0.5, acc, y, ws, x_offset=offset)
    ref = torch.nn.functional.conv2d((x.cpu().double() + offset).permute(0, 3, 1, 2).contiguous(), w.cpu().double().permute(0, 3, 1, 2).contiguous(),
                                     stride=stride, padding=pad).permute(0, 2, 3, 1)
    assert bool((acc.cpu().double() == ref).all()) and bool((y.cpu().double() == ref * 0.125).all())
    assert bool((buf[:shift] == 7.0).all()) and bool((buf[shift + B * P * Q * N:] == 7.0).all())
