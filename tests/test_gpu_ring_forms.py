"""GPU forward products in every form of tile with direct loads: 256 x 256, 256 x 128, 256 x 64, 128 x 128, 128 x 64 outputs, of matrices, of windows whose taps are whole K-tiles and of
windows whose taps are not (a K-tile across taps, contractions that end inside one); rows and columns that end inside a tile, images smaller than a tile, several tiles to a block, operands
stored with an offset, accumulators beside the outputs.  Every accumulator is compared with a product in double on the host's side of the GPU (whole numbers: exactly)."""
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu

MATRICES = [(3700, 1990, 1280), (8324, 1300, 1536), (100_003, 100, 1152), (60_001, 128, 640), (8324, 192, 1536), (18_304, 189, 256), (5469, 768, 448), (1146, 1341, 1280), (982, 1408, 640),
            (4033, 320, 1024), (100_352, 61, 576), (65_537, 250, 320)]


@pytest.mark.parametrize("M,N,K", MATRICES)
@pytest.mark.parametrize("offsets", [(0, 0), (128, 128)])
def test_matrix(M, N, K, offsets):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N)
    a = torch.randint(-128, 128, (M, K), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)
    b = torch.randint(-128, 128, (N, K), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)
    ws = gu.workspace(cdl.qgemm_fwd_offset_workspace_bytes(M, N, K))
    y, acc = gu.empty((M, N), torch.float32), gu.empty((M, N), torch.int32)
    ref = ((a.double() + offsets[0]) @ (b.double() + offsets[1]).t().contiguous()).to(torch.int64)
    want = (ref.float() * 0.125)
    for out in (None, acc):
        y.fill_(float("nan"))
        cdl.cdl_qgemm_fwd_offset(a, b, M, N, K, 0.25, 0.5, *offsets, out, y, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, want)
    assert torch.equal(acc.long(), ref)


# B, H, W, C, N, R, S, stride, pad
LAYERS = [(60, 56, 56, 64, 64, 3, 3, 1, 1), (41, 51, 49, 128, 20, 3, 3, 1, 1), (128, 28, 28, 128, 128, 3, 3, 1, 1), (64, 28, 28, 128, 250, 3, 3, 2, 1), (80, 14, 14, 256, 256, 3, 3, 1, 1),
          (185, 29, 18, 48, 148, 3, 3, 1, 1), (30, 55, 55, 48, 468, 3, 3, 1, 1), (229, 26, 26, 32, 84, 5, 5, 1, 2), (138, 25, 25, 448, 52, 3, 3, 2, 1), (30, 19, 53, 288, 412, 3, 3, 1, 1),
          (82, 34, 18, 16, 420, 3, 3, 1, 1), (175, 30, 30, 144, 132, 1, 1, 1, 0), (21, 51, 51, 96, 328, 1, 1, 1, 0), (60, 40, 40, 112, 416, 1, 1, 1, 0), (72, 24, 24, 64, 160, 3, 3, 1, 1),
          (3000, 3, 5, 80, 136, 3, 2, 1, 1), (90, 31, 29, 16, 132, 4, 5, 2, 3), (1, 300, 301, 48, 200, 3, 3, 1, 1), (200, 40, 40, 32, 128, 1, 1, 1, 0), (128, 7, 7, 512, 512, 3, 3, 1, 1)]


@pytest.mark.parametrize("geom", LAYERS)
@pytest.mark.parametrize("offset", [0, 128])
def test_windows(geom, offset):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    B, H, W, C, N, R, S, stride, pad = geom
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(C + N)
    x = torch.randint(-128, 128, (B, H, W, C), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)
    w = torch.randint(-127, 128, (N, R, S, C), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)
    xp = torch.zeros((B, H + 2 * pad + stride, W + 2 * pad + stride, C), dtype=torch.float64, device="cuda")
    xp[:, pad:pad + H, pad:pad + W] = x.double() + offset
    ref = torch.zeros((B * P * Q, N), dtype=torch.float64, device="cuda")
    for r in range(R):
        for s in range(S):
            ref += xp[:, r:r + stride * P:stride, s:s + stride * Q:stride][:, :P, :Q].reshape(-1, C) @ w[:, r, s].double().t().contiguous()
    ref = ref.to(torch.int64)
    want = ref.float() * 0.125
    ws = gu.workspace(cdl.qconv_fwd_workspace_bytes(N, offset))
    y, acc = gu.empty((B * P * Q, N), torch.float32), gu.empty((B * P * Q, N), torch.int32)
    for out in (None, acc):
        y.fill_(float("nan"))
        cdl.cdl_qconv_fwd(x, w, *geom, 0.25, 0.5, out, y, ws, x_offset=offset)
        torch.cuda.synchronize()
        assert torch.equal(y, want)
    assert torch.equal(acc.long(), ref)
