"""GPU forward products in every form of tile with direct loads, with stores that stay in the caches and that go past them, over contractions of fewer K-tiles than a ring holds (the stores of several tiles and the
loads of the next ones under way together), rows and columns that end inside a tile, few rows, operands stored with an offset (ring_cases.py: which form each takes is checked without a GPU).  Sums are integers:
exact; y is one rounded product."""
import pytest

import gpu_util as gu
from ring_cases import LAYERS, MATRICES

pytestmark = pytest.mark.gpu


def _compare(acc, y, want, rows, first):
    torch = gu.torch_mod()
    scale = torch.tensor(0.3, device="cuda") * torch.tensor(0.07, device="cuda")      # (in fp32, as the call forms it)
    part = want.to(torch.int32)
    if acc is not None:
        assert torch.equal(acc[first:first + rows], part), first
    assert torch.equal(y[first:first + rows], part.float() * scale), first


@pytest.mark.parametrize("shape,form,stream", MATRICES, ids=str)
@pytest.mark.parametrize("offsets", [(0, 0), (128, 128)])
def test_matrix(shape, form, stream, offsets):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    M, N, K = shape
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randint(-128, 128, (M, K), device="cuda", generator=gen, dtype=torch.int8)
    b = torch.randint(-128, 128, (N, K), device="cuda", generator=gen, dtype=torch.int8)
    y = torch.full((M, N), 7e7, device="cuda")
    acc = None if stream else gu.empty((M, N), torch.int32)      # (accumulators as well: no stores past the caches)
    ws = gu.workspace(cdl.qgemm_fwd_offset_workspace_bytes(M, N, K))
    for _ in range(2):
        cdl.cdl_qgemm_fwd_offset(a, b, M, N, K, 0.3, 0.07, *offsets, acc, y, ws)
    torch.cuda.synchronize()
    bt = (b.double() + offsets[1]).t().contiguous()
    for m in range(0, M, 8192):
        rows = min(8192, M - m)
        _compare(acc, y, (a[m:m + rows].double() + offsets[0]) @ bt, rows, m)


@pytest.mark.parametrize("geom,form,stream", LAYERS, ids=str)
@pytest.mark.parametrize("offset", [0, 128])
def test_windows(geom, form, stream, offset):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    B, H, W, C, N, R, S, stride, pad = geom
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    gen = torch.Generator(device="cuda").manual_seed(H * W + C)
    x = torch.randint(-128, 128, (B, H, W, C), device="cuda", generator=gen, dtype=torch.int8)
    w = torch.randint(-127, 128, (N, R, S, C), device="cuda", generator=gen, dtype=torch.int8)
    y = torch.full((B * P * Q, N), 7e7, device="cuda")
    acc = None if stream else gu.empty((B * P * Q, N), torch.int32)
    ws = gu.workspace(cdl.qconv_fwd_workspace_bytes(N, offset))
    for _ in range(2):
        cdl.cdl_qconv_fwd(x, w, *geom, 0.3, 0.07, acc, y, ws, x_offset=offset)
    torch.cuda.synchronize()
    some = max(1, 40_000 // (P * Q))      # images at a time
    for b0 in range(0, B, some):
        images = x[b0:b0 + some]
        padded = torch.zeros((images.shape[0], H + 2 * pad, W + 2 * pad, C), dtype=torch.float64, device="cuda")      # (level index 0 outside the image)
        padded[:, pad:pad + H, pad:pad + W] = images.double() + offset
        want = torch.zeros((images.shape[0] * P * Q, N), dtype=torch.float64, device="cuda")
        for r in range(R):
            for s in range(S):
                tap = padded[:, r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride].reshape(-1, C)
                want += tap @ w[:, r, s].double().t().contiguous()
        _compare(acc, y, want, want.shape[0], b0 * P * Q)
