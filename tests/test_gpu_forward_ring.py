"""GPU forward product whose blocks go through tile after tile: contractions of one K-tile to more than the ring holds, one tile a block and
many, ragged rows and columns (whole tiles and cut ones mixed in a block), operands stored with offsets, both outputs, an output beyond the
caches.  Sums are integers: exact; y is one rounded product."""
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu


def _check(M, N, K, want_acc, oa=0, ob=0):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randint(-128, 128, (M, K), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)
    b = torch.randint(-128, 128, (N, K), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)
    y = gu.empty((M, N), torch.float32)
    y.fill_(7e7)
    acc = gu.empty((M, N), torch.int32) if want_acc else None
    ws = gu.workspace(cdl.qgemm_fwd_offset_workspace_bytes(M, N, K))
    for _ in range(2):
        if oa or ob:
            cdl.cdl_qgemm_fwd_offset(a, b, M, N, K, 0.3, 0.07, oa, ob, acc, y, ws)
        else:
            cdl.cdl_qgemm_fwd(a, b, M, N, K, 0.3, 0.07, acc, y, ws)
    torch.cuda.synchronize()
    scale = torch.tensor(0.3, device="cuda") * torch.tensor(0.07, device="cuda")      # (in fp32, as the call forms it)
    bt = (b.double() + ob).t().contiguous()
    for m in range(0, M, 8192):
        want = (a[m:m + 8192].double() + oa) @ bt      # exact: below 2^53
        if want_acc:
            assert torch.equal(acc[m:m + 8192], want.to(torch.int32)), m
        assert torch.equal(y[m:m + 8192], want.to(torch.int32).float() * scale), m


@pytest.mark.parametrize("K", [64, 128, 192, 256, 320, 832])
@pytest.mark.parametrize("M,N", [(9_001, 999), (60_000, 320), (24_064, 1500), (2_049, 2_303)])
def test_tiles_one_after_the_other(M, N, K):
    _check(M, N, K, want_acc=K == 192)


def test_output_beyond_the_caches():
    _check(70_000, 1_024, 256, want_acc=False)


@pytest.mark.parametrize("oa,ob", [(128, 0), (128, 128), (0, 128)])
def test_offsets(oa, ob):
    _check(30_001, 700, 192, want_acc=True, oa=oa, ob=ob)


@pytest.mark.parametrize("B,H,W,C,N,R,S,stride,pad,off", [
    (41, 28, 27, 64, 256, 3, 3, 1, 1, 0), (90, 29, 31, 192, 260, 3, 3, 2, 1, 128), (33, 30, 30, 128, 700, 1, 1, 1, 0, 0), (70, 19, 23, 320, 192, 5, 3, 1, 2, 0),
    (64, 56, 55, 64, 200, 3, 5, 2, 2, 128), (130, 14, 14, 256, 256, 3, 3, 1, 1, 0)])
def test_windows(B, H, W, C, N, R, S, stride, pad, off):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    gen = torch.Generator(device="cuda").manual_seed(H * W + C)
    x = torch.randint(-128, 28, (B, H, W, C), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)
    w = torch.randint(-128, 128, (N, R, S, C), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    y, acc = gu.empty((B, P, Q, N), torch.float32), gu.empty((B, P, Q, N), torch.int32)
    y.fill_(7e7)
    ws = gu.workspace(cdl.qconv_fwd_workspace_bytes(N, off))
    for _ in range(2):
        cdl.cdl_qconv_fwd(x, w, B, H, W, C, N, R, S, stride, pad, 0.3, 0.07, acc, y, ws, x_offset=off)
    torch.cuda.synchronize()
    padded = torch.zeros((B, H + 2 * pad, W + 2 * pad, C), dtype=torch.float64, device="cuda")      # (level index 0 outside the image)
    padded[:, pad:pad + H, pad:pad + W] = x.double() + off
    want = torch.zeros((B * P * Q, N), dtype=torch.float64, device="cuda")
    for r in range(R):
        for s in range(S):
            tap = padded[:, r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride].reshape(-1, C)
            want += tap @ w[:, r, s].double().t().contiguous()
    want = want.to(torch.int32).reshape(B, P, Q, N)
    assert torch.equal(acc, want)
    assert torch.equal(y, want.float() * (torch.tensor(0.3, device="cuda") * torch.tensor(0.07, device="cuda")))
