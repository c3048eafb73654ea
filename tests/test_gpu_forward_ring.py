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
