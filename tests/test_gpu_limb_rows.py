"""GPU activation gradient of linear layers over contractions of up to 384 entries: every number of k-steps, row tiles of 64 and 32, ragged
rows, columns and contractions, columns of less than one pass and of many, outputs beyond the caches, a stored offset, three to six limbs.

Tolerance: the rounding of g to limbs changes an output by at most 9e-7 (six limbs may not reach that: then what they leave, 2^-47 of
the largest entry times the step and the sum of |w|), rounding to fp32 by 2^-24 of it."""
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = [(12_000, 64, 577), (40_001, 36, 300), (9_001, 128, 1000), (5_003, 192, 900), (7_001, 100, 1100), (4_001, 256, 2304), (3_001, 320, 1500),
         (3_001, 384, 1501), (20_003, 384, 65), (40_000, 260, 128), (1_031, 300, 3001), (50_200, 48, 1344)]


def _inputs(M, N, K, scale):
    torch = gu.torch_mod()
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    G = torch.randn((M, N), device="cuda", generator=gen) * scale
    return G, torch.randint(-128, 128, (N, K), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)


def _check(got, G, b, step, offset=0):
    torch = gu.torch_mod()
    six = 2.0 ** -46 * float(G.abs().max()) * step * 128.0 * b.shape[0]
    for m in range(0, G.shape[0], 8192):      # (in parts: a product of doubles)
        ref = step * (G[m:m + 8192].double() @ (b.double() + offset))
        off = (got[m:m + 8192].double() - ref).abs()
        assert bool((off <= max(9e-7, six) + 2.0 ** -23 * ref.abs()).all()), (m, float((off - 2.0 ** -23 * ref.abs()).max()))


@pytest.mark.parametrize("M,N,K", CASES)
@pytest.mark.parametrize("scale", [2.0e-5, 1.0, 3.0e4, 1.0e7])
def test_activation_gradient(M, N, K, scale):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    G, b = _inputs(M, N, K, scale)
    da = gu.empty((M, K), torch.float32)
    da.fill_(123.0)
    ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    ws.fill_(0x77)
    for _ in range(2):
        cdl.cdl_qgemm_bwd(G, None, b, M, N, K, 1.0, 0.0625, da, None, ws)
    torch.cuda.synchronize()
    _check(da, G, b, 0.0625)


@pytest.mark.parametrize("M,N,K", [CASES[2], CASES[5], CASES[7]])
def test_stored_with_an_offset(M, N, K):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    G, b = _inputs(M, N, K, 1.0)
    a = torch.randint(0, 16, (M, K), device="cuda").to(torch.int8)
    da, db = gu.empty((M, K), torch.float32), gu.empty((N, K), torch.float32)
    ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    cdl.cdl_qgemm_bwd_offset(G, a, b, M, N, K, 0.125, 0.0625, 0, 128, da, db, ws)
    torch.cuda.synchronize()
    _check(da, G, b, 0.0625, 128)
    _check(db, G.t().contiguous(), a, 0.125)
