"""GPU activation gradient of short contractions asked for alone and together with the weight gradient, where the two calls take different kernels and where they take the same: both are sums in double (or of exact
digits) rounded once, so that an output differs by the last bit of fp32 at most, where a sum lies next to the middle of two floats."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,same", [(50_000, 16, 64, False), (16_384, 16, 144, False), (2048, 16, 1500, False), (32_768, 32, 36, False), (100_000, 32, 40, True), (65_536, 17, 60, False), (65_537, 48, 64, False), (65_537, 48, 32, True),
                                        (131_072, 16, 27, True), (131_072, 16, 144, True), (20_000, 16, 40, True), (65_536, 64, 33, True)])
def test_alone_and_together(M, N, K, same):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    g = torch.randn(M, N, device="cuda", generator=gen)
    a = torch.randint(0, 16, (M, K), dtype=torch.int8, device="cuda", generator=gen)
    b = torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda", generator=gen)
    alone, both, db = torch.empty(M, K, device="cuda"), torch.empty(M, K, device="cuda"), torch.empty(N, K, device="cuda")
    ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    cdl.cdl_qgemm_bwd(g, a, b, M, N, K, 0.5, 0.3, alone, None, ws)
    cdl.cdl_qgemm_bwd(g, a, b, M, N, K, 0.5, 0.3, both, db, ws)
    torch.cuda.synchronize()
    if same:
        assert torch.equal(alone, both)
        return
    off = (alone.double() - both.double()).abs()
    ulp = torch.exp2(torch.floor(torch.log2(both.double().abs().clamp_min(2.0 ** -126))) - 23)
    assert bool((off <= ulp).all())
    # two sums in double, each off by (N + 2) 2^-53 of the sum of magnitudes (about 4 sqrt N outputs), on either side of a middle: 2 (N + 2) 4 sqrt(N) 2^-53 / 2^-24 of the outputs of a typical size, and
    # as many times more where an output has cancelled: below one in 10^5 with room to spare
    assert int((off != 0).sum()) <= max(1, M * K // 100_000)
