"""Activation gradient of short contractions (at most 32 entries, 64 in long layers): every way in which the outputs are stored, contractions and columns that do and do not fill their tiles, one and several
groups of columns, rows that do not fill a tile, both sides of the line on the number of outputs."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu

# (M, N, K, offset of the outputs in entries): 2^21 outputs or more of one product alone; 2^24 through LDS for rows of any length, 65 M for whole words
CASES = [
    (131072, 16, 16), (131072, 16, 15), (131072, 1, 17), (65537, 3, 32), (20_001, 16, 144), (20_001, 13, 160), (20_001, 16, 164), (20_001, 16, 163), (13_000, 5, 333), (20_001, 12, 144),
    (65_536, 32, 64), (65_535, 17, 68), (60_000, 32, 63), (60_000, 31, 65), (300, 32, 8000), (17, 16, 250_000), (150, 20, 20_003),
    (600_000, 16, 28), (600_001, 16, 29), (600_001, 32, 29), (160_003, 9, 105), (270_001, 32, 63), (160_003, 16, 161), (460_001, 16, 144), (250_001, 30, 264), (2_200_001, 8, 32),
    (32767, 16, 64), (32768, 16, 64), (32768, 32, 32), (32767, 32, 33), (116_509, 3, 9),
    (65536, 33, 32), (65535, 33, 32), (65537, 48, 64), (65537, 48, 65), (65539, 47, 63), (65537, 49, 31), (65536, 64, 32), (65536, 64, 33), (70_003, 64, 1), (131_075, 61, 27), (2_100_001, 64, 31),
]


@pytest.mark.parametrize("M,N,K", CASES)
def test_da_direct(M, N, K):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    g = torch.randn(M, N, device="cuda", generator=gen) * 10.0 ** torch.randint(-6, 7, (M, N), device="cuda", generator=gen)
    b = torch.randint(-128, 128, (N, K), dtype=torch.int8, device="cuda", generator=gen)
    a = torch.empty(M * K, dtype=torch.int8, device="cuda")
    delta = 0.0625
    for off in (0, 128):
        guard = torch.full((M * K + 8,), 7.0, device="cuda")
        da = guard[4:4 + M * K].view(M, K)
        ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
        cdl.cdl_qgemm_bwd_offset(g, a, b, M, N, K, delta, delta, 0, off, da, None, ws)
        torch.cuda.synchronize()
        assert bool((guard[:4] == 7.0).all()) and bool((guard[4 + M * K:] == 7.0).all())
        bd = b.double() + off
        step = max(1, (1 << 24) // K)
        for r in range(0, M, step):
            rows = g[r:r + step].double()
            ref = delta * (rows @ bd)
            # one rounding to fp32 (2^-24 of the result) and N + 1 in double of the sum of magnitudes (both sums)
            bound = 2.0 ** -23 * ref.abs() + (N + 2) * 2.0 ** -51 * delta * (rows.abs() @ bd.abs()) + 2.0 ** -140
            assert bool(((da[r:r + step].double() - ref).abs() <= bound).all()), (off, r)


def test_infinities():
    """An entry that is not finite reaches its own row and no other."""
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    M, N, K = 32_771, 16, 144
    g = torch.ones(M, N, device="cuda")
    g[5, 3], g[M - 1, 15] = float("inf"), float("nan")
    b = torch.ones(N, K, dtype=torch.int8, device="cuda")
    da = torch.zeros(M, K, device="cuda")
    cdl.cdl_qgemm_bwd(g, torch.empty(M * K, dtype=torch.int8, device="cuda"), b, M, N, K, 1.0, 1.0, da, None, gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K)))
    bad = torch.zeros(M, dtype=torch.bool, device="cuda")
    bad[5] = bad[M - 1] = True
    assert bool(torch.isinf(da[5]).all()) and bool(torch.isnan(da[M - 1]).all()) and bool((da[~bad] == N).all())


@pytest.mark.parametrize("M,N,K", [(65536, 16, 16), (65535, 16, 17), (65536, 17, 40), (65536, 17, 41), (70_001, 5, 63), (131072, 32, 9), (131072, 3, 27), (65536, 33, 32), (65536, 48, 33), (65541, 64, 27)])
def test_both(M, N, K):
    """Both products of one call, on both sides of the lines on rows, contraction and columns."""
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    g = torch.randn(M, N, device="cuda", generator=gen)
    a = torch.randint(0, 16, (M, K), dtype=torch.int8, device="cuda", generator=gen)
    b = torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda", generator=gen)
    da, db = torch.empty(M, K, device="cuda"), torch.empty(N, K, device="cuda")
    cdl.cdl_qgemm_bwd(g, a, b, M, N, K, 0.5, 0.25, da, db, gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K)))
    G, A, B = g.double(), a.double(), b.double()
    # one rounding to fp32, and sums in double or on six digits (2^-44 of the largest entry of a row of g)
    ref, mag = 0.25 * (G @ B), 0.25 * (G.abs() @ B.abs())
    assert bool(((da.double() - ref).abs() <= 2.0 ** -23 * ref.abs() + 2.0 ** -40 * mag + 1e-30).all())
    ref = 0.5 * (G.t().contiguous() @ A)
    mag = 0.5 * M * float(g.abs().max()) * 15
    assert bool(((db.double() - ref).abs() <= 2.0 ** -23 * ref.abs() + 2.0 ** -40 * mag).all())
