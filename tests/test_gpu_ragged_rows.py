"""GPU products over index rows that do not start on 16-byte boundaries: every remainder of a 16-byte chunk and of a 64-byte step, each tile
shape of the forward product, the transposed copies of the backward products, and the sums that operands stored with an offset need.

Tolerance: the forward product is a sum of integers below 2^24 in magnitude, exact, times one step product (exact powers of two here).
Backward: as in test_gpu_limb_rows, the rounding of g to limbs changes an output by at most 9e-7, fp32 rounding by 2^-24 of it."""
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu

K_EDGES = [1, 15, 16, 17, 31, 33, 47, 63, 65, 79, 81, 127, 129, 191, 193, 1000, 1023, 1025]


def _indices(rows, cols, seed, lo=-128, hi=128):
    torch = gu.torch_mod()
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(lo, hi, (rows, cols), device="cuda", generator=gen, dtype=torch.int32).to(torch.int8)


# 256-, 128- and 64-row tiles, 64 and 128 columns wide; ragged in both directions
@pytest.mark.parametrize("M,N", [(70_001, 33), (20_003, 64), (9_001, 61), (40_007, 130), (20_001, 129), (5_003, 300)])
@pytest.mark.parametrize("K", K_EDGES)
@pytest.mark.parametrize("offsets", [(0, 0), (128, 0), (128, 128)])
def test_forward(M, N, K, offsets):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    a, b = _indices(M, K, M + K), _indices(N, K, N + K)
    y, acc = gu.empty((M, N), torch.float32), gu.empty((M, N), torch.int32)
    y.fill_(7.0)
    ws = gu.workspace(cdl.qgemm_fwd_offset_workspace_bytes(M, N, K))
    cdl.cdl_qgemm_fwd_offset(a, b, M, N, K, 0.25, 0.5, *offsets, acc, y, ws)
    ref = (a.double() + offsets[0]) @ (b.double() + offsets[1]).t()
    assert bool((acc.double() == ref).all())
    assert bool((y.double() == (ref.float() * 0.125).double()).all())


@pytest.mark.parametrize("M,N,K", [(30_011, 64, 2646), (9_001, 260, 1001), (12_007, 73, 999), (40_003, 5, 1003), (3_001, 1025, 515), (30_003, 148, 432), (5_000, 2052, 258)])
def test_both_gradients_of_an_unsigned_layer(M, N, K):
    """Column sums of g with fewer and with more columns than threads, in groups of four and singly."""
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    G = torch.randn((M, N), device="cuda", generator=torch.Generator(device="cuda").manual_seed(M)) * 0.5
    a, b = _indices(M, K, M), _indices(N, K, N, -7, 8)
    da, db = gu.empty((M, K), torch.float32), gu.empty((N, K), torch.float32)
    ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    ws.fill_(0x77)
    for _ in range(2):
        cdl.cdl_qgemm_bwd_offset(G, a, b, M, N, K, 2.0 ** -7, 2.0 ** -6, 128, 0, da, db, ws)
    ref_a = 2.0 ** -6 * (G.double() @ b.double())
    ref_b = 2.0 ** -7 * (G.double().t().contiguous() @ (a.double() + 128.0))
    for got, ref in ((da, ref_a), (db, ref_b)):
        assert bool(((got.double() - ref).abs() <= 9e-7 + 2.0 ** -23 * ref.abs()).all())


# more tiles of 32 x 32 than a thousand: short and long rows, at multiples of four bytes and not, few columns with and without an offset
@pytest.mark.parametrize("M,N", [(2003, 517), (270, 5000), (36_001, 31), (50_007, 16)])
@pytest.mark.parametrize("K", [17, 129, 147, 516, 769])
@pytest.mark.parametrize("offsets", [(0, 0), (128, 0), (0, 128)])
def test_forward_of_middling_products(M, N, K, offsets):
    test_forward(M, N, K, offsets)


# (transposed in tiles of 128 columns: rows that end at every place of a chunk, in the first tile and behind it)
@pytest.mark.parametrize("K", [112 + i for i in range(1, 16)] + [144 + i for i in range(1, 16, 2)])
def test_both_gradients_of_rows_that_end_anywhere(K):
    test_both_gradients_of_an_unsigned_layer(90_001, 72, K)


# (sums of rows beside an operand with an offset: from one lane a row to a wave, more rows than a grid takes at once)
@pytest.mark.parametrize("M,N,K", [(1_100_003, 3, 16), (600_011, 5, 17), (530_003, 3, 33), (70_003, 7, 5), (40_001, 17, 63), (40_001, 9, 64), (40_001, 9, 65), (9_001, 70, 1024), (9_001, 70, 1025), (3_003, 300, 2049)])
def test_forward_with_row_sums(M, N, K):
    test_forward(M, N, K, (0, 128))


# (results beyond the last-level cache: copies with padded rows for the kernel of direct loads, and what lies next to them)
@pytest.mark.parametrize("M,N,K", [(58_601, 1_025, 63), (20_003, 3_077, 121), (20_003, 3_073, 249), (30_001, 2_051, 1_013), (155_009, 401, 50), (155_009, 401, 47), (20_003, 3_077, 129)])
@pytest.mark.parametrize("offsets", [(0, 0), (128, 128)])
def test_forward_of_padded_copies(M, N, K, offsets):
    test_forward(M, N, K, offsets)
