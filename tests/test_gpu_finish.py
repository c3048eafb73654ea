"""Where the per-block partial results of the quantizer kernels are added up: inside the kernel for grids of few blocks, by
a second launch beyond - marginal PMF, entropy and scalar gradients on both sides of the line, in a dirty workspace, twice."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu


# grids of 1, 2, the last one that finishes itself and the first one that does not, for few and for many levels
@pytest.mark.parametrize("n,bits", [(2045, 4), (2049, 4), (524284, 4), (524292, 4), (131068, 8), (131076, 8), (700001, 2)])
def test_block_sums(oracle, n, bits):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    half = 2 ** (bits - 1) - 1
    lo, levels, delta, alpha = -half, 2 * half + 1, 0.0625, 4.0 / 0.0625 ** 2
    rng = np.random.default_rng(n)
    theta = (rng.standard_normal(n) * 0.4 * delta * half).astype(np.float32)
    g = rng.standard_normal(n).astype(np.float32)
    th_d, g_d = gu.dev(theta), gu.dev(g)
    ws = gu.workspace(cdl.quantize_workspace_bytes(n, levels))
    seen = []
    for fill in (255, 0):
        ws.fill_(fill)
        idx, soft = gu.empty((n,), torch.int8), gu.empty((n,), torch.float32)
        marg, H = gu.empty((levels,), torch.float32), gu.empty((1,), torch.float32)
        dth, dd, da = gu.empty((n,), torch.float32), gu.empty((1,), torch.float32), gu.empty((1,), torch.float32)
        cdl.cdl_quantize_fwd(th_d, n, lo, levels, delta, alpha, idx, soft, marg, H, ws)
        cdl.cdl_quantize_bwd(th_d, g_d, n, lo, levels, delta, alpha, dth, dd, da, ws)
        torch.cuda.synchronize()
        seen.append([t.cpu().numpy() for t in (marg, H, dd, da)])
    for a, b in zip(*seen):
        assert np.array_equal(a, b)
    r_m, r_h = oracle.marginal_entropy(theta, lo, levels, delta, alpha)
    gu.assert_close(seen[0][0], r_m, "marginal PMF")
    gu.assert_close(seen[0][1], [r_h], "entropy")
    r = oracle.quantize_bwd(theta, g, lo, levels, delta, alpha)
    scale = np.abs(g).sum() * half
    assert abs(seen[0][2][0] - r["d_delta"]) <= 1e-6 + 1e-5 * abs(r["d_delta"]) + 2e-7 * scale
    assert abs(seen[0][3][0] - r["d_alpha"]) <= 1e-6 + 1e-5 * abs(r["d_alpha"])


# one block, few, the last grid that finishes itself, the first that does not; skewed counts (many levels of the tree) and flat ones
@pytest.mark.parametrize("n", [15, 40_001, 2_097_152, 2_129_937])
@pytest.mark.parametrize("skewed", [False, True])
def test_huffman_blocks(oracle, n, skewed):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    rng = np.random.default_rng(n)
    idx = (np.minimum(rng.geometric(0.3, n), 255) - 128).astype(np.int8) if skewed else rng.integers(-127, 128, n).astype(np.int8)
    ws = gu.workspace(cdl.huffman_workspace_bytes(n))
    ws.fill_(255)
    counts, total, rate = gu.empty((256,), torch.int64), gu.empty((1,), torch.int64), gu.empty((1,), torch.float32)
    for _ in range(2):
        cdl.cdl_huffman_bits(gu.dev(idx), n, -128, 256, counts, total, rate, ws)
    r_counts, r_total, r_rate = oracle.huffman_bits(idx, -128, 256)
    assert np.array_equal(counts.cpu().numpy(), np.asarray(r_counts).astype(np.int64)) and int(total.item()) == int(r_total)
    assert float(rate.item()) == pytest.approx(float(r_rate), rel=1e-6)
