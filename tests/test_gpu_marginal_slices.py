"""Marginal PMF and entropy whose blocks' histograms the last blocks add up, a slice of the levels each: on both sides of every line between that
form, the last block alone and a second launch, level counts that are and are not multiples of four, whole and ragged tensors, dirty workspaces, replays."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu

# (n, lo, levels): blocks of 2048 entries, up to 256 of them; the last block alone up to 4096 records, slices up to 16384 and wherever blocks make several trips
CASES = [
    (17 * 2048 - 4, -127, 255), (16 * 2048 - 4, 0, 256), (17 * 2048 - 1, 0, 256),
    (64 * 2048 - 4, 0, 256), (64 * 2048, 0, 256),
    (131 * 2048 + 3, -15, 31), (132 * 2048 + 3, -15, 31), (256 * 2048 - 4, -31, 63), (256 * 2048 + 4, -31, 63), (700_001, -3, 30),
    (524_289, -127, 255), (2_097_152, -127, 255), (2_097_153, -127, 255), (2_000_001, -8, 17), (1_300_002, 0, 66),
]


def _parameters(levels):
    delta = 0.0625
    return delta, 4.0 / delta ** 2


@pytest.mark.parametrize("n,lo,levels", CASES)
@pytest.mark.parametrize("soft", [False, True])
def test_slices(oracle, n, lo, levels, soft):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    delta, alpha = _parameters(levels)
    rng = np.random.default_rng(n + levels)
    theta = ((rng.standard_normal(n) * 0.25 * levels + lo + 0.5 * levels) * delta).astype(np.float32)
    th = gu.dev(theta)
    ws = gu.workspace(cdl.quantize_workspace_bytes(n, levels))
    seen = []
    for fill in (255, 0):
        ws.fill_(fill)
        idx, sv = gu.empty((n,), torch.int8), gu.empty((n,), torch.float32) if soft else None
        marg, H = gu.empty((levels,), torch.float32), gu.empty((1,), torch.float32)
        cdl.cdl_quantize_fwd(th, n, lo, levels, delta, alpha, idx, sv, marg, H, ws)
        torch.cuda.synchronize()
        seen.append((marg.cpu().numpy(), H.cpu().numpy()))
    assert np.array_equal(seen[0][0], seen[1][0]) and np.array_equal(seen[0][1], seen[1][1])
    r_m, r_h = oracle.marginal_entropy(theta, lo, levels, delta, alpha)
    gu.assert_close(seen[0][0], r_m, "marginal PMF")
    gu.assert_close(seen[0][1], [r_h], "entropy")
    only = gu.empty((1,), torch.float32)       # the entropy alone, and the PMF alone
    cdl.cdl_quantize_fwd(th, n, lo, levels, delta, alpha, idx, None, None, only, ws)
    m2 = gu.empty((levels,), torch.float32)
    cdl.cdl_quantize_fwd(th, n, lo, levels, delta, alpha, idx, None, m2, None, ws)
    torch.cuda.synchronize()
    gu.assert_close(only.cpu().numpy(), [r_h], "entropy alone")
    gu.assert_close(m2.cpu().numpy(), r_m, "PMF alone")
    cdl.cdl_marginal_entropy(th, n, lo, levels, delta, alpha, m2, only, ws)      # (the pass that only builds the histogram)
    torch.cuda.synchronize()
    gu.assert_close(m2.cpu().numpy(), r_m, "PMF pass")
    gu.assert_close(only.cpu().numpy(), [r_h], "PMF pass, entropy")


def test_replays():
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    n, lo, levels = 600_001, -31, 63
    delta, alpha = _parameters(levels)
    rng = np.random.default_rng(3)
    th = gu.dev((rng.standard_normal(n) * 16 * delta).astype(np.float32))
    idx, marg, H = gu.empty((n,), torch.int8), gu.empty((levels,), torch.float32), gu.empty((1,), torch.float32)
    ws = gu.workspace(cdl.quantize_workspace_bytes(n, levels))

    def run():
        cdl.cdl_quantize_fwd(th, n, lo, levels, delta, alpha, idx, None, marg, H, ws)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for rep in range(4):
        if rep != 2:      # (once the same input again)
            th.copy_(gu.dev((rng.standard_normal(n) * (4 + 8 * rep) * delta).astype(np.float32)))
        run()
        torch.cuda.synchronize()
        want = marg.cpu().numpy().copy(), H.cpu().numpy().copy()
        marg.zero_()
        H.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(marg.cpu().numpy(), want[0]) and np.array_equal(H.cpu().numpy(), want[1])
