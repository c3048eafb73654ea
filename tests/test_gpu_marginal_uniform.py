"""Marginal PMF of levels that are nearly all live: every level's sum over a block, for the smallest and the largest set of each unrolled width (6 - 9, 10 - 17 and
18 - 33 levels), fewer entries than a block has threads, ragged tensors, one and several blocks; dirty workspaces."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [6, 9, 10, 17, 18, 33])
@pytest.mark.parametrize("n", [1, 1021, 1025, 30_001])
@pytest.mark.parametrize("alpha", [0.01, 0.5])
def test_uniform(oracle, levels, n, alpha):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    delta, lo = 0.25, -(levels // 2)
    theta = (np.random.default_rng(n + levels).standard_normal(n) * 0.25 * levels * delta).astype(np.float32)
    th, ws = gu.dev(theta), gu.workspace(cdl.quantize_workspace_bytes(n, levels))
    r_m, r_h = oracle.marginal_entropy(theta, lo, levels, delta, alpha)
    seen = []
    for fill in (255, 0):
        ws.fill_(fill)
        idx, marg, H = gu.empty((n,), torch.int8), gu.empty((levels,), torch.float32), gu.empty((1,), torch.float32)
        cdl.cdl_quantize_fwd(th, n, lo, levels, delta, alpha, idx, None, marg, H, ws)
        torch.cuda.synchronize()
        gu.assert_close(marg.cpu().numpy(), r_m, "marginal PMF")
        gu.assert_close(H.cpu().numpy(), [r_h], "entropy")
        seen.append(marg.cpu().numpy())
    assert np.array_equal(seen[0], seen[1])
