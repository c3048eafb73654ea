"""GPU weight gradients over long contractions, where the column tiles of a block share the digits of g: two to six tiles, one and several groups of
tiles, one and several rounds of steps, last steps that are not whole, widths that are no multiple of four; entries far apart in size, rows that grow from round to round,
non-finite entries, an operand stored with an offset, a 1 x 1 convolution.

Tolerance: as of the other products on digits (every product exact, sums in double): n 2^-52 of the sum of magnitudes and 2^-23 of the output."""
import numpy as np
import pytest

import cdl_inputs
import gpu_util as gu
from test_gpu_digit_tiles import _check
from test_gpu_dispatch import _recorded

pytestmark = pytest.mark.gpu

SHAPES = [(79_701, 18, 124), (131_009, 16, 146), (119_370, 25, 242), (207_871, 17, 283), (93_389, 19, 356), (34_214, 25, 923)]


def _product(g, a, offset):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    (M, N), K = g.shape, a.shape[1]
    b = gu.dev(np.zeros((N, K), np.int8))
    out = gu.empty((N, K), torch.float32)
    ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    ws.fill_(255)
    G, A, names, seen = gu.dev(g), gu.dev(a), set(), []
    for _ in range(2):
        out.fill_(float("nan"))
        names = _recorded(lambda: cdl.cdl_qgemm_bwd_offset(G, A, b, M, N, K, 0.5, 0.25, offset, 0, None, out, ws))
        torch.cuda.synchronize()
        seen.append(out.cpu().numpy())
    assert "dw_shared_kernel" in names, names
    assert np.array_equal(seen[0], seen[1], equal_nan=True)
    assert ws[:8].view(torch.int32).tolist() == [0, 0]      # (the diagnostic words: no limbs)
    return seen[0]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("kind,offset", [("normal", 0), ("normal", 128), ("column", 0), ("mixed", 128), ("growing", 0), ("zeros", 128)])
def test_shared_digits(M, N, K, kind, offset):
    rng = np.random.default_rng(M + N)
    g = rng.standard_normal((M, N))
    a = cdl_inputs.draw_indices((M, K), -128, 127, seed=K)
    if kind == "column":            # one row and one column 2^30 times the rest
        g[:, 5] *= 2.0 ** 30
        g[70, :] *= 2.0 ** 30
        a[70, ::2] = -offset
    elif kind == "mixed":           # entries of every size in every step: whole steps in double
        g *= np.exp2(rng.uniform(-60, 0, (M, N))) * (rng.random((M, N)) < 0.7)
    elif kind == "growing":         # from round to round
        g *= np.exp2(np.minimum(np.arange(M)[:, None] // 512 % 64, 40))
    elif kind == "zeros":
        g *= (rng.random((M, N)) < 0.01) * (rng.random((M, 1)) < 0.5)
    g = g.astype(np.float32)
    _check(_product(g, a, offset), np.ascontiguousarray(g.astype(np.float64).T), a.astype(np.float64) + offset, 0.5, "d_b_hat")


@pytest.mark.parametrize("offset", [0, 128])
def test_non_finite_entries(offset):
    M, N, K = SHAPES[1]
    rng = np.random.default_rng(5)
    g = rng.standard_normal((M, N)).astype(np.float32)
    a = cdl_inputs.draw_indices((M, K), -128, 127, seed=K)
    a[17, ::3] = -offset
    g[17, 3], g[M - 1, 9], g[4000, 9], g[4001, 11] = np.inf, -np.inf, np.nan, -np.inf
    got = _product(g, a, offset)
    idx = a.astype(np.float64) + offset
    with np.errstate(invalid="ignore"):
        for n, ms in ((3, [17]), (9, [4000, M - 1]), (11, [4001])):
            ref = sum(np.float64(g[m, n]) * idx[m] for m in ms)
            assert np.array_equal(np.isnan(got[n]), np.isnan(ref)) and np.array_equal(got[n][np.isinf(ref)], ref[np.isinf(ref)].astype(np.float32))
    good = np.setdiff1d(np.arange(N), [3, 9, 11])
    _check(got[good], np.ascontiguousarray(g.astype(np.float64).T)[good], idx, 0.5, "d_b_hat")


# the same on a 1 x 1 convolution with more than 32 output channels
def test_pointwise_convolution():
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    B, H, W, C, N = 53, 45, 45, 224, 48
    geom = (B, H, W, C, N, 1, 1, 1, 0)
    rng = np.random.default_rng(1)
    g = rng.standard_normal((B * H * W, N)).astype(np.float32)
    x = cdl_inputs.draw_indices((B * H * W, C), -128, 127, seed=2)
    out = gu.empty((N, C), torch.float32)
    ws = gu.workspace(cdl.qconv_bwd_weights_workspace_bytes(*geom))
    G, X = gu.dev(g), gu.dev(x)
    assert "dw_shared_kernel" in _recorded(lambda: cdl.cdl_qconv_bwd_weights(G, X, *geom, 0.5, out, ws))
    torch.cuda.synchronize()
    _check(out.cpu().numpy(), np.ascontiguousarray(g.astype(np.float64).T), x.astype(np.float64), 0.5, "d_w_hat")


# on the other side of the rule: short contractions, few columns
@pytest.mark.parametrize("M,N,K", [(13_296, 17, 384), (39_007, 24, 319), (270_320, 19, 69)])
def test_not_served(M, N, K):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    g, a = torch.randn((M, N), device="cuda"), gu.dev(cdl_inputs.draw_indices((M, K), -8, 7, seed=K))
    out, ws = gu.empty((N, K), torch.float32), gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    assert "dw_shared_kernel" not in _recorded(lambda: cdl.cdl_qgemm_bwd(g, a, a[:N], M, N, K, 0.5, 0.25, None, out, ws))
