"""Products of small layers: the forward kernel that splits the contraction over the waves of a block, and the backward
products formed directly in double - ragged tiles, rows that are not aligned, contractions shorter and longer than a step,
operands stored with an offset, contractions cut into pieces - and backward products just too large for that."""
import numpy as np
import pytest

import cdl_inputs
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 1, 16), (33, 31, 17), (32, 32, 127), (64, 65, 129), (31, 33, 143), (100, 37, 1005), (7, 300, 640), (1000, 33, 255)])
@pytest.mark.parametrize("oa,ob", [(0, 0), (128, 0), (128, 128)])
def test_forward(M, N, K, oa, ob):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    a, b = cdl_inputs.draw_indices((M, K), -128, 127, seed=M), cdl_inputs.draw_indices((N, K), -128, 127, seed=N)
    acc, y = gu.empty((M, N), torch.int32), gu.empty((M, N), torch.float32)
    ws = gu.workspace(cdl.qgemm_fwd_offset_workspace_bytes(M, N, K))
    cdl.cdl_qgemm_fwd_offset(gu.dev(a), gu.dev(b), M, N, K, 0.5, 0.25, oa, ob, acc, y, ws)
    ref = (a.astype(np.int64) + oa) @ (b.astype(np.int64) + ob).T
    assert np.array_equal(acc.cpu().numpy(), ref)
    assert np.array_equal(y.cpu().numpy(), ref.astype(np.float32) * np.float32(0.125))


@pytest.mark.parametrize("M,N,K", [(1, 1, 4), (17, 5, 7), (16, 16, 64), (15, 33, 65), (33, 40, 6), (130, 1, 68), (260, 34, 129), (5000, 20, 70), (5121, 31, 64),
                                   (700, 250, 300), (300, 700, 77), (5003, 61, 131),      # with the diagnostic words
                                   (6001, 130, 333), (9001, 301, 333)])                   # limbs: the two products side by side, one after the other
@pytest.mark.parametrize("oa,ob", [(0, 0), (128, 128)])
def test_backward(oracle, M, N, K, oa, ob):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    rng = np.random.default_rng(M + N + K)
    g = rng.standard_normal((M, N)).astype(np.float32)
    a, b = cdl_inputs.draw_indices((M, K), -128, 127, seed=M), cdl_inputs.draw_indices((N, K), -128, 127, seed=N)
    d_a, d_b = gu.empty((M, K), torch.float32), gu.empty((N, K), torch.float32)
    ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    ws.fill_(255)
    for _ in range(2):
        d_a.fill_(float("nan"))
        d_b.fill_(float("nan"))
        cdl.cdl_qgemm_bwd_offset(gu.dev(g), gu.dev(a), gu.dev(b), M, N, K, 0.015625, 0.0078125, oa, ob, d_a, d_b, ws)
    g64 = g.astype(np.float64)
    gu.assert_close(d_a.cpu().numpy(), 0.0078125 * (g64 @ (b.astype(np.float64) + ob)), "d_a_hat")
    gu.assert_close(d_b.cpu().numpy(), 0.015625 * (g64.T @ (a.astype(np.float64) + oa)), "d_b_hat")
    only = gu.empty((N, K), torch.float32)
    cdl.cdl_qgemm_bwd_offset(gu.dev(g), gu.dev(a), gu.dev(b), M, N, K, 0.015625, 0.0078125, oa, ob, None, only, ws)
    gu.assert_close(only.cpu().numpy(), 0.015625 * (g64.T @ (a.astype(np.float64) + oa)), "d_b_hat alone")


# few and many channels, one and four classes of pixels, and just too large for the direct kernels
@pytest.mark.parametrize("B,H,W,C,N,R,S,stride,pad", [(2, 9, 7, 16, 4, 3, 3, 1, 1), (3, 8, 11, 48, 20, 5, 3, 2, 2), (1, 13, 13, 80, 12, 1, 1, 2, 0),
                                                      (40, 17, 19, 112, 36, 3, 3, 1, 1), (12, 57, 57, 48, 100, 3, 3, 1, 1)])
@pytest.mark.parametrize("x_offset", [0, 128])
def test_convolution_gradients(oracle, B, H, W, C, N, R, S, stride, pad, x_offset):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    rng = np.random.default_rng(C + N)
    x = cdl_inputs.draw_indices((B, H, W, C), -128, 127, seed=C)
    w = cdl_inputs.draw_indices((N, R, S, C), -127, 127, seed=N)
    g = rng.standard_normal((B, P, Q, N)).astype(np.float32)
    dX, dW = gu.empty((B, H, W, C), torch.float32), gu.empty((N, R, S, C), torch.float32)
    geom = (B, H, W, C, N, R, S, stride, pad)
    ws = gu.workspace(max(cdl.qconv_bwd_weights_workspace_bytes(*geom), cdl.qconv_bwd_activations_workspace_bytes(*geom)))
    ws.fill_(255)
    for _ in range(2):
        cdl.cdl_qconv_bwd_weights(gu.dev(g), gu.dev(x), *geom, 0.015625, dW, ws, x_offset=x_offset)
        cdl.cdl_qconv_bwd_activations(gu.dev(g), gu.dev(w), *geom, 0.0078125, dX, ws)
    r_x, r_w = oracle.qconv_bwd(g, x.astype(np.int16) + x_offset, w, stride, pad, 0.015625, 0.0078125)
    gu.assert_close(dX.cpu().numpy(), r_x, "d_x_hat")
    gu.assert_close(dW.cpu().numpy(), r_w, "d_w_hat")


@pytest.mark.parametrize("M,N,K", [(32, 128, 256), (512, 256, 256), (5000, 16, 144), (131072, 16, 144), (20000, 32, 100)])
@pytest.mark.parametrize("want", ["both", "a", "b"])
def test_diagnostic_words_of_products_without_limbs(M, N, K, want):
    """A call that forms its products directly says so in the workspace - no limbs, bounds of zero - whatever lay there before."""
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    ws.fill_(0x5a)
    g = torch.randn((M, N), device="cuda")
    a, b = torch.randint(0, 16, (M, K), dtype=torch.int8, device="cuda"), torch.randint(-7, 8, (N, K), dtype=torch.int8, device="cuda")
    da, db = gu.empty((M, K), torch.float32), gu.empty((N, K), torch.float32)
    cdl.cdl_qgemm_bwd(g, a, b, M, N, K, 0.5, 0.02, da if want != "b" else None, db if want != "a" else None, ws)
    torch.cuda.synchronize()
    limbs, bounds = ws[:8].view(torch.int32).tolist(), ws[32:48].view(torch.float64).tolist()
    assert limbs == [0, 0] and bounds == [0.0, 0.0]
