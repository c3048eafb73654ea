"""GPU backward products on digits scaled by row: ends of the contraction, scales that grow inside a row, far apart rows, small entries next to
far larger ones, non-finite entries, and the products that are cut into pieces together with the diagnostic words.

Tolerance.  Every product of an entry of g and an index is exact, so an output is off by what its sum of n products in double is, at most
n 2^-53 of the sum of their magnitudes, and by 2^-24 of the output for fp32.  Checked entry by entry with bounds twice as large (the reference
is summed in double, in another order)."""
import numpy as np
import pytest

import cdl_inputs
import gpu_util as gu

pytestmark = pytest.mark.gpu


def _check(got, g64, idx64, step, what):
    ref = g64 @ idx64
    bound = step * (g64.shape[1] * 2.0 ** -52 * (np.abs(g64) @ np.abs(idx64)) + 2.0 ** -23 * np.abs(ref))
    off = np.abs(got.astype(np.float64) - step * ref)
    assert np.all(off <= bound + 1.5e-45), "%s: %.3g of the bound" % (what, np.max(off / (bound + 1e-300)))


def _run(g, a, b, oa=0, ob=0, apart=False):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    M, N, K = g.shape[0], g.shape[1], a.shape[1]
    d_a, d_b = gu.empty((M, K), torch.float32), gu.empty((N, K), torch.float32)
    ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    ws.fill_(255)
    for _ in range(2):
        d_a.fill_(float("nan"))
        d_b.fill_(float("nan"))
        for x, y in ((d_a, None), (None, d_b)) if apart else ((d_a, d_b),):
            cdl.cdl_qgemm_bwd_offset(gu.dev(g), gu.dev(a), gu.dev(b), M, N, K, 0.5, 0.25, oa, ob, x, y, ws)
    torch.cuda.synchronize()
    return d_a.cpu().numpy(), d_b.cpu().numpy(), ws


def _indices(M, N, K):
    return cdl_inputs.draw_indices((M, K), -128, 127, seed=M), cdl_inputs.draw_indices((N, K), -128, 127, seed=N)


# contraction lengths around a step of 64 and a quarter of it; more than seven steps for a wave (5000); widths that are no multiple of four
@pytest.mark.parametrize("M,N,K", [(700, 63, 400), (700, 64, 400), (700, 65, 400), (63, 700, 400), (65, 700, 402), (640, 79, 401), (641, 81, 399), (640, 128, 403),
                                   (100, 5000, 80), (5000, 100, 80), (33, 2100, 500), (300, 129, 1030)])
@pytest.mark.parametrize("oa,ob", [(0, 0), (128, 128)])
def test_ends(M, N, K, oa, ob):
    rng = np.random.default_rng(M * N + K)
    g = rng.standard_normal((M, N)).astype(np.float32)
    a, b = _indices(M, N, K)
    d_a, d_b, _ = _run(g, a, b, oa, ob)
    g64 = g.astype(np.float64)
    _check(d_a, g64, b.astype(np.float64) + ob, 0.25, "d_a_hat")
    _check(d_b, np.ascontiguousarray(g64.T), a.astype(np.float64) + oa, 0.5, "d_b_hat")


# growing: every 64 entries of a row (and of a column) are larger than the ones before; rows of very different size, down to subnormal numbers;
# rows that are zero; one step of huge numbers
@pytest.mark.parametrize("kind", ["growing", "shrinking", "rows", "zeros", "huge"])
@pytest.mark.parametrize("M,N,K", [(600, 650, 300), (4000, 200, 256)])
def test_scales(kind, M, N, K):
    rng = np.random.default_rng(len(kind))
    g = rng.standard_normal((M, N))
    i, j = np.arange(M)[:, None], np.arange(N)[None, :]
    if kind == "growing":
        g *= np.exp2(3.0 * (j // 64) + 1.0 * (i // 64))
    elif kind == "shrinking":
        g *= np.exp2(-5.0 * (j // 64) - 2.0 * (i // 64))
    elif kind == "rows":
        g *= np.exp2(rng.uniform(-140, 100, (M, 1)))
    elif kind == "zeros":
        g *= (rng.random((M, N)) < 0.01) * (rng.random((M, 1)) < 0.5)
    else:
        g[:, 64:128] *= 2.0 ** 100      # (4000 products of 2^103 and 2^7 stay below 2^128: with 2^115 an fp32 output overflows)
    g = g.astype(np.float32)
    a, b = _indices(M, N, K)
    d_a, d_b, _ = _run(g, a, b)
    g64 = g.astype(np.float64)
    with np.errstate(over="ignore"):
        _check(d_a, g64, b.astype(np.float64), 0.25, "d_a_hat")
        _check(d_b, np.ascontiguousarray(g64.T), a.astype(np.float64), 0.5, "d_b_hat")


# One row and one column of g far larger than the rest, with zeros among the indices that they meet: what the others contribute to those outputs
# keeps all its bits.  "mixed": entries of every size in every step, zeros among them.
@pytest.mark.parametrize("kind", [2.0 ** 18, 2.0 ** 24, 2.0 ** 30, 2.0 ** 60, "mixed"])
@pytest.mark.parametrize("M,N,K", [(2048, 64, 256), (256, 1000, 512), (600, 650, 300), (700, 63, 400), (5120, 64, 192)])
@pytest.mark.parametrize("oa,ob", [(0, 0), (128, 128)])
def test_small_entries_next_to_large_ones(kind, M, N, K, oa, ob, apart=False):
    rng = np.random.default_rng(K)
    g = rng.standard_normal((M, N))
    a, b = _indices(M, N, K)
    if kind == "mixed":
        g *= np.exp2(rng.uniform(-60, 0, (M, N))) * (rng.random((M, N)) < 0.7)
    else:
        g[:, 5] *= kind
        g[70 % M, :5] *= kind
        g[70 % M, 6:] *= kind
    b[5, ::2] = -ob
    a[70 % M, ::2] = -oa
    g = g.astype(np.float32)
    d_a, d_b, _ = _run(g, a, b, oa, ob, apart)
    g64 = g.astype(np.float64)
    _check(d_a, g64, b.astype(np.float64) + ob, 0.25, "d_a_hat")
    _check(d_b, np.ascontiguousarray(g64.T), a.astype(np.float64) + oa, 0.5, "d_b_hat")


# up to 0.7 * 10^9 multiply-adds of what is asked for, in whole tiles: directly, also where limbs would take less time by the estimate.  apart: one
# product to a call, layers that are too large for both
@pytest.mark.parametrize("M,N,K,apart", [(40, 5376, 128, False), (136, 385, 5631, False), (16, 3687, 3605, False), (1583, 75, 2702, False), (25, 2624, 4032, False),
                                         (489, 512, 2112, True), (74, 3648, 1728, True), (2208, 64, 4672, True)])
@pytest.mark.parametrize("kind", [1.0, 2.0 ** 30])
def test_few_multiplications(M, N, K, apart, kind):
    test_small_entries_next_to_large_ones(kind, M, N, K, 0, 0, apart)


# the same for the gradients of a convolution, 16 x 28 x 28 x 64 -> 64, with stride 2, a 1 x 1 kernel (a linear layer of 10240 rows), 48 channels in double
@pytest.mark.parametrize("geom", [(16, 28, 28, 64, 64, 3, 3, 1, 1), (24, 33, 31, 96, 64, 3, 3, 2, 1), (40, 16, 16, 128, 128, 1, 1, 1, 0),
                                  (34, 60, 60, 48, 32, 3, 3, 2, 1)])
@pytest.mark.parametrize("size,scale", [(1.0, 1.0), (2.0 ** 30, 1.0), (2.0 ** 30, 2.0 ** -40)])
def test_small_entries_next_to_large_ones_conv(geom, size, scale):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    B, H, W, C, N, R, S, stride, pad = geom
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    gen = torch.Generator().manual_seed(H)
    g = torch.randn((B, P, Q, N), generator=gen) * scale
    g[..., 5] *= size                       # a channel (activations' gradient) and a pixel (weights')
    g[1, 2, 3, :5] *= size
    x = torch.randint(-128, 128, (B, H, W, C), generator=gen, dtype=torch.int32)
    w = torch.randint(-128, 128, (N, R, S, C), generator=gen, dtype=torch.int32)
    w[5, :, :, ::2] = 0
    x[1, 2 * stride - pad:2 * stride - pad + R, 3 * stride - pad:3 * stride - pad + S, ::2] = 0
    G, X, Wi = g.cuda(), x.to(torch.int8).cuda(), w.to(torch.int8).cuda()
    dx, dw = gu.empty((B, H, W, C), torch.float32), gu.empty((N, R, S, C), torch.float32)
    ws = gu.workspace(max(cdl.qconv_bwd_weights_workspace_bytes(*geom), cdl.qconv_bwd_activations_workspace_bytes(*geom)))
    cdl.cdl_qconv_bwd_activations(G, Wi, *geom, 0.25, dx, ws)
    cdl.cdl_qconv_bwd_weights(G, X, *geom, 0.5, dw, ws)
    torch.cuda.synchronize()
    g2, xp = g.double().reshape(-1, N), torch.zeros((B, H + 2 * pad + R, W + 2 * pad + S, C), dtype=torch.float64)
    xp[:, pad:pad + H, pad:pad + W] = x.double()
    sums = []
    for f in (lambda t: t, torch.abs):      # the products, and the sums of their magnitudes
        out, dw_ref = torch.zeros_like(xp), torch.zeros((N, R, S, C), dtype=torch.float64)
        for r in range(R):
            for s in range(S):
                out[:, r:r + stride * P:stride, s:s + stride * Q:stride] += (f(g2) @ f(w.double())[:, r, s].contiguous()).reshape(B, P, Q, C)
                dw_ref[:, r, s] = f(g2).t().contiguous() @ f(xp)[:, r:r + stride * P:stride, s:s + stride * Q:stride].reshape(-1, C)
        sums.append((out[:, pad:pad + H, pad:pad + W], dw_ref))
    for got, ref, mag, step, n in ((dx, sums[0][0], sums[1][0], 0.25, R * S * N), (dw, sums[0][1], sums[1][1], 0.5, B * P * Q)):
        off, bound = (got.cpu().double() - step * ref).abs(), step * (n * 2.0 ** -52 * mag + 2.0 ** -23 * ref.abs())
        assert bool((off <= bound).all()), float((off / (bound + 1e-300)).max())


# an infinity or a NaN shows in the outputs it enters, as a sum in double has it, and in no other
@pytest.mark.parametrize("M,N,K", [(600, 650, 300), (4000, 200, 256)])
@pytest.mark.parametrize("offset", [0, 128])
def test_non_finite_entries(M, N, K, offset):
    rng = np.random.default_rng(M)
    g = rng.standard_normal((M, N)).astype(np.float32)
    places = [(0, 0, np.inf), (17, 63, np.nan), (M - 1, N - 1, -np.inf), (300, 64, np.inf), (300, 190, -np.inf)]
    for m, n, v in places:
        g[m, n] = v
    a, b = _indices(M, N, K)
    d_a, d_b, _ = _run(g, a, b, offset, offset)
    finite = np.where(np.isfinite(g), g, 0.0).astype(np.float64)
    rows, cols = sorted({p[0] for p in places}), sorted({p[1] for p in places})
    with np.errstate(invalid="ignore"):
        for got, gg, idx, bad in ((d_a, g, b, rows), (d_b, g.T, a, cols)):
            for r in bad:
                ref = sum(np.float64(v) * (idx[k].astype(np.float64) + offset) for k, v in enumerate(gg[r]) if not np.isfinite(v))
                assert np.array_equal(np.isnan(got[r]), np.isnan(ref)) and np.array_equal(got[r][np.isinf(ref)], ref[np.isinf(ref)].astype(np.float32))
    good_r, good_c = np.setdiff1d(np.arange(M), rows), np.setdiff1d(np.arange(N), cols)
    _check(d_a[good_r], finite[good_r], b.astype(np.float64) + offset, 0.25, "d_a_hat")
    _check(d_b[good_c], np.ascontiguousarray(finite.T)[good_c], a.astype(np.float64) + offset, 0.5, "d_b_hat")


# long contractions over few output tiles, cut into pieces: the diagnostic words come from the kernel that adds them up; spread: entries of many sizes
@pytest.mark.parametrize("M,N,K", [(6001, 40, 333), (12000, 64, 192), (20000, 64, 100), (9000, 48, 79)])      # (more than 2^25 multiply-adds: fewer have no such words)
@pytest.mark.parametrize("spread", [0, 16])
def test_pieces_and_diagnostic_words(M, N, K, spread):
    rng = np.random.default_rng(M)
    g = (rng.standard_normal((M, N)) * np.exp2(rng.uniform(-spread, 0, (M, N)))).astype(np.float32)
    a, b = _indices(M, N, K)
    d_a, d_b, ws = _run(g, a, b)
    g64 = g.astype(np.float64)
    _check(d_a, g64, b.astype(np.float64), 0.25, "d_a_hat")
    _check(d_b, np.ascontiguousarray(g64.T), a.astype(np.float64), 0.5, "d_b_hat")
    torch = gu.torch_mod()
    limbs, bounds = ws[:8].view(torch.int32).tolist(), ws[32:48].view(torch.float64).tolist()
    e = np.frexp(np.float32(np.max(np.abs(g)) * np.float32(1.01)))[1]
    for k, (step, idx) in enumerate(((0.25, b), (0.5, a))):
        unit = step * float(np.max(np.sum(np.abs(idx.astype(np.int64)), axis=0)))
        want = next((c for c in range(3, 7) if unit * 2.0 ** (e - 8 * c) <= 9e-7), 6)
        assert limbs[k] == want and bounds[k] == unit * 2.0 ** (e - 8 * want)
