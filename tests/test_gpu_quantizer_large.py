"""Quantizer kernels on tensors that are taken in one trip of all blocks, and the marginal PMF: remainders of a block, small, middling and larger sets
for every band width, bins filled by equal entries."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu

LINE = 2_097_152      # more entries: one trip, blocks of 2048 entries


@pytest.mark.parametrize("n", [LINE, LINE + 1, LINE + 2047, LINE + 2048 + 1027, 4 * LINE - 1, 4 * LINE + 1027])
def test_one_trip_remainders(oracle, n):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    lo, levels, delta, alpha = -7, 15, 0.0625, 4.0 / 0.0625 ** 2
    rng = np.random.default_rng(n)
    theta = (rng.standard_normal(n) * 0.2).astype(np.float32)
    g, u = rng.standard_normal(n).astype(np.float32), rng.random(n).astype(np.float32)
    th_d, g_d = gu.dev(theta), gu.dev(g)
    ws = gu.workspace(cdl.quantize_workspace_bytes(n, levels))
    ws.fill_(255)
    # (one entry more than asked for in every output: it stays as it is)
    idx, soft = torch.full((n + 1,), 99, dtype=torch.int8, device="cuda"), torch.full((n + 1,), 7.0, device="cuda")
    dth, dent, drawn = torch.full((n + 1,), 7.0, device="cuda"), torch.full((n + 1,), 7.0, device="cuda"), torch.full((n + 1,), 99, dtype=torch.int8, device="cuda")
    dd, da, marg = gu.empty((1,), torch.float32), gu.empty((1,), torch.float32), gu.empty((levels,), torch.float32)
    cdl.cdl_quantize_fwd(th_d, n, lo, levels, delta, alpha, idx, soft)
    cdl.cdl_quantize_bwd(th_d, g_d, n, lo, levels, delta, alpha, dth, dd, da, ws)
    cdl.cdl_quantize_draw(th_d, gu.dev(u), n, lo, levels, delta, alpha, drawn)
    cdl.cdl_marginal_entropy(th_d, n, lo, levels, delta, alpha, marg, gu.empty((1,), torch.float32), ws)
    cdl.cdl_entropy_bwd(th_d, marg, n, lo, levels, delta, alpha, 0.01 * n, g_d, dent, None, None, ws)
    torch.cuda.synchronize()
    assert int(idx[n]) == 99 and float(soft[n]) == 7.0 and float(dth[n]) == 7.0 and float(dent[n]) == 7.0 and int(drawn[n]) == 99
    r_idx, r_soft, r_gap = oracle.quantize_fwd(theta, lo, levels, delta, alpha)[:3]
    gu.assert_indices(idx[:n].cpu().numpy(), r_idx, r_gap, "indices")
    gu.assert_close(soft[:n].cpu().numpy(), r_soft, "soft")
    r = oracle.quantize_bwd(theta, g, lo, levels, delta, alpha)
    gu.assert_close(dth[:n].cpu().numpy(), r["dtheta"], "dtheta")
    gu.check_quantizer_scalars(oracle, "one trip %d" % n, theta, g, (lo, levels, delta, alpha), dd.item(), da.item(), r)
    r_draw, margin = oracle.quantize_draw(theta, u, lo, levels, delta, alpha)
    assert np.all(np.asarray(margin)[drawn[:n].cpu().numpy() != r_draw] < 1e-6)
    tail = slice(n - 5000, n)
    r_e = oracle.entropy_bwd(theta, marg.cpu().numpy().astype(np.float64), lo, levels, delta, alpha, scale=0.01 * n)
    gu.assert_close(dent[:n].cpu().numpy()[tail], (r_e["dtheta"] + g)[tail], "entropy gradient")


# indices without soft values go in one trip from more entries on; draws and soft values of wider bands from fewer
@pytest.mark.parametrize("n,kappa", [(8 * LINE - 3, 4.0), (8 * LINE + 1027, 4.0), (8 * LINE + 2, 1.5), (3 * LINE - 1, 1.5), (3 * LINE + 1026, 2.5)])
def test_indices_and_draws(oracle, n, kappa):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    q = (-7, 15, 0.0625, kappa / 0.0625 ** 2)
    gen = torch.Generator(device="cuda").manual_seed(n)
    theta, u = 0.2 * torch.randn(n, device="cuda", generator=gen), torch.rand(n, device="cuda", generator=gen)
    idx, both, drawn = (torch.full((n + 1,), 99, dtype=torch.int8, device="cuda") for _ in range(3))
    soft = torch.full((n + 1,), 7.0, device="cuda")
    cdl.cdl_quantize_fwd(theta, n, *q, idx)
    cdl.cdl_quantize_fwd(theta, n, *q, both, soft)
    cdl.cdl_quantize_draw(theta, u, n, *q, drawn)
    torch.cuda.synchronize()
    assert torch.equal(idx, both) and int(idx[n]) == 99 and int(drawn[n]) == 99 and float(soft[n]) == 7.0
    at = np.r_[0:4100, n // 2 // 2048 * 2048 - 50:n // 2 // 2048 * 2048 + 50, n - 5000:n]
    th = theta.cpu().numpy()[at]
    r_idx, r_soft, r_gap = oracle.quantize_fwd(th, *q)[:3]
    gu.assert_indices(idx.cpu().numpy()[:n][at], r_idx, r_gap, "indices")
    gu.assert_close(soft.cpu().numpy()[:n][at], r_soft, "soft")
    r_draw, margin = oracle.quantize_draw(th, u.cpu().numpy()[at], *q)
    assert np.all(np.asarray(margin)[drawn.cpu().numpy()[:n][at] != r_draw] < 1e-6)


# the gradient of the entropy without the scalar ones, large sets: one trip as well; entries at both ends of the tensor and of blocks
@pytest.mark.parametrize("kappa", [16.0, 4.0, 2.5, 1.5])
@pytest.mark.parametrize("add", [False, True])
def test_entropy_gradient_alone(oracle, kappa, add):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    n, lo, levels, delta = 4 * LINE + 2051, -127, 255, 0.02
    alpha = kappa / delta ** 2
    theta = torch.randn(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    g = 0.5 * theta if add else None
    marg = np.random.default_rng(1).random(levels) + 0.1
    marg = (marg / marg.sum()).astype(np.float32)
    out, ws = torch.full((n + 1,), 7.0, device="cuda"), gu.workspace(cdl.quantize_workspace_bytes(n, levels))
    cdl.cdl_entropy_bwd(theta, gu.dev(marg), n, lo, levels, delta, alpha, 0.1 * n, g, out, None, None, ws)
    torch.cuda.synchronize()
    assert float(out[n]) == 7.0
    at = np.r_[0:4100, n // 2 // 2048 * 2048 - 50:n // 2 // 2048 * 2048 + 50, n - 5000:n]
    th, got = theta.cpu().numpy()[at], out[:n].cpu().numpy()[at]
    # (an entry's gradient has a factor scale / n, and nothing else of the other entries)
    want = oracle.entropy_bwd(th, marg.astype(np.float64), lo, levels, delta, alpha, scale=0.1 * at.size)["dtheta"]
    gu.assert_close(got, want + 0.5 * th if add else want, "entropy gradient")


# a last vector of one to three entries: alone, behind whole ones of the same wave, first of a wave or a block, in the second trip of a loop and in the last block of one trip
@pytest.mark.parametrize("n", [1, 2, 3, 5, 1_023, 1_025, 66_051, LINE - 1, LINE + 2, LINE + 1_026, 4 * LINE + 4_097])
@pytest.mark.parametrize("levels,kappa", [(15, 4.0), (15, 1.5), (127, 0.5)])
def test_last_vector_of_gradients(oracle, n, levels, kappa):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    lo, delta = -(levels // 2), 2.0 / levels
    alpha = kappa / delta ** 2
    rng = np.random.default_rng(n + levels)
    theta, g = (rng.standard_normal(n) * 0.3).astype(np.float32), rng.standard_normal(n).astype(np.float32)
    marg = rng.random(levels) + 0.1
    marg = (marg / marg.sum()).astype(np.float32)
    th_d, g_d, m_d, ws = gu.dev(theta), gu.dev(g), gu.dev(marg), gu.workspace(cdl.quantize_workspace_bytes(n, levels))
    ws.fill_(255)
    at = np.unique(np.r_[0:min(n, 500), n // 2048 * 2048 - 3:n // 2048 * 2048 + 3, max(0, n - 500):n].clip(0, n - 1))
    want = oracle.quantize_bwd(theta[at], g[at], lo, levels, delta, alpha)["dtheta"]
    want_e = oracle.entropy_bwd(theta[at], marg.astype(np.float64), lo, levels, delta, alpha, scale=0.1 * at.size)["dtheta"]
    for scalars in (False, True):
        dd = [gu.empty((1,), torch.float32) if scalars else None for _ in range(4)]
        outs = [torch.full((n + 1,), 7.0, device="cuda") for _ in range(3)]      # (one more entry than asked for: it stays as it is)
        cdl.cdl_quantize_bwd(th_d, g_d, n, lo, levels, delta, alpha, outs[0], dd[0], dd[1], ws)
        cdl.cdl_entropy_bwd(th_d, m_d, n, lo, levels, delta, alpha, 0.1 * n, g_d, outs[1], dd[2], dd[3], ws)
        cdl.cdl_entropy_bwd(th_d, m_d, n, lo, levels, delta, alpha, 0.1 * n, None, outs[2], dd[2], dd[3], ws)
        torch.cuda.synchronize()
        for got, ref in zip(outs, (want, want_e + g[at], want_e)):
            assert float(got[n]) == 7.0
            gu.assert_close(got.cpu().numpy()[:n][at], ref, "gradient")
        if scalars and n <= 66_051:
            gu.check_quantizer_scalars(oracle, "last vector %d" % n, theta, g, (lo, levels, delta, alpha), dd[0].item(), dd[1].item(), oracle.quantize_bwd(theta, g, lo, levels, delta, alpha))


# (kappa of band widths 1 .. 4; sets of which every level is live)
@pytest.mark.parametrize("n", [3001, 90_001, LINE + 5])
@pytest.mark.parametrize("levels,kappa", [(2, 16.0), (97, 16.0), (98, 16.0), (72, 4.0), (73, 4.0), (48, 2.5), (49, 2.5), (36, 1.5), (37, 1.5), (72, 3.82), (3, 0.05), (5, 0.05), (5, 3.9)])
def test_marginal_of_pairs(oracle, n, levels, kappa):
    lo, delta = -(levels // 2), 0.05
    alpha = kappa / delta ** 2
    rng = np.random.default_rng(levels)
    theta = (rng.uniform(-0.6, 0.6, n) * levels * delta).astype(np.float32)      # (beyond both ends too)
    q = gu.Quantizer(type("S", (), dict(lo=lo, n_levels=levels, delta=delta, alpha=alpha))())
    got = q.fwd(gu.dev(theta))
    r_idx, r_soft, r_gap = oracle.quantize_fwd(theta, lo, levels, delta, alpha)[:3]
    r_m, r_h = oracle.marginal_entropy(theta, lo, levels, delta, alpha)
    gu.assert_indices(got[0], r_idx, r_gap, "indices")
    gu.assert_close(got[1], r_soft, "soft")
    gu.assert_close(got[2], r_m, "marginal PMF")
    gu.assert_close([got[3]], [r_h], "entropy")


# one bin of one copy takes everything its threads see: at a level, halfway between two, next to the ends and far outside
@pytest.mark.parametrize("n", [4099, 16_777_215])
@pytest.mark.parametrize("at", [0.0, 0.5, -0.5, 6.5, 7.0, -7.4, 40.0])
@pytest.mark.parametrize("kappa", [3.82, 16.0, 2.5])
def test_marginal_of_equal_entries(oracle, n, at, kappa):
    torch = gu.torch_mod()
    lo, levels, delta = -7, 15, 0.0625
    alpha = kappa / delta ** 2
    q = gu.Quantizer(type("S", (), dict(lo=lo, n_levels=levels, delta=delta, alpha=alpha))())
    marg, H = q.marginal(torch.full((n,), at * delta, device="cuda"))
    r_m, r_h = oracle.marginal_entropy(np.full(4, at * delta, np.float32), lo, levels, delta, alpha)
    # (all entries round alike: half a unit of 2^-21 each, which the tolerance of 1e-6 holds)
    gu.assert_close(marg, r_m, "marginal PMF")
    assert abs(H - r_h) <= 2e-5      # (-m log2 m of a probability rounded by 2^-22: 2^-22 (22 + 1.5), three levels)
