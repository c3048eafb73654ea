"""Soft regime from a table: both sides of the first size that uses it, ragged tails, the smallest and largest level sets on
both sides of 33 levels, the lowest and the highest sharpness, entries at the edges of the table's intervals, at the end of its
range, beyond it and infinite - forward, marginal PMF, entropy and backward, in a dirty workspace, twice."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu

FROM = 1 << 16


@pytest.mark.parametrize("n,levels,lo,kappa,spread", [
    (FROM - 1, 31, -15, 0.28, 0.4), (FROM, 31, -15, 0.28, 0.4), (FROM + 3, 31, -15, 0.0077, 0.4), (FROM + 4097, 15, -7, 0.3, 0.4),
    (FROM + 1, 7, -3, 0.05, 0.5), (FROM + 2, 6, 0, 0.3, 0.5), (FROM, 33, -16, 1.2, 0.4), (FROM, 34, -17, 1.2, 0.4), (FROM, 16, 0, 1.25, 0.6),
    (FROM, 255, -127, 0.01, 0.4), (FROM, 256, 0, 0.05, 0.4), (FROM, 256, 0, 0.06, 0.4), (3 * FROM + 1, 31, -15, 0.5, 3.0), (FROM + 1, 63, -31, 0.9, 3.0),
    (40 * FROM + 3, 31, -15, 0.28, 0.0), ((1 << 24) // 15, 31, -15, 0.28, 0.4), ((1 << 24) // 15 + 2, 31, -15, 0.0077, 0.4), (96 * FROM, 6, 0, 0.3, 0.5), (40 * FROM, 33, -16, 0.28, 1.5), (FROM, 31, -15, 0.28, "edges"), (20 * FROM, 31, -15, 0.28, "edges"), (FROM, 127, -63, 0.3, "edges")])
def test_soft_table(oracle, n, levels, lo, kappa, spread):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    delta = 0.03
    alpha = kappa / delta ** 2
    rng = np.random.default_rng(n + levels)
    c0, half = lo + 0.5 * (levels - 1), 0.5 * (levels - 1)
    if spread == "edges":
        r = np.linspace(-(levels + 3.0) * 1.001, (levels + 3.0) * 1.001, n)
        r[:4] = [np.inf, -np.inf, levels + 3.0, -(levels + 3.0)]
    else:
        r = c0 * 0 + rng.standard_normal(n) * spread * half + 0.3
    theta = ((r + c0) * delta).astype(np.float32)
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
        only_m, only_h = gu.empty((levels,), torch.float32), gu.empty((1,), torch.float32)
        cdl.cdl_marginal_entropy(th_d, n, lo, levels, delta, alpha, only_m, only_h, ws)
        torch.cuda.synchronize()
        assert torch.equal(only_m, marg) and torch.equal(only_h, H)
        seen.append([t.cpu().numpy() for t in (idx, soft, marg, H, dth, dd, da)])
    for a, b in zip(*seen):
        assert np.array_equal(a, b, equal_nan=True)
    idx, soft, marg, H, dth, dd, da = seen[0]
    finite = np.isfinite(theta)
    step, sharp = float(np.float32(delta)), float(np.float32(alpha))
    r = (theta[finite].astype(np.float64) / step - c0)[:, None]
    o = np.arange(levels) - half
    e = -sharp * step * step * (r - o) ** 2
    P = np.exp(e - e.max(1, keepdims=True))
    P /= P.sum(1, keepdims=True)
    mu = P @ o
    dev = o - mu[:, None]
    var, c3 = (P * dev ** 2).sum(1), (P * dev ** 3).sum(1)
    k = sharp * step * step
    gf = g[finite].astype(np.float64)
    r = r[:, 0]
    fine = levels <= 33      # sums in double whatever the place of an entry
    assert np.abs(soft[finite] - step * (c0 + mu)).max() <= (1e-6 if fine else 2e-6) * step * levels
    assert (np.abs(dth[finite] - gf * 2 * k * var) <= np.abs(gf) * 2 * k * (1e-6 * var + (2e-7 if fine else 1e-5) * var.max())).all()
    assert np.array_equal(idx[finite], np.clip(np.ceil(theta[finite].astype(np.float64) / step - 0.5), lo, lo + levels - 1).astype(np.int64).astype(np.int16) - (128 if lo + levels - 1 > 127 else 0))
    if finite.all():
        m = P.mean(0)
        assert np.abs(marg - m).max() <= 3e-7
        assert H[0] == pytest.approx(-(m[m > 0] * np.log2(m[m > 0])).sum(), rel=3e-6)
        t_d, t_a = (c0 + mu) + 2 * k * ((r - c0 - 2 * mu) * var - c3), 2 * (r - mu) * var - c3
        assert abs(dd[0] - (gf * t_d).sum()) <= (1e-8 if fine else 2e-7) * (np.abs(gf) * (np.abs(c0 + mu) + 2 * k * np.abs(r - c0 - 2 * mu) * var)).sum() + 1e-7 * abs((gf * t_d).sum())
        assert abs(da[0] - step ** 3 * (gf * t_a).sum()) <= step ** 3 * (np.abs(gf) * (2e-6 * np.abs(2 * (r - mu) * var) + 2e-6 * np.abs(c3) + 1e-9 * (np.abs(r) + np.abs(mu)) * var)).sum()


def _moments(r, levels, kappa):
    """P, mean, variance and third central moment of the level offset from the centre, in extended precision."""
    o = np.arange(levels).astype(np.longdouble) - np.longdouble(levels - 1) / 2
    r = r.astype(np.longdouble)[:, None]
    e = -np.longdouble(kappa) * (r - o) ** 2
    P = np.exp(e - e.max(1, keepdims=True))
    P /= P.sum(1, keepdims=True)
    mu = (P * o).sum(1)
    dev = o - mu[:, None]
    return P, mu, (P * dev ** 2).sum(1), (P * dev ** 3).sum(1)


@pytest.mark.parametrize("levels", [6, 7, 15, 31, 33])
@pytest.mark.parametrize("kappa", [1.0, 0.0077, 1e-4, 1e-6, 1e-8])
def test_scalar_gradients_of_the_table_at_any_sharpness(levels, kappa):
    """The scalar sums just above the size from which the table serves, down to sharpness at which the CPMF hardly leaves the
    uniform one, with gradients that cancel and gradients that do not."""
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    n = (3 << 23) // (levels // 2) + 5
    if kappa == 1.0:      # the highest sharpness that the table serves
        kappa = {6: 1.2, 7: 1.2, 15: 0.8, 31: 0.15, 33: 0.13}[levels]
    lo = -(levels // 2)
    step = np.float64(np.float32(0.03))
    sharp = np.float64(np.float32(kappa / step ** 2))
    k, c0 = sharp * step * step, lo + 0.5 * (levels - 1)
    rng = np.random.default_rng(levels)
    values = ((rng.standard_normal(4001) * 0.4 * (levels - 1) / 2 + 0.3 + c0) * step).astype(np.float32)
    place = np.arange(n) % values.size
    theta = values[place]
    r = values.astype(np.float64) / step - c0
    _, mu, var, c3 = _moments(r, levels, k)
    t_d, t_a = (c0 + mu) + 2 * k * ((r - c0 - 2 * mu) * var - c3), 2 * (r - mu) * var - c3
    size_d = np.abs(c0 + mu) + 2 * k * (np.abs(r - c0 - 2 * mu) * var + np.abs(c3))
    size_a = 2 * np.abs(r - mu) * var + np.abs(c3)
    ws = gu.workspace(cdl.quantize_workspace_bytes(n, levels))
    th_d = gu.dev(theta)
    for sign in (None, np.sign(r)):
        g = rng.standard_normal(n).astype(np.float32)
        if sign is not None:
            g = (np.abs(g) * sign[place]).astype(np.float32)
        dth, dd, da = gu.empty((n,), torch.float32), gu.empty((1,), torch.float32), gu.empty((1,), torch.float32)
        cdl.cdl_quantize_bwd(th_d, gu.dev(g), n, lo, levels, float(step), float(sharp), dth, dd, da, ws)
        torch.cuda.synchronize()
        g_sum = np.bincount(place, g.astype(np.float64))
        g_abs = np.bincount(place, np.abs(g.astype(np.float64)))
        # per term: roundings of double sums over the levels (mean: of the size of the set; 1e-12 of the other parts); the result is a float
        bound_d = (g_abs * (1e-12 * size_d + 4 * 2.2e-16 * levels / 2)).sum()
        bound_a = (g_abs * (1e-12 * size_a + 2 * var * 4 * 2.2e-16 * levels / 2)).sum()
        ref_d, ref_a = (g_sum * t_d).sum(), (g_sum * t_a).sum()
        assert abs(dd.item() - ref_d) <= bound_d + 6e-8 * abs(ref_d), (dd.item(), ref_d)
        assert abs(da.item() - step ** 3 * ref_a) <= step ** 3 * (bound_a + 6e-8 * abs(ref_a)), (da.item(), ref_a)
        want = g[:values.size] * (2 * k * var).astype(np.float64)
        assert (np.abs(dth[:values.size].cpu().numpy() - want) <= 1.2e-7 * np.abs(want)).all()


@pytest.mark.parametrize("levels,kappa", [(6, 1.2), (7, 0.05), (15, 0.8), (15, 0.0077), (31, 0.15), (31, 0.0077), (33, 0.13), (31, 1e-6)])
def test_marginal_pmf_of_equal_entries(levels, kappa):
    """Where every entry is the same nothing averages out: the marginal PMF is the entry's CPMF rounded to fp32, inside the table's range
    (next to a node, at an interval's edge, anywhere) and beyond it."""
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    n = (5 << 23) // (levels // 2) + 3
    lo = -(levels // 2)
    step = np.float64(np.float32(0.03))
    sharp = np.float64(np.float32(kappa / step ** 2))
    k, c0 = sharp * step * step, lo + 0.5 * (levels - 1)
    ws = gu.workspace(cdl.quantize_workspace_bytes(n, levels))
    idx, marg, H = gu.empty((n,), torch.int8), gu.empty((levels,), torch.float32), gu.empty((1,), torch.float32)
    values = np.float32([0.0, 0.013, -0.4 * (levels - 1) * step, 0.31 * step * levels, (levels + 4.0) * step, (-levels - 9.3) * step])
    P = _moments(values.astype(np.float64) / step - c0, levels, k)[0]
    for v, want in zip(values, P):
        theta = torch.full((n,), float(v), device="cuda")
        cdl.cdl_quantize_fwd(theta, n, lo, levels, float(step), float(sharp), idx, None, marg, H, ws)
        torch.cuda.synchronize()
        m = marg.cpu().numpy().astype(np.longdouble)
        # half a unit of the fp32 result; interpolation: 1e-12 of the largest probability; 64 partial sums rounded to 2^-21
        assert (np.abs(m - want) <= 6e-8 * want + 1e-12 * want.max() + 64 * 2.0 ** -22 / n).all(), (float(v), np.abs(m - want).max())
        w = want[want > 0]
        assert abs(H.item() + float((w * np.log2(w)).sum())) <= 1.2e-7 * abs(H.item()) + 1e-9


@pytest.mark.parametrize("levels,lo,kappa", [(34, -17, 0.3), (63, -31, 0.05), (127, -63, 0.9), (255, -127, 0.01), (256, 0, 0.05)])
def test_gradient_of_wide_sets_entry_by_entry(levels, lo, kappa):
    """dtheta of sets above 33 levels against the variance of each entry, not the largest one; inside the set and a little beyond it.
    The weights are fp32: base-2 exponents down to -28 and their factors carry 2^-24 each, 3 x 28 x 2^-24 = 5e-6 of a weight, and the
    weights that far down do not count; a beyond entry's variance is one neighbour's weight, whose exponent grows with its distance."""
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    n = FROM + 5
    step = np.float64(np.float32(0.03))
    sharp = np.float64(np.float32(kappa / step ** 2))
    k, c0, half = sharp * step * step, lo + 0.5 * (levels - 1), 0.5 * (levels - 1)
    rng = np.random.default_rng(levels)
    values = ((np.linspace(-half - 1.5, half + 1.5, 3001) + c0) * step).astype(np.float32)
    theta = values[np.arange(n) % values.size]
    g = rng.standard_normal(n).astype(np.float32)
    dth, sc = gu.empty((n,), torch.float32), gu.empty((2,), torch.float32)
    cdl.cdl_quantize_bwd(gu.dev(theta), gu.dev(g), n, lo, levels, float(step), float(sharp), dth, sc[0:1], sc[1:2],
                         gu.workspace(cdl.quantize_workspace_bytes(n, levels)))
    var = _moments(values.astype(np.float64) / step - c0, levels, k)[2]
    want = g.astype(np.float64) * (2 * k * var).astype(np.float64)[np.arange(n) % values.size]
    got = dth.cpu().numpy()
    worst = (np.abs(got - want) / np.abs(want)).max()
    assert worst <= 1e-5, worst


@pytest.mark.parametrize("n,levels,kappa", [((3 << 23) // 15 + 1, 31, 0.0077), ((3 << 23) // 3 + 2, 7, 0.8), (5000, 31, 0.0077), (300_003, 15, 0.3)])
def test_scalar_sums_with_infinite_entries(n, levels, kappa):
    """An infinite entry sits on the outermost level: it adds g times that level to the step's sum, nothing to the sharpness's sum, and
    nothing of it is NaN - with the table and with the loop over the levels."""
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    lo = -(levels // 2)
    step = np.float64(np.float32(0.03))
    sharp = np.float64(np.float32(kappa / step ** 2))
    k, c0, half = sharp * step * step, lo + 0.5 * (levels - 1), 0.5 * (levels - 1)
    rng = np.random.default_rng(n)
    values = ((rng.standard_normal(997) * 0.4 * half + c0) * step).astype(np.float32)
    values[[3, 500, 996]] = np.inf
    values[[7, 501]] = -np.inf
    place = np.arange(n) % values.size
    g = rng.standard_normal(n).astype(np.float32)
    g_sum, g_abs = np.bincount(place, g.astype(np.float64)), np.bincount(place, np.abs(g.astype(np.float64)))
    dth, sc = gu.empty((n,), torch.float32), gu.empty((2,), torch.float32)
    cdl.cdl_quantize_bwd(gu.dev(values[place]), gu.dev(g), n, lo, levels, float(step), float(sharp), dth, sc[0:1], sc[1:2],
                         gu.workspace(cdl.quantize_workspace_bytes(n, levels)))
    fin = np.isfinite(values)
    r = np.where(fin, values, 0.0).astype(np.float64) / step - c0
    _, mu, var, c3 = _moments(r, levels, k)
    t_d = np.where(fin, (c0 + mu) + 2 * k * ((r - c0 - 2 * mu) * var - c3), c0 + np.sign(values) * half)
    t_a = np.where(fin, 2 * (r - mu) * var - c3, 0.0)
    size_d = np.where(fin, np.abs(c0 + mu) + 2 * k * (np.abs(r - c0 - 2 * mu) * var + np.abs(c3)), half)
    size_a = np.where(fin, 2 * np.abs(r - mu) * var + np.abs(c3), half ** 3)
    dd, da = sc.cpu().numpy().astype(np.float64)
    # the entry is held where its CPMF is one level to e^-30 / kappa
    assert abs(dd - (g_sum * t_d).sum()) <= 6e-8 * abs(dd) + 1e-11 * (g_abs * size_d).sum()
    assert abs(da - step ** 3 * (g_sum * t_a).sum()) <= 6e-8 * abs(da) + step ** 3 * 1e-10 * (g_abs * size_a).sum()
    assert np.array_equal(np.abs(dth.cpu().numpy()[:values.size][~fin]) <= 1e-9 * np.abs(g[:values.size][~fin]), np.ones((~fin).sum(), bool))


@pytest.mark.parametrize("n,levels,kappa", [((1 << 28) + 6, 31, 0.0077), ((1 << 26) + 4096 * 256 + 1, 255, 0.02)])
def test_marginal_pmf_of_a_large_tensor(n, levels, kappa):
    """Beyond 2^26 entries the moments are rounded to fewer bits, so that a block's sums stay inside 64; also the index and the ragged tail."""
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    lo = -(levels // 2)
    step = np.float64(np.float32(0.03))
    sharp = np.float64(np.float32(kappa / step ** 2))
    k, c0 = sharp * step * step, lo + 0.5 * (levels - 1)
    rng = np.random.default_rng(levels)
    values = ((rng.standard_normal(1009) * 0.35 * (levels - 1) / 2 + c0) * step).astype(np.float32)
    theta = gu.dev(values).repeat(n // values.size + 1)[:n].contiguous()
    idx, marg, H = gu.empty((n,), torch.int8), gu.empty((levels,), torch.float32), gu.empty((1,), torch.float32)
    cdl.cdl_quantize_fwd(theta, n, lo, levels, float(step), float(sharp), idx, None, marg, H, gu.workspace(cdl.quantize_workspace_bytes(n, levels)))
    torch.cuda.synchronize()
    count = np.full(values.size, n // values.size, np.longdouble)
    count[: n % values.size] += 1
    P = _moments(values.astype(np.float64) / step - c0, levels, k)[0]
    want = (P * count[:, None]).sum(0) / n
    # (wide sets: interpolation of sixth order)
    assert (np.abs(marg.cpu().numpy() - want) <= 6e-8 * want + (1e-12 if levels <= 33 else 3e-9) * P.max()).all()
    w = want[want > 0]
    assert abs(H.item() + float((w * np.log2(w)).sum())) <= 1.2e-7 * H.item() + (1e-9 if levels <= 33 else 1e-7)
    r = values.astype(np.float64) / step
    near = np.clip(np.ceil(r - 0.5), lo, lo + levels - 1).astype(np.int8)
    last = np.arange(n - 5000, n) % values.size
    assert np.array_equal(idx[-5000:].cpu().numpy(), near[last])
