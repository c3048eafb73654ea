"""GPU marginal PMF where roundings do not average out or entries are no numbers: tensors of equal entries at the sharpness of each band width whose
probabilities round worst, tensors of which half are zero, and NaNs between ordinary entries.

Tolerance: a probability is added as a multiple of 2^-21, off by at most 2^-22 and 2^-25 of the sum before it is cut; what is added has at most
eight roundings of 2^-24 (weights, their sum, reciprocal, product) and the output one."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu

SIZES = [3001, 90_001, 2_200_003, 7_000_001, 17_000_002]
BANDS = {1: (10.9, 16.0), 2: (3.82, 10.8), 3: (1.99, 3.81), 4: (1.23, 1.97)}      # half-widths of the unrolled bands and their sharpness


def _tolerance(p):
    return 2.0 ** -22 + 2.0 ** -25 + 9 * 2.0 ** -24 * p


def _worst_kappa(width):
    """The sharpness at which the neighbours of an entry at a level, rounded to 2^-21, are together furthest from their sum."""
    j = np.arange(1, width + 1)
    best = (0.0, 0.0)
    for kappa in np.linspace(*BANDS[width], 2001):
        w = np.exp(-kappa * j * j)
        p = w / (1.0 + 2.0 * w.sum()) * 2.0 ** 21
        best = max(best, (abs(float((np.rint(p) - p).sum())), float(kappa)))
    return best[1]


def _quantizer(levels, kappa, delta=0.0625):
    return gu.Quantizer(type("S", (), dict(lo=-(levels // 2), n_levels=levels, delta=delta, alpha=kappa / delta ** 2))())


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("width", sorted(BANDS))
def test_equal_entries(oracle, n, width):
    torch = gu.torch_mod()
    q = _quantizer(15, _worst_kappa(width))
    marg = q.marginal(torch.zeros(n, device="cuda"))[0].astype(np.float64)
    ref = np.asarray(oracle.marginal_entropy(np.zeros(4, np.float32), *q.args)[0])
    assert np.all(np.abs(marg - ref) <= _tolerance(ref)), np.abs(marg - ref).max()


@pytest.mark.parametrize("width", sorted(BANDS))
def test_half_of_the_entries_zero(oracle, width):
    q = _quantizer(15, _worst_kappa(width))
    theta = (np.random.default_rng(width).standard_normal(2_200_003) * 0.2).astype(np.float32)
    theta[::2] = 0.0
    idx, soft, marg, _ = q.fwd(gu.dev(theta))
    ref = np.asarray(oracle.marginal_entropy(theta, *q.args)[0])
    assert np.all(np.abs(marg - ref) <= _tolerance(ref)), np.abs(marg - ref).max()


@pytest.mark.parametrize("n", SIZES[1:])
@pytest.mark.parametrize("levels", [15, 63, 96])
@pytest.mark.parametrize("kappa", [16.0, 2.5, 1.5])
def test_nan_adds_nothing(n, levels, kappa):
    torch = gu.torch_mod()
    q = _quantizer(levels, kappa)
    theta = torch.randn(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(levels)) * 0.3
    finite = torch.ones(n, dtype=torch.bool, device="cuda")
    finite[::10] = False
    want, _ = q.marginal(theta[finite].contiguous())
    got, _ = q.marginal(torch.where(finite, theta, float("nan")))
    want = want.astype(np.float64) * (int(finite.sum()) / n)
    assert np.all(np.abs(got - want) <= 2.0 ** -22 * want)      # (the same whole numbers over n; each output rounded once)
