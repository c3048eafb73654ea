"""GPU Huffman-coded sizes: the merge takes up to 64 weights, many pairs, at a time; here at the counts where a round ends, and with 64-bit weights.
The expected size comes from a heap (the oracle counts a host copy of the indices, which 2^31 entries would make slow)."""
import heapq

import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu


def _size(counts):
    h = [int(c) for c in counts if c > 0]
    if len(h) == 1:
        return h[0]
    heapq.heapify(h)
    total = 0
    while len(h) > 1:
        w = heapq.heappop(h) + heapq.heappop(h)
        total += w
        heapq.heappush(h, w)
    return total


def _gpu(counts):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    n = int(sum(counts))
    values = torch.arange(-128, -128 + len(counts), dtype=torch.int8, device="cuda")
    if n < 1 << 24:
        idx = torch.repeat_interleave(values, torch.tensor(np.asarray(counts, np.int64), device="cuda"))
    else:
        idx = torch.empty(n, dtype=torch.int8, device="cuda")
        ends = np.cumsum(np.asarray(counts, np.int64))
        for i, c in enumerate(counts):
            idx[int(ends[i]) - int(c):int(ends[i])].fill_(i - 128)
    out, total = gu.empty((len(counts),), torch.int64), gu.empty((1,), torch.int64)
    ws = gu.workspace(cdl.huffman_workspace_bytes(n))
    cdl.cdl_huffman_bits(idx, n, -128, len(counts), out, total, None, ws)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), np.asarray(counts))
    return int(total.item())


# symbols around a window of 64 and its multiples; counts: all one, few values (ties between leaves and nodes), spread over octaves, a bell
@pytest.mark.parametrize("symbols", [2, 3, 4, 63, 64, 65, 127, 128, 129, 191, 193, 255, 256])
@pytest.mark.parametrize("kind", ["ones", "ties", "octaves", "bell"])
def test_rounds(symbols, kind):
    rng = np.random.default_rng(symbols)
    if kind == "ones":
        counts = np.ones(symbols, np.int64)
    elif kind == "ties":
        counts = rng.choice([1, 2, 3, 4, 6, 8], symbols)
    elif kind == "octaves":
        counts = np.exp2(rng.uniform(0, 14, symbols)).astype(np.int64)
    else:
        counts = np.maximum(1, 20000 * np.exp(-0.5 * (np.linspace(-3.5, 3.5, symbols)) ** 2)).astype(np.int64)
    assert _gpu(counts) == _size(counts)


# the largest weights of 32 bits and the smallest tensors whose weights take 64
@pytest.mark.parametrize("n", [2 ** 31 - 1, 2 ** 31 + 13])
def test_weights_of_a_large_tensor(n):
    counts = np.exp2(np.random.default_rng(5).uniform(0, 22, 256)).astype(np.int64)
    counts[200] += n - counts.sum()
    assert _gpu(counts) == _size(counts)
