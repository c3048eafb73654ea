"""GPU Huffman-coded size where one launch does it all: counts of 16 bits in the blocks' records at their largest (a constant tensor, the last entries of a ragged one in the last
block), grids of one to 64 blocks and trips that are not whole groups, a dirty workspace of just the size asked for, replays."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu


def _call(idx, ws, out):
    import paper_2501_09849_amd as cdl
    cdl.cdl_huffman_bits(idx, idx.numel(), -128, 256, out[0], out[1], None, ws)


def _outputs():
    torch = gu.torch_mod()
    return gu.empty((256,), torch.int64), gu.empty((1,), torch.int64)


@pytest.mark.parametrize("n", [65_535, 65_536, 70_001, 131_072, 500_003, 1_048_592, 2_097_152, 2_097_167, 2_097_168])
@pytest.mark.parametrize("kind", ["constant", "two", "all"])
def test_counts(oracle, n, kind):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    rng = np.random.default_rng(n)
    idx = np.full(n, 77, np.int8) if kind == "constant" else rng.choice(np.array([-128, 127], np.int8), n) if kind == "two" else rng.integers(-128, 128, n).astype(np.int8)
    ws = gu.workspace(cdl.huffman_workspace_bytes(n))
    out = _outputs()
    for fill in (255, 0):
        ws.fill_(fill)
        _call(gu.dev(idx), ws, out)
        torch.cuda.synchronize()
        r_counts, r_total, _ = oracle.huffman_bits(idx, -128, 256)
        assert np.array_equal(out[0].cpu().numpy(), np.asarray(r_counts).astype(np.int64)) and int(out[1].item()) == int(r_total)


def test_replays():
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    n = 800_001
    idx = torch.zeros(n, dtype=torch.int8, device="cuda")
    ws, out = gu.workspace(cdl.huffman_workspace_bytes(n)), _outputs()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        _call(idx, ws, out)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _call(idx, ws, out)
    for rep in range(4):
        if rep != 2:
            idx.copy_((torch.randn(n, device="cuda") * (3.0 + 20.0 * rep)).clamp(-128, 127).to(torch.int8))
        _call(idx, ws, out)
        torch.cuda.synchronize()
        want = [t.cpu().numpy().copy() for t in out]
        for t in out:
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(np.array_equal(t.cpu().numpy(), w) for t, w in zip(out, want))
