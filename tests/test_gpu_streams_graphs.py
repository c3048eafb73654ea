"""The library only enqueues kernels on the stream it is given: no allocation, no memset, no synchronisation,
and every counter a kernel uses is reset by the kernels themselves.  Two consequences are checked here on a
whole layer step (quantizer forward on W and X, the three index products, quantizer backward on X and W):
the step gives bit-identical results on a side stream, and it can be captured into a HIP graph whose
replays - with other work and fresh inputs in between - give what the eager calls give.
"""
import numpy as np
import pytest

import cdl_inputs
import gpu_util as gu

pytestmark = pytest.mark.gpu

M, N, K = 700, 300, 260          # several tiles, ragged in every dimension, K not a multiple of 16
W_SPEC = (-7, 15, 0.02, 1.0e4)   # lo, n_levels, delta, alpha
X_SPEC = (0, 16, 0.25, 64.0)


class Layer:
    def __init__(self, seed):
        import paper_2501_09849_amd as cdl
        torch = gu.torch_mod()
        self.cdl, self.torch = cdl, torch
        rng = np.random.default_rng(seed)
        f32, i8 = torch.float32, torch.int8
        self.W = gu.dev((rng.standard_normal((N, K)) * 0.05).astype(np.float32))
        self.X = gu.dev(np.abs(rng.standard_normal((M, K))).astype(np.float32))
        self.G = gu.dev(rng.standard_normal((M, N)).astype(np.float32))
        self.out = {
            "Wi": gu.empty(N * K, i8), "Xi": gu.empty(M * K, i8),
            "Wsoft": gu.empty(N * K, f32), "Xsoft": gu.empty(M * K, f32),
            "margW": gu.empty(W_SPEC[1], f32), "margX": gu.empty(X_SPEC[1], f32),
            "scal": gu.empty(8, f32),
            "Y": gu.empty((M, N), f32), "acc": gu.empty((M, N), torch.int32),
            "dXh": gu.empty((M, K), f32), "dWh": gu.empty((N, K), f32),
            "dX": gu.empty(M * K, f32), "dW": gu.empty(N * K, f32),
        }
        need = max(cdl.quantize_workspace_bytes(M * K, 16), cdl.quantize_workspace_bytes(N * K, 15),
                   cdl.qgemm_fwd_workspace_bytes(M, N, K), cdl.qgemm_bwd_workspace_bytes(M, N, K))
        self.ws = gu.workspace(need)

    def run(self):
        cdl, o, s = self.cdl, self.out, self.out["scal"]
        cdl.cdl_quantize_fwd(self.W, N * K, *W_SPEC, o["Wi"], o["Wsoft"], o["margW"], s[0:1], self.ws)
        cdl.cdl_quantize_fwd(self.X, M * K, *X_SPEC, o["Xi"], o["Xsoft"], o["margX"], s[1:2], self.ws)
        cdl.cdl_qgemm_fwd(o["Xi"], o["Wi"], M, N, K, X_SPEC[2], W_SPEC[2], o["acc"], o["Y"], self.ws)
        cdl.cdl_qgemm_bwd(self.G, o["Xi"], o["Wi"], M, N, K, X_SPEC[2], W_SPEC[2], o["dXh"], o["dWh"], self.ws)
        cdl.cdl_quantize_bwd(self.X, o["dXh"], M * K, *X_SPEC, o["dX"], s[4:5], s[5:6], self.ws)
        cdl.cdl_quantize_bwd(self.W, o["dWh"], N * K, *W_SPEC, o["dW"], s[2:3], s[3:4], self.ws)

    def scramble(self):
        """Other work on the same buffers between runs: every output is overwritten with junk."""
        for name, t in self.out.items():
            if t.dtype.is_floating_point:
                t.fill_(float("nan"))
            else:
                t.fill_(77)
        self.out["scal"].zero_()

    def results(self):
        self.torch.cuda.synchronize()
        return {k: v.detach().cpu().numpy().copy() for k, v in self.out.items()}


def same(a, b):
    for k in a:
        x, y = a[k], b[k]
        if k == "scal":
            x, y = x[:6], y[:6]
        assert np.array_equal(x, y, equal_nan=False), k


def test_step_on_a_side_stream_is_bit_identical():
    torch = gu.torch_mod()
    layer = Layer(seed=5)
    layer.scramble()
    layer.run()
    want = layer.results()
    side = torch.cuda.Stream()
    layer.scramble()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        layer.run()
    side.synchronize()
    same(layer.results(), want)


def test_step_replayed_from_a_graph_matches_eager_every_time():
    torch = gu.torch_mod()
    layer = Layer(seed=6)
    # warm-up on a side stream, then capture
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        layer.run()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer.run()
    rng = np.random.default_rng(9)
    for rep in range(4):
        if rep:
            # fresh inputs in the same buffers: the graph must read them, and size the limbs from them again
            layer.X.copy_(gu.dev(np.abs(rng.standard_normal((M, K))).astype(np.float32)))
            layer.G.copy_(gu.dev((rng.standard_normal((M, N)) * 10.0 ** rep).astype(np.float32)))
        layer.scramble()
        layer.run()
        want = layer.results()
        layer.scramble()
        torch.cuda.synchronize()
        graph.replay()
        same(layer.results(), want)


def _replayed(run, outputs, refresh, replays=4):
    """Captures run(), and for each replay - fresh inputs, junk in the outputs, eager work in between - compares every output with what
    the eager call gives."""
    torch = gu.torch_mod()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()

    def junk():
        for t in outputs:
            t.fill_(float("nan") if t.dtype.is_floating_point else 77)
    for rep in range(replays):
        if rep != 1:
            refresh(rep)
        junk()
        run()
        torch.cuda.synchronize()
        want = [t.clone() for t in outputs]
        junk()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for i, (t, w) in enumerate(zip(outputs, want)):
            assert torch.equal(t, w), (rep, i)


@pytest.mark.parametrize("n,levels,kappa", [((5 << 23) // 15 + 3, 31, 0.008), ((5 << 23) // 7 + 1, 15, 0.5), (70_001, 63, 0.05), (300_000, 255, 0.02),
                                            (40_001, 31, 0.008), (900_000, 31, 0.008)])
def test_soft_regime_replayed_from_a_graph(n, levels, kappa):
    """The table, its moments and the sums of the scalar gradients: kernels of cdl_soft.hip on both sides of the sizes that they serve."""
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    spec = (-(levels // 2), levels, 0.01, kappa / 0.01 ** 2)
    theta, g = gu.empty(n, torch.float32), gu.empty(n, torch.float32)
    idx, soft, dth = gu.empty(n, torch.int8), gu.empty(n, torch.float32), gu.empty(n, torch.float32)
    marg, only, sc = gu.empty(levels, torch.float32), gu.empty(levels, torch.float32), gu.empty(8, torch.float32)
    ws = gu.workspace(cdl.quantize_workspace_bytes(n, levels))

    def run():
        cdl.cdl_quantize_fwd(theta, n, *spec, idx, soft, marg, sc[0:1], ws)
        cdl.cdl_quantize_bwd(theta, g, n, *spec, dth, sc[1:2], sc[2:3], ws)
        cdl.cdl_marginal_entropy(theta, n, *spec, only, sc[3:4], ws)
        sc[4:].zero_()

    def refresh(rep):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(rep)
        theta.copy_(torch.randn(n, device="cuda", generator=gen) * (0.002 * levels * (1 + rep)))
        g.copy_(torch.randn(n, device="cuda", generator=gen))
    refresh(9)
    _replayed(run, [idx, soft, marg, dth, only, sc], refresh)


@pytest.mark.parametrize("n,levels", [(3000, 15), (200_000, 255), (2_359_296, 255)])
def test_huffman_size_replayed_from_a_graph(n, levels):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    idx = gu.empty(n, torch.int8)
    counts, bits, rate = gu.empty(levels, torch.int64), gu.empty(1, torch.int64), gu.empty(1, torch.float32)
    ws = gu.workspace(cdl.huffman_workspace_bytes(n))

    def refresh(rep):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(rep)
        half = levels // 2
        idx.copy_((torch.randn(n, device="cuda", generator=gen) * half / (2 + rep)).clamp(-half, half).to(torch.int8))
    refresh(9)
    _replayed(lambda: cdl.cdl_huffman_bits(idx, n, -(levels // 2), levels, counts, bits, rate, ws), [counts, bits, rate], refresh)


# limb products with the plan made at the end of the transpositions, one and several pieces of the contraction; direct products whose
# last block fills the diagnostic words; direct products of a few outputs each
@pytest.mark.parametrize("M,N,K", [(2048, 640, 1024), (60000, 96, 144), (256, 1000, 512), (32, 128, 256), (131072, 16, 144)])
@pytest.mark.parametrize("offset", [0, 128])
def test_backward_products_replayed_from_a_graph(M, N, K, offset):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    g = gu.empty((M, N), torch.float32)
    a, b = gu.empty((M, K), torch.int8), gu.empty((N, K), torch.int8)
    da, db = gu.empty((M, K), torch.float32), gu.empty((N, K), torch.float32)
    ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    words = gu.empty(2, torch.int32)

    def run():
        cdl.cdl_qgemm_bwd_offset(g, a, b, M, N, K, 0.25, 0.02, offset, 0, da, db, ws)
        words.copy_(ws[:8].view(torch.int32))

    def refresh(rep):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(rep)
        g.copy_(torch.randn((M, N), device="cuda", generator=gen) * 10.0 ** (rep % 5))
        a.copy_(torch.randint(-128, 128, (M, K), device="cuda", generator=gen))
        b.copy_(torch.randint(-7, 8, (N, K), device="cuda", generator=gen))
    refresh(9)
    _replayed(run, [da, db, words], refresh)


# digit planes at stride 1 and 2, the direct product, a linear layer
@pytest.mark.parametrize("B,H,W,C,N,R,stride", [(16, 14, 14, 256, 256, 3, 1), (16, 28, 29, 64, 128, 3, 2), (32, 32, 32, 16, 16, 3, 1), (16, 28, 28, 128, 64, 1, 1)])
def test_convolution_gradients_replayed_from_a_graph(B, H, W, C, N, R, stride):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    pad = R // 2
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    geom = (B, H, W, C, N, R, R, stride, pad)
    g, x, w = gu.empty((B, P, Q, N), torch.float32), gu.empty((B, H, W, C), torch.int8), gu.empty((N, R, R, C), torch.int8)
    y, dx, dw = gu.empty((B, P, Q, N), torch.float32), gu.empty((B, H, W, C), torch.float32), gu.empty((N, R, R, C), torch.float32)
    ws = gu.workspace(max(cdl.qconv_fwd_workspace_bytes(N, 0), cdl.qconv_bwd_weights_workspace_bytes(*geom), cdl.qconv_bwd_activations_workspace_bytes(*geom)))

    def run():
        cdl.cdl_qconv_fwd(x, w, *geom, 0.25, 0.02, None, y, ws)
        cdl.cdl_qconv_bwd_weights(g, x, *geom, 0.25, dw, ws)
        cdl.cdl_qconv_bwd_activations(g, w, *geom, 0.02, dx, ws)

    def refresh(rep):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(rep)
        g.copy_(torch.randn(g.shape, device="cuda", generator=gen) * 10.0 ** (rep % 5))
        x.copy_(torch.randint(0, 16, x.shape, device="cuda", generator=gen))
        w.copy_(torch.randint(-7, 8, w.shape, device="cuda", generator=gen))
    refresh(9)
    _replayed(run, [y, dx, dw], refresh)
