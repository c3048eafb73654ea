"""GPU backward products of 33 to 64 output channels in long layers of few columns, whose activation gradient is formed in double: the diagnostic words tell the limb counts and bounds of the limb rule all the
same, for the activation gradient alone, together with the weight gradient (directly, in pieces and on limbs) and in the call that also takes the quantizers' backward passes; on both sides of 2^25 multiply-adds
and of the lines on rows and columns; dirty workspaces, replays."""
import numpy as np
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu

STEP_A, STEP_B = 0.5, 0.25


def _inputs(M, N, K, scale):
    torch = gu.torch_mod()
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    g = torch.randn(M, N, device="cuda", generator=gen) * scale
    g[M // 3, N - 1] = -7.5 * scale
    a = torch.randint(-128, 128, (M, K), dtype=torch.int8, device="cuda", generator=gen)
    b = torch.randint(-20, 21, (N, K), dtype=torch.int8, device="cuda", generator=gen)
    b[:, K - 1] = -128      # (the last column has the largest sum)
    return g, a, b


def _words(ws):
    torch = gu.torch_mod()
    return ws[:8].view(torch.int32).tolist(), ws[32:48].view(torch.float64).tolist()


def _rule(g, step, idx):
    torch = gu.torch_mod()
    e = int(np.frexp(np.float32(float(g.abs().max()) * np.float32(1.01)))[1])
    unit = step * float(idx.double().abs().sum(0).max())
    limbs = next((c for c in range(3, 7) if unit * 2.0 ** (e - 8 * c) <= 9e-7), 6)
    return limbs, unit * 2.0 ** (e - 8 * limbs)


@pytest.mark.parametrize("M,N,K", [(65536, 64, 32), (65536, 33, 16), (65541, 48, 31), (65536, 47, 64), (65537, 48, 63), (65536, 64, 9), (65535, 64, 32), (65536, 49, 33), (400_003, 64, 32), (1_400_000, 33, 32)])
@pytest.mark.parametrize("want", ["a", "both"])
@pytest.mark.parametrize("scale,offsets", [(1.0, (0, 0)), (2.0 ** 14, (0, 128))])
def test_words(M, N, K, want, scale, offsets):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    g, a, b = _inputs(M, N, K, scale)
    da, db = torch.empty(M, K, device="cuda"), torch.empty(N, K, device="cuda")
    ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    for fill in (255, 0, 0x5a):
        ws.fill_(fill)
        cdl.cdl_qgemm_bwd_offset(g, a, b, M, N, K, STEP_A, STEP_B, *offsets, da, db if want == "both" else None, ws)
        torch.cuda.synchronize()
        limbs, bounds = _words(ws)
        if M * N * K <= 1 << 25:
            assert limbs == [0, 0] and bounds == [0.0, 0.0]
            continue
        assert (limbs[0], bounds[0]) == _rule(g, STEP_B, b)
        if want == "both":
            assert (limbs[1], bounds[1]) == _rule(g, STEP_A, a)
    ref, mag = STEP_B * (g.double() @ (b.double() + offsets[1])), STEP_B * (g.double().abs() @ (b.double() + offsets[1]).abs())
    # one rounding to fp32 (2^-24 of the result), sums in double
    assert bool(((da.double() - ref).abs() <= 2.0 ** -23 * ref.abs() + 2.0 ** -40 * mag).all())


def test_words_of_the_call_with_the_quantizers():
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    M, N, K = 65536, 64, 32
    g, a, b = _inputs(M, N, K, 1.0)
    theta = a.float() * STEP_A
    dx, ds, dal = torch.empty(M, K, device="cuda"), gu.empty((1,), torch.float32), gu.empty((1,), torch.float32)
    ws = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K))
    ws.fill_(255)
    cdl.cdl_qgemm_bwd_quantize_bwd(g, a, b, M, N, K, theta, -128, 256, STEP_A, 4.0 / STEP_A ** 2, STEP_B, dx, ds, dal, None, ws)
    torch.cuda.synchronize()
    limbs, bounds = _words(ws)
    assert (limbs[0], bounds[0]) == _rule(g, STEP_B, b)


def test_replays():
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    M, N, K = 131072, 64, 9
    g, a, b = _inputs(M, N, K, 1.0)
    da = torch.empty(M, K, device="cuda")
    ws, words = gu.workspace(cdl.qgemm_bwd_workspace_bytes(M, N, K)), torch.zeros(48, dtype=torch.uint8, device="cuda")

    def run():
        cdl.cdl_qgemm_bwd(g, a, b, M, N, K, STEP_A, STEP_B, da, None, ws)
        words.copy_(ws[:48])

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for rep in range(4):
        if rep != 2:
            g.mul_(16.0)
        words.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        limbs, bounds = _words(words)
        assert (limbs[0], bounds[0]) == _rule(g, STEP_B, b)
