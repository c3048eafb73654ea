"""GPU dispatch of the kernels for few channels and columns, by the names that the library's own profile records: one call on each side of their rules."""
import pytest

import gpu_util as gu

pytestmark = pytest.mark.gpu


def _recorded(call):
    import paper_2501_09849_amd as cdl
    gu.torch_mod().cuda.synchronize()
    cdl.cdl_profile_enable(True)
    try:
        call()
        return {name for name, _ in cdl.cdl_profile_collect()}
    finally:
        cdl.cdl_profile_enable(False)


def _i8(*shape):
    torch = gu.torch_mod()
    return torch.randint(-7, 8, shape, device="cuda", dtype=torch.int32).to(torch.int8)


@pytest.mark.parametrize("M,N,K,offsets,thin", [(40_000, 16, 144, (0, 0), True), (131_072, 20, 768, (0, 0), True), (70_000, 20, 448, (0, 0), True), (50_007, 16, 147, (0, 0), True), (36_001, 32, 50, (128, 0), True),
                                                (65_536, 16, 1040, (0, 0), True), (40_000, 22, 144, (128, 0), True), (40_000, 16, 144, (0, 128), False), (70_000, 20, 464, (0, 0), False),
                                                (40_000, 22, 144, (0, 0), False), (65_537, 16, 1040, (0, 0), True), (65_537, 16, 1680, (0, 0), False), (65_537, 8, 1680, (0, 0), True), (65_537, 8, 2064, (0, 0), False), (40_000, 16, 301, (0, 0), False), (40_000, 33, 144, (0, 0), False),
                                                (1000, 16, 144, (0, 0), False)])
def test_forward_product(M, N, K, offsets, thin):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    a, b, y = _i8(M, K), _i8(N, K), gu.empty((M, N), torch.float32)
    ws = gu.workspace(cdl.qgemm_fwd_offset_workspace_bytes(M, N, K))
    names = _recorded(lambda: cdl.cdl_qgemm_fwd_offset(a, b, M, N, K, 0.25, 0.5, *offsets, None, y, ws))
    assert ("fwd_thin_kernel" in names) == thin, names


# B, H, W, C, N, R, stride; the forward product and the activation gradient of the same layer
@pytest.mark.parametrize("case,forward,gradient", [((40, 32, 32, 16, 16, 3, 1), True, True), ((60, 25, 24, 32, 16, 5, 1), False, True), ((16, 32, 32, 16, 16, 3, 1), True, False), ((32, 32, 32, 16, 32, 3, 1), False, True), ((33, 32, 32, 32, 32, 3, 1), True, True),
                                                   ((64, 28, 28, 32, 32, 3, 2), False, False), ((40, 32, 32, 16, 36, 3, 1), False, False), ((64, 32, 32, 32, 16, 3, 1), True, True), ((63, 32, 32, 32, 16, 3, 1), True, False), ((130, 32, 32, 16, 8, 3, 1), True, True),
                                                   ((130, 32, 32, 32, 8, 3, 1), True, False), ((130, 32, 32, 16, 4, 3, 1), True, False), ((66, 32, 32, 16, 24, 3, 1), True, True), ((130, 32, 32, 32, 20, 3, 1), True, True), ((16, 72, 72, 32, 20, 3, 1), True, False), ((30, 72, 72, 16, 12, 3, 1), True, True), ((25, 72, 72, 16, 12, 3, 1), True, False),
                                                   ((20, 72, 72, 16, 32, 3, 1), True, False), ((26, 72, 72, 16, 32, 3, 1), True, True),
                                                   ((80, 32, 32, 32, 16, 5, 1), False, False), ((26, 56, 56, 32, 16, 5, 1), False, True), ((36, 31, 33, 32, 12, 5, 1), False, True), ((90, 14, 14, 48, 4, 1, 1), True, False)], ids=str)
def test_convolution(case, forward, gradient):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    B, H, W, C, N, R, stride = case
    pad = R // 2
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    geom = (B, H, W, C, N, R, R, stride, pad)
    x, w, y, dx = _i8(B, H, W, C), _i8(N, R, R, C), gu.empty((B, P, Q, N), torch.float32), gu.empty((B, H, W, C), torch.float32)
    g = torch.randn((B, P, Q, N), device="cuda")
    ws = gu.workspace(cdl.qconv_bwd_activations_workspace_bytes(*geom))
    assert ("fwd_thin_kernel(windows)" in _recorded(lambda: cdl.cdl_qconv_fwd(x, w, *geom, 0.25, 0.5, None, y, None))) == forward
    assert ("conv_dx_thin_kernel" in _recorded(lambda: cdl.cdl_qconv_bwd_activations(g, w, *geom, 0.125, dx, ws))) == gradient
