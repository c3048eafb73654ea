"""Host-side checks of the C boundary that need no GPU: the library loads, exports every symbol the
header declares, sizes its workspaces sensibly and rejects bad arguments before touching the device."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def cdl():
    import paper_2501_09849_amd as pkg
    import paper_2501_09849_amd.build as b
    if not os.path.exists(b.LIB_PATH):
        b.build_lib()
    pkg.load()
    return pkg


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "cdl.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(cdl_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_entry_point(cdl):
    lib = cdl.load()
    declared = _declared_functions()
    assert {"cdl_quantize_fwd", "cdl_quantize_bwd", "cdl_marginal_entropy", "cdl_qgemm_fwd", "cdl_qgemm_bwd"} <= set(declared)
    for name in declared:
        assert hasattr(lib, name), name
    assert sorted(cdl.EXPORTS) == declared
    assert lib.cdl_version() >= 100
    assert lib.cdl_status_string(0) == b"ok" and lib.cdl_status_string(-3) != lib.cdl_status_string(-2)


def test_workspace_queries(cdl):
    assert cdl.quantize_workspace_bytes(0, 15) > 0
    assert cdl.quantize_workspace_bytes(10**9, 255) >= cdl.quantize_workspace_bytes(10, 15)
    assert cdl.quantize_workspace_bytes(10, 1) == 0 and cdl.quantize_workspace_bytes(-1, 15) == 0
    assert cdl.qgemm_fwd_workspace_bytes(64, 64, 64) == 0
    assert cdl.qgemm_fwd_workspace_bytes(64, 64, 70) >= (64 + 64) * 80
    small, big = cdl.qgemm_bwd_workspace_bytes(32, 128, 256), cdl.qgemm_bwd_workspace_bytes(65536, 3072, 768)
    assert 0 < small < big
    assert cdl.qgemm_bwd_workspace_bytes(0, 3, 4) == 0


def _q(lo, n, delta, alpha, top_k=0):
    from paper_2501_09849_amd.binding import QParams
    return ctypes.byref(QParams(lo, n, delta, alpha, top_k))


OK, NULL, PARAM, RANGE, ALIGN, WS = 0, -1, -2, -3, -4, -5
FAKE = 0x1000   # a well-aligned non-NULL address that is never dereferenced: every call below must fail first


def test_quantizer_argument_validation_happens_before_any_gpu_work(cdl):
    lib = cdl.load()
    good = _q(-7, 15, 0.02, 1e4)
    f = lib.cdl_quantize_fwd
    assert f(FAKE, 16, None, FAKE, None, None, None, None, 0, None) == NULL
    assert f(FAKE, 16, _q(-7, 1, 0.02, 1e4), FAKE, None, None, None, None, 0, None) == PARAM
    assert f(FAKE, 16, _q(-7, 15, 0.0, 1e4), FAKE, None, None, None, None, 0, None) == PARAM
    assert f(FAKE, 16, _q(-7, 15, 0.02, -1.0), FAKE, None, None, None, None, 0, None) == PARAM
    assert f(FAKE, 16, _q(-7, 15, float("nan"), 1.0), FAKE, None, None, None, None, 0, None) == PARAM
    assert f(FAKE, 16, _q(-7, 15, 0.02, float("inf")), FAKE, None, None, None, None, 0, None) == PARAM
    assert f(FAKE, 16, _q(0, 257, 0.02, 1e4), FAKE, None, None, None, None, 0, None) == RANGE    # beyond the unsigned 8-bit set
    assert f(FAKE, 16, _q(-5, 140, 0.02, 1e4), FAKE, None, None, None, None, 0, None) == RANGE   # inside neither [-128,127] nor [0,255]
    assert f(FAKE, 16, _q(-129, 4, 0.02, 1e4), FAKE, None, None, None, None, 0, None) == RANGE
    # the offset a level set is stored with: 0 inside [-128, 127], 128 for sets that reach beyond 127
    assert lib.cdl_index_offset(_q(-128, 256, 0.02, 1e4)) == 0 and lib.cdl_index_offset(_q(0, 128, 0.02, 1e4)) == 0
    assert lib.cdl_index_offset(_q(0, 256, 0.02, 1e4)) == 128 and lib.cdl_index_offset(_q(100, 29, 0.02, 1e4)) == 128
    assert lib.cdl_index_offset(_q(-1, 130, 0.02, 1e4)) == RANGE and lib.cdl_index_offset(None) == NULL
    assert f(FAKE, -1, good, FAKE, None, None, None, None, 0, None) == PARAM
    assert f(None, 16, good, FAKE, None, None, None, None, 0, None) == NULL
    assert f(FAKE, 16, good, None, None, None, None, None, 0, None) == NULL
    assert f(FAKE + 4, 16, good, FAKE, None, None, None, None, 0, None) == ALIGN
    assert f(FAKE, 16, good, FAKE + 1, None, None, None, None, 0, None) == ALIGN
    assert f(FAKE, 16, good, FAKE, FAKE + 8, None, None, None, 0, None) == ALIGN
    assert f(FAKE, 16, good, FAKE, None, FAKE, None, None, 0, None) == WS                       # marginal needs scratch
    assert f(FAKE, 16, good, FAKE, None, FAKE, None, FAKE, 16, None) == WS
    need = cdl.quantize_workspace_bytes(16, 15)
    assert f(FAKE, 16, good, FAKE, None, FAKE, None, FAKE + 64, need, None) == ALIGN
    b = lib.cdl_quantize_bwd
    assert b(FAKE, FAKE, 16, good, None, None, None, None, 0, None) == NULL                     # no output requested
    assert b(FAKE, None, 16, good, FAKE, None, None, None, 0, None) == NULL
    assert b(FAKE, FAKE, 16, good, FAKE, FAKE, None, None, 0, None) == WS
    assert b(FAKE, FAKE + 8, 16, good, FAKE, None, None, None, 0, None) == ALIGN
    m = lib.cdl_marginal_entropy
    assert m(FAKE, 16, good, None, None, FAKE, need, None) == NULL
    assert m(FAKE, 16, good, FAKE, None, None, 0, None) == WS


def test_extension_argument_validation_happens_before_any_gpu_work(cdl):
    lib = cdl.load()
    good = _q(-7, 15, 0.02, 1e4)
    for k in (2, 4, 10, 11, -1):
        bad = _q(0, 16, 0.25, 64.0, top_k=k)
        assert lib.cdl_quantize_fwd(FAKE, 16, bad, FAKE, None, None, None, None, 0, None) == PARAM
    d = lib.cdl_quantize_draw
    assert d(FAKE, FAKE, 16, None, FAKE, None) == NULL
    assert d(FAKE, None, 16, good, FAKE, None) == NULL
    assert d(FAKE, FAKE, 16, good, None, None) == NULL
    assert d(FAKE, FAKE, -2, good, FAKE, None) == PARAM
    assert d(FAKE, FAKE + 4, 16, good, FAKE, None) == ALIGN
    assert d(FAKE, FAKE, 16, good, FAKE + 2, None) == ALIGN
    h = lib.cdl_huffman_bits
    assert h(FAKE, 16, 0, 16, None, None, None, FAKE, 4096, None) == NULL                       # no output requested
    assert h(None, 16, 0, 16, FAKE, None, None, FAKE, 4096, None) == NULL
    assert h(FAKE, -1, 0, 16, FAKE, None, None, FAKE, 4096, None) == PARAM
    assert h(FAKE, 16, 0, 257, FAKE, None, None, FAKE, 4096, None) == RANGE
    assert h(FAKE + 8, 16, 0, 16, FAKE, None, None, FAKE, 4096, None) == ALIGN
    assert h(FAKE, 16, 0, 16, FAKE, None, None, None, 0, None) == WS
    assert cdl.huffman_workspace_bytes(0) > 0 and cdl.huffman_workspace_bytes(10**9) >= cdl.huffman_workspace_bytes(100)
    e = lib.cdl_entropy_bwd
    assert e(FAKE, FAKE, None, 16, good, 1.0, None, None, None, None, 0, None) == NULL          # no output requested
    assert e(FAKE, None, None, 16, good, 1.0, FAKE, None, None, None, 0, None) == NULL
    assert e(None, FAKE, None, 16, good, 1.0, FAKE, None, None, None, 0, None) == NULL
    assert e(FAKE, FAKE, None, 16, good, float("nan"), FAKE, None, None, None, 0, None) == PARAM
    assert e(FAKE, FAKE, FAKE + 4, 16, good, 1.0, FAKE, None, None, None, 0, None) == ALIGN
    assert e(FAKE, FAKE, None, 16, good, 1.0, FAKE, FAKE, None, None, 0, None) == WS            # scalar outputs need scratch


def test_gemm_argument_validation_happens_before_any_gpu_work(cdl):
    lib = cdl.load()
    f = lib.cdl_qgemm_fwd
    assert f(FAKE, FAKE, -1, 4, 4, 1.0, 1.0, FAKE, None, None, 0, None) == PARAM
    assert f(FAKE, FAKE, 4, 4, 16, 0.0, 1.0, FAKE, None, None, 0, None) == PARAM
    assert f(FAKE, FAKE, 4, 4, 16, 1.0, float("nan"), FAKE, None, None, 0, None) == PARAM
    assert f(FAKE, FAKE, 4, 4, 16, 1.0, 1.0, None, None, None, 0, None) == NULL
    assert f(None, FAKE, 4, 4, 16, 1.0, 1.0, FAKE, None, None, 0, None) == NULL
    assert f(FAKE, FAKE, 4, 4, 131072, 1.0, 1.0, FAKE, None, None, 0, None) == RANGE             # int32 could overflow
    assert f(FAKE + 4, FAKE, 4, 4, 16, 1.0, 1.0, FAKE, None, None, 0, None) == ALIGN
    assert f(FAKE, FAKE, 4, 4, 20, 1.0, 1.0, FAKE, None, None, 0, None) == WS                    # ragged K needs staging
    b = lib.cdl_qgemm_bwd
    assert b(FAKE, FAKE, FAKE, 4, 4, 16, 1.0, 1.0, None, None, None, 0, None) == NULL
    assert b(None, FAKE, FAKE, 4, 4, 16, 1.0, 1.0, FAKE, FAKE, None, 0, None) == NULL
    assert b(FAKE, FAKE, FAKE, 4, 4, 16, 1.0, 1.0, FAKE, FAKE, None, 0, None) == WS
    assert b(FAKE, FAKE, FAKE, 4, 131072, 16, 1.0, 1.0, FAKE, None, None, 0, None) == RANGE      # contraction over N, int32
    assert b(FAKE, FAKE, FAKE, 262145, 4, 16, 1.0, 1.0, None, FAKE, None, 0, None) == WS         # contraction over M is cut up
    assert b(FAKE, FAKE, FAKE, 11000001, 4, 16, 1.0, 1.0, None, FAKE, None, 0, None) == RANGE    # 32-bit offsets inside
    assert lib.cdl_profile_collect(None, 4) == PARAM


def test_layer_entry_points_validate_before_any_gpu_work(cdl):
    lib = cdl.load()
    good = _q(0, 16, 0.25, 64.0)
    # the convolution: geometry, channel multiple, offsets, contraction length, pointers, workspace with an offset
    c = lib.cdl_qconv_fwd
    ok = dict(B=1, H=8, W=8, C=16, N=4, R=3, S=3, stride=1, pad=1)
    def conv(x=FAKE, w=FAKE, acc=FAKE, y=None, off=0, ws=None, ws_bytes=0, **kw):
        g = dict(ok, **kw)
        return c(x, w, g["B"], g["H"], g["W"], g["C"], g["N"], g["R"], g["S"], g["stride"], g["pad"], 0.1, 0.1, off, acc, y, ws, ws_bytes, None)
    assert conv(C=3) == PARAM and conv(C=24) == PARAM
    assert conv(pad=3) == PARAM and conv(stride=0) == PARAM and conv(H=1, W=1, R=5, S=5, pad=1) == PARAM
    assert conv(off=64) == PARAM
    assert conv(C=4096) == RANGE                              # contraction beyond the tap table
    assert conv(acc=None) == NULL and conv(x=None) == NULL
    assert conv(x=FAKE + 8) == ALIGN
    assert conv(off=128) == WS
    assert lib.cdl_qconv_fwd_workspace_bytes(64, 0) == 0 and lib.cdl_qconv_fwd_workspace_bytes(64, 128) >= 256 + 64 * 4
    # the forward product with the quantizer in its prologue
    f = lib.cdl_qgemm_fwd_quantize
    assert f(FAKE, None, FAKE, 4, 4, 128, 0.1, FAKE, None) == NULL
    assert f(FAKE, good, FAKE, 4, 4, 100, 0.1, FAKE, None) == PARAM            # whole K-tiles only
    assert f(FAKE, _q(0, 256, 0.25, 64.0), FAKE, 4, 4, 128, 0.1, FAKE, None) == PARAM   # indices stored with an offset
    assert f(FAKE, good, FAKE, 4, 4, 131072, 0.1, FAKE, None) == RANGE
    assert f(FAKE, good, None, 4, 4, 128, 0.1, FAKE, None) == NULL
    assert f(FAKE + 4, good, FAKE, 4, 4, 128, 0.1, FAKE, None) == ALIGN
    # the backward step in one call
    b = lib.cdl_qgemm_bwd_quantize_bwd
    def bwd(M=64, N=64, K=64, theta_a=FAKE, d_theta_a=FAKE, delta_b=0.25, b_off=0, theta_b=None, p_b=None, d_theta_b=None, ws=None, ws_bytes=0):
        return b(FAKE, FAKE, FAKE, M, N, K, theta_a, good, delta_b, b_off, d_theta_a, None, None, None, theta_b, p_b, d_theta_b, None, None,
                 ws, ws_bytes, None)
    assert bwd(K=62) == PARAM and bwd(N=32) == PARAM and bwd(M=0) == PARAM
    assert bwd(d_theta_a=None) == NULL
    assert bwd(theta_b=FAKE, p_b=good) == NULL                                   # no place for dL/dtheta of the weights
    assert bwd(theta_b=FAKE, p_b=_q(0, 16, 0.3, 64.0), d_theta_b=FAKE) == PARAM  # not the step the product was told
    assert bwd(theta_b=FAKE, p_b=good, d_theta_b=FAKE, b_off=128) == PARAM       # not the storage offset of that quantizer
    assert bwd(theta_b=FAKE, p_b=good, d_theta_b=FAKE) == WS
    assert bwd() == WS
    # the two gradients of the convolution
    cw, ca = lib.cdl_qconv_bwd_weights, lib.cdl_qconv_bwd_activations
    def wgrad(g=FAKE, x=FAKE, out=FAKE, C=16, pad=1, off=0, ws=None, ws_bytes=0, B=1):
        return cw(g, x, B, 8, 8, C, 4, 3, 3, 1, pad, 0.1, off, out, ws, ws_bytes, None)
    assert wgrad(C=8) == PARAM and wgrad(pad=3) == PARAM and wgrad(off=5) == PARAM and wgrad(B=0) == PARAM
    assert wgrad(out=None) == NULL and wgrad(g=FAKE + 4) == ALIGN and wgrad() == WS
    assert lib.cdl_qconv_bwd_weights_workspace_bytes(1, 8, 8, 16, 4, 3, 3, 1, 1) > 64 * 144
    def xgrad(g=FAKE, w=FAKE, out=FAKE, N=128, stride=1, pad=1, C=16, ws=None, ws_bytes=0):
        return ca(g, w, 1, 8, 8, C, N, 3, 3, stride, pad, 0.1, out, ws, ws_bytes, None)
    assert xgrad(N=6) == PARAM and xgrad(stride=3) == PARAM and xgrad(pad=3) == PARAM and xgrad(C=6) == PARAM
    assert xgrad(N=16384) == RANGE
    assert xgrad(w=None) == NULL and xgrad(out=FAKE + 8) == ALIGN and xgrad() == WS
    assert lib.cdl_qconv_bwd_activations_workspace_bytes(1, 8, 8, 16, 128, 3, 3, 1, 1) >= 16 * 9 * 128
    assert lib.cdl_qconv_bwd_activations_workspace_bytes(1, 8, 8, 16, 6, 3, 3, 1, 1) == 0
    assert lib.cdl_profile_only(None) == OK and lib.cdl_profile_only(b"limb_gemm_kernel(d_b_hat)") == OK and lib.cdl_profile_only(b"") == OK


def test_binding_fails_loudly_without_the_library(monkeypatch):
    import paper_2501_09849_amd.binding as binding
    monkeypatch.setattr(binding, "_LIB", None)
    monkeypatch.setattr(binding, "_LIB_PATH", "/nonexistent/libcdl.so")
    with pytest.raises(RuntimeError, match="not built"):
        binding.load()


def test_window_rule_matches_the_documented_bound():
    """Levels beyond the band must carry less than 3e-9 (times m^3) of the weight of the nearest level."""
    import math
    for kappa, want in ((1e4, 1), (30.0, 1), (11.0, 1), (10.8, 2), (4.0, 2), (3.8, 3), (2.0, 3), (1.9, 4), (1.3, 4)):
        W = 1
        while True:
            m = W + 1
            if kappa * m * (m - 1) > 19.6 + 3 * math.log(m):
                break
            W += 1
        assert W == want, (kappa, W, want)
        m = W + 1
        assert m ** 3 * math.exp(-kappa * m * (m - 1)) < 3.1e-9


def test_a_stale_binary_is_detected_by_content(monkeypatch):
    """The loader refuses a libcdl.so that was not built from the sources in the tree: the check hashes file
    contents and compiler flags, so it survives a copy of the tree that resets every time stamp."""
    import paper_2501_09849_amd.build as b
    assert not b.is_stale(), "the library in the tree must have been built from the tree's sources (run the build)"
    h = b.source_hash()
    assert h == b.source_hash()
    monkeypatch.setattr(b, "HIPCC_FLAGS", b.HIPCC_FLAGS + ["-DSOMETHING_ELSE"])
    assert b.source_hash() != h and b.is_stale()


def test_activation_gradient_asks_for_digit_planes_only_where_they_are_made(cdl):
    """Six bytes per entry of g for the limb product; small layers (in double) and 1 x 1 kernels (a linear layer) have no planes."""
    f = cdl.qconv_bwd_activations_workspace_bytes
    planes = 6 * 256 * 14 * 14 * 256
    assert planes < f(256, 14, 14, 256, 256, 3, 3, 1, 1) < planes + 2 * 9 * 256 * 256 + (1 << 20)
    assert f(128, 32, 32, 16, 16, 3, 3, 1, 1) < 1 << 20        # 131072 x 16 outputs: six bytes each would be 12.6 MB
    assert f(4096, 32, 32, 16, 16, 3, 3, 1, 1) < 1 << 20       # any number of pixels where a limb tile would be padding
    assert f(128, 32, 32, 16, 16, 3, 3, 2, 1) < 1 << 20
    assert f(64, 56, 56, 64, 256, 1, 1, 1, 0) == cdl.qgemm_bwd_workspace_bytes(64 * 56 * 56, 256, 64)
    assert f(64, 56, 56, 64, 256, 1, 1, 2, 0) > 6 * 64 * 28 * 28 * 256      # stride 2: the limb product


def test_combined_backward_call_refuses_outputs_over_its_inputs(cdl):
    """d_theta_a holds dL/dQ(a) before theta_a is read: in place it would be wrong without a word.  (What is allowed is called
    without a workspace and ends at that check, so nothing is ever launched.)"""
    f = cdl.load().cdl_qgemm_bwd_quantize_bwd
    M, N, K = 128, 64, 256
    qa, qb = _q(0, 16, 0.25, 64.0), _q(-7, 15, 0.02, 1e4)
    G, XI, WI, X, W, DX, DW, DWH = (FAKE + (i << 20) for i in range(8))

    def call(x=X, w=W, dx=DX, dw=DW, dwh=DWH):
        return f(G, XI, WI, M, N, K, x, qa, 0.02, 0, dx, None, None, dwh, w, qb, dw, None, None, *ws, None)

    ws = (None, 0)
    assert call() == WS and call(dwh=None) == WS and call(dwh=DW) == WS
    assert call(dx=X + 4 * M * K) == WS and call(dx=X - 4 * M * K) == WS
    ws = (FAKE + (8 << 20), 1 << 40)
    assert call(dx=X) == PARAM and call(dx=X + 64) == PARAM and call(dx=X - 4 * M * K + 64) == PARAM
    assert call(dw=W) == PARAM and call(dw=W, dwh=None) == PARAM and call(dwh=W) == PARAM
    assert call(dx=W) == PARAM and call(dw=X) == PARAM and call(dwh=X) == PARAM
