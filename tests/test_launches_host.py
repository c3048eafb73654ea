"""Which kernels a call launches and how, on both sides of the rules that choose them, without a GPU (launch_recorder.py)."""
import shutil

import pytest

import launch_recorder as lr
import ring_cases

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or shutil.which("c++filt") is None, reason="no host compiler")


def test_convolutions_with_an_offset_look_no_device_variable_up(tmp_path):
    """Their padding comes from the workspace, so that the first call on a GPU may be one that is captured into a graph; the header asks for a call before a capture only without an offset."""
    geoms = [(64, 28, 28, 48, 96, 3, 3, 1, 1), (128, 56, 56, 16, 64, 3, 3, 1, 1), (128, 28, 28, 128, 128, 3, 3, 1, 1), (53, 19, 53, 288, 412, 3, 3, 1, 1), (4, 9, 9, 16, 20, 3, 3, 1, 1)]
    seen = lr.record(tmp_path, [lr.conv_fwd(*g, x_offset=128) for g in geoms] + [lr.conv_fwd(*geoms[0]), lr.conv_fwd(*geoms[0])])
    assert [s[1] for s in seen] == [0] * len(geoms) + [1, 0]      # (without an offset once)
    assert any("ChunkSource" in l.name or ", true>(" in l.name for l in seen[0][0]), seen[0]


@pytest.mark.parametrize("form,products", [
    # up to 64 columns over few K-tiles: every form with direct loads is slower there; from eight K-tiles on, and with fewer rows than fill the chip from seventeen (64 columns: eight), faster
    ("staged", [(662125, 63, 128), (240573, 43, 128), (1254090, 46, 128), (147875, 36, 448), (203841, 43, 192), (23877, 38, 576), (16514, 64, 448), (454824, 64, 128)]),
    ("low", [(73034, 46, 512), (16514, 64, 960)]), ("narrow", [(1344058, 33, 512)]),
    # outputs beyond the memory-side cache over few K-tiles
    ("wide", [(252312, 1189, 64), (522648, 574, 64), (131072, 1024, 128), (131072, 1500, 192), (70000, 1024, 256)]),
    ("tall", [(100352, 128, 1152)]), ("square", [(60000, 128, 1152)])])
def test_forms_of_matrix_products(tmp_path, form, products):
    assert [(p, lr.tile_form(s[0])) for p, s in zip(products, lr.record(tmp_path, [lr.gemm_fwd(*p) for p in products]))] == [(p, form) for p in products]


@pytest.mark.parametrize("form,layers", [
    ("wide", [(370, 19, 22, 64, 460, 1, 1, 1, 0), (164, 99, 25, 128, 196, 1, 1, 1, 0), (256, 14, 14, 256, 256, 3, 3, 1, 1)]), ("narrow", [(128, 56, 56, 64, 64, 3, 3, 1, 1)]), ("tall", [(128, 28, 28, 128, 128, 3, 3, 1, 1)])])
def test_forms_of_layers(tmp_path, form, layers):
    assert [(g, lr.tile_form(s[0])) for g, s in zip(layers, lr.record(tmp_path, [lr.conv_fwd(*g) for g in layers]))] == [(g, form) for g in layers]


def _ring(launches):
    """form, stores past the caches, K-tiles across taps"""
    form = lr.tile_form(launches)
    flags = [l.name.split(">, ", 1)[1].split(">", 1)[0].split(", ") for l in launches if "dma_kernel" in l.name]
    return (form,) + tuple(f == "true" for f in flags[0]) if flags else (form,)


def test_cases_of_the_rings_take_the_forms_that_they_name(tmp_path):
    """Every form of matrices and of layers, of both kinds of K-tiles, and every one that stores past the caches, is among them."""
    seen = [_ring(s[0]) for s in lr.record(tmp_path, [lr.gemm_fwd(*c[0]) for c in ring_cases.MATRICES] + [lr.conv_fwd(*c[0]) for c in ring_cases.LAYERS])]
    matrices, layers = seen[:len(ring_cases.MATRICES)], seen[len(ring_cases.MATRICES):]
    assert matrices == [(form, stream) for _, form, stream in ring_cases.MATRICES]
    assert layers == [(form, stream, geom[3] % 64 != 0) for geom, form, stream in ring_cases.LAYERS]
    forms = {"wide", "tall", "narrow", "square", "low"}
    assert {m[0] for m in matrices} == forms and {m[0] for m in matrices if m[1]} == forms - {"low"}
    assert {(l[0], l[2]) for l in layers} == {(f, across) for f in forms for across in (False, True)}
    assert sum(shape[2] <= 192 and form == "wide" for shape, form, _ in ring_cases.MATRICES) >= 4


def _direct(launches):
    """Rows of the contraction that a wave of da_direct_kernel holds and how it stores (0: words, 1: scalars, 2, 3: through LDS in rows of whole words, of any length); None: another kernel."""
    names = [l.name for l in launches if "da_direct_kernel" in l.name]
    if not names:
        return None
    held, store = names[0].split("da_direct_kernel<", 1)[1].split(">", 1)[0].split(", ", 1)
    return int(held), int(store.rsplit(")", 1)[1])


def test_cases_of_the_activation_gradient_of_short_contractions(tmp_path):
    """test_gpu_da_direct.py: every way of storing for every length that has it, and both sides of the lines on outputs, rows, contraction and columns."""
    import test_gpu_da_direct as cases
    seen = dict(zip(cases.CASES, (_direct(s[0]) for s in lr.record(tmp_path, [lr.gemm_bwd(*c, "a") for c in cases.CASES]))))
    others = {(32767, 16, 64), (32767, 32, 33), (65535, 33, 32), (65537, 48, 65), (65536, 64, 33)}
    assert {c for c in cases.CASES if seen[c] is None} == others
    assert {v for v in seen.values() if v} == {(16, 0), (16, 1), (16, 2), (16, 3), (32, 0), (32, 1), (32, 2), (32, 3), (48, 0), (48, 1), (64, 0), (64, 1)}
    both = next(m for m in cases.test_both.pytestmark if m.name == "parametrize").args[1]
    seen = dict(zip(both, (_direct(s[0]) for s in lr.record(tmp_path, [lr.gemm_bwd(*c, "both") for c in both]))))
    assert {c for c in both if seen[c] is None} == {(65535, 16, 17), (65536, 17, 41), (65536, 48, 33)}


# contraction, rows, columns of the weight gradient of a 1 x 1 layer
@pytest.mark.parametrize("shared,layers", [
    (False, [(7259, 320, 608), (12354, 120, 528), (5201, 192, 912), (4554, 136, 1024), (13333, 160, 576), (6597, 56, 896), (15508, 76, 976), (2543, 264, 112)]),
    (True, [(104_394, 48, 224), (131_072, 16, 144), (84_130, 20, 1376), (12_608, 268, 240), (9840, 284, 112)])])
def test_weight_gradients_that_share_digits(tmp_path, shared, layers):
    """Not short contractions, whose operands stay in the caches: each of those named here was slower (5 to 22 %) so."""
    seen = lr.record(tmp_path, [lr.conv_bwd_weights(1, M, 1, K, N, 1, 1, 1, 0) for M, N, K in layers])
    assert [any("dw_shared_kernel" in l.name for l in s[0]) for s in seen] == [shared] * len(layers)


def test_activation_gradients_by_columns(tmp_path):
    import test_gpu_da_columns as cases
    assert not any("da_columns_kernel" in l.name for l in lr.record(tmp_path, [lr.gemm_bwd(2, 3, 70_000_004, "a")])[0][0])      # (more blocks than a grid has in y)
    seen = lr.record(tmp_path, [lr.gemm_bwd(*c[:3], want) for c in cases.CASES for want in ("a", "both")])
    assert [any("da_columns_kernel" in l.name for l in s[0]) for s in seen] == [c[3] for c in cases.CASES for _ in range(2)]
    for c, (launches, _) in zip([c for c in cases.CASES for _ in range(2)], seen):
        for l in launches:
            if "da_columns_kernel" in l.name:
                assert l.grid == (-(-c[0] // 128), -(-(c[2] // 4) // 256), 1), (c, l)
