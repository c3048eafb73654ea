"""Which kernels a call launches and how, on both sides of the rules that choose them, without a GPU (launch_recorder.py)."""
import shutil

import pytest

import launch_recorder as lr

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
