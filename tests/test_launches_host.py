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
