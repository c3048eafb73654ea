"""The Python calls of the library, without a GPU: what they take as a number.  Every call here fails the library's own validation
(negative size), so that nothing is launched wherever the test runs."""
import os

import numpy as np
import pytest
import torch

FAKE = 1 << 20


@pytest.fixture(scope="module")
def cdl():
    import paper_2501_09849_amd as pkg
    import paper_2501_09849_amd.build as b
    if not os.path.exists(b.LIB_PATH):
        b.build_lib()
    pkg.load()
    return pkg


def _status(cdl, f, *args, **kw):
    with pytest.raises(cdl.CdlError) as e:
        f(*args, stream=0, **kw)
    return e.value.status


@pytest.mark.parametrize("bad", [-1.0, 3.7, "-1", np.float32(-1), None])
def test_a_size_is_an_integer(cdl, bad):
    with pytest.raises(TypeError):
        cdl.cdl_quantize_draw(FAKE, FAKE, bad, -7, 15, 0.02, 1e4, FAKE, stream=0)
    with pytest.raises(TypeError):
        cdl.cdl_qgemm_fwd(FAKE, FAKE, -1, bad, 16, 1.0, 1.0, None, FAKE, stream=0)
    with pytest.raises(TypeError):
        cdl.cdl_huffman_bits(FAKE, -1, bad, 16, FAKE, stream=0)
    with pytest.raises(TypeError):
        cdl.cdl_qconv_fwd(FAKE, FAKE, -1, 8, 8, 16, 16, 3, bad, 1, 1, 0.1, 0.1, None, FAKE, stream=0)


@pytest.mark.parametrize("size", [-1, np.int64(-1), np.int32(-1), torch.tensor(-1)])
def test_what_python_takes_as_an_index_is_a_size(cdl, size):
    assert _status(cdl, cdl.cdl_quantize_draw, FAKE, FAKE, size, -7, 15, 0.02, 1e4, FAKE) == -2
    assert _status(cdl, cdl.cdl_qgemm_fwd, FAKE, FAKE, size, 16, 16, 1.0, 1.0, None, FAKE) == -2


def test_quantizers_and_offsets_are_converted_as_int_and_float_do(cdl):
    for lo, levels, delta, alpha in ((-7.0, "15", "0.02", 10000), (np.float32(-7), np.int64(15), np.float64(0.02), torch.tensor(1e4))):
        assert _status(cdl, cdl.cdl_quantize_draw, FAKE, FAKE, -1, lo, levels, delta, alpha, FAKE) == -2
    assert _status(cdl, cdl.cdl_qgemm_fwd_offset, FAKE, FAKE, -1, 16, 16, 1.0, 1.0, 128.0, "0", None, FAKE) == -2
    assert _status(cdl, cdl.cdl_entropy_bwd, FAKE, FAKE, -1, -7, 15, 0.02, 1e4, scale="0.5", dtheta=FAKE) == -2
    with pytest.raises(TypeError):       # a step of a product is a number
        cdl.cdl_qgemm_fwd(FAKE, FAKE, -1, 16, 16, "1.0", 1.0, None, FAKE, stream=0)


def test_current_stream_without_the_internal_queries_of_torch(cdl, monkeypatch):
    """The address of the current stream comes from torch's public functions where the internal ones are missing."""
    import types
    from paper_2501_09849_amd import _marshal, binding
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d=None: types.SimpleNamespace(cuda_stream=0x1000 + d))
    stream_of, device = binding._stream_queries()
    assert device() == 3 and stream_of(device()) == 0x1003
    lib = cdl.load()
    import ctypes
    table = {name: ctypes.cast(getattr(lib, name), ctypes.c_void_p).value for name in binding._MARSHALLED}
    _marshal.init(table, stream_of, device)
    try:
        with pytest.raises(cdl.CdlError) as e:      # (reaches the library: no stream given)
            cdl.cdl_quantize_draw(FAKE, FAKE, -1, -7, 15, 0.02, 1e4, FAKE)
        assert e.value.status == -2
    finally:
        monkeypatch.undo()
        _marshal.init(table, *binding._stream_queries())


def test_native_module_belongs_to_one_interpreter(cdl, monkeypatch):
    import sysconfig
    import paper_2501_09849_amd.build as b
    from paper_2501_09849_amd import _marshal
    assert os.path.basename(b.MARSHAL_PATH) == "_marshal" + sysconfig.get_config_var("EXT_SUFFIX") != "_marshal.so"
    assert os.path.samefile(_marshal.__file__, b.MARSHAL_PATH)
    assert not b.is_stale()
    monkeypatch.setattr(b, "MARSHAL_SUFFIX", ".cpython-399-x86_64-linux-gnu.so")
    assert b.is_stale()
