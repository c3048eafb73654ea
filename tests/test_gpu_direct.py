"""Products of small layers: the forward kernel that splits the contraction over the waves of a block, and the backward
products formed directly in double - ragged tiles, rows that are not aligned, contractions shorter and longer than a step,
operands stored with an offset, contractions cut into pieces - and backward products just too large for that."""
import numpy as np
import pytest

import cdl_inputs
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 1, 16), (33, 31, 17), (32, 32, 127), (64, 65, 129), (31, 33, 143), (100, 37, 1005), (7, 300, 640), (1000, 33, 255)])
@pytest.mark.parametrize("oa,ob", [(0, 0), (128, 0), (128, 128)])
def test_forward(M, N, K, oa, ob):
    import paper_2501_09849_amd as cdl
    torch = gu.torch_mod()
    a, b = cdl_inputs.draw_indices((M, K), -128, 127, seed=M), cdl_inputs.draw_indices((N, K), -128, 127, seed=N)
    acc, y = gu.empty((M, N), torch.int32), gu.empty((M, N), torch.float32)
    ws = gu.workspace(cdl.qgemm_fwd_offset_workspace_bytes(M, N, K))
    cdl.cdl_qgemm_fwd_offset(gu.dev(a), gu.dev(b), M, N, K, 0.5, 0.25, oa, ob, acc, y, ws)
    ref = (a.astype(np.int64) + oa) @ (b.astype(np.int64) + ob).T
    assert np.array_equal(acc.cpu().numpy(), ref)
    assert np.array_equal(y.cpu().numpy(), ref.astype(np.float32) * np.float32(0.125))
