"""Forward product where its output has fewer tiles of 128 rows than the chip has compute units (tiles of 64 rows, chunks asked for
two steps ahead): one step of the contraction, odd and even numbers of them, ragged rows and columns - accumulators exact."""
import numpy as np
import pytest

import cdl_inputs
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [16, 64, 80, 128, 192, 336])
@pytest.mark.parametrize("M,N", [(17_001, 64), (25_000, 33), (8_193, 130), (9_100, 128)])
def test_few_row_tiles(oracle, M, N, K):
    a = cdl_inputs.draw_indices((M, K), -128, 127, seed=M + K)
    b = cdl_inputs.draw_indices((N, K), -128, 127, seed=N + K)
    acc, y = gu.qgemm_fwd(a, b, 0.15092, 0.0028209)
    want = (a.astype(np.float32) @ b.astype(np.float32).T).astype(np.int32)      # exact: every sum stays below 2^24
    assert np.array_equal(acc, want), "int32 accumulators differ at %d places" % int((acc != want).sum())
    gu.assert_close(y, want.astype(np.float64) * float(np.float32(0.15092) * np.float32(0.0028209)), "y")
