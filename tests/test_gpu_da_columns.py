"""GPU activation gradient of up to 16 output channels whose results don't fit the memory-side cache, in rows of more than 160 columns that are no whole pieces of 64 bytes: a thread per four columns; rows of fewer and of more
columns than a block's threads take, last rows that do not fill a block, both sides of the rule (which kernel serves is checked without a GPU)."""
import pytest

import gpu_util as gu
from test_gpu_da_direct import test_da_direct as check

pytestmark = pytest.mark.gpu

# M, N, K, whether it serves
CASES = [(220_603, 16, 408, True), (441_201, 1, 204, True), (90_403, 5, 996, True), (1385, 16, 65_004, True), (548_801, 13, 164, True), (555, 3, 162_500, True), (225_001, 16, 400, False), (220_603, 17, 408, False),
         (562_501, 9, 160, False), (220_585, 16, 408, False)]


@pytest.mark.parametrize("M,N,K,served", CASES)
def test_columns(M, N, K, served):
    check(M, N, K)
