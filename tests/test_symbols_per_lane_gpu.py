"""GPU tests of the softmax launch of large alphabets around the sizes at which the symbols per lane change, with rows that start at
every place within 16 bytes (the batch is odd) and with activations and gradient that start at different places."""
import pytest
import torch

from paper_1512_02595_amd import ctc

import parity_checks as pc
from test_block_edges_gpu import batch_of
from test_row_vectors_gpu import check_off_boundary

pytestmark = pytest.mark.gpu

SIZES = [191, 192, 193, 383, 384, 385, 767, 768, 769, 1535, 1536, 1537, 3071, 3072, 3073, 6143, 6144, 6145]


@pytest.mark.parametrize("dtype", [ctc.DTYPE_F32, ctc.DTYPE_BF16])
@pytest.mark.parametrize("A", SIZES)
def test_rows_around_symbols_per_lane(A, dtype):
    pc.check(batch_of([19, 7, 16, 3, 12], [4, 3, 0, 9, 6], A, blank=A - 1, T=33, seed=A), dtype)


@pytest.mark.parametrize("dtype,torch_dtype", [(ctc.DTYPE_F32, torch.float32), (ctc.DTYPE_BF16, torch.bfloat16)])
@pytest.mark.parametrize("A", [192, 384, 768, 1536, 3072, 6144])
@pytest.mark.parametrize("x_at,g_at", [(0, 0), (1, 0), (3, 6)])
def test_full_rows_off_a_boundary(A, dtype, torch_dtype, x_at, g_at):
    check_off_boundary(A, dtype, torch_dtype, x_at, g_at)
