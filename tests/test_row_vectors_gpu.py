"""GPU tests of the softmax launch of large alphabets at the sizes where it can go wrong: rows around the sizes at which
the lanes per row change, rows that start at every place within 16 bytes, activations and gradient that start at
different places, zero rows left to the lattice launch."""
import numpy as np
import pytest
import torch

from oracle import ctc_oracle as orc
from paper_1512_02595_amd import ctc
from paper_1512_02595_amd import workloads as wl

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu

SIZES = [65, 71, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2049, 4095, 4096, 4097, 8191, 8192, 8193]


@pytest.mark.parametrize("dtype", [ctc.DTYPE_F32, ctc.DTYPE_BF16])
@pytest.mark.parametrize("A", SIZES)
def test_rows_around_lane_counts(A, dtype):
    pc.check(batch_of([19, 7, 16, 3, 12], [4, 3, 0, 9, 6], A, blank=A - 1, T=33, seed=A), dtype)


@pytest.mark.parametrize("dtype,torch_dtype", [(ctc.DTYPE_F32, torch.float32), (ctc.DTYPE_BF16, torch.bfloat16)])
@pytest.mark.parametrize("A", [77, 300, 1200, 2600])
@pytest.mark.parametrize("x_at,g_at", [(1, 1), (3, 3), (5, 5), (0, 1), (2, 0)])
def test_tensors_off_a_16_byte_boundary(A, dtype, torch_dtype, x_at, g_at):
    check_off_boundary(A, dtype, torch_dtype, x_at, g_at)


@pytest.mark.parametrize("dtype,torch_dtype", [(ctc.DTYPE_F32, torch.float32), (ctc.DTYPE_BF16, torch.bfloat16)])
@pytest.mark.parametrize("A", [65, 513, 4097, 8191, 8192])
@pytest.mark.parametrize("x_at,g_at", [(0, 3), (1, 0), (3, 6), (7, 4)])
def test_gradient_at_another_place_than_the_activations(A, dtype, torch_dtype, x_at, g_at):
    check_off_boundary(A, dtype, torch_dtype, x_at, g_at)


def check_off_boundary(A, dtype, torch_dtype, x_at, g_at):
    batch = batch_of([21, 13, 18], [5, 4, 7], A, T=24, seed=A)
    n = batch.logits.size
    logits = batch.logits if dtype == ctc.DTYPE_F32 else wl.to_bf16_grid(batch.logits)
    x = torch.zeros(n + 8, dtype=torch_dtype, device="cuda")
    x[x_at:x_at + n] = torch.from_numpy(logits).reshape(-1).to("cuda", torch_dtype)
    g = torch.full((n + 16,), 7.0, dtype=torch_dtype, device="cuda")
    costs = torch.zeros(batch.B, device="cuda")
    ws = torch.empty(ctc.workspace_size(batch.T, batch.B, A, batch.label_lengths, batch.input_lengths, dtype),
                     dtype=torch.uint8, device="cuda")
    size = x.element_size()
    ctc.loss_and_grad(x.data_ptr() + x_at * size, batch.flat_labels, batch.label_lengths, batch.input_lengths, batch.T,
                      batch.B, A, batch.blank, dtype, costs.data_ptr(), g.data_ptr() + g_at * size, ws.data_ptr(), ws.numel())
    torch.cuda.synchronize()
    ref_c, ref_g = orc.ctc_loss_and_grad(logits, batch.flat_labels, batch.label_lengths, batch.input_lengths, batch.blank)
    got = g.float().cpu().numpy()
    assert (got[:g_at] == 7.0).all() and (got[g_at + n:] == 7.0).all()
    assert np.abs(got[g_at:g_at + n].reshape(ref_g.shape) - ref_g).max() <= (pc.GRAD_ATOL if dtype == ctc.DTYPE_F32 else pc.BF16_GRAD_ATOL)
    np.testing.assert_allclose(costs.cpu().numpy(), ref_c, rtol=1e-4 if dtype == ctc.DTYPE_F32 else 2e-2)


@pytest.mark.parametrize("A", [90, 3001])
def test_zero_rows_beside_the_chains(A):
    """Most of the tensor is padding, by far more than the chains give time for; some utterances have no alignment."""
    pc.check(batch_of([40, 1, 37, 2, 16, 17], [4, 5, 3, 1, 30, 2], A, T=217, seed=A))
