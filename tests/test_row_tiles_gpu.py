"""GPU tests of the order in which the softmax launch of large alphabets takes its rows: tiles of eight frames that end
beyond the last frame or the last utterance, fewer tiles than dies, runs of whole rows around the number of rounds from
which they are used and behind the last whole round, and rows that are loaded past the caches."""
import numpy as np
import pytest
import torch

from paper_1512_02595_amd import ctc

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("A,B", [(70, 1), (70, 17), (200, 550), (600, 1), (600, 5), (600, 128), (600, 129), (600, 133), (700, 200)])
@pytest.mark.parametrize("T", [1, 8, 57, 64])
def test_tiles_end_beyond_the_tensor(A, B, T):
    frames = np.random.default_rng(A + B).integers(0, T + 1, B)
    pc.check(batch_of(frames, [min(3, f // 3) for f in frames], A, T=T, seed=A + B + T))


def softmax_of_rows(T, B, A, seed):
    """Utterances without a symbol: the gradient is y but for the blank's column, which is y - 1."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    x = torch.randn((T, B, A), generator=gen, device="cuda")
    frames = np.random.default_rng(seed).integers(0, T + 1, B).astype(np.int32)
    nothing = np.zeros(B, dtype=np.int32)
    costs, grads = torch.zeros(B, device="cuda"), torch.full_like(x, 7.0)
    ws = torch.empty(ctc.workspace_size(T, B, A, nothing, frames, ctc.DTYPE_F32), dtype=torch.uint8, device="cuda")
    print(f"rows T={T} B={B} A={A} seed={seed}", flush=True)
    ctc.loss_and_grad(x.data_ptr(), np.zeros(0, dtype=np.int32), nothing, frames, T, B, A, 0, ctc.DTYPE_F32, costs.data_ptr(),
                      grads.data_ptr(), ws.data_ptr(), ws.numel())
    torch.cuda.synchronize()
    for t in range(0, T, 64):                  # in slices: the tensor is large
        y = torch.softmax(x[t:t + 64], dim=2)
        y[:, :, 0] -= 1.0
        valid = torch.arange(t, min(t + 64, T), device="cuda")[:, None] < torch.from_numpy(frames).to("cuda")[None, :]
        error = (grads[t:t + 64] - y * valid[:, :, None]).abs().max().item()
        # y is off by a few ulp of 1 in the blank's column and by a relative 1e-6 (exponent times 6e-8) elsewhere
        assert error <= 2e-6, (t, error)


# 24 rounds of 8 runs of 64 rows: 12288
@pytest.mark.parametrize("T,B", [(2457, 5), (2458, 5), (12288, 1), (12289, 1), (1117, 11), (175, 73)])
def test_runs_of_whole_rows(T, B):
    softmax_of_rows(T, B, 2049, T)


# 512 million bytes: 160 frames of 100 utterances of 8000 symbols
@pytest.mark.parametrize("T,B,A", [(160, 100, 8000), (161, 199, 4000), (159, 100, 8000)])
def test_rows_past_the_caches(T, B, A):
    softmax_of_rows(T, B, A, A)


# Zero rows left to the launch of the label columns: few and all of those that the lattice launch does not write, frames that
# end within the sixteen of a round, more utterances than chains leave compute units for
@pytest.mark.parametrize("dtype", [ctc.DTYPE_F32, ctc.DTYPE_BF16])
@pytest.mark.parametrize("T,B", [(17, 1), (41, 300), (31, 140), (160, 7)])
def test_zero_rows_beside_the_label_columns(T, B, dtype):
    frames = np.random.default_rng(T).integers(0, max(2, T // 4), B)
    frames[0] = T
    pc.check(batch_of(frames, [min(3, f // 3) for f in frames], 2050, T=T, seed=T), dtype)
