"""GPU tests of the order in which the softmax launch of large alphabets takes its rows: tiles of eight frames that end
beyond the last frame or the last utterance, fewer tiles than dies, runs of whole rows around the number of rounds from
which they are used and behind the last whole round, and rows that are loaded past the caches."""
import os
import subprocess

import numpy as np
import pytest
import torch

from paper_1512_02595_amd import ctc, harness

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


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
@pytest.mark.parametrize("T,B,A", [(160, 100, 8000), (161, 199, 4000), (159, 100, 8000), (210, 200, 3072)])
def test_rows_past_the_caches(T, B, A):
    softmax_of_rows(T, B, A, A)


# Zero rows left to the launch of the label columns, some of them after those that the lattice launch writes: rows off 16 bytes, frames
# that end within the sixteen of a round before, among and behind the ones left over, few utterances and so many that the lattice launch
# leaves none; what is left to whom is asked of the rules themselves (ctc_internal.h).
RULES = r"""
#include <cstdio>
#include "ctc_internal.h"
int main()
{
    double zero_bytes;
    int longest, chains, A;
    while (std::scanf("%lf %d %d %d", &zero_bytes, &longest, &chains, &A) == 4) {
        const int defer = ctc::deferred_frames(zero_bytes, longest, chains, 256);
        std::printf("%d %d\n", defer, ctc::columns_frames(zero_bytes, A, defer));
    }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(RULES)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1512_02595_amd", "csrc"),
                    str(d / "rules.cpp"), "-o", str(d / "rules")], check=True)

    def ask(*args):
        out = subprocess.run([str(d / "rules")], input=" ".join(map(str, args)), capture_output=True, text=True, check=True).stdout
        return tuple(map(int, out.split()))
    return ask


def padded_batch(T, B, A):
    frames = np.random.default_rng(T).integers(1, max(2, T // 4), B)
    frames[0] = T
    return batch_of(frames, [min(3, f // 3) for f in frames], A, T=T, seed=T)


@pytest.mark.parametrize("T,B,A,dtype", [
    (113, 90, 2051, ctc.DTYPE_F32), (127, 90, 2053, ctc.DTYPE_F32), (121, 80, 2052, ctc.DTYPE_F32), (401, 20, 4097, ctc.DTYPE_F32),
    (118, 170, 2050, ctc.DTYPE_F32), (113, 170, 2051, ctc.DTYPE_BF16), (127, 90, 4099, ctc.DTYPE_BF16), (124, 90, 4098, ctc.DTYPE_BF16),
    (399, 40, 5001, ctc.DTYPE_BF16)])
def test_zero_rows_beside_the_label_columns(T, B, A, dtype, rules):
    batch = padded_batch(T, B, A)
    zero_bytes = (T * B - int(batch.input_lengths.sum())) * A * (4 if dtype == ctc.DTYPE_F32 else 2)
    defer, columns = rules(zero_bytes, T, 2 * B, A)
    assert columns > 0 and (defer > 0 or B > 96)
    pc.check(batch, dtype)


@pytest.mark.parametrize("T,B,A", [(303, 40, 4099), (305, 40, 4099)])
def test_zero_rows_beside_the_label_columns_with_metadata_on_the_gpu(T, B, A, rules):
    batch = padded_batch(T, B, A)
    defer, columns = rules(T * B * A * 4 / 3, T // 2, 2 * B, A)
    assert columns > 0 and defer > 0
    dm = harness.DeviceMetaBatch(T, B, A, 3, batch.blank)
    dm.load(batch)
    dm.poison()
    dm.run()
    status, costs, grads = dm.results()
    want_costs, want = pc.orc.ctc_loss_and_grad(batch.logits, batch.flat_labels, batch.label_lengths, batch.input_lengths, batch.blank)
    assert status == ctc.STATUS_SUCCESS and np.abs(grads - want).max() <= pc.GRAD_ATOL
    assert (np.abs(costs - want_costs) <= pc.COST_RTOL * np.maximum(np.abs(want_costs), 1e-2)).all()
    for b in range(B):
        assert not grads[batch.input_lengths[b]:, b].any()
