"""GPU tests of how small a probability may be before an utterance's chains leave the linear domain (2^-100), and of the classes on
the way there (2^-32 and 2^-79: how often chains look after their lanes' exponents).  Frames are only powers of two, so a class must not
show in the results: with the same emissions and a symbol that no label uses at 2^-20, 2^-33, ... 2^-99, costs and the other columns of
the gradient are the same bit for bit (alphabets of at most 64 symbols look at all of their symbols).  And sustained stretches of such
frames stay as close to the oracle as everything else."""
import numpy as np
import pytest

from paper_1512_02595_amd import ctc, harness
from paper_1512_02595_amd import workloads as wl

import parity_checks as pc
from probability_stretches import batch_of_stretches

pytestmark = pytest.mark.gpu

LABELS = [0, 1, 30, 63, 64, 100, 143, 160, 207, 232, 248, 300, 352, 416]


def unused_symbol_batch(bits, A, copies, seed=3):
    rng = np.random.default_rng([seed, A])
    labels = np.asarray(LABELS * copies, dtype=np.int32)
    frames = (2 * labels + 40 + rng.integers(0, 30, len(labels))).astype(np.int32)
    T, B = int(frames.max()), len(labels)
    flat = rng.integers(1, A - 1, int(labels.sum())).astype(np.int32)        # (symbol A - 1 is in no label)
    x = rng.normal(0, 2, (T, B, A)).astype(np.float32)
    # (under the row's largest by so much that the sum does not depend on it; the largest is above 2^-5)
    x[:, :, A - 1] = x[:, :, :A - 1].max(axis=2) - np.float32(40 * np.log(2))
    for b in range(B):
        t = rng.integers(0, frames[b], 3)
        x[t, b, A - 1] = x[t, b, :A - 1].max(axis=1) - np.float32(bits * np.log(2))
    return wl.CTCBatch(f"unused symbol at 2^-{bits}", T, B, A, 0, x, flat, labels, frames, seed=seed)


@pytest.mark.parametrize("A,copies", [(29, 1), (29, 10), (60, 1)])           # beside the chains, and in a launch behind them
def test_classes_give_the_same_bits(A, copies):
    results = {}
    for bits in (40, 50, 75, 85, 94):
        batch = unused_symbol_batch(bits, A, copies)
        print(f"case {batch.name} A={A} B={batch.B}", flush=True)
        on_gpu = harness.DeviceBatch(batch)
        on_gpu.run()
        costs, grads = on_gpu.results()
        on_gpu.run_loss()
        results[bits] = costs, grads[:, :, :A - 1], on_gpu.results()[0]
    for bits, got in results.items():
        for one, other in zip(got, results[40]):
            assert np.array_equal(one, other), bits


@pytest.mark.parametrize("bits", [31, 33, 78, 81, 99])
@pytest.mark.parametrize("who", ["blank", "labels"])
@pytest.mark.parametrize("A,copies,dtype", [(24, 1, ctc.DTYPE_F32), (24, 14, ctc.DTYPE_F32), (60, 1, ctc.DTYPE_BF16), (80, 1, ctc.DTYPE_F32)])
def test_sustained_stretches(bits, who, A, copies, dtype):
    batch = batch_of_stretches(bits, who, A, copies=copies)
    pc.check(batch, dtype)
    if copies == 1:
        pc.check_loss(batch, dtype)


@pytest.mark.parametrize("bits", [33, 99])
def test_sustained_stretches_of_a_very_wide_alphabet(bits):
    pc.check(batch_of_stretches(bits, "labels", 8300, labels=[1, 40, 130]))


@pytest.mark.parametrize("bits", [33, 81, 99])
@pytest.mark.parametrize("A", [24, 80])
def test_sustained_stretches_with_metadata_on_the_gpu(bits, A):
    batch = batch_of_stretches(bits, "blank", A)
    dm = harness.DeviceMetaBatch(batch.T, batch.B, batch.A, int(batch.label_lengths.max()), batch.blank)
    dm.load(batch)
    dm.poison()
    dm.run()
    status, costs, grads = dm.results()
    want_costs, want = pc.orc.ctc_loss_and_grad(batch.logits, batch.flat_labels, batch.label_lengths, batch.input_lengths, batch.blank)
    assert status == ctc.STATUS_SUCCESS
    assert (np.abs(costs - want_costs) <= pc.COST_RTOL * np.maximum(np.abs(want_costs), 1e-2)).all()
    assert np.abs(grads - want).max() <= pc.GRAD_ATOL
