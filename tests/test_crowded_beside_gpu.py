"""GPU tests of the gradient beside the chains where there are more chains than compute units: the same bits as in a launch of its own, and
the oracle's gradient, with one wavefront and several to a chain, two and four tiles of symbols, the log domain, steep utterances, empty labels, chains that
come late, and two such calls at once."""
import numpy as np
import pytest
import torch

from oracle import ctc_oracle as orc
from paper_1512_02595_amd import ctc, harness
from paper_1512_02595_amd import workloads as wl
from probability_stretches import batch_of_stretches

pytestmark = pytest.mark.gpu


def buffers_of(batch, dtype, device):
    if not device:
        return harness.DeviceBatch(batch, dtype)
    db = harness.DeviceMetaBatch(batch.T, batch.B, batch.A, max(int(batch.label_lengths.max()), 1), batch.blank, dtype)
    db.load(batch)
    return db


def run_with(batch, dtype, percent, device):
    """Costs, gradient, and whether the gradient was written in the chains' launch."""
    ctc.debug_set_overlap(percent)
    try:
        db = buffers_of(batch, dtype, device)
        db.run()
        costs, grads = db.results()[-2:]
        kernel_ms = np.zeros(ctc.NUM_KERNELS, dtype=np.float32)
        db.run(kernel_ms=kernel_ms)
        return costs, grads, kernel_ms[2] == 0
    finally:
        ctc.debug_set_overlap(-1)


def check_crowded(batch, dtype, device):
    assert 2 * batch.B > torch.cuda.get_device_properties(0).multi_processor_count
    print(f"crowded case {batch.name} T={batch.T} B={batch.B} A={batch.A} labels up to {batch.label_lengths.max()} device={device}", flush=True)
    ref_c, ref_g, beside = run_with(batch, dtype, 0, device)
    assert not beside
    logits = batch.logits if dtype == ctc.DTYPE_F32 else wl.to_bf16_grid(batch.logits)
    orc_c, orc_g = orc.ctc_loss_and_grad(logits, batch.flat_labels, batch.label_lengths, batch.input_lengths, batch.blank)
    assert not np.isinf(orc_c).any()                     # every utterance has its two chains
    rtol, atol = (1e-4, 1e-4) if dtype == ctc.DTYPE_F32 else (2e-2, 1e-2)       # (the parity tests' bounds)
    err = np.abs(ref_c - orc_c) / np.maximum(np.abs(orc_c), 1e-2)
    assert not np.isnan(ref_c).any() and err.max() <= rtol
    assert np.abs(ref_g - orc_g).max() <= atol
    for percent in (101, 30):
        c, g, beside = run_with(batch, dtype, percent, device)
        assert beside and np.array_equal(c, ref_c) and np.array_equal(g, ref_g), percent


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("seed,T,B,A,most,least,sigma,dtype", [
    (11, 33, 129, 29, 12, 1, 2.0, ctc.DTYPE_F32),        # two chains more than compute units
    (12, 90, 300, 32, 30, 10, 2.0, ctc.DTYPE_F32),
    (13, 90, 260, 33, 30, 10, 2.0, ctc.DTYPE_BF16),
    (14, 180, 140, 64, 150, 40, 2.0, ctc.DTYPE_F32),     # several wavefronts, two pieces
    (15, 500, 130, 20, 420, 300, 2.0, ctc.DTYPE_F32),    # more than four
    (16, 60, 200, 7, 25, 30, 60.0, ctc.DTYPE_F32),       # log domain
    (18, 150, 140, 40, 110, 120, 60.0, ctc.DTYPE_F32),   # ... of several wavefronts
    (17, 20, 512, 29, 0, 3, 2.0, ctc.DTYPE_F32),         # empty labels
])
def test_beside_crowded_chains(seed, T, B, A, most, least, sigma, dtype, device):
    check_crowded(wl.make_random(seed, T=T, B=B, A=A, max_label=most, min_input=least, sigma=sigma, feasible_only=True), dtype, device)


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("A,labels,copies", [(29, (1, 20, 62), 45), (40, (20, 90, 130, 230), 33)])
def test_steep_utterances_beside_crowded_chains(A, labels, copies, device):
    """Probabilities from 2^-79 to 2^-100: frames looked after every four steps, in the chains and in the blocks that are computed beside them."""
    check_crowded(batch_of_stretches(95, "blank", A, labels=labels, copies=copies), ctc.DTYPE_F32, device)


@pytest.mark.parametrize("percent", [-1, 40])            # of the chains' workgroups come late: others leave them their places
def test_two_crowded_calls_at_once(percent):
    """Either call alone has more workgroups that wait than the chip has places."""
    calls = [buffers_of(wl.make_random(21, T=160, B=300, A=29, max_label=40, min_input=20, feasible_only=True), ctc.DTYPE_F32, False),
             buffers_of(wl.make_random(22, T=200, B=140, A=50, max_label=120, min_input=60, feasible_only=True), ctc.DTYPE_BF16, True)]
    alone = []
    for c in calls:
        c.run()
        alone.append(c.results()[-2:])
        kernel_ms = np.zeros(ctc.NUM_KERNELS, dtype=np.float32)
        c.run(kernel_ms=kernel_ms)
        assert kernel_ms[2] == 0                         # (beside the chains by default)
    streams = [torch.cuda.Stream() for _ in calls]
    torch.cuda.synchronize()
    ctc.debug_set_overlap(percent)
    try:
        for _ in range(4):
            for c, s in zip(calls, streams):
                c.run(s.cuda_stream)
    finally:
        ctc.debug_set_overlap(-1)
    for c, (costs, grads) in zip(calls, alone):
        got = c.results()[-2:]
        assert np.array_equal(got[0], costs) and np.array_equal(got[1], grads)
