"""GPU tests of the frames' norms: probabilities around the two bounds below which a chain looks after its lanes' exponents more
often (2^-32) or runs on logarithms (2^-79), for the blank and for label symbols, over label lengths at the edges of the plans.
Costs and gradients within 1e-4 of the oracle's, as everywhere (costs relative, gradients absolute)."""
import numpy as np
import pytest

from oracle import ctc_oracle as orc
from paper_1512_02595_amd import harness
from paper_1512_02595_amd import workloads as wl

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 62, 63, 64, 95, 111, 112, 143, 159, 160, 207, 208, 231, 232, 239, 240, 247, 248, 352, 415, 416]


@pytest.mark.parametrize("A", [24, 80])
@pytest.mark.parametrize("bits", [20, 33, 78, 81, 110])
@pytest.mark.parametrize("who", ["blank", "label", "both"])
def test_small_probabilities(A, bits, who):
    rng = np.random.default_rng([A, bits, len(who)])
    blank = A - 1
    lengths = np.asarray(LENGTHS, dtype=np.int32)
    frames = np.maximum(2 * lengths + 20, 40) + rng.integers(0, 40, len(lengths))
    flat = np.concatenate([rng.integers(0, blank, n) for n in lengths]).astype(np.int32)
    B, T = len(lengths), int(frames.max())
    x = rng.normal(0, 1, (T, B, A)).astype(np.float32)
    # (the row's largest logit less bits ln 2: a probability of a little under 2^-bits)
    depth = np.float32(bits * np.log(2))
    for b in range(B):
        at = rng.integers(0, frames[b], 6)
        if who in ("blank", "both"):
            x[at[:3], b, blank] = x[at[:3], b, :].max(axis=1) - depth
        if who in ("label", "both"):
            first = int(lengths[:b].sum())
            symbols = flat[first:first + lengths[b]]
            if len(symbols):
                x[at[3:], b, symbols[rng.integers(0, len(symbols), 3)]] = x[at[3:], b, :].max(axis=1) - depth
    batch = wl.CTCBatch("small probabilities", T, B, A, blank, x, flat, lengths, frames.astype(np.int32), seed=0)
    want_costs, want = orc.ctc_loss_and_grad(x, flat, lengths, batch.input_lengths, blank)
    on_gpu = harness.DeviceBatch(batch)
    on_gpu.poison()
    on_gpu.run()
    costs, grads = on_gpu.results()
    bound = 1e-4 * np.maximum(np.abs(want_costs), 1e-2)
    assert (np.abs(costs - want_costs) <= bound).all()
    assert np.abs(grads - want).max() <= 1e-4
    on_gpu.poison()
    on_gpu.run_loss()
    only, _ = on_gpu.results()
    assert (np.abs(only - want_costs) <= bound).all()
