"""GPU tests of the gradient beside the chains where there are more chains than compute units: the same bits as in a launch of its own, and
the oracle's gradient, with one wavefront and several to a chain, two and four tiles of symbols, the log domain, empty labels, and chains that come
late."""
import numpy as np
import pytest

from oracle import ctc_oracle as orc
from paper_1512_02595_amd import ctc, harness
from paper_1512_02595_amd import workloads as wl

pytestmark = pytest.mark.gpu


def run_with(batch, dtype, percent, device):
    ctc.debug_set_overlap(percent)
    try:
        if device:
            db = harness.DeviceMetaBatch(batch.T, batch.B, batch.A, max(int(batch.label_lengths.max()), 1), batch.blank, dtype)
            db.load(batch)
        else:
            db = harness.DeviceBatch(batch, dtype)
        db.run()
        return db.results()[-2:]
    finally:
        ctc.debug_set_overlap(-1)


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("seed,T,B,A,most,least,sigma,dtype", [
    (11, 33, 129, 29, 12, 1, 2.0, ctc.DTYPE_F32),        # a chain more than compute units, two of them
    (12, 90, 300, 32, 30, 10, 2.0, ctc.DTYPE_F32),
    (13, 90, 260, 33, 30, 10, 2.0, ctc.DTYPE_BF16),
    (14, 180, 140, 64, 150, 40, 2.0, ctc.DTYPE_F32),     # several wavefronts, two pieces
    (15, 500, 130, 20, 420, 300, 2.0, ctc.DTYPE_F32),    # more than four
    (16, 60, 200, 7, 25, 30, 60.0, ctc.DTYPE_F32),       # log domain
    (17, 20, 512, 29, 0, 3, 2.0, ctc.DTYPE_F32),         # empty labels
])
def test_beside_crowded_chains(seed, T, B, A, most, least, sigma, dtype, device):
    batch = wl.make_random(seed, T=T, B=B, A=A, max_label=most, min_input=least, sigma=sigma)
    print(f"crowded case T={T} B={B} A={A} labels up to {most} device={device}", flush=True)
    ref_c, ref_g = run_with(batch, dtype, 0, device)
    logits = batch.logits if dtype == ctc.DTYPE_F32 else wl.to_bf16_grid(batch.logits)
    orc_c, orc_g = orc.ctc_loss_and_grad(logits, batch.flat_labels, batch.label_lengths, batch.input_lengths, batch.blank)
    inf = np.isinf(orc_c)
    assert np.array_equal(np.isinf(ref_c) & (ref_c > 0), inf) and not np.isnan(ref_c).any()
    rtol, atol = (1e-4, 1e-4) if dtype == ctc.DTYPE_F32 else (2e-2, 1e-2)       # (the parity tests' bounds)
    err = np.abs(ref_c[~inf] - orc_c[~inf]) / np.maximum(np.abs(orc_c[~inf]), 1e-2)
    assert err.size == 0 or err.max() <= rtol
    assert np.abs(ref_g - orc_g).max() <= atol
    for percent in (101, 30):
        c, g = run_with(batch, dtype, percent, device)
        assert np.array_equal(c, ref_c, equal_nan=True) and np.array_equal(g, ref_g), percent
