"""GPU tests of the workgroups that write the gradient inside the lattice launch and wait for the chains of their utterance."""
import numpy as np
import pytest
import torch

from oracle import ctc_oracle as orc
from paper_1512_02595_amd import ctc, harness
from paper_1512_02595_amd import workloads as wl

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_label", [40, 200])        # chains of one wavefront, of several
def test_a_wait_that_gives_up_is_reported_as_nan_cost(max_label):
    """No look at the chains but the first: a workgroup that finds them under way writes zeros, and the cost is NaN even
    though the chains go on to their end and store one.  Whatever else is there is right."""
    batch = wl.make_random(71, T=500, B=6, A=29, max_label=max_label, min_input=400, sigma=2.0, feasible_only=True)
    ref_c, ref_g = orc.ctc_loss_and_grad(batch.logits, batch.flat_labels, batch.label_lengths, batch.input_lengths, batch.blank)
    db = harness.DeviceBatch(batch)
    db.poison()
    ctc.debug_set_end_polls(0)
    try:
        db.run()
    finally:
        ctc.debug_set_end_polls(-1)
    costs, grads = db.results()
    lost = np.isnan(costs)
    print(f"  costs {costs}", flush=True)
    assert lost.any()                                    # (the first workgroups look before a chain has made its steps)
    assert (np.abs(costs - ref_c)[~lost] <= pc.COST_RTOL * ref_c[~lost]).all()
    assert np.isfinite(grads).all()
    close = np.abs(grads - ref_g).max(axis=2) <= pc.GRAD_ATOL                  # [frame][utterance]
    assert close[:, ~lost].all() and (close | (grads == 0).all(axis=2)).all()
    # and the next call on the same buffers is none the worse for it
    db.run()
    costs, grads = db.results()
    assert (np.abs(costs - ref_c) <= pc.COST_RTOL * ref_c).all() and np.abs(grads - ref_g).max() <= pc.GRAD_ATOL


@pytest.mark.parametrize("percent", [-1, 40, 100])      # of the chains' workgroups come late: others leave them their places
@pytest.mark.parametrize("dtype", [ctc.DTYPE_F32, ctc.DTYPE_BF16])
def test_calls_on_two_streams_at_once(percent, dtype):
    """Each of two calls in flight fills the chip with workgroups that wait; both end, with the results each has alone."""
    batches = [wl.make_config(1, seed=5, B=48), wl.make_random(72, T=600, B=70, A=29, max_label=60, min_input=16, sigma=2.0)]
    host = harness.DeviceBatch(batches[0], dtype)
    device = harness.DeviceMetaBatch(600, 70, 29, 60, batches[1].blank, dtype)
    device.load(batches[1])
    calls = [host, device]
    alone = []
    for c in calls:
        c.run()
        alone.append(c.results()[-2:])
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
        assert np.array_equal(got[0], costs, equal_nan=True) and np.array_equal(got[1], grads)


@pytest.mark.parametrize("frames,labels", [([16, 9, 3], [4, 0, 3]),                # one block: a single workgroup waits
                                           ([700, 90, 1], [300, 20, 1])])          # several wavefronts a chain
def test_places_left_to_late_chains(frames, labels):
    ctc.debug_set_overlap(100)
    try:
        pc.check(batch_of(frames, labels, 29))
    finally:
        ctc.debug_set_overlap(-1)
