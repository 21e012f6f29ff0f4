"""GPU test of labels longer than their utterance, which get no room in the workspace's lattice: alone and beside others, by
host metadata and by bounds far beyond the frames, with every byte around the workspace's own watched."""
import numpy as np
import pytest
import torch

from oracle import ctc_oracle as orc
from paper_1512_02595_amd import ctc, harness

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("A", [29, 90])
@pytest.mark.parametrize("frames,labels", [([5, 20, 17, 1, 33, 16], [60, 21, 4, 2, 33, 0]), ([3], [60]), ([1, 1], [1, 60])])
def test_no_room_for_labels_beyond_frames(A, frames, labels):
    batch = batch_of(frames, labels, A, T=35)
    pc.check(batch)
    pc.check_loss(batch)
    pc.check_best(batch)
    ref_c, ref_g = orc.ctc_loss_and_grad(batch.logits, batch.flat_labels, batch.label_lengths, batch.input_lengths, batch.blank)
    db = harness.DeviceMetaBatch(35, len(frames), A, 60, batch.blank)
    guard = 4096
    ws = torch.full((db.ws_bytes + 2 * guard + 256,), 0xA5, dtype=torch.uint8, device=db.device)
    db.ws_ptr = (ws.data_ptr() + guard + 255) // 256 * 256
    at = db.ws_ptr - ws.data_ptr()
    db.load(batch)
    db.run()
    status, costs, grads = db.results()
    assert status == ctc.STATUS_SUCCESS
    assert np.array_equal(np.isinf(costs), np.isinf(ref_c)) and np.abs(grads - ref_g).max() <= pc.GRAD_ATOL
    fin = np.isfinite(ref_c)
    assert (np.abs(costs[fin] - ref_c[fin]) <= pc.COST_RTOL * np.maximum(np.abs(ref_c[fin]), 1e-2)).all()
    assert bool((ws[:at] == 0xA5).all()) and bool((ws[at + db.ws_bytes:] == 0xA5).all())
