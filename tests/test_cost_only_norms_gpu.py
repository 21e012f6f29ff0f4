"""GPU test of the workgroups that see to the norms of cost-only launches: one utterance to a wavefront, so numbers of utterances around
what a workgroup of one, two and more wavefronts takes, among them utterances without frames, without an alignment, without a symbol,
and in the log domain, whose forward chain sees to its own."""
import numpy as np
import pytest

from paper_1512_02595_amd import workloads as wl

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("longest", [20, 100, 200, 330])
@pytest.mark.parametrize("B", [1, 2, 3, 4, 5, 7, 64, 65, 131, 300])
@pytest.mark.parametrize("A", [29, 70])
def test_every_utterance_has_its_norms(longest, B, A):
    rng = np.random.default_rng([longest, B, A])
    labels = rng.integers(0, longest + 1, B)
    labels[-1] = longest
    frames = 2 * labels + rng.integers(17, 60, B)
    if B > 3:
        frames[0], labels[1], frames[2] = 0, 0, max(1, labels[2] // 2)
    batch = batch_of(frames, labels, A, seed=B, T=int(frames.max()))
    x = batch.logits.copy()
    for b in range(3, B, 4):                             # (log domain)
        x[: frames[b], b, :] *= 40
    pc.check_loss(wl.CTCBatch("norms", batch.T, B, A, batch.blank, x, batch.flat_labels, batch.label_lengths, batch.input_lengths, seed=B))
