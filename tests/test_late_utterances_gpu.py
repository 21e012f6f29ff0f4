"""Launches of many blocks give several wavefronts to a block only in the utterances that end last (shared_utterances in ctc_kernels.hip): batches in which some have
them and others do not, with labels of one to six pieces, beside the chains and apart (the same sums), against the oracle; metadata on the host and on the GPU."""
import numpy as np
import pytest

from paper_1512_02595_amd import ctc, harness

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,longest,A", [(60, 1100, 530, 29), (60, 1100, 300, 50), (150, 450, 200, 29), (330, 320, 130, 33)])
def test_some_have_several_wavefronts_to_a_block(B, T, longest, A):
    rng = np.random.default_rng(B)
    labels = rng.integers(0, longest + 1, B)
    labels[0] = longest
    frames = np.minimum(T, labels + labels // 8 + rng.integers(17, T // 2, B))
    frames[1], frames[2] = T, 0
    batch = batch_of(frames, labels, A, seed=B, T=T)
    results = []
    try:
        for overlap in (0, 101):
            ctc.debug_set_overlap(overlap)
            results.append(pc.check(batch)[:2] if overlap == 0 else harness.run_batch(batch))
    finally:
        ctc.debug_set_overlap(-1)
    for one, other in zip(*results):
        assert np.array_equal(one, other)
    on_gpu = harness.DeviceMetaBatch(batch.T, batch.B, batch.A, longest, batch.blank)
    on_gpu.load(batch)
    on_gpu.run()
    # (the plans, and so who ends last, follow from bounds there)
    _, costs, grads = on_gpu.results()
    finite = np.isfinite(results[0][0])
    assert np.array_equal(np.isfinite(costs), finite)
    assert np.max(np.abs(costs[finite] - results[0][0][finite]) / results[0][0][finite].clip(1e-2)) <= 1e-6 and np.max(np.abs(grads - results[0][1])) <= 1e-5
