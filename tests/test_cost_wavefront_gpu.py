"""GPU test of the wavefront that writes an utterance's cost in the gradient's launch (alphabets of at most 64 symbols), the first one
behind the utterance's blocks of 16 frames: utterances that fill all blocks of the tensor and utterances that leave some, block
counts around what a workgroup of four wavefronts takes, with one, two and four wavefronts to a block, beside the chains and apart."""
import numpy as np
import pytest

from paper_1512_02595_amd import ctc, harness

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [1, 2, 3, 4, 5, 7, 8, 9, 12, 31, 32])
@pytest.mark.parametrize("longest,A", [(5, 29), (128, 29), (200, 29), (300, 64)])
@pytest.mark.parametrize("copies", [1, 150])               # (150: blocks are not shared)
def test_behind_the_last_block(blocks, longest, A, copies):
    T = 16 * blocks
    frames = sorted({T, T - 1, T - 15, max(1, T - 16), max(1, T // 2), 1}, reverse=True)
    labels = [min(longest, f // 2) for f in frames]
    copies = min(copies, 1 + 12000 // T)
    batch = batch_of(frames, labels, A, T=T, seed=blocks, copies=copies)
    results = []
    try:
        for overlap in (0, 101):
            ctc.debug_set_overlap(overlap)
            results.append(pc.check(batch)[:2] if overlap == 0 else harness.run_batch(batch))
    finally:
        ctc.debug_set_overlap(-1)
    for one, other in zip(*results):
        assert np.array_equal(one, other)
