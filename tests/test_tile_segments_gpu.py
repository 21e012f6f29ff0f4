"""Utterances get as many of the gradient's workgroups as the longest of their segment needs (TileArgs::segment_tile), and the rows behind those are divided among them:
fewer utterances than segments, one to a segment and more, most of them far shorter than the tensor, beside the chains and apart, against the oracle."""
import numpy as np
import pytest

from paper_1512_02595_amd import ctc

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("overlap", [0, 101])
@pytest.mark.parametrize("B,T,longest,A", [(1, 700, 40, 29), (7, 333, 150, 29), (8, 64, 10, 64), (9, 1000, 300, 29), (520, 64, 12, 29), (300, 257, 90, 40)])
def test_rows_of_every_utterance(B, T, longest, A, overlap):
    rng = np.random.default_rng([B, T])
    frames = np.minimum(T, (T * rng.random(B) ** 3).astype(int) + 1)
    frames[0] = T if B > 1 else 100
    frames[B // 2] = 0 if B > 2 else frames[B // 2]
    labels = np.minimum(longest, frames // 3)
    try:
        ctc.debug_set_overlap(overlap)
        pc.check(batch_of(frames, labels, A, seed=B, T=T))
    finally:
        ctc.debug_set_overlap(-1)
