"""GPU tests of the gradient of wide alphabets at the edges of what its workgroups take: label pieces of 128 positions (96 further
ones each), one piece or several to a wavefront, symbols that fill one or several rounds of the wavefronts, runs of one symbol, last
blocks of 1 to 16 frames, more utterances than one and fewer.  Costs and gradients as close to the oracle's as everywhere
(parity_checks)."""
import numpy as np
import pytest

import parity_checks as pc
from paper_1512_02595_amd import ctc
from paper_1512_02595_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", [[0, 1, 3, 4, 5, 63, 64, 65, 127, 128], [128, 129, 0, 130, 2], [223, 224, 225, 319, 320, 321, 16],
                                     [415, 416, 417, 511, 512, 513, 1], [1000, 705, 9], [77]])
@pytest.mark.parametrize("A,few", [(66, 66), (66, 3), (700, 700)])
@pytest.mark.parametrize("dtype", [ctc.DTYPE_F32, ctc.DTYPE_BF16])
def test_edges(lengths, A, few, dtype):
    rng = np.random.default_rng([len(lengths), lengths[0], A, few])
    lengths = np.asarray(lengths, dtype=np.int32)
    blank = int(rng.integers(0, A))
    symbols = np.setdiff1d(np.arange(A), [blank])[:few]
    flat = symbols[rng.integers(0, len(symbols), int(lengths.sum()))].astype(np.int32)
    starts = np.concatenate([[0], np.cumsum(lengths)])
    repeats = np.asarray([int((np.diff(flat[starts[b]:starts[b + 1]]) == 0).sum()) for b in range(len(lengths))])
    frames = (lengths + repeats + 1 + rng.integers(18, 60, len(lengths))).astype(np.int32)
    T, B = int(frames.max()) + 3, len(lengths)
    x = rng.normal(0, 1.5, (T, B, A)).astype(np.float32)
    batch = wl.CTCBatch("label columns", T, B, A, blank, x, flat, lengths, frames, seed=0)
    pc.check(batch, dtype)
