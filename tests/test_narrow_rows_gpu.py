"""GPU tests of the softmax launch of small alphabets at the sizes where it can go wrong: symbols around what a lane of a
quad holds (two, eight and sixteen times four), blank in the first, last and a middle column, frames around the 64 of a
workgroup and the chunks of 8, labels longer than a workgroup has threads, cost, gradient and alignment."""
import pytest

from paper_1512_02595_amd import ctc

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu

FRAMES = [1, 3, 8, 9, 63, 64, 65, 71, 72, 128, 129]


@pytest.mark.parametrize("dtype", [ctc.DTYPE_F32, ctc.DTYPE_BF16])
@pytest.mark.parametrize("A", [2, 3, 4, 5, 7, 8, 9, 31, 32, 33, 36, 37, 63, 64])
@pytest.mark.parametrize("copies", [1, 13])                # (13: 143 utterances, behind an upload launch)
def test_symbols_around_a_lanes_share(A, dtype, copies):
    for blank in {0, A // 2, A - 1}:
        pc.check(batch_of(FRAMES, [f // 4 for f in FRAMES], A, blank=blank, T=130, seed=A, copies=copies), dtype)


@pytest.mark.parametrize("A", [5, 32, 64])
def test_cost_and_alignment(A):
    batch = batch_of(FRAMES, [f // 4 for f in FRAMES], A, blank=A - 1, T=130, seed=A)
    pc.check_loss(batch)
    pc.check_best(batch)


@pytest.mark.parametrize("labels", [[255, 256, 257], [511, 513, 1], [0, 700, 0]])
def test_labels_longer_than_a_workgroup(labels):
    pc.check(batch_of([2 * n + 30 for n in labels], labels, 29, seed=labels[1]))
