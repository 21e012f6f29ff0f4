"""GPU tests of the chains' checkpoints and the gradient's recomputation between them, at the sizes where they can
go wrong: utterances around whole blocks of 16 frames and chunks of 8, labels around the pieces of 128 and 96 positions
that one wavefront recomputes, blocks shared by several wavefronts and not, more symbols than one pair of matrix tiles."""
import numpy as np
import pytest

from paper_1512_02595_amd import ctc
from paper_1512_02595_amd import workloads as wl

import parity_checks as pc

pytestmark = pytest.mark.gpu


def batch_of(frames, labels, A, blank=0, seed=0, T=None, sigma=2.0, copies=1):
    rng = np.random.default_rng(seed)
    frames = np.asarray(list(frames) * copies, dtype=np.int32)
    labels = np.asarray(list(labels) * copies, dtype=np.int32)
    T = int(frames.max()) if T is None else T
    symbols = rng.integers(0, A - 1, int(labels.sum()))
    symbols = symbols + (symbols >= blank)
    x = (rng.standard_normal((T, len(frames), A)) * sigma).astype(np.float32)
    x[:, :, blank] += 2.0
    return wl.CTCBatch("edges", T, len(frames), A, blank, x, symbols.astype(np.int32), labels, frames, seed=seed)


@pytest.mark.parametrize("A,blank", [(29, 0), (33, 32), (64, 5), (65, 0), (300, 7)])
def test_frames_around_blocks_and_chunks(A, blank):
    frames = [1, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 47, 48, 49]
    pc.check(batch_of(frames, [min(5, f // 3) for f in frames], A, blank, T=50))


@pytest.mark.parametrize("A", [29, 64, 90])
def test_labels_around_pieces(A):
    labels = [0, 1, 63, 64, 65, 127, 128, 129, 223, 224, 225, 319, 320, 321]
    pc.check(batch_of([2 * n + 40 for n in labels], labels, A))


@pytest.fixture(params=[0, 101], ids=["apart", "beside"])
def form(request):
    """The gradient in a launch of its own, and beside the chains."""
    ctc.debug_set_overlap(request.param)
    yield request.param
    ctc.debug_set_overlap(-1)


@pytest.mark.parametrize("A", [29, 40])
def test_blocks_of_many_utterances_are_not_shared(A, form):
    """Enough blocks times pieces for every wavefront to take a whole block of its own."""
    pc.check(batch_of([560, 530], [230, 129], A, copies=64, sigma=1.0))


@pytest.mark.parametrize("A", [29, 40])
def test_log_domain_blocks_of_many_utterances_are_not_shared(A, form):
    pc.check(batch_of([560, 530], [230, 129], A, copies=64, sigma=60.0))


@pytest.mark.parametrize("A", [29, 90])
def test_longest_labels_and_bf16(A):
    pc.check(batch_of([1500, 1130], [600, 1023 if A > 64 else 900], A, sigma=1.0), ctc.DTYPE_BF16)


@pytest.mark.parametrize("A,copies", [(29, 1), (64, 1), (90, 1), (40, 12)])     # (12: more chains than compute units)
def test_log_domain_around_blocks_and_pieces(A, copies, form):
    """Logits so steep that every utterance has emissions below the linear domain's range."""
    frames = [1, 15, 16, 17, 33, 150, 300, 290, 480, 470, 700]
    labels = [1, 2, 0, 5, 9, 63, 127, 128, 223, 225, 321]
    pc.check(batch_of(frames, labels, A, copies=copies, sigma=60.0))
