"""Host-side checks of sizes at the edge of what the calls take: workspaces lay utterances out in whole blocks of 16 frames,
which must not take away shapes that fit without the rounding."""
import numpy as np
import pytest

from paper_1512_02595_amd import ctc


# Shapes of 60 to 64 MiB, and the most utterances there may be, when rows are counted in frames and no block is rounded up:
# the static workspace took them before there were blocks.
SHAPES = [(100, 350, 29, 100), (100, 370, 29, 100), (33, 2210, 64, 33), (33, 2250, 60, 33), (49, 2190, 50, 20), (17, 4096, 64, 17),
          (2, 4096, 64, 2), (1, 4096, 64, 400), (3, 930, 80, 1000), (750, 21, 29, 250), (1500, 5, 29, 540), (65, 735, 1000, 65),
          (17, 4096, 300, 17), (500, 43, 750, 150), (1009, 4, 29, 1009)]


@pytest.mark.parametrize("T,B,A,max_label", SHAPES)
def test_the_static_workspace_holds_what_it_held(T, B, A, max_label):
    assert ctc.workspace_size_device(T, B, A, max_label) <= ctc.STATIC_WORKSPACE_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("T,B,A,max_label", SHAPES)
def test_the_static_call_takes_what_it_took(T, B, A, max_label):
    # (refused for the null pointers, not for the size, which is looked at first)
    assert ctc.loss_and_grad_device_static_status(0, 0, 0, 0, max_label, T, B, A, 0, ctc.DTYPE_F32, 0, 0, 0) == ctc.STATUS_INVALID_VALUE


def test_limits_count_frames_as_the_caller_does():
    most = (2**31 - 1) // (2 * 8)                        # frames of an utterance without symbols
    assert ctc.workspace_size_device(most, 1, 2, 0) > 0
    assert ctc.workspace_size_device_status(most + 1, 1, 2, 0)[0] == ctc.STATUS_UNSUPPORTED
    assert ctc.workspace_size(most, 1, 2, [0], [most]) > 0
    assert ctc.workspace_size_status(most + 1, 1, 2, [0], [most + 1])[0] == ctc.STATUS_UNSUPPORTED
    frames, B = 35791, 60000                             # just below 2^31 frames together, just above in whole blocks
    assert B * frames < 2**31 < B * ((frames + 15) // 16 * 16)
    assert ctc.workspace_size(frames, B, 2, np.zeros(B, dtype=np.int32), np.full(B, frames, dtype=np.int32)) > 0
