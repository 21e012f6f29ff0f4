"""GPU tests of the backtrace by segments of 32 frames: utterances whose halves end around a segment's and a chunk's end, more
segments than a workgroup has wavefronts, origins that do not fit the LDS, labels of one wavefront, of several and of those
that exchange at every step."""
import pytest

from paper_1512_02595_amd import ctc

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("A,dtype", [(29, ctc.DTYPE_F32), (300, ctc.DTYPE_BF16)])
def test_halves_around_segments(A, dtype):
    frames = [1, 2, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64, 65, 80, 96, 97, 112, 127, 128, 129, 144, 145, 255, 256, 257]
    pc.check_best(batch_of(frames, [f // 4 for f in frames], A, T=260), dtype)


@pytest.mark.parametrize("frames,labels", [([1300, 1111, 700], [90, 300, 40]),            # 21 segments, 16 wavefronts
                                           ([2500, 2200], [600, 900]),                    # origins beyond the LDS
                                           ([2300, 2100, 40], [1023, 1010, 3])])          # an exchange at every step
def test_many_segments(frames, labels):
    pc.check_best(batch_of(frames, labels, 40, sigma=1.0), min_same=0.0)
