"""How often a linear-domain chain's wavefronts hand over (Exchange in ctc_kernels.hip) follows from the halo of its plan: labels at the ends of
the plans' ranges, in few frames to spare and in more blocks than the ring of hand-overs holds, with the gradient and for the cost alone, against the oracle."""
import pytest

import parity_checks as pc
from test_block_edges_gpu import batch_of

pytestmark = pytest.mark.gpu

# one wavefront; a pair to a lane, halos of 32 and 16 pairs, two to four wavefronts; two pairs to a lane, two to five wavefronts
LABELS = [0, 1, 63, 64, 95, 96, 111, 112, 127, 128, 159, 160, 207, 208, 221, 222, 240, 301, 302, 420, 453]


@pytest.mark.parametrize("A", [29, 90])
@pytest.mark.parametrize("spare", [17, 80, 700])
def test_every_way_of_handing_over(spare, A):
    batch = batch_of([n + n // 8 + spare for n in LABELS], LABELS, A, seed=spare)
    pc.check(batch)
    pc.check_loss(batch)
