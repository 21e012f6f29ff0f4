"""GPU tests of the profiled calls: they time the launches that the plain call makes.  Where the lattice launch writes the
gradient too there is no third launch, and its time is 0 -- unless ctc_debug_set_overlap(0) gives the gradient one."""
import numpy as np
import pytest

from paper_1512_02595_amd import ctc, harness
from paper_1512_02595_amd import workloads as wl

pytestmark = pytest.mark.gpu


def plain_and_profiled(device, B, A):
    batch = wl.make_random(60 + B + A, T=90, B=B, A=A, max_label=30, min_input=50, sigma=2.0)
    if device:
        db = harness.DeviceMetaBatch(batch.T, batch.B, batch.A, 30, batch.blank, ctc.DTYPE_F32)
        db.load(batch)
    else:
        db = harness.DeviceBatch(batch)
    db.run()
    plain = db.results()[-2:]
    kernel_ms = np.full(ctc.NUM_KERNELS, -1.0, dtype=np.float32)
    db.run(kernel_ms=kernel_ms)
    profiled = db.results()[-2:]
    print(f"  {kernel_ms}", flush=True)
    assert np.array_equal(profiled[0], plain[0], equal_nan=True) and np.array_equal(profiled[1], plain[1])
    return plain, kernel_ms


@pytest.mark.parametrize("B,A,launches", [(6, 29, 2), (6, 64, 2), (6, 65, 3), (300, 29, 3)])
@pytest.mark.parametrize("device", [False, True])
def test_the_launches_of_the_plain_call(device, B, A, launches):
    _, kernel_ms = plain_and_profiled(device, B, A)
    assert (kernel_ms[:launches] > 0).all() and (kernel_ms[launches:] == 0).all()


@pytest.mark.parametrize("device", [False, True])
def test_the_overlap_switch_gives_the_gradient_a_launch(device):
    default, _ = plain_and_profiled(device, 6, 29)
    ctc.debug_set_overlap(0)
    try:
        apart, kernel_ms = plain_and_profiled(device, 6, 29)
    finally:
        ctc.debug_set_overlap(-1)
    assert (kernel_ms > 0).all()
    assert np.array_equal(apart[0], default[0], equal_nan=True) and np.array_equal(apart[1], default[1])
