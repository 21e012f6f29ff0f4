"""GPU test of the probabilities in the gradient of small alphabets, which are stored as ratios to the blank's and multiplied by it again:
with empty labels the gradient is the softmax but for the blank's column.  The yardstick is the same product of roundings in numpy's fp32
(exponential over sum, divided by the blank's, times the blank's); the GPU's exponential is good to an ulp where numpy's is rounded, and
its sums have another order, which may cost a tenth of the whole."""
import numpy as np
import pytest

from paper_1512_02595_amd import harness
from paper_1512_02595_amd import workloads as wl

pytestmark = pytest.mark.gpu


def in_fp32(x, blank):
    f = np.float32
    e = np.exp2((x - x.max(axis=2, keepdims=True)) * f(1.4426950408889634)).astype(f)
    quarter = [e[:, :, i::4].cumsum(axis=2, dtype=f)[:, :, -1:] for i in range(4)]
    y = e * (f(1) / ((quarter[0] + quarter[1]) + (quarter[2] + quarter[3])))
    norm = y[:, :, blank:blank + 1]
    return (y / norm) * norm


@pytest.mark.parametrize("A", [29, 60])
@pytest.mark.parametrize("sigma", [1.0, 2.0, 6.0])
def test_probabilities_of_symbols_in_no_label(A, sigma):
    T, B, blank = 300, 48, 0
    x = np.random.default_rng([A, int(sigma)]).normal(0, sigma, (T, B, A)).astype(np.float32)
    x[:, :, blank] += 1.5 * sigma
    nothing = np.zeros(B, dtype=np.int32)
    batch = wl.CTCBatch("empty labels", T, B, A, blank, x, np.zeros(0, dtype=np.int32), nothing, np.full(B, T, dtype=np.int32), seed=0)
    _, grads = harness.run_batch(batch)
    x64 = x.astype(np.float64)
    y = np.exp(x64 - x64.max(axis=2, keepdims=True))
    y /= y.sum(axis=2, keepdims=True)

    def error(got):
        return np.linalg.norm(got[:, :, 1:] - y[:, :, 1:]) / np.linalg.norm(y[:, :, 1:])

    got, yardstick = error(grads.astype(np.float64)), error(in_fp32(x, blank).astype(np.float64))
    print(f"  A={A} sigma={sigma}: error {got:.3e}, in numpy's fp32 {yardstick:.3e}", flush=True)
    assert got <= 1.1 * yardstick
