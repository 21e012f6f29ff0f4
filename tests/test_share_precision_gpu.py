"""GPU test of how exactly the shares of label positions are summed (alphabets of at most 64 symbols: matrix cores, two fp16
halves a share).  Equal logits over 32 symbols make every emission 2^-5 exactly, so that alpha and beta are numbers of paths
times a power of two: exact in the chains and, while there are fewer than 2^21, in the 20 bits that the recomputation keeps of
alpha.  A share is such a number over that of all paths."""
from math import comb

import numpy as np
import pytest

from oracle import ctc_oracle as orc
from paper_1512_02595_amd import harness
from paper_1512_02595_amd import workloads as wl

pytestmark = pytest.mark.gpu

A = 32


def test_shares_keep_their_bits():
    def paths(t, n):                             # of t frames through n different symbols
        return comb(t + n, 2 * n)

    # (16 frames to spare at least: fewer run the log domain)
    frames, labels = zip(*[(t, n) for n in (1, 2, 3, 4) for t in range(n + 16, 161, 3) if paths(t, n) < 1 << 53])
    B, T = len(frames), max(frames)
    flat = np.concatenate([(np.arange(n) * 7 + b) % (A - 1) + 1 for b, n in enumerate(labels)]).astype(np.int32)
    batch = wl.CTCBatch("equal logits", T, B, A, 0, np.zeros((T, B, A), dtype=np.float32), flat,
                        np.asarray(labels, dtype=np.int32), np.asarray(frames, dtype=np.int32), seed=0)
    _, ref = orc.ctc_loss_and_grad(batch.logits, flat, batch.label_lengths, batch.input_lengths, 0)
    _, got = harness.run_batch(batch)
    # Of a label's column, in units u = 2^-24 of the occupancy: rounding the share to fp32 1, its two halves 2, the product with
    # 1 / p 1; the difference from y 1 of the result.  (Halves rounded toward zero: up to 6 in place of 2.)  1 / p itself keeps
    # the top 20 bits of its mantissa, a factor common to the utterance.
    u, worst = 2.0 ** -24, 0.0
    at = 0
    for b, n in enumerate(labels):
        symbols = flat[at:at + n]
        at += n
        mantissa = np.frexp(float(paths(frames[b], n)))[0]
        factor = np.floor(2.0 ** 20 / mantissa) / 2.0 ** 20 * mantissa
        exact = [t for t in range(frames[b]) if paths(t + 1, n) < 1 << 21]
        grad, want = got[exact][:, b, symbols].astype(np.float64), ref[exact][:, b, symbols]
        occupancy = 2.0 ** -5 - want
        error = np.abs(2.0 ** -5 - grad - factor * occupancy) / (4 * u * occupancy + u * np.abs(want) + 1e-14)
        worst = max(worst, error.max())
    print(f"  largest error, of the bound: {worst:.2f}", flush=True)
    assert worst <= 1.0
