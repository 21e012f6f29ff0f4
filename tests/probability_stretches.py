"""Minibatches with stretches of 16 to 64 consecutive frames in which the blank lies at 2^-bits under the label's symbols, or the
label's symbols under the blank: on block boundaries (16 frames) and 8 frames off them.  For the tests of the chains' frames."""
import numpy as np

from paper_1512_02595_amd import workloads as wl


def batch_of_stretches(bits, who, A, labels=(1, 20, 62, 63, 90, 130, 180, 230, 250, 420), copies=1, seed=0):
    rng = np.random.default_rng([bits, A, len(who), seed])
    blank = A - 1
    labels = np.asarray(list(labels) * copies, dtype=np.int32)
    frames = (2 * labels + 200 + rng.integers(0, 16, len(labels))).astype(np.int32)
    T, B = int(frames.max()), len(labels)
    flat = rng.integers(0, blank, int(labels.sum())).astype(np.int32)
    x = rng.normal(0, 0.5, (T, B, A)).astype(np.float32)
    depth = np.float32(bits * np.log(2))
    at = 0
    for b in range(B):
        symbols = np.unique(flat[at:at + labels[b]])
        at += int(labels[b])
        for start, length in ((16 + 8 * (b % 2), 64), (112 + 8 * (b % 2), 16), (150, 32)):
            t = np.arange(start, start + length)
            if who == "blank":
                x[t, b, blank] = x[t, b, :blank].max(axis=1) - depth
            else:
                rows = x[t, b]
                rows[:, symbols] = (rows[:, blank] - depth)[:, None]
                rows[:, blank] += 6.0                    # (the blank has nearly all of the frame)
                rows[:, symbols] += 6.0
                x[t, b] = rows
    return wl.CTCBatch(f"{who} at 2^-{bits}", T, B, A, blank, x, flat, labels, frames, seed=seed)
