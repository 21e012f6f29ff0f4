"""Minibatches whose symbols are held against the blank for dozens of frames, and transcripts that lack some of them."""
import numpy as np

from paper_1512_02595_amd import workloads as wl


def held_batch(hold, depth, blanks, A=29, B=24, T=750, seed=0):
    """Nothing but stretches of about `hold` frames of one of three symbols (blanks: or the blank, as often), `depth` nats above the rest;
    the transcripts lack about 40 % of them."""
    rng = np.random.default_rng([hold, depth, blanks, seed])
    x = rng.normal(0, 1, (T, B, A)).astype(np.float32)
    labels = []
    for b in range(B):
        t, said = 0, []
        while t < T:
            symbol = 0 if blanks and rng.random() < 0.5 else int(rng.integers(1, 4))
            frames = int(rng.integers(hold // 2, hold * 3 // 2 + 1))
            x[t:t + frames, b, symbol] += depth
            t += frames
            if symbol:
                said.append(symbol)
        labels.append([s for s in said if rng.random() > 0.4])
    lengths = np.asarray([len(s) for s in labels], dtype=np.int32)
    flat = np.asarray([k for s in labels for k in s], dtype=np.int32)
    return wl.CTCBatch(f"held for {hold} frames at {depth} nats", T, B, A, 0, x, flat, lengths, np.full(B, T, dtype=np.int32), seed=seed)


def speech_with_held_symbols(symbols, A, B, hold=60, depth=16.0, every=None, blank=0, seed=0):
    """Every symbol of the text has two frames and the blank one or two between them; after some symbols three held ones, of which
    the transcript lacks about a third."""
    every = every or min(25, symbols // 3)
    rng = np.random.default_rng([symbols, A, B, hold, seed])
    utterances = []
    for b in range(B):
        rows, said = [], []
        n = int(symbols * rng.uniform(0.8, 1.0))
        for i in range(n):
            k = int(rng.integers(0, A - 1))
            k += k >= blank
            rows += [(k, 6.0)] * 2 + [(blank, 5.0)] * int(rng.integers(1, 3))
            said.append(k)
            if i % every == every - 1:
                for _ in range(3):
                    k = int(rng.integers(0, 3))
                    k += k >= blank
                    rows += [(k, depth)] * int(rng.integers(hold // 2, hold * 3 // 2 + 1))
                    if rng.random() > 0.35:
                        said.append(k)
        utterances.append((rows, said))
    frames = np.asarray([len(rows) for rows, _ in utterances], dtype=np.int32)
    lengths = np.asarray([len(said) for _, said in utterances], dtype=np.int32)
    x = rng.normal(0, 1, (int(frames.max()), B, A)).astype(np.float32)
    for b, (rows, _) in enumerate(utterances):
        for t, (k, up) in enumerate(rows):
            x[t, b, k] += up
    flat = np.asarray([k for _, said in utterances for k in said], dtype=np.int32)
    return wl.CTCBatch(f"speech of {symbols} symbols with held ones", int(frames.max()), B, A, blank, x, flat, lengths, frames, seed=seed)
