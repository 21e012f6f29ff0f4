"""What users of this library have it compute, as cases that can be timed and compared.

A case is one call through the public binding (`paper_1512_02595_amd.ctc`) on a synthetic minibatch whose
activations sit on the GPU.  Fields of a case:

  call      "grad"    cost and gradient, labels and lengths in host arrays (ctc.loss_and_grad)
            "device"  the same with labels and lengths on the GPU (ctc.loss_and_grad_device)
            "cost"    costs only (ctc.loss_and_grad without a gradient buffer)
            "align"   most probable alignment (ctc.best_path)
  dtype     "f32" or "bf16": type of the activations and of the gradient
  B, T, A   utterances, frames of the tensor, symbols including blank; `blank` is the blank's id
  shortest  input lengths are uniform in [shortest, T]
  dense_lo, dense_hi   an utterance has a fraction of its frames as label symbols, uniform in this range

Logits are normal with the blank's column raised by 3, as in `workloads`: standard deviation 2 for alphabets of
characters and character pairs, 1 for wide ones.  Label symbols are uniform for alphabets of at most 64 symbols and
Zipf-like for larger ones; one position in twenty repeats its predecessor.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1512_02595_amd import ctc

NARROW = 64                  # alphabets of characters
CHARACTERS = 2048            # beyond this: alphabets of thousands of ideographs
MOST_VALUES = 192_000_000    # of an activation tensor (64 utterances of 500 frames over 6000 symbols)
MOST_LATTICE = 86_000_000    # utterances x frames x label symbols (512 utterances of 750 frames, 0.3 symbols a frame)
MOST_SYMBOLS = 49_000        # of a drawn minibatch's transcripts together (about those of the same 512 utterances)


def _case(name, call, dtype, B, T, A, shortest, dense_lo, dense_hi, blank=0):
    return {"name": name, "call": call, "dtype": dtype, "B": B, "T": T, "A": A, "blank": blank,
            "shortest": shortest, "dense_lo": dense_lo, "dense_hi": dense_hi}


def listed():
    return [
        # a whole 512-utterance minibatch on one GPU, unsorted
        _case("sweep", "grad", "f32", 512, 750, 29, 100, 0.15, 0.30),
        # four short snippets: what a test, a demonstration or the first epoch of a curriculum sorted by length calls
        _case("tiny", "grad", "f32", 4, 50, 29, 30, 0.15, 0.30),
        # one utterance of 15 s: validation or debugging of a single recording
        _case("one utterance", "grad", "f32", 1, 750, 29, 700, 0.15, 0.30),
        # the per-GPU English training minibatch (64 utterances of up to 15 s), the benchmark's workload
        _case("english", "grad", "f32", 64, 750, 29, 100, 0.15, 0.30),
        # the same from a training step in bf16 whose batch metadata never leaves the GPU
        _case("english bf16 device", "device", "bf16", 64, 750, 29, 100, 0.15, 0.30),
        # the same for validation: the cost alone
        _case("english cost", "cost", "f32", 64, 750, 29, 100, 0.15, 0.30),
        # the same in dataset construction: every recording aligned with its transcript
        _case("english align", "align", "f32", 64, 750, 29, 100, 0.15, 0.30),
        # utterances of up to 30 s with long transcripts
        _case("long", "grad", "f32", 32, 1500, 29, 1200, 0.20, 0.36),
        # an output layer of character pairs, time stride 3
        _case("bigram", "grad", "f32", 64, 500, 750, 67, 0.15, 0.35),
        # the Mandarin output layer
        _case("mandarin", "grad", "f32", 64, 500, 6000, 100, 0.03, 0.20),
        # the same in bf16
        _case("mandarin bf16", "grad", "bf16", 64, 500, 6000, 100, 0.03, 0.20),
        # a character set whose size is no multiple of anything, blank last, in an odd batch
        _case("odd alphabet", "grad", "f32", 27, 333, 4733, 80, 0.03, 0.20, blank=4732),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["grad", "grad", "grad", "grad", "grad", "device", "device", "cost", "align", "align"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    kind = rng.choice(["characters", "characters", "characters", "pairs", "ideographs", "ideographs"])
    if kind == "characters":
        A = rng.randint(20, NARROW)
    elif kind == "pairs":
        A = _log_uniform(rng, NARROW + 1, CHARACTERS)
    else:
        A = _log_uniform(rng, CHARACTERS + 1, 8000)
        if rng.random() < 0.5:
            A -= A % 8
    T = _log_uniform(rng, 40, 1500)
    B = _log_uniform(rng, 1, 512)
    dense_hi = rng.uniform(0.1, 0.36) if kind != "ideographs" else rng.uniform(0.05, 0.2)
    dense_lo = dense_hi * rng.uniform(0.2, 0.8)
    B = max(1, min(B, int(MOST_VALUES * 0.8) // (T * A), int(MOST_LATTICE * 0.8 / (T * T * dense_hi))))
    shortest = max(1, int(T * rng.uniform(0.1, 0.9)))
    # (at 5 bytes a symbol and 100 an utterance the metadata of one call stays near 256 KiB)
    B = max(1, min(B, int(5 * MOST_SYMBOLS / (5 * (dense_lo + dense_hi) / 2 * (shortest + T) / 2 + 100))))
    case = _case("", call, dtype, B, T, A, shortest, round(dense_lo, 4), round(dense_hi, 4),
                 blank=0 if rng.random() < 0.75 else A - 1)
    del case["name"]
    return case


def _labels(rng, case, input_lengths):
    """Flat label strings and their lengths; every utterance has an alignment."""
    A, blank = case["A"], case["blank"]
    lengths = np.floor(rng.uniform(case["dense_lo"], case["dense_hi"], case["B"]) * input_lengths).astype(np.int32)
    n = int(lengths.sum())
    if A <= NARROW:
        symbols = rng.integers(0, A - 1, n)
    else:
        weights = np.arange(1, A, dtype=np.float64) ** (-1.1 if A > CHARACTERS else -1.0)
        symbols = np.searchsorted(np.cumsum(weights / weights.sum()), rng.random(n)).clip(0, A - 2)
    symbols = symbols + (symbols >= blank)
    repeat = rng.random(n) < 0.05
    first = np.zeros(n, dtype=bool)
    starts = np.concatenate([[0], np.cumsum(lengths)[:-1]])
    first[starts[lengths > 0]] = True
    for i in np.nonzero(repeat & ~first)[0]:
        symbols[i] = symbols[i - 1]
    return symbols.astype(np.int32), lengths


def prepare(case, seed):
    B, T, A, blank = case["B"], case["T"], case["A"], case["blank"]
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(seed)
    input_lengths = rng.integers(case["shortest"], T + 1, B).astype(np.int32)
    flat, label_lengths = _labels(rng, case, input_lengths)
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    x = torch.randn((T, B, A), generator=gen, device=dev, dtype=torch.float32)
    if A <= CHARACTERS:
        x *= 2.0
    x[:, :, blank] += 3.0
    dtype = ctc.DTYPE_F32
    if case["dtype"] == "bf16":
        x = x.to(torch.bfloat16)
        dtype = ctc.DTYPE_BF16
    s = {"case": case, "x": x, "dtype": dtype, "flat": flat, "label_lengths": label_lengths,
         "input_lengths": input_lengths, "costs": torch.empty(B, dtype=torch.float32, device=dev)}
    if case["call"] in ("grad", "device"):
        s["grads"] = torch.empty_like(x)
    if case["call"] == "align":
        s["alignment"] = torch.empty((B, T), dtype=torch.int32, device=dev)
    if case["call"] == "device":
        # the padded label matrix of a training program: as wide as its longest transcript may be
        bound = max(1, int(case["dense_hi"] * T))
        padded = np.zeros((B, bound), dtype=np.int32)
        at = 0
        for b in range(B):
            padded[b, :label_lengths[b]] = flat[at:at + label_lengths[b]]
            at += int(label_lengths[b])
        s["bound"] = bound
        s["labels"] = torch.from_numpy(padded).to(dev)
        s["dev_label_lengths"] = torch.from_numpy(label_lengths).to(dev)
        s["dev_input_lengths"] = torch.from_numpy(input_lengths).to(dev)
        s["status"] = torch.empty(1, dtype=torch.int32, device=dev)
        s["ws_bytes"] = ctc.workspace_size_device(T, B, A, bound, dtype)
    else:
        s["ws_bytes"] = ctc.workspace_size(T, B, A, label_lengths, input_lengths, dtype)
    s["ws"] = torch.empty(s["ws_bytes"] + 256, dtype=torch.uint8, device=dev)
    s["ws_ptr"] = (s["ws"].data_ptr() + 255) // 256 * 256
    return s


def run(s):
    try:
        return _call(s)
    except ctc.CTCError as e:
        if e.status != ctc.STATUS_NOT_READY:
            raise
        # so far ahead of the GPU that the pinned metadata buffers are full: what the header asks a caller to do
        torch.cuda.current_stream().synchronize()
        return _call(s)


def _call(s):
    c = s["case"]
    T, B, A, blank, call = c["T"], c["B"], c["A"], c["blank"], c["call"]
    stream = torch.cuda.current_stream().cuda_stream
    if call == "device":
        ctc.loss_and_grad_device(s["x"].data_ptr(), s["labels"].data_ptr(), s["dev_label_lengths"].data_ptr(),
                                 s["dev_input_lengths"].data_ptr(), s["bound"], T, B, A, blank, s["dtype"],
                                 s["costs"].data_ptr(), s["grads"].data_ptr(), s["status"].data_ptr(),
                                 s["ws_ptr"], s["ws_bytes"], stream)
        return {"costs": s["costs"], "grads": s["grads"], "status": s["status"]}
    if call == "align":
        ctc.best_path(s["x"].data_ptr(), s["flat"], s["label_lengths"], s["input_lengths"], T, B, A, blank,
                      s["dtype"], s["costs"].data_ptr(), s["alignment"].data_ptr(), s["ws_ptr"], s["ws_bytes"], stream)
        return {"scores": s["costs"], "alignment": s["alignment"]}
    grads = s["grads"].data_ptr() if call == "grad" else None
    ctc.loss_and_grad(s["x"].data_ptr(), s["flat"], s["label_lengths"], s["input_lengths"], T, B, A, blank,
                      s["dtype"], s["costs"].data_ptr(), grads, s["ws_ptr"], s["ws_bytes"], stream)
    return {"costs": s["costs"], "grads": s["grads"]} if call == "grad" else {"costs": s["costs"]}


def work(case):
    """Every valid row of logits read once, what the call returns written once; the recursions' additions and products."""
    B, T, A = case["B"], case["T"], case["A"]
    elem = 4 if case["dtype"] == "f32" else 2
    frames = B * (case["shortest"] + T) / 2
    nbytes = frames * A * elem + 4 * B
    if case["call"] in ("grad", "device"):
        nbytes += T * B * A * elem
    if case["call"] == "align":
        nbytes += 4 * B * T
    mean_square = (case["shortest"] ** 2 + case["shortest"] * T + T ** 2) / 3          # of the input lengths
    pair_steps = B * mean_square * (case["dense_lo"] + case["dense_hi"]) / 2
    directions = 2 if case["call"] in ("grad", "device") else 1
    return {"bytes": nbytes, "flops": 4 * frames * A + 7 * pair_steps * directions}


def tolerance(case):
    # Costs and fp32 gradients: sums of 32-bit terms.  bf16: the rounding of the stored gradient.  Alignments: frames of
    # utterances that have several equally probable alignments, common only among bf16 logits.
    if case["call"] == "align":
        return {"rel": 1e-5, "differ": 1e-3 if case["dtype"] == "f32" else 1e-2}
    if case["call"] == "cost" or case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 5e-3, "max": 2e-2}
