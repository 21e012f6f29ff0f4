"""The linear domain's chains (run_chain_linear, run_chain_linear2 in ctc_kernels.hip) replayed on the CPU in fp64 with the constants of the source: their classes
of utterances, one pair and two to a lane, one wavefront and several with what they hand up, looks a step before a chunk ends, renewals, headroom and shifts.
A wavefront finds what it asks for here (in the kernel it waits until it does); what leaves the recursion is not followed."""
import os
import re

import numpy as np

from oracle import ctc_oracle as orc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NOTHING = -(1 << 28)
CHUNK = 8


def constants():
    found = {}
    for name in ("ctc_kernels.hip", "ctc_internal.h"):
        text = open(os.path.join(ROOT, "paper_1512_02595_amd", "csrc", name)).read()
        for m in re.finditer(r"\b(k[A-Z]\w*) = (-?\d+)(?:\.\d*f?)?[,;]", text):
            found.setdefault(m[1], int(m[2]))
    return found


def class_of(bits):
    """bits: the smallest probability is 2^-bits."""
    k = constants()
    return "gentle" if bits <= -k["kGentleMinLog2"] else ("rough" if bits <= -k["kRoughMinLog2"] else "steep")


class Chain:
    """One chain.  `x`: [frames, symbols]; halo, waves: as the plans give them (lanes); `lanes` of a wavefront.  `behind`: pairs from L on read the last symbol's
    emissions, where they have none."""

    def __init__(self, x, label, blank, kind, pairs=1, waves=1, halo=0, backward=False, lanes=64, behind=False, **changed):
        k = {**constants(), **changed}
        self.k, self.kind, self.pairs, self.waves, self.halo, self.L = k, kind, pairs, waves, halo, len(label)
        lp = x.astype(np.float64) - np.logaddexp.reduce(x.astype(np.float64), axis=1)[:, None]
        if backward:
            lp, label = lp[::-1], label[::-1]
        self.norms = lp[:, blank].sum()
        self.lanes = lanes
        self.first = pairs * (np.arange(waves)[:, None] * (lanes - halo) + np.arange(lanes)[None, :])
        self.pair = self.first[:, :, None] + np.arange(pairs)
        assert self.pair.max() >= self.L and halo <= lanes - halo
        T, blocks = len(x), (len(x) + 15) // 16
        ratio = np.zeros((blocks * 16, self.L + 1))
        ratio[:T, :self.L] = np.exp(lp[:, label] - lp[:, [blank]])
        reads = np.where(self.pair < self.L, self.pair, self.L - 1 if behind and self.L else self.L)
        self.emission = ratio[:, reads]                  # [frame, wavefront, lane, pair]
        skip = np.zeros(self.L + 1, dtype=bool)
        skip[1:self.L] = label[1:] != label[:-1]
        self.skip = skip[np.minimum(self.pair, self.L)].astype(float)
        self.blank, self.label = (self.pair == 0).astype(float), np.zeros(self.pair.shape)
        self.frame = np.zeros((waves, lanes), dtype=np.int64)
        self.scale = np.ones((waves, lanes))
        self.rough = np.ones(waves, dtype=bool)
        gentle, steep = kind == "gentle", kind == "steep"
        name = "kGentle" if gentle else ("kEasy" if steep else "kRough")
        self.low, self.high = k[name + "Low"], k[name + "High"]
        self.smooth = pairs * (k["kGentleSmooth"] if gentle else (k["kSteepSmoothFrames"] if steep else k["kSmoothFrames"]))
        self.headroom = k["kHeadroom"] if gentle else 0
        self.reach = (k["kSteepSteps"] if steep else CHUNK) // pairs
        self.shift_down, self.shift_up = (k["kShiftDown"], k["kShiftUp"]) if gentle else (0, 0)
        self.strained_below = k["kGentleStrained"] if gentle and "kGentleStrained" in k else k["kStrained"]
        self.exchange = 0 if waves == 1 else (1 if pairs * halo < 32 else 2)     # blocks between hand-overs
        self.renewals = self.unusual = 0
        self.lowest = 0                                  # exponent of the least first blank that a shift down has left, before any wavefront would have left the recursion
        self.strained = self.overflowed = False
        with np.errstate(over="ignore", under="ignore", invalid="ignore"):
            self.run(blocks)

    def top(self):
        return np.fmax(self.blank, self.label).max(axis=-1)

    def outside(self, top):
        e = np.where(np.isfinite(top), np.frexp(np.where(np.isfinite(top), top, 0.0))[1], 0) - 1
        return (e < self.low) | (e > self.high)

    def step(self, t):
        prev = np.concatenate([np.zeros((self.waves, 1)), self.label[:, :-1, -1]], axis=1)
        e = self.emission[t]
        blank, label = self.blank.copy(), self.label.copy()
        self.label[..., 0] = ((prev * (self.skip[..., 0] * self.scale)) + (blank[..., 0] + label[..., 0])) * e[..., 0]
        self.blank[..., 0] = prev * self.scale + blank[..., 0]
        if self.pairs == 2:
            self.label[..., 1] = (label[..., 0] * self.skip[..., 1] + (blank[..., 1] + label[..., 1])) * e[..., 1]
            self.blank[..., 1] = blank[..., 1] + label[..., 0]
        of_label = self.pair <= self.L
        self.overflowed = self.overflowed or not (np.isfinite(self.blank[of_label]).all() and np.isfinite(self.label[self.pair < self.L]).all())

    def rescale(self, w, massless):
        down = np.concatenate([[NOTHING], self.frame[w, :-1]]) - self.frame[w]
        self.scale[w] = np.ldexp(1.0, np.clip(down, -1100, 1023))
        self.rough[w] = bool((down > self.smooth).any() or ((down < -self.smooth) & massless)[1:].any())

    def renew(self, w):
        k = self.k
        self.renewals += 1
        top = self.top()[w]
        mass = top > 0
        mine = np.where(mass, self.frame[w] + np.frexp(top)[1], NOTHING)
        window, below = mine.copy(), mine
        for _ in range(self.reach):
            below = np.concatenate([[NOTHING], below[:-1]])
            window = np.maximum(window, below)
        new = self.frame[w].copy()
        front = max(self.halo - 1, 0)
        if mass.any():
            new = window + self.headroom - np.minimum(np.maximum(window - mine - (k["kFrameSlack"] - self.headroom), 0), k["kFrameDrop"] + self.headroom)
            front = np.nonzero(mass)[0].max()
        new[front + 1:] = new[front]
        rise = self.frame[w] - new
        first = self.blank[w, :, 0]
        self.strained = self.strained or bool(((np.frexp(first)[1] + rise < self.strained_below) & (self.first[w] <= self.L)).any())
        self.blank[w] = np.ldexp(self.blank[w], rise[:, None])
        self.label[w] = np.ldexp(self.label[w], rise[:, None])
        self.frame[w] = new
        self.rescale(w, ~mass)

    def renew_if_due(self, w):
        if self.outside(self.top()[w]).any() or self.rough[w]:
            self.renew(w)

    def end_block(self, w, outside, exchange):
        k, halo = self.k, self.halo
        unusual = bool(outside[w].any() or self.rough[w] or self.kind == "steep")
        due = bool(outside[w].any() or self.rough[w])
        handed = None
        if exchange and w > 0:
            blank, label, frame, theirs = self.handed[w - 1]
            shift = frame - self.frame[w, :halo]
            unusual = unusual or theirs or bool(((shift < -self.shift_down) | (shift > self.shift_up)).any())
        if exchange:
            if unusual and w > 0:
                self.frame[w, :halo] = frame
            up = slice(self.lanes - halo, self.lanes)
            handed = (self.blank[w, up].copy(), self.label[w, up].copy(), self.frame[w, up].copy(), due and unusual)
            if w > 0:
                shift = (frame - self.frame[w, :halo])[:, None]
                lower = (self.first[w, :halo] <= self.L) & (blank[:, 0] > 0) & (shift[:, 0] < 0)
                if lower.any() and not self.strained:
                    self.lowest = min(self.lowest, int((np.frexp(blank[:, 0])[1] + shift[:, 0])[lower].min()))
                self.blank[w, :halo], self.label[w, :halo] = np.ldexp(blank, shift), np.ldexp(label, shift)
        self.handed[w] = handed
        self.unusual += unusual
        if unusual:
            top = self.top()[w]
            renews = bool(self.outside(top).any())
            if not renews:
                if exchange:
                    self.rescale(w, ~(top > 0))
                renews = bool(self.rough[w])
            if renews:
                self.renew(w)

    def run(self, blocks):
        steep, ahead = self.kind == "steep", self.k["kLookAhead"]
        self.handed = [None] * self.waves
        for c in range(2 * blocks):
            for q in range(CHUNK):
                self.step(c * CHUNK + q)
                if steep and q == self.k["kSteepSteps"] - 1:
                    for w in range(self.waves):
                        self.renew_if_due(w)
                if q == CHUNK - 1 - ahead:
                    outside = self.outside(self.top())
            for w in range(self.waves):
                if c % 2:
                    self.end_block(w, outside, self.exchange == 1 or (self.exchange == 2 and c % 4 == 3))
                elif steep:
                    self.renew_if_due(w)
                elif outside[w].any() or self.rough[w]:
                    self.renew(w)
        w, lane, k = (int(v[0]) for v in np.nonzero((self.pair == self.L) & (np.arange(self.lanes) >= np.where(np.arange(self.waves) > 0, self.halo, 0)[:, None])[:, :, None]))
        below = self.label[w, lane, 0] if k else (self.label[w, lane - 1, -1] * self.scale[w, lane] if lane else 0.0)
        p = self.blank[w, lane, k] + below
        self.cost = -(np.log(p) + self.frame[w, lane] * np.log(2.0)) - self.norms if p > 0 and not self.overflowed else np.inf


def utterances_of(batch):
    costs = orc.ctc_loss_and_grad(batch.logits, batch.flat_labels, batch.label_lengths, batch.input_lengths, batch.blank, want_grad=False)[0]
    at = 0
    for b in range(batch.B):
        label = batch.flat_labels[at:at + batch.label_lengths[b]]
        at += int(batch.label_lengths[b])
        yield batch.logits[:batch.input_lengths[b], b], label, batch.blank, costs[b]
