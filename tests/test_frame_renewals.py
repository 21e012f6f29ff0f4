"""The rule by which the chains of the linear domain look after their lanes' exponents (ChainFrames in ctc_kernels.hip), replayed on the
CPU in fp64 with the constants of the source: looks every 16, 8 or 4 frames keep the values of an utterance within fp64 where its
probabilities are above 2^-32, 2^-79 and 2^-100, and the inputs of the GPU tests (probability_stretches) are such that looking too
seldom does not.  And the rule by which they notice that a lane's exponent does not hold its states, on symbols held against the blank."""
import os
import re

import numpy as np
import pytest

from oracle import ctc_oracle as orc
from held_symbols import held_batch
from probability_stretches import batch_of_stretches

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def constants():
    found = {}
    for name in ("ctc_kernels.hip", "ctc_internal.h"):
        text = open(os.path.join(ROOT, "paper_1512_02595_amd", "csrc", name)).read()
        for key in ("kFrameSlack", "kFrameDrop", "kEasyLow", "kEasyHigh", "kSmoothFrames", "kSteepSmoothFrames", "kGentleMinLog2",
                    "kRoughMinLog2", "kLinearMinLog2", "kSteepSteps", "kStrained"):
            m = re.search(r"\b%s = (-?[\d.]+)f?[,;]" % key, text)
            if m:
                found[key] = float(m[1])
    return found


K = constants()
NOTHING = -(1 << 28)


def chain_cost(x, label, blank, every):
    """-ln p of one utterance by a chain of one pair per lane that looks after its frames every `every` steps: a block's, a chunk's
    or a steep one's rule (renewals between the looks of a block where lanes are rough, as the chain does).  And whether it has noticed (strains)."""
    T, L = len(x), len(label)
    lp = x.astype(np.float64) - np.logaddexp.reduce(x.astype(np.float64), axis=1)[:, None]
    ratio = np.zeros((T, L + 1))
    ratio[:, :L] = np.exp(lp[:, label] - lp[:, [blank]])
    skip = np.zeros(L + 1)
    skip[1:L] = label[1:] != label[:-1]
    steep = every == K["kSteepSteps"]
    smooth, reach = (K["kSteepSmoothFrames"], every) if steep else (K["kSmoothFrames"], 8)
    vb, vl = np.zeros(L + 1), np.zeros(L + 1)
    vb[0] = 1.0
    frame = np.zeros(L + 1, dtype=np.int64)
    scale, rough, strained = np.ones(L + 1), True, False

    def shifted(v, fill):
        return np.concatenate([[fill], v[:-1]])

    def rescale(massless):
        nonlocal scale, rough
        down = shifted(frame, NOTHING) - frame
        scale = np.ldexp(1.0, np.clip(down, -1100, 1023))
        rough = bool((down > smooth).any() or ((down < -smooth) & massless)[1:].any())

    def renew():
        nonlocal frame, vb, vl, strained
        top = np.maximum(vb, vl)
        mass = top > 0
        mine = np.where(mass, frame + np.frexp(top)[1], NOTHING)
        window = mine.copy()
        below = mine
        for _ in range(reach):
            below = shifted(below, NOTHING)
            window = np.maximum(window, below)
        new = window - np.minimum(np.maximum(window - mine - int(K["kFrameSlack"]), 0), int(K["kFrameDrop"]))
        front = np.nonzero(mass)[0].max()
        new[front + 1:] = new[front]
        strained = strained or bool((np.frexp(vb)[1] + frame - new < K["kStrained"]).any())
        vb, vl = np.ldexp(vb, frame - new), np.ldexp(vl, frame - new)
        frame = new
        rescale(~mass)

    def due():
        top = np.maximum(vb, vl)
        mass = top > 0
        with np.errstate(divide="ignore"):
            e = np.frexp(top)[1] - 1
        return rough or bool((mass & ((e < K["kEasyLow"]) | (e > K["kEasyHigh"]) | ~np.isfinite(top))).any())

    with np.errstate(over="ignore", under="ignore", invalid="ignore"):
        for t in range(T):
            prev = shifted(vl, 0.0)
            i_label = prev * skip * scale + (vb + vl)
            vb = prev * scale + vb
            vl = i_label * ratio[t]
            if not np.isfinite(vb).all() or not np.isfinite(vl).all():
                return np.inf, strained
            if (t + 1) % every == 0:
                if due():
                    renew()
            elif (t + 1) % 8 == 0 and rough and due():
                renew()
        p = vb[L] + shifted(vl, 0.0)[L] * scale[L]
    if not p > 0:
        return np.inf, strained
    return -(np.log(p) + frame[L] * np.log(2.0)) - lp[:, blank].sum(), strained


def utterances_of(batch):
    costs = orc.ctc_loss_and_grad(batch.logits, batch.flat_labels, batch.label_lengths, batch.input_lengths, batch.blank, want_grad=False)[0]
    at = 0
    for b in range(batch.B):
        label = batch.flat_labels[at:at + batch.label_lengths[b]]
        at += int(batch.label_lengths[b])
        yield batch.logits[:batch.input_lengths[b], b], label, batch.blank, costs[b]


def utterances(bits, who):
    return utterances_of(batch_of_stretches(bits, who, 24))


@pytest.mark.parametrize("who", ["blank", "labels"])
@pytest.mark.parametrize("bits,every", [(31, 16), (33, 8), (78, 8), (81, 4), (99, 4)])
def test_looking_as_often_as_the_probabilities_ask_for(bits, every, who):
    for x, label, blank, want in utterances(bits, who):
        got, _ = chain_cost(x, label, blank, every)
        assert abs(got - want) <= 1e-9 * abs(want), (len(label), got, want)


@pytest.mark.parametrize("bits", [78, 99])
def test_the_inputs_ask_for_it(bits):
    """Looked after once a block only, the chains of these inputs leave fp64's range."""
    lost = [not abs(chain_cost(x, label, blank, 16)[0] - want) <= 1e-9 * abs(want) for x, label, blank, want in utterances(bits, "blank")]
    assert np.mean(lost) >= 0.5


def test_constants_are_those_of_the_classes():
    assert (K["kGentleMinLog2"], K["kRoughMinLog2"], K["kLinearMinLog2"], K["kSteepSteps"]) == (-32, -79, -100, 4)


# (every: of utterances with probabilities below 2^-32, which these are)
@pytest.mark.parametrize("hold,depth,blanks,most", [(10, 10, True, 2), (60, 20, True, 24), (100, 14, True, 24), (60, 14, False, 24)])
def test_chains_notice_states_that_their_frames_do_not_hold(hold, depth, blanks, most):
    """Wherever the cost is wrong the chain has noticed; and it hardly notices anything where symbols are held for ten frames only."""
    noticed = wrong = 0
    for x, label, blank, want in utterances_of(held_batch(hold, depth, blanks)):
        got, strained = chain_cost(x, label, blank, 8)
        right = abs(got - want) <= 1e-6 * abs(want) + 1e-9
        assert right or strained, (len(label), got, want)
        noticed += strained
        wrong += not right
    print(f"  {noticed} noticed, {wrong} wrong")
    assert noticed <= most and (wrong > 0) == (blanks and most == 24)
