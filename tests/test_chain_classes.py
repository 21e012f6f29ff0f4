"""The chains' replay (chain_replay) for each class of utterances, with the constants of the source: gentle ones (no probability below 2^-32), rough ones (2^-79) and steep ones,
one pair to a lane and two, a wavefront and as many as the plans give, both directions.  Their costs are the oracle's, and with a limit moved past what it is for they are not: upper
limits and limits between frames, that is; the blank's ratio is 1, so that a lane's largest value falls no further than its blank."""
import numpy as np
import pytest

from chain_replay import Chain, class_of, utterances_of
from held_symbols import held_batch
from probability_stretches import batch_of_stretches
from test_block_edges_gpu import batch_of


def plan(L, pairs):
    """Wavefronts and halo (lanes): the fewest whose halo lasts for a block."""
    lanes, step = (L + pairs) // pairs, 16 // pairs
    if lanes <= 64:
        return 1, 0
    for waves in range(2, 17):
        halo = min((64 * waves - lanes) // (waves - 1), 2 * step)
        if halo >= step:
            return waves, halo - halo % step
    raise AssertionError((L, pairs))


def chains(batch, kind, **changed):
    for x, label, blank, want in utterances_of(batch):
        for pairs in (1, 2):
            waves, halo = plan(len(label), pairs)
            for backward in (False, True):
                yield Chain(x, label, blank, kind, pairs, waves, halo, backward, **changed), want


def wrong(batch, kind, **changed):
    return [not abs(chain.cost - want) <= 1e-9 * abs(want) for chain, want in chains(batch, kind, **changed)]


LABELS = (1, 20, 63, 130, 250)


@pytest.mark.parametrize("who", ["blank", "labels"])
@pytest.mark.parametrize("bits,kind", [(31, "gentle"), (33, "rough"), (78, "rough"), (81, "steep"), (99, "steep")])
def test_costs_of_each_class(bits, kind, who):
    assert class_of(bits) == kind
    assert not any(wrong(batch_of_stretches(bits, who, 24, labels=LABELS), kind))


@pytest.mark.parametrize("deviation,kind", [(2, "gentle"), (4, "rough"), (6, "rough")])
def test_costs_of_random_logits(deviation, kind):
    assert not any(wrong(batch_of([400, 150, 330, 480], [40, 64, 150, 225], 29, sigma=deviation), kind))


@pytest.mark.parametrize("bits,past", [(31, dict(kGentleHigh=800)), (31, dict(kGentleSmooth=1000)), (31, dict(kShiftUp=1200)), (78, dict(kRoughHigh=400)),
                                       (78, dict(kSmoothFrames=1000)), (78, dict(kLookAhead=7)), (99, dict(kEasyHigh=800))])
def test_limits_matter(bits, past):
    assert any(wrong(batch_of_stretches(bits, "blank", 24), class_of(bits), **past))


@pytest.mark.parametrize("hold,depth,blanks", [(10, 10, True), (60, 20, True), (100, 14, True), (60, 14, False)])
def test_each_class_notices_states_that_its_frames_do_not_hold(hold, depth, blanks):
    """Symbols held against the blank, whatever the class: wherever the cost is wrong the chain has noticed."""
    batch = held_batch(hold, depth, blanks, B=8)
    kind = "gentle" if depth / np.log(2) < 25 else "rough"
    for chain, want in chains(batch, kind):
        assert chain.strained or abs(chain.cost - want) <= 1e-6 * abs(want) + 1e-9, (chain.L, chain.cost, want)


def held_and_dropped(seed, L, symbols, T=420, B=4):
    """For 4 to 40 frames at a time some symbols at 2^31 to the blank, or at 2^-31, and the others as probable as it."""
    rng = np.random.default_rng([seed, L, symbols])
    batch = batch_of([T] * B, [L] * B, symbols + 1, seed=seed)
    batch.logits[:] = rng.normal(0, 0.05, batch.logits.shape)
    for b in range(B):
        t = 0
        while t < T:
            frames, up = int(rng.integers(4, 41)), rng.random() < 0.5
            some = np.nonzero(rng.random(symbols) < rng.choice([0.2, 0.5, 0.9]))[0] + 1
            batch.logits[t:t + frames, b, some] += (31 if up else -31) * np.log(2)
            t += frames
    return batch


def test_a_shift_rounds_no_blank():
    """Of the states that are taken by a shift a lane's first blank is the least; what it gives its label in the next step is 2^-32 of it at worst."""
    lowest = []
    for seed in range(6):
        for x, label, blank, _ in utterances_of(held_and_dropped(seed, 60 + 30 * (seed % 3), 2 + seed % 4)):
            for pairs, halo in ((1, 16), (1, 32), (2, 8), (2, 16)):
                lanes = (len(label) + pairs) // pairs
                waves = max(2, -(-(lanes - halo) // (64 - halo)))
                lowest += [Chain(x, label, blank, "gentle", pairs, waves, halo, backward).lowest for backward in (False, True)]
    print(f"  lowest first blanks after a shift: 2^{sorted(lowest)[:5]}")
    assert min(lowest) >= -1022 + 32
    assert min(lowest) < -500                            # (these inputs ask for it)
