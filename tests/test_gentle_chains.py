"""Gentle utterances (no probability below 2^-32): their chains look after their frames before the last step of every chunk, in a wider range than
others, and take what is handed up by a shift.  The rule, with the constants of the source, keeps values within fp64: replayed on the CPU over nine steps
between looks, every value as far out as a shift may have put it."""
import os
import re

import pytest

import test_frame_renewals as renewals

SOURCE = os.path.join(renewals.ROOT, "paper_1512_02595_amd", "csrc", "ctc_kernels.hip")


def constant(name):
    return float(re.search(r"\b%s = (-?[\d.]+)[,;]" % name, open(SOURCE).read())[1])


@pytest.mark.parametrize("who", ["blank", "labels"])
@pytest.mark.parametrize("bits", [20, 31])
def test_nine_steps_between_looks(bits, who, monkeypatch):
    monkeypatch.setitem(renewals.K, "kEasyLow", constant("kGentleLow") - constant("kShiftDown"))
    monkeypatch.setitem(renewals.K, "kEasyHigh", constant("kGentleHigh") + constant("kShiftUp"))
    monkeypatch.setitem(renewals.K, "kSmoothFrames", constant("kGentleSmooth"))
    for x, label, blank, want in renewals.utterances(bits, who):
        got, _ = renewals.chain_cost(x, label, blank, 9)
        assert abs(got - want) <= 1e-9 * abs(want), (len(label), got, want)
