"""Lanes of a linear-domain chain behind the label's end have no label states: their emissions lie past the end of the buffer (emission_column in ctc_internal.h), whose loads
give 0, so that they hold no mass and a wavefront renews its frames as often as if there were none of them.  The rule on the CPU, for every label length, and the chains' replay."""
import os
import subprocess

import numpy as np
import pytest

from chain_replay import ROOT, Chain

PROGRAM = r"""
#include <cstdio>
#include "ctc_internal.h"
int main()
{
    for (int L = 0; L <= CTC_MAX_LABEL_LENGTH; ++L)
        for (int j = 0; j < 1100; ++j) {
            const unsigned at = ctc::emission_column(j, L, j + 3);
            if (j < L ? at != 32u * (j + 3) : (at < ctc::kNoColumn || at + 32u < at)) std::printf("%d %d %u\n", L, j, at);
        }
    std::printf("%u\n", ctc::kNoColumn);
}
"""


def test_pairs_without_a_label_state_read_past_the_end(tmp_path):
    src, exe = tmp_path / "columns.cpp", tmp_path / "columns"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1512_02595_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split() == [str(1 << 31)]
    # (the buffer ends one byte before; nobody who reads emissions takes another column)
    text = open(os.path.join(ROOT, "paper_1512_02595_amd", "csrc", "ctc_kernels.hip")).read()
    emissions = text[text.index("struct ChainEmissions"):text.index("struct ChainEmissions") + 2500]
    assert "static_cast<int>(kNoColumn - 1)" in emissions and "return emission_column(j, m.L, " in emissions


def utterance(symbols, deviation, seed, T=750, A=29):
    rng = np.random.default_rng([symbols, seed])
    x = (deviation * rng.standard_normal((T, A))).astype(np.float32)
    x[:, 0] += 3.0
    return x, rng.integers(1, A, symbols)


# (40 symbols and 20: their wavefronts' 64 lanes are mostly behind the label; 190, 240: in the plans' last wavefront 17 of 64 and 36 of 64 are)
@pytest.mark.parametrize("symbols,pairs,lanes,deviation", [(20, 1, 64, 4), (40, 1, 64, 4), (40, 1, 64, 6), (190, 1, 208, 2), (240, 2, 160, 2), (240, 2, 160, 4)])
def test_they_call_for_no_renewal(symbols, pairs, lanes, deviation):
    counts = np.zeros(3, dtype=int)
    for seed in range(4):
        x, label = utterance(symbols, deviation, seed)
        kind = "gentle" if deviation <= 2 else "rough"
        for backward in (False, True):
            have = dict(pairs=pairs, backward=backward)
            without = Chain(x, label, 0, kind, lanes=(symbols + pairs) // pairs, **have)
            given = [Chain(x, label, 0, kind, lanes=lanes, behind=behind, **have) for behind in (False, True)]
            assert abs(given[0].cost - without.cost) <= 1e-12 * without.cost and given[0].renewals == without.renewals
            counts += [without.renewals, given[0].renewals, given[1].renewals]
    print(f"  renewals without lanes behind, with them, where those read the last symbol's emissions: {counts}")
    assert counts[2] > counts[0]                         # (these inputs ask for it)
