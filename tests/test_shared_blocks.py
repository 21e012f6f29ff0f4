"""The rule by which late utterances get several wavefronts to a block of the gradient (blocks_to_share in ctc_internal.h), on the CPU: batches as they were measured. One whose
late utterances alone fill the chip shares nothing."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include "ctc_internal.h"
int main()
{
    long late;
    int chains;
    while (std::scanf("%ld %d", &late, &chains) == 2) std::printf("%d\n", ctc::blocks_to_share(late, chains, 256));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("share")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1512_02595_amd", "csrc"),
                    str(d / "rule.cpp"), "-o", str(d / "rule")], check=True)
    return lambda late, chains: int(subprocess.run([str(d / "rule")], input=f"{late} {chains}", capture_output=True, text=True, check=True).stdout)


@pytest.mark.parametrize("utterances,frames,symbols,pieces", [(64, 750, 225, 3), (128, 750, 225, 3), (128, 750, 300, 3), (32, 1500, 540, 6), (48, 1500, 400, 4), (128, 750, 130, 2)])
def test_utterances_that_end_together_share_nothing(rule, utterances, frames, symbols, pieces):
    """us a call, none shared and 8192 blocks times pieces: 61.8 and 72.3, 82.1 and 92.6, 92.5 and 101.8, 152.7 and 166.1, 116.5 and 119.9, 62.5 and 66.9."""
    assert rule(utterances * ((frames + 15) // 16) * pieces, 2 * utterances) == 0


@pytest.mark.parametrize("late,chains,share", [(2847, 64, 8192), (2770, 64, 8192), (1305, 256, 8192), (4096, 256, 8192), (4097, 256, 0), (2000, 258, 2048), (-1, 64, 2048), (-1, 1024, 2048)])
def test_mixed_batches(rule, late, chains, share):
    """32 x 1500, lengths from 1200 and from 400 on, and 128 x 750: 122.9 and 111.2, 120.3 and 108.5, 49.2 and 45.0; crowded launches and unknown lengths in between."""
    assert rule(late, chains) == share
