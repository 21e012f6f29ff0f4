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
    int A, chains;
    while (std::scanf("%ld %d %d", &late, &A, &chains) == 3) std::printf("%d\n", ctc::blocks_to_share(late, A, chains, 256));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("share")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1512_02595_amd", "csrc"),
                    str(d / "rule.cpp"), "-o", str(d / "rule")], check=True)
    return lambda late, A, chains: int(subprocess.run([str(d / "rule")], input=f"{late} {A} {chains}", capture_output=True, text=True, check=True).stdout)


@pytest.mark.parametrize("utterances,frames,symbols,pieces", [(64, 750, 225, 3), (128, 750, 225, 3), (128, 750, 300, 3), (32, 1500, 540, 6), (48, 1500, 400, 4), (128, 750, 130, 2)])
def test_utterances_that_end_together_share_nothing(rule, utterances, frames, symbols, pieces):
    """us a call, none shared and 8192 blocks times pieces: 61.8 and 72.3, 82.1 and 92.6, 92.5 and 101.8, 152.7 and 166.1, 116.5 and 119.9, 62.5 and 66.9."""
    assert rule(utterances * ((frames + 15) // 16) * pieces, 29, 2 * utterances) == 0


@pytest.mark.parametrize("late,A,chains,share", [(2847, 29, 64, 4096), (1305, 32, 256, 4096), (4096, 29, 256, 4096), (4097, 29, 256, 0), (1162, 37, 256, 2048), (1104, 60, 64, 2048), (4097, 60, 64, 0),
                                                 (2000, 29, 258, 2048), (-1, 29, 64, 2048), (-1, 40, 1024, 2048)])
def test_mixed_batches(rule, late, A, chains, share):
    """us a call with none, this many and 8192: 32 x 1500 x 29 122.1, 109.8, 109.5; 128 x 750 x 29 48.5, 44.7, 44.8; 128 x 768 x 37 59.3, 58.3, 69.1; 32 x 1500 x 60 134.6, 129.4, 148.7.
    Crowded launches and unknown lengths: 2048."""
    assert rule(late, A, chains) == share
