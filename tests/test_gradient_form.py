"""Host-side checks of the rule by which the gradient is written beside the chains or in a launch of its own: that it takes the
batches it was made for to the form that was measured to be quicker, and that more work left at the end never favours the other."""
import subprocess
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "ctc_internal.h"
#include <cstdio>
int main()
{
    double early, late, us;
    int waves, chains;
    while (std::scanf("%lf %lf %lf %d %d", &early, &late, &us, &waves, &chains) == 5)
        std::printf("%d\n", ctc::gradient_beside_chains(early, late, us, waves, chains, 256));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1512_02595_amd", "csrc"),
                    str(d / "rule.cpp"), "-o", str(d / "rule")], check=True)

    def ask(*args):
        return subprocess.run([str(d / "rule")], input=" ".join(map(str, args)), capture_output=True, text=True, check=True).stdout == "1\n"
    return ask


@pytest.mark.parametrize("beside,early,late,us,waves,chains", [
    # blocks x pieces of the utterances that end early and late, the longest chain, wavefronts, chains
    (True, 8, 4, 2, 4, 8),                      # four short snippets
    (True, 0, 94, 45, 4, 2),                    # one utterance of 750 frames
    (True, 2200, 600, 45, 4, 128),              # 64 utterances of up to 750 frames, spread from 100: 59.9 us, apart 66.4
    (False, 700, 5600, 46, 4, 128),             # the same, spread from 640: 74.4, apart 70.7
    (False, 0, 11000, 46, 4, 256),              # 128 utterances, spread from 640: 105, apart 87
    (True, 10300, 1970, 131, 12, 64),           # 32 long transcripts among shorter ones: 157.6, apart 169.6
    (False, 35000, 19600, 131, 12, 256),        # 128 long transcripts: 468, apart 294
])
def test_measured_batches_take_the_quicker_form(rule, beside, early, late, us, waves, chains):
    assert rule(early, late, us, waves, chains) == beside


def test_more_late_work_never_favours_the_chains_launch(rule):
    for waves in (1, 4, 8, 9, 12):
        for chains in (2, 100, 256):
            forms = [rule(1000, late, 40, waves, chains) for late in range(0, 20000, 500)]
            assert forms == sorted(forms, reverse=True)


GRID_PROGRAM = r"""
#include "ctc_internal.h"
#include <cstdio>
int main()
{
    int T, B, waves, chains;
    while (std::scanf("%d %d %d %d", &T, &B, &waves, &chains) == 4)
        std::printf("%d\n", ctc::can_fuse_gradient(2, waves, chains, 256, T, B));
}
"""


# Forms by the size of the grid alone: at worst a workgroup of 64 max(waves, 4) threads to a block of 16 frames, and one more.
@pytest.mark.parametrize("T,B,waves,chains,beside", [
    (750, 512, 1, 1024, True),
    (2_100_000, 512, 1, 1024, False),           # (67 million workgroups of 256 threads)
    (1_500_000, 352, 5, 704, False),            # (33 million of 320)
    (500_000, 512, 4, 1024, True),
    (2**31 - 1, 1, 4, 2, False),
])
def test_launches_beside_the_chains_fit_a_grid(tmp_path, T, B, waves, chains, beside):
    (tmp_path / "grid.cpp").write_text(GRID_PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1512_02595_amd", "csrc"),
                    str(tmp_path / "grid.cpp"), "-o", str(tmp_path / "grid")], check=True)
    out = subprocess.run([str(tmp_path / "grid")], input=f"{T} {B} {waves} {chains}", capture_output=True, text=True, check=True).stdout
    assert (out == "1\n") == beside
    if beside:
        assert (T // 16 + 2) * B * 64 * max(waves, 4) < 2**32
