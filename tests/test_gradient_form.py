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
    int frames, waves, chains;
    while (std::scanf("%lf %lf %lf %d %d %d", &early, &late, &us, &frames, &waves, &chains) == 6)
        std::printf("%d\n", ctc::gradient_in_lattice_launch(early, late, us, frames, waves, chains, 256));
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


@pytest.mark.parametrize("beside,early,late,us,frames,waves,chains", [
    # blocks x pieces of the utterances that end early and late, the longest chain, its frames, wavefronts, chains
    (True, 8, 4, 2, 50, 4, 8),                          # four short snippets
    (True, 0, 94, 45, 750, 4, 2),                       # one utterance of 750 frames
    (True, 2200, 600, 45, 750, 4, 128),                 # 64 utterances of up to 750 frames, spread from 100
    (True, 700, 5600, 46, 750, 4, 128),                 # the same, spread from 640
    (True, 0, 11000, 46, 750, 4, 256),                  # 128 utterances, spread from 640
    (True, 10300, 1970, 131, 1500, 12, 64),             # 32 long transcripts among shorter ones: 157.6 us, apart 169.6
    (False, 35000, 19600, 131, 1500, 12, 256),          # 128 long transcripts: 468, apart 294
    (True, 20000, 8000, 45, 750, 4, 1024),              # 512 utterances of up to 750 frames: 115.5, apart 127.3
])
def test_measured_batches_take_the_quicker_form(rule, beside, early, late, us, frames, waves, chains):
    assert rule(early, late, us, frames, waves, chains) == beside


# More chains than the 256 compute units: the limits on frames, on chains to a compute unit, and, from five wavefronts on, on late work.
@pytest.mark.parametrize("beside,early,late,frames,waves,chains", [
    (True, 0, 0, 100, 4, 256), (False, 0, 0, 100, 4, 257), (True, 0, 0, 101, 4, 257),
    (True, 0, 0, 750, 1, 1024), (False, 0, 0, 750, 1, 1025), (True, 0, 0, 750, 4, 1024), (False, 0, 0, 750, 4, 1025),
    (True, 10, 10, 750, 5, 704), (False, 10, 10, 750, 5, 705), (False, 10, 11, 750, 5, 704), (False, 10, 10, 100, 8, 300), (True, 10, 10, 101, 8, 300),
    (True, 0, 10, 750, 8, 256),
])
def test_limits_of_crowded_launches(rule, beside, early, late, frames, waves, chains):
    assert rule(early, late, 40, frames, waves, chains) == beside


def test_work_counts_for_long_chains_and_crowded_ones_of_several_wavefronts_only(rule):
    """Where beside_by_work says that the sums are not asked for, the host leaves them zero: the answer must not depend on them."""
    for waves, chains in ((1, 2), (4, 256), (8, 256), (1, 300), (4, 1024), (4, 1100)):
        assert len({rule(early, late, us, 750, waves, chains) for early in (0, 50000) for late in (0, 50000) for us in (0, 150)}) == 1


def test_more_late_work_never_favours_the_chains_launch(rule):
    for waves in (1, 4, 8, 9, 12):
        for chains in (2, 100, 256, 300, 700):
            forms = [rule(1000, late, 40, 750, waves, chains) for late in range(0, 20000, 500)]
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
