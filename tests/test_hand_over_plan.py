"""The plans that linear-domain chains run by (ctc_internal.h: linear_plan2, linear_two_pairs), checked on the CPU for every label
length: they hand over at the ends of blocks, so what a halo keeps exact must last for one, and every pair needs a lane."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "ctc_internal.h"
int main()
{
    for (int crowded = 0; crowded < 2; ++crowded)
        for (int L = 0; L <= CTC_MAX_LABEL_LENGTH; ++L) {
            const ctc::WavePlan one = ctc::plan_waves(L, crowded != 0), two = ctc::linear_plan2(L, crowded != 0);
            std::printf("%d %d %d %d %d %d %d\n", L, one.waves, one.halo, one.barrier ? 1 : 0, two.waves, two.halo,
                        ctc::linear_two_pairs(L, crowded != 0) ? 1 : 0);
        }
    std::printf("%d\n", ctc::kBlockFrames);
}
"""


def test_halos_last_for_a_block(tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1512_02595_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    *rows, block = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(rows) == 2 * 1024
    for L, waves, halo, barrier, waves2, halo2, two in (map(int, row.split()) for row in rows):
        pairs, lanes = L + 1, (L + 2) // 2
        if not two:
            assert not barrier and waves <= 4
            assert waves == 1 or halo >= int(block), (L, waves, halo)
            continue
        assert waves2 * (64 - halo2) + halo2 >= lanes and waves2 <= 16, (L, waves2, halo2)
        assert halo2 <= 16 and (waves2 == 1 or 2 * halo2 >= int(block)), (L, waves2, halo2)
        assert pairs > 64
