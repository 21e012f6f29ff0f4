"""Utterances of more than a million frames over more than 64 symbols: the label columns' launch has a workgroup per block of 16 frames,
more than one dimension of a grid takes."""
import os
import subprocess

import numpy as np
import pytest

from paper_1512_02595_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include "ctc_internal.h"
int main()
{
    for (int rows; std::scanf("%d", &rows) == 1;) {
        const ctc::WideRows w = ctc::wide_rows(rows);
        std::printf("%d %d\n", w.y, w.z);
    }
}
"""


def test_a_grid_takes_every_number_of_blocks(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1512_02595_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    most = (2**31 - 1) // 16 // 16 + 256                 # blocks of the longest utterance that is accepted, and rounds of zero rows
    counts = [1, 2, 32, 65534, 65535, 65536, 65537, 131070, 131071, 131072, 2621440, most]
    out = subprocess.run([str(exe)], input="\n".join(map(str, counts)), capture_output=True, text=True, check=True).stdout.split()
    for n, y, z in zip(counts, map(int, out[::2]), map(int, out[1::2])):
        assert 1 <= y <= 65535 and 1 <= z <= 65535 and n <= y * z < n + z, (n, y, z)
        assert n > 65535 or (y, z) == (n, 1)


@pytest.mark.gpu
def test_more_blocks_than_one_dimension_of_a_grid():
    import parity_checks as pc
    T, A = 16 * 65535 + 37, 65
    frames = np.asarray([T], dtype=np.int32)
    labels = np.asarray([3, 9], dtype=np.int32)
    x = np.random.default_rng(5).normal(0, 1, (T, 1, A)).astype(np.float32)
    x[:, :, 0] += 3.0
    pc.check(wl.CTCBatch("many frames", T, 1, A, 0, x, labels, np.asarray([2], dtype=np.int32), frames, seed=5))
