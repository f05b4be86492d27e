"""Where the lanes of the redundancy stream put the streamed rows' weights: the kernel's own index map on the CPU."""
import subprocess

import paper_2412_08521_amd.build as build

PROGRAM = r"""
#include <cstdio>
#include "ems_red_weights.h"
int main()
{
    using W = ems::RedWeights;
    std::printf("%d %d %d\n", W::kFloats, W::kSecond, (int)W::sound());
    for (int lane = 0; lane < W::kLanes; ++lane) std::printf("%d %d\n", W::slot(lane), (int)W::holds(lane));
}
"""


def test_every_store_of_a_weight_lies_in_its_stage(tmp_path):
    """Both stores of all 64 lanes inside the stage's array, each of the 32 rows written by the one lane that holds it."""
    assert "ems_red_weights.h" in build.HEADERS            # a change to it rebuilds the kernel
    src, exe = tmp_path / "weights.cpp", tmp_path / "weights"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", f"-I{build.CSRC}", str(src), "-o", str(exe)], check=True)
    first, *lanes = [tuple(map(int, x.split())) for x in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()]
    n_floats, second, sound = first
    assert len(lanes) == 64
    written = {}
    for lane, (slot, holds) in enumerate(lanes):
        # lane l of a 16x16 accumulator: rows 4 (l / 16) .. + 3 of column l % 16
        assert holds == (lane % 16 in range(4 * (lane // 16), 4 * (lane // 16) + 4))
        for at in (slot, slot + second):
            assert 0 <= at < n_floats, (lane, at, n_floats)
            if at < 32:
                assert holds and at % 16 == lane % 16
                assert written.setdefault(at, lane) == lane
    assert sorted(written) == list(range(32))
    assert sound

