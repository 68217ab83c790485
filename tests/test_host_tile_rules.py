"""The sizes at which a handle changes to launches of the library's own follow the
device's compute units (host build of the rules): 256 of a whole MI355X, 128 to
32 of a partition.
"""
import os
import subprocess

import pytest

import test_host_replay as R

PROGRAM = r"""
#include <cstdio>
#include "lbm_node.h"
#include "lbm_tiles.h"
using namespace lbm;
int main() {
    for (int cu : {256, 128, 64, 32}) {
        int deep = 0, three = 0;
        while (deep_fits(deep + 1, cu)) ++deep;
        while (!three_steps(ST_F64, {three, three, three}, cu)) ++three;
        printf("%d %d %d %d %d\n", cu, deep, three, (int)three_steps(ST5_F64, {1, 1, 1}, cu),
               (int)three_steps(ST_F32, {9999, 0, 99999}, cu));
    }
    // beyond one round: the fullest CU's tiles, or few at walls
    auto q9 = [](int64_t three, int64_t wall, int64_t two) { return (int)three_steps(ST_F64, {three, wall, two}); };
    printf("%d %d %d %d %d %d %d %d\n", kDeepTiles, q9(384, 384, 384), q9(512, 512, 512), q9(513, 513, 1024),
           q9(513, 513, 1025), q9(768, 230, 768), q9(768, 231, 768), q9(4096, 4096, 6560));
}
"""


def test_own_launches_follow_the_compute_units(tmp_path):
    if not os.path.exists(R.CXX):
        pytest.skip("no host clang++")
    src, exe = tmp_path / "rules.cpp", str(tmp_path / "rules")
    src.write_text(PROGRAM)
    subprocess.check_call([R.CXX, "-std=c++17", "-O0", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + R.CSRC,
                           "-o", exe, str(src)])
    code, out = R._run(exe, "")
    assert code == 0, out
    rows = [[int(v) for v in line.split()] for line in out.splitlines()]
    # CUs, most deep tiles, fewest three-step FP64 D2Q9 tiles, D2Q5 always, others never
    assert rows[:4] == [[256, 256, 384, 1, 0], [128, 128, 192, 1, 0], [64, 64, 96, 1, 0], [32, 32, 48, 1, 0]]
    assert rows[4] == [256, 1, 1, 0, 1, 1, 0, 1]
