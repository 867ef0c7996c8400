"""Which staged tiles run drained (plain C++, compiled and run here): by rows
that are no whole sectors and by the rounds a launch takes, on both sides of
the lines that the measurements drew."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "lbfss_plan.hpp"
int main(int, char **v) {  // fp16 tx ty tz snap L replicas
    const std::vector<int> L(atoi(v[7]), atoi(v[6]));
    std::vector<lbfss::FusedTile> t;
    const int tx = atoi(v[2]), ty = atoi(v[3]);
    if (lbfss::make_fused_tiles(L, tx, ty, atoi(v[4]), t)) return 1;
    printf("%d\n", lbfss::drained_plan(L, atoi(v[1]), tx, ty, (int64_t)t.size(), atoi(v[5])));
}
"""


@pytest.fixture(scope="module")
def drained(tmp_path_factory):
    d = tmp_path_factory.mktemp("drained")
    (d / "t.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_1202_4748_amd", "csrc"), "-o",
                    str(d / "t"), str(d / "t.cpp")], check=True)

    def run(L, tile, fp16=False, snap=False, replicas=1):
        a = [int(fp16), *tile, int(snap), L, replicas]
        return bool(int(subprocess.run([str(d / "t"), *map(str, a)], capture_output=True, text=True, check=True).stdout))

    return run


@pytest.mark.parametrize("L,tile,kw,want", [
    (504, (64, 8, 84), dict(fp16=True), True), (512, (64, 8, 86), dict(fp16=True), False),
    (216, (64, 8, 54), dict(fp16=True), False), (168, (32, 8, 16), dict(fp16=True), True),
    (132, (32, 8, 16), {}, True), (256, (32, 8, 16), {}, False), (100, (32, 8, 16), {}, False),
    (132, (64, 4, 16), {}, False), (196, (64, 4, 66), {}, True),
    (308, (64, 8, 77), {}, True), (300, (64, 8, 75), {}, False), (512, (64, 8, 86), {}, False),
    (256, (64, 8, 64), {}, True), (256, (64, 8, 64), dict(snap=True), False), (192, (64, 8, 48), {}, False),
    (256, (64, 8, 64), dict(replicas=2), False), (100, (32, 8, 16), dict(replicas=4), True)])
def test_drained(drained, L, tile, kw, want):
    assert drained(L, tile, **kw) is want
