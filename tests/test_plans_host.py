"""The plan of a new handle (plain C++, compiled and run here) at edges whose
rows are no whole sectors and beside them, and for batches: the kernel and
tile that were measured fastest there, or at most a few per cent behind."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "lbfss_plan.hpp"
int main(int argc, char **v) {  // fp16 eq L...
    std::vector<int> L;
    for (int i = 3; i < argc; ++i) L.push_back(atoi(v[i]));
    const lb_plan p = lbfss::default_plan(L, atoi(v[1]), atoi(v[2]));
    printf("%d %d %d %d\n", p.kernel, p.tile_x, p.tile_y, p.tile_z);
}
"""

SPLIT = (0, 0, 0, 0)


def rows(tx, ty, tz):
    return 3, tx, ty, tz


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plans")
    (d / "t.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1202_4748_amd", "csrc"), "-o", str(d / "t"), str(d / "t.cpp")], check=True)

    def run(Ls, fp16=False, eq=False):
        a = [int(fp16), int(eq), *Ls]
        r = subprocess.run([str(d / "t"), *map(str, a)], capture_output=True, text=True, check=True)
        return tuple(map(int, r.stdout.split()))

    return run


@pytest.mark.parametrize("L,want", [
    (132, SPLIT), (148, SPLIT), (164, rows(64, 8, 21)), (172, rows(64, 8, 25)), (176, rows(64, 8, 16)),
    (180, rows(64, 8, 26)), (188, rows(64, 8, 27)), (192, rows(64, 8, 28)), (196, rows(64, 8, 40)),
    (204, rows(64, 8, 51)), (208, rows(64, 8, 52)), (212, rows(64, 8, 53)), (220, rows(64, 8, 55)),
    (228, rows(64, 8, 57)), (236, rows(64, 8, 59)), (240, rows(64, 8, 60)), (244, rows(64, 8, 61)),
    (252, rows(64, 8, 63)), (256, rows(64, 8, 64)), (260, SPLIT), (264, rows(64, 8, 66)), (300, SPLIT),
    (500, rows(64, 8, 125)), (512, rows(64, 8, 86)), (250, SPLIT)])
def test_force_fp32(plan, L, want):
    assert plan([L]) == want


@pytest.mark.parametrize("L,want", [
    (120, rows(64, 8, 8)), (128, rows(64, 8, 8)), (136, SPLIT), (152, SPLIT), (168, rows(64, 8, 21)),
    (200, rows(64, 8, 40)), (216, SPLIT), (232, rows(64, 8, 58)), (256, rows(64, 8, 64)), (264, SPLIT),
    (328, rows(64, 8, 55)), (496, rows(64, 8, 32)), (504, rows(64, 8, 84)), (512, rows(64, 8, 86)), (252, SPLIT)])
def test_force_fp16(plan, L, want):
    assert plan([L], fp16=True) == want


@pytest.mark.parametrize("L,want", [
    (116, rows(32, 8, 2)), (124, rows(64, 8, 8)), (132, SPLIT), (144, rows(64, 8, 16)), (148, SPLIT),
    (152, rows(64, 8, 38)), (160, rows(64, 8, 20)), (164, SPLIT), (176, rows(64, 8, 16)), (196, SPLIT),
    (208, rows(64, 8, 52)), (220, SPLIT), (248, rows(64, 8, 62)), (256, rows(64, 8, 32)), (260, SPLIT),
    (300, SPLIT), (376, rows(64, 8, 47)), (500, SPLIT), (512, rows(64, 8, 64))])
def test_equilibrium(plan, L, want):
    assert plan([L], eq=True) == want


@pytest.mark.parametrize("Ls,kw,want", [
    ([96] * 2, {}, SPLIT), ([96] * 3, {}, rows(32, 8, 16)), ([64] * 12, {}, rows(32, 8, 16)),
    ([64] * 16, {}, rows(32, 8, 12)), ([100] * 4, {}, SPLIT), ([60] * 33, {}, SPLIT),
    ([L for L in (8, 12, 16, 24, 32, 48) for _ in range(16)], {}, rows(32, 8, 12)),
    ([128] * 2, {}, rows(64, 8, 16)), ([192] * 3, {}, rows(64, 8, 16)), ([256] * 2, {}, rows(64, 8, 64)),
    ([256, 128, 64], {}, rows(64, 8, 64)), ([112] * 9, dict(fp16=True), rows(64, 8, 16)),
    ([56] * 33, dict(fp16=True), rows(32, 8, 12)), ([104] * 3, dict(fp16=True), SPLIT),
    ([144] * 3, dict(fp16=True), rows(64, 8, 16)), ([100] * 2, dict(eq=True), SPLIT),
    ([160] * 3, dict(eq=True), rows(64, 8, 16)), ([128] * 9, dict(eq=True), rows(64, 8, 16))],
    ids=lambda v: f"{len(v)}x{v[0]}" if isinstance(v, list) else None)
def test_batches(plan, Ls, kw, want):
    assert plan(Ls, **kw) == want
