"""The tile tables of the launch plans (plain C++, compiled and run here): the
lists of a batch, one per XCD, hold every tile once and share the work, for
few and for uneven replicas as well as for many."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "lbfss_plan.hpp"
int main(int argc, char **argv) {  // tx ty tz L...
    std::vector<int> L;
    for (int i = 4; i < argc; ++i) L.push_back(atoi(argv[i]));
    std::vector<lbfss::FusedTile> t;
    if (lbfss::make_fused_tiles(L, atoi(argv[1]), atoi(argv[2]), atoi(argv[3]), t)) return 1;
    for (const auto &k : t) printf("%d %d %d %d %d %d %d\n", k.rep, k.x0, k.y0, k.z0, k.nx, k.ny, k.nz);
}
"""

SWEEP = [L for L in (8, 12, 16, 24, 32, 48) for _ in range(16)]


@pytest.fixture(scope="module")
def table(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    (d / "t.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1202_4748_amd", "csrc"), "-o", str(d / "t"), str(d / "t.cpp")], check=True)

    def run(tile, Ls):
        r = subprocess.run([str(d / "t"), *map(str, tile), *map(str, Ls)], capture_output=True, text=True, check=True)
        return [tuple(map(int, line.split())) for line in r.stdout.splitlines()]

    return run


@pytest.mark.parametrize("Ls", [[50], [4, 36, 8], [48] * 9, [64, 32, 16], SWEEP], ids=lambda v: f"{len(v)}x{v[0]}")
@pytest.mark.parametrize("tile", [(32, 8, 12), (64, 8, 16), (16, 8, 1), (32, 4, 4)])
def test_every_site_once(table, tile, Ls):
    tiles = [t for t in table(tile, Ls) if t[6]]
    assert len(set(tiles)) == len(tiles)
    for r, L in enumerate(Ls):
        mine = [t for t in tiles if t[0] == r]
        assert sum(t[4] * t[5] * t[6] for t in mine) == L ** 3
        assert all(t[1] + t[4] <= L and t[2] + t[5] <= L and t[3] + t[6] <= L for t in mine)


@pytest.mark.parametrize("Ls", [[128] * 2, [256] * 2, [128] * 3, [128] * 4, [48] * 9, [100] * 12, [64] * 33,
                                [256, 128, 64], [256] + [16] * 7, SWEEP], ids=lambda v: f"{len(v)}x{v[0]}")
@pytest.mark.parametrize("tile", [(32, 8, 12), (64, 8, 16), (32, 4, 4)])
def test_batch_shares_the_xcds(table, tile, Ls):
    """The fullest list holds at most a tenth, or one tile, more planes than
    the even share; so is the length of the table bounded that every list is
    padded to."""
    t = table(tile, Ls)
    assert len(t) % 8 == 0
    per = len(t) // 8
    lists = [[k for k in t[x * per:(x + 1) * per] if k[6]] for x in range(8)]
    work = [sum(k[6] + 4 for k in ls) for ls in lists]
    share, biggest = sum(work) / 8, max(k[6] + 4 for k in t)
    assert max(work) <= max(1.1 * share, share + biggest)


@pytest.mark.parametrize("Ls", [[128] * 2, [100] * 3, [48] * 9, [64] * 33], ids=lambda v: f"{len(v)}x{v[0]}")
def test_equal_replicas_are_hardly_padded(table, Ls):
    t = table((32, 8, 12), Ls)
    n = sum(1 for k in t if k[6])
    assert len(t) <= 1.1 * n + 8


@pytest.mark.parametrize("tile,Ls,whole", [((16, 8, 1), [16] * 7, True), ((16, 8, 1), [16] * 8, True),
                                           ((32, 4, 4), [8] * 33, True), ((16, 8, 4), [32] * 2, False),
                                           ((32, 8, 16), [64] * 2, False)])
def test_blocks_with_a_cu_each_stay_together(table, tile, Ls, whole):
    """Block plans whose fullest list has a CU for every block keep replicas on
    one XCD; more blocks, and marching tiles, are cut."""
    t = table(tile, Ls)
    per = len(t) // 8
    where = [{x for x in range(8) for k in t[x * per:(x + 1) * per] if k[6] and k[0] == r} for r in range(len(Ls))]
    assert all(len(w) == 1 for w in where) is whole
