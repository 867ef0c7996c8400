// Host side of the launch plans: the tile table of a plan (plain C++, no HIP).
#pragma once

#include <algorithm>
#include <array>
#include <cstdint>
#include <numeric>
#include <vector>

namespace lbfss {

struct FusedTile {
    int32_t rep, x0, y0, z0, nx, ny, nz, pad;
};

constexpr int kXcds = 8;

// The tile table of a plan over replicas of edges Ls: of one replica x
// fastest, then y, then z, which xcd_tile deals to the XCDs in contiguous
// runs.  For a batch the table holds a list per XCD, the shorter lists filled
// with empty tiles (nz = 0).  Replicas, the largest first, go whole to the XCD
// with the least work so far where that leaves the fullest one within 5% of
// the even share (96-replica sweep on 32 x 8 x 12: 136 us a step with its
// tiles in one run, 130 us dealt whole), or where the tiles are blocks and the
// fullest one has a CU for each (7 x 16^3 in 16 x 8 x 1: 7.8 us cut, 7.4 whole:
// neighbours share an L2); where it does not, the lists are runs of equal work
// over all tiles, cut where they end (2 x 256^3: whole replicas would keep two
// XCDs of eight, 3597 us a step against 1247 in one run).
inline int make_fused_tiles(const std::vector<int> &Ls, int tx, int ty, int tz, std::vector<FusedTile> &out) {
    if (tx < 1 || ty < 1 || tz < 1 || tz > 1024) return -1;
    out.clear();
    std::vector<size_t> order(Ls.size());
    std::iota(order.begin(), order.end(), size_t(0));
    std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return Ls[a] > Ls[b]; });
    auto work_of = [](const FusedTile &t) { return (int64_t)t.nz + 4; };  // planes marched
    std::vector<FusedTile> run;  // all tiles in order
    std::vector<size_t> ends;    // of each replica's tiles there
    int64_t total = 0;
    for (size_t r : order) {
        const int L = Ls[r], nx = std::min(tx, L), ny = std::min(ty, L), nz = std::min(tz, L);
        for (int z0 = 0; z0 < L; z0 += nz)
            for (int y0 = 0; y0 < L; y0 += ny)
                for (int x0 = 0; x0 < L; x0 += nx) {
                    run.push_back(FusedTile{(int32_t)r, x0, y0, z0, std::min(nx, L - x0), std::min(ny, L - y0),
                                            std::min(nz, L - z0), 0});
                    total += work_of(run.back());
                }
        ends.push_back(run.size());
    }
    if (Ls.size() < 2) {
        out = std::move(run);
        return 0;
    }
    std::array<std::vector<FusedTile>, kXcds> lists;
    std::array<int64_t, kXcds> work{};
    size_t first = 0;
    for (size_t end : ends) {
        const int k = (int)(std::min_element(work.begin(), work.end()) - work.begin());
        for (; first < end; ++first) {
            lists[k].push_back(run[first]);
            work[k] += work_of(run[first]);
        }
    }
    size_t fullest = 0;
    for (const auto &l : lists) fullest = std::max(fullest, l.size());
    const bool one_each = tz <= 4 && fullest <= 32;
    if (!one_each && 20 * kXcds * *std::max_element(work.begin(), work.end()) > 21 * total) {
        for (auto &l : lists) l.clear();
        int64_t before = 0;
        for (const FusedTile &t : run) {  // by the middle of the tile's share of the run
            const int64_t w = work_of(t);
            lists[(2 * before + w) * kXcds / (2 * total)].push_back(t);
            before += w;
        }
    }
    size_t per = 0;
    for (const auto &l : lists) per = std::max(per, l.size());
    out.assign(per * kXcds, FusedTile{0, 0, 0, 0, 0, 0, 0, 0});
    for (int k = 0; k < kXcds; ++k) std::copy(lists[k].begin(), lists[k].end(), out.begin() + per * k);
    return 0;
}

// Most sites in rows that are no whole 64 bytes (FP16: 32)?
inline bool ragged_rows(const std::vector<int> &Ls) {
    int64_t sites = 0, ragged = 0;
    for (int L : Ls) {
        sites += (int64_t)L * L * L;
        if (L % 16) ragged += (int64_t)L * L * L;
    }
    return 2 * ragged > sites;
}

// Do the staged tiles (tx, ty), n of them, run drained (k_fused_staged)?  Us a
// step, copies left in flight against drained.
inline bool drained_plan(const std::vector<int> &Ls, bool fp16, int tx, int ty, int64_t n, bool snap) {
    const int maxL = *std::max_element(Ls.begin(), Ls.end());
    const bool ragged = ragged_rows(Ls);
    // ragged FP16 rows: 504^3 4800, 4299, 264^3 745, 699, 216^3 417, 432 on 64 x 8
    // tiles; 168^3 230, 217 on 32 x 8.  Others: 512^3 3547, 3810, 240^3 465, 490
    if (fp16) return ragged && (tx * ty < 512 || maxL >= 232);
    // ragged FP32 rows on tiles of 256 threads: 132^3 149, 136, 220^3 814, 760 on
    // 32 x 8; 196^3 521, 466, 132^3 165, 173 on 64 x 4; fewer tiles than two on
    // most CUs: 116^3 95, 98.  Whole rows: 256^3 715, 763
    if (tx * ty < 512) return ragged && n > 480 && (tx < 64 || maxL >= 196);
    // 64 x 8: ragged rows 308^3 1749, 1670, 404^3 3821, 3644, 300^3 1482, 1504; and
    // where all tiles are resident at once, nearly two on each CU: 256^3 630, 606,
    // 228^3 648, 584, 240^3 547, 532, 192^3 276, 273 in one round, 192^3 in six
    // slabs (288 tiles) 392, 394, 256^3 in 16-plane slabs 645, 671; not with the
    // snapshot's stores (256^3 798, 853) nor in FP16 (256^3 438, 473) or with the
    // equilibrium model (256^3 562, 617)
    return (ragged && maxL >= 308) || (!snap && n > 384 && n <= 512);
}

}  // namespace lbfss
