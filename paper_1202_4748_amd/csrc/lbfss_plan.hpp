// Host side of the launch plans: the plan of a new handle and the tile table of
// a plan (plain C++, no HIP).
#pragma once

#include <algorithm>
#include <array>
#include <cstdint>
#include <numeric>
#include <vector>

#include "../../include/lbfss.h"

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

// The rows staging copies 16-byte chunks that must not straddle the periodic
// seam: every lattice edge a multiple of 4 (FP32) or 8 (FP16 storage).
inline bool rows_edges(const std::vector<int> &Ls, bool fp16) {
    for (int L : Ls)
        if (L % (fp16 ? 8 : 4)) return false;
    return true;
}

// Tiles (or blocks) of a shape over all replicas.
inline int64_t count_tiles(const std::vector<int> &Ls, int tx, int ty, int tz) {
    int64_t n = 0;
    for (int L : Ls) n += (int64_t)((L + tx - 1) / tx) * ((L + ty - 1) / ty) * ((L + tz - 1) / tz);
    return n;
}

// Planes a 64 x 8 tile marches where two workgroups a CU hold all tiles at once,
// which then start and end together: as few as that allows, at most a quarter
// of the edge, or 0 where that does not fit.
inline int round_depth(const std::vector<int> &Ls, int maxL) {
    auto depth = [&](int k) { return (maxL + k - 1) / k; };
    int k = 3;
    while (depth(k + 1) >= 8 && count_tiles(Ls, 64, 8, depth(k + 1)) <= 512) ++k;
    return k > 3 ? depth(k) : 0;
}

// The plan of a new handle, by size: blocks while they are resident in one
// round of the 256 CUs, then two passes, then marching tiles (us a step, force
// model FP32 unless stated).
inline lb_plan default_plan(const std::vector<int> &Ls, bool fp16, bool eq) {
    const lb_plan split{LB_KERNEL_SPLIT, 0, 0, 0, 0, 0};
    const bool rows = rows_edges(Ls, fp16);
    int64_t sites = 0;
    for (int L : Ls) sites += (int64_t)L * L * L;
    // the stores of neighbouring tiles meet in a line, which the marching
    // kernels write around the L2 and the two passes in it
    const bool ragged = ragged_rows(Ls);
    const int maxL = *std::max_element(Ls.begin(), Ls.end());
    const int march = rows ? LB_KERNEL_ROWS : LB_KERNEL_FUSED;
    auto tiles64 = [&](int tz) { return lb_plan{LB_KERNEL_ROWS, 64, 8, tz, 0, 0}; };
    if (eq) {
        if (!rows) return split;
        // 32^3: 7.4, marching 45; 64^3: 13.3, 46; 112^3: 59 against 70; 128^3: 113 against 80
        if (count_tiles(Ls, 32, 8, 1) <= 256) return lb_plan{march, 32, 8, 1, 0, 0};
        if (sites < 118 * 118 * 118) return lb_plan{march, 32, 8, 2, 0, 0};
        // ragged rows: 132^3 112 against 122 on the best tiles, 164^3 218 against
        // 228, 196^3 361 against 426, 220^3 509 against 550, 300^3 1239 against
        // 1377; up to 128^3 the tiles are ahead (124^3 82 against 86).  Multiples
        // of 8 come off better on the tiles: 152^3 156 in four slabs against 174,
        // 248^3 672 against 699 (200^3 387 against 379), 376^3 2371 against 2425
        if (ragged && maxL > 128) {
            const bool four = (maxL > 144 && maxL <= 168) || (maxL > 224 && maxL < 256);
            if (maxL % 8 || (!four && maxL < 368)) return split;
            return tiles64(four ? (maxL + 3) / 4 : (maxL + 7) / 8);
        }
    } else {
        // 32^3: 7.7 as 256 blocks of 16 x 8 x 1, 8.7 as 128 of twice the
        // depth, 10.3 in three passes, marching 54
        if (count_tiles(Ls, 16, 8, 1) <= 256) return lb_plan{march, 16, 8, 1, 0, 0};
        // deeper blocks where the lattice's edge leaves few of their threads
        // idle: 48^3 12.1 against 15.2 in two passes (40^3, padded by a
        // fifth: 13.4 against 11.4), 64^3 15.4 against 16.2 (FP16 13.5, 15.9)
        for (int tx : {16, 32}) {
            const int64_t n = count_tiles(Ls, tx, 8, 4);
            if (n <= 256 && 5 * n * tx * 32 < 6 * sites) return lb_plan{march, tx, 8, 4, 0, 0};
        }
        // two passes read the populations twice, but every CU is at work:
        // 96^3 38 against 51 on the best marching tiles, 144^3 147 against
        // 156, 160^3 188 against 192, 176^3 279 against 237; FP16 112^3 54
        // against 58, 128^3 69 against 60.  Without rows staging (an edge
        // that is no multiple of 4, FP16 of 8) they stay ahead: 250^3 844
        // against 1183.  A batch of small lattices marches from 2^21 sites
        // (96-replica sweep: 130 against 139).
        const int64_t two = fp16 ? 116 * 116 * 116 : (maxL < 128 ? 128 * 128 * 128 : 161 * 161 * 161);
        if (!rows || sites < two) return split;
        // FP16, two passes: 136^3 92 against 106 on the best tiles, 152^3 118
        // against 145, 160^3 134 against 140, 2 x 152^3 255 against 286 (168^3 178
        // against 161, 3 x 144^3 339 against 324)
        if (fp16 && maxL > 128 && maxL < 168 && sites < 200 * 200 * 200) return split;
        // ragged rows.  FP16: 216^3 362 against 371, 264^3 680 against 699, 280^3
        // 785 against 881, 296^3 947 against 1002; 328^3 1288 to 1318 against 1305,
        // 376^3 1869 against 1846.  FP32: 260^3 949 against 1077, 308^3 1590 against
        // 1670, 340^3 2115 against 2410, 404^3 3557 against 3644 where the edge is
        // no multiple of 8; 264^3 965 against 994, 296^3 1378 against 1302, 376^3
        // 2798 against 2678, 408^3 3564 against 3344 where it is
        if (ragged && fp16 && ((maxL > 200 && maxL < 232) || (maxL > 256 && maxL < 308))) return split;
        if (ragged && !fp16 && maxL > 256 && maxL < 424 && maxL % 8) return split;
    }
    if (maxL < 116) {
        // batches of small lattices.  Ragged rows: 33 x 100^3 1850 in two
        // passes, 2486 on 32 x 8 tiles, 33 x 60^3 365, 533; FP16 3 x 104^3 125,
        // 157, 33 x 72^3 531, 560, but 33 x 56^3 226, 206
        if (ragged && (!fp16 || maxL > 64)) return split;
        // 64 wide where that leaves no more lanes idle: FP16 9 x 112^3 407
        // against 541 on 32 x 8 x 16, 16 x 64^3 105 against 119 (33 x 48^3 148
        // against 139 in 12 planes, 9 x 96^3 282 against 241); eq 9 x 112^3 458
        // against 537
        if (((fp16 && maxL >= 64) || (eq && maxL > 64)) && (maxL + 31) / 32 % 2 == 0) return tiles64(16);
        if (fp16) return lb_plan{LB_KERNEL_ROWS, 32, 8, 12, 0, 0};  // 33 x 80^3 697, 725 in 16
        // 32 x 8 tiles of 16 planes, or of 12 where the rounds they take
        // (three workgroups a CU, the equilibrium model four) then march fewer
        // planes: sweep 130 in 12, 147 in 16; 12 x 64^3 138, 127; 33 x 96^3 1143,
        // 1114; eq 5 x 96^3 168, 178, 12 x 64^3 125, 109
        const int64_t resident = eq ? 1024 : 768;
        auto planes = [&](int tz) { return (count_tiles(Ls, 32, 8, tz) + resident - 1) / resident * (tz + 4); };
        return lb_plan{LB_KERNEL_ROWS, 32, 8, planes(12) < planes(16) ? 12 : 16, 0, 0};
    }
    // 64 x 8 tiles stage the fewest halo rows a site (512 threads, two
    // workgroups per CU).  Up to 128^3 eight planes while sixteen leave CUs
    // idle: eq 80.7, 81.8 in sixteen; 9 x 128^3 644, 629
    if (maxL <= 128) return tiles64(count_tiles(Ls, 64, 8, 16) < 512 ? 8 : 16);
    // whole rows from 161 to 191, which is 176^3: sixteen planes 237, in one
    // round 242; eq 203, 210; FP16 174, 175
    if (!ragged && maxL > 160 && maxL < 192) return tiles64(16);
    // one round: 196^3 410 (496 in sixteen planes, 600 on 32 x 8 x 16), 192^3 273
    // (313), 220^3 525 (642, 816), 240^3 532 (584 in 32 planes), 256^3 606 (626);
    // FP16 200^3 302 (339 in sixteen planes), 192^3 191 (214), 208^3 327 (328),
    // 240^3 438 (481), 256^3 438 (445 in six slabs); eq 144^3 127 (150 on 32 x 8
    // x 16), 160^3 160 (187 in sixteen planes), 192^3 241 (263), 224^3 422 (430)
    if (maxL < (eq ? 240 : 257)) {
        if (const int tz = round_depth(Ls, maxL)) return tiles64(tz);
        // batches of more: 2 x 192^3 542 (585 in seven slabs), 5 x 192^3 1297
        // (1381 in five), eq 3 x 160^3 468 (481 in five); 2 x 240^3 1083 in four
        // slabs (1160 in 32 planes)
        if (fp16 || maxL < 208) return tiles64(16);
    }
    if (eq) return tiles64((maxL + 7) / 8);  // 256^3 550, in one round 562
    if (fp16) {
        // six slabs; slabs of 32 for rows of whole 32- but not 64-byte sectors:
        // 368^3 1636 against 1672, 400^3 2149 against 2255, 496^3 3829 against
        // 3993 (336^3 1286 against 1272, 384^3 1523 against 1476)
        if (maxL > 256) return tiles64(maxL % 32 == 16 && maxL >= 368 ? 32 : (maxL + 5) / 6);
    }
    // four slabs while a layer of tiles cannot fill a round, else six (512^3:
    // 7% faster than four)
    return tiles64((maxL + 63) / 64 * ((maxL + 7) / 8) >= 512 ? (maxL + 5) / 6 : (maxL + 3) / 4);
}

}  // namespace lbfss
