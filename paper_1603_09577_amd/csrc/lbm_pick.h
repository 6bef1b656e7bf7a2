// Which pass a run starts with: pure functions of the grid, the storage
// type and the number of CUs (no HIP types, so that they run on the host alone).
#pragma once

#include <stdint.h>

namespace lbm {

// Passes of several time steps, D2Q9: steps per pass, rows of the region (tile
// and halo), waves per workgroup and width of the region of shape `shape`;
// false past the last shape.  Shapes 0 to 2 run 8, 6 and 4 steps with one row
// per wave (16 x 16), 3 and 4 six and four steps on more rows, 5 to 7 are 32
// nodes wide.
inline bool multi_shape_of(int prec, int shape, int *steps, int *rows, int *waves, int *width = nullptr) {
    constexpr int t[3][5][3] = {{{8, 16, 16}, {6, 16, 16}, {4, 16, 16}, {6, 32, 16}, {4, 16, 8}},     // FP64
                                {{8, 16, 16}, {6, 16, 16}, {4, 16, 16}, {6, 32, 16}, {4, 32, 16}},    // FP32
                                {{8, 16, 16}, {6, 16, 16}, {4, 16, 16}, {6, 48, 16}, {4, 32, 16}}};   // FP16
    constexpr int half[3] = {8, 6, 4};   // steps of the 32-wide shapes, 16 rows on 8 waves
    if (prec < 0 || prec > 2 || shape < 0 || shape >= 8) return false;
    if (width) *width = shape < 5 ? 64 : 32;
    if (shape >= 5) {
        *steps = half[shape - 5];
        *rows = 16;
        *waves = 8;
        return true;
    }
    *steps = t[prec][shape][0];
    *rows = t[prec][shape][1];
    *waves = t[prec][shape][2];
    return true;
}

// Columns of the tiles of shape `shape` and all of its tiles on a grid.
inline uint64_t multi_columns(int prec, int shape, uint32_t nx) {
    int t = 2, tr = 4, nw = 0, tx = 64;
    multi_shape_of(prec, shape, &t, &tr, &nw, &tx);
    const uint32_t tw = (uint32_t)(tx - 2 * (t - 1));
    return (nx + tw - 1) / tw;
}

inline uint64_t multi_tiles(int prec, int shape, uint32_t nx, uint32_t ny) {
    int t = 2, tr = 4, nw = 0, tx = 64;
    multi_shape_of(prec, shape, &t, &tr, &nw, &tx);
    const uint32_t th = (uint32_t)(tr - 2 * (t - 1));
    return multi_columns(prec, shape, nx) * ((ny + th - 1) / th);
}

// Shape of the D2Q9 passes of several steps.  A pass costs one launch (1.6 us
// between dependent launches, plus the first loads and the last stores), one
// collision per step on the chain of its waves, and the halo: T - 1 nodes on
// each side of a region of 64 x TR or 32 x TR nodes.
//  - While the grid gives every CU at most one workgroup, nothing else runs on
//    that CU and the halo is free; a step costs about 0.9 us with the four rows
//    per SIMD of a 64 x 16 region and 0.5 us with half of them (FP64).  So the
//    32-wide region with the most steps that still fits one round wins: us per
//    step, FP64 without / FP32 with a source, 64^2 32-wide T = 8 0.89 / 0.82, 6
//    1.03 / 0.93, 64-wide T = 8 1.14 / 1.01; 128^2 32-wide T = 8, two rounds,
//    1.24 / 1.03, 6 1.07 / 0.95, 64-wide 8 1.21 / 1.04; FP64 200^2 32-wide 4
//    1.40, 64-wide 6 1.44.
//  - FP32 and FP16 gain less from the shorter steps, and their second and third
//    32-wide workgroup on a CU costs less: six steps up to two of them (200^2
//    1.19, one 64 x 16 region with six steps 1.21), and up to three rather than
//    four steps in 64 x 16 (300^2 1.53 against 1.62).
//  - Then 64 x 16 with six, then with four steps in one round (256^2 1.26 / 1.76
//    against 1.46 / 2.09 32-wide with four).
//  - Then the tall region with six steps (512^2 FP32 2.18 against 2.43 for four
//    steps in 16 rows, FP64 3.35 against 3.92), or with four where that fits
//    one round of resident workgroups and six steps do not (1000 x 723 FP32
//    with walls 5.14 against 5.65).
//  - FP16 takes four steps in 32 rows up to eight workgroups per CU (512^2 3.07
//    against 3.24 for six in 48 rows, 1024^2 6.02 / 6.79, 1600^2 12.2 / 12.6; 2048^2
//    19.2 / 18.2).
//  - Beyond one round the halo work counts: FP32 and FP16 keep six steps in the
//    tall region (2048^2 FP32 18.9 against 22.3 for four), FP64, whose tall region
//    leaves one workgroup per CU, takes four steps in 16 rows (1024^2 12.0 against
//    12.6).  FP32 takes four steps too where their 58-node columns are at most
//    three for four of the 54-node ones (57 x 10000 4.1 against 5.3, 112 x 50000
//    30.3 / 34.6, 170 x 30000 27.8 / 28.3).
inline int pick_multi(int prec, uint32_t nx, uint32_t ny, uint64_t ncu) {
    auto fits = [&](int shape, uint64_t per_cu) { return multi_tiles(prec, shape, nx, ny) <= per_cu * ncu; };
    const bool f64 = prec == 0;
    if (fits(5, 1)) return 5;
    if (fits(6, f64 ? 1 : 2)) return 6;
    if (fits(0, 1)) return 0;
    if (f64 && fits(7, 1)) return 7;
    if (fits(1, 1)) return 1;
    if (!f64 && fits(6, 3)) return 6;
    if (fits(2, 1)) return 2;
    if (prec == 2) return fits(4, 8) ? 4 : 3;
    if (fits(3, f64 ? 1 : 2)) return 3;
    if (fits(4, 2)) return 4;
    return f64 || 5 * multi_columns(prec, 4, nx) < 4 * multi_columns(prec, 3, nx) ? 4 : 3;
}

// Whether two-step passes, whose columns are 62 nodes wide, beat passes in
// `shape` on a grid that its columns fit badly.  They do where several
// workgroups share a CU, so that the work counts:
//  - FP64 and FP16 with two columns for one (nx 55 or 59 to 62).  us per step
//    several / two steps, FP64 with a source 60 x 2200 2.94 / 3.43 (one round),
//    59 x 3000 4.6 / 3.7, 60 x 20000 20.0 / 16.2, 60 x 60000 64.5 / 56.5; FP16 60 x
//    6000 3.95 / 4.09, 60 x 8000 5.6 / 5.0, 60 x 20000 11.1 / 7.8, 60 x 150000 61.5 / 49.1.
//  - FP16 with three columns for two (nx 109 or 117 to 124), from four workgroups
//    per CU up and while the state stays in the Infinity Cache: 120 x 6000 5.7 / 6.0,
//    120 x 14000 11.3 / 9.4, but 120 x 60000 38.5 / 51.9.
//  - FP32, whose two-step passes cost more, keeps the passes of several steps
//    (60 x 20000 9.7 / 9.6, 60 x 100000 43 / 53) unless a step costs more too: with
//    two columns for one, walls or rates other than 1 while the state stays in
//    the cache (60 x 20000 11.3 / 10.7 and 10.5 / 9.7), Scheme B (11.9 / 10.6, 62 x
//    60000 31.5 / 27.0).
//  - FP64 with Scheme B also with three columns for two, in the cache (120 x 14000
//    25.3 / 21.0, 124 x 10000 18.7 / 16.1; Scheme A 17.6 / 17.5).
// sb: Scheme B with a source; plain: periodic, all non-flux rates 1.
inline bool two_steps_fit_better(int prec, int shape, uint32_t nx, uint32_t ny, uint64_t ncu, bool beyond_cache,
                                 bool sb, bool plain) {
    const uint64_t c = multi_columns(prec, shape, nx), c2 = (nx + 61) / 62, tiles = multi_tiles(prec, shape, nx, ny);
    if (shape != 3 && shape != 4) return false;
    const bool twice = c >= 2 * c2, half_more = 2 * c >= 3 * c2 && !beyond_cache;
    switch (prec) {
        case 0: return (twice && tiles > 2 * ncu) || (sb && half_more && tiles > 8 * ncu);
        case 1: return twice && tiles > 4 * ncu && (sb || (!plain && !beyond_cache));
        default: return (twice && tiles > 2 * ncu) || (half_more && tiles > 4 * ncu);
    }
}

// D3Q19: single sweeps, two-step passes in 62-node columns or in 64-node lines,
// for n nodes on lines of nx (src: a Scheme-A source).
// A pass has one workgroup per column and chunk of planes, a wave computes 64
// nodes whether the grid has them or not, and the planes of the halo are extra.
//  - It wins over single sweeps once enough nodes share that, more of them the
//    emptier the lines are: with f the filled part of the lines (FP64: of the
//    62-node columns where it takes those), N f^2 separates the two.  us per step single / lines, FP64 with a source and walls, 56^3
//    (143k) 11.4 / 13.7, 72^3 (126k) 20.9 / 25.6, 58^3 (171k) 12.0 / 13.8, 60^3 (202k)
//    14.3 / 14.0 (without 13.3 / 12.0), 80^3 (213k) 27.8 / 28.5 (25.6 / 24.4); periodic
//    58^3 with a source 13.6 / 12.9,
//    without 12.2 / 11.2, 60^2 x 30 (101k) 8.3 / 8.9; FP32 100 x 60^2 (220k) 11.3 / 11.9, 64^3 (262k) 9.1 / 9.4, 50 x
//    100 x 80 (244k) 12.7 / 11.9, 64^2 x 80 (327k) 11.0 / 10.0; FP16 with walls 100^3 (610k) 19.2 / 18.9,
//    80 x 120 x 140 (525k) 26.4 / 28.1; without, where single sweeps move half the
//    bytes at full occupancy, 130^3 (1.0M) 31 / 43, 128^3 (2.1M) 30.5 / 30.0.
//  - Lines where they save a column (256^3 FP32 291 against 325, FP64 82 against 108
//    on 128^3).  Where they do not, a 62-node column is the better one in FP64 (its
//    lines have an odd wave: 200 x 180 x 160 224 / 215, with a source 247 / 228), in
//    FP32 without walls or beyond a million nodes (lines / columns 216 x 157 x 128
//    105 / 82; periodic 60 x 80^2 10.3 / 9.7, 180 x 60 x 90 18.5 / 17.4, with a source
//    100 x 80 x 60 15.3 / 13.4; with walls 96^3 17.5 / 18.7) and in FP16 with a
//    source beyond four million (216 x 157 x 128 87 / 72; 130^3 43 / 46).
enum class Pass3 { single, columns, lines };

inline Pass3 pick_pass3(int prec, uint32_t nx, uint32_t n, bool src, bool wall) {
    const uint32_t lines = (nx + 63) / 64, columns = (nx + 61) / 62;
    const bool saves = lines < columns;
    const double f = prec == 0 && !saves ? (double)nx / (62.0 * columns) : (double)nx / (64.0 * lines);
    const double small64 = wall ? 190e3 : (src ? 165e3 : 130e3);
    const double small = prec == 0 ? small64 : (prec == 1 ? 240e3 : (wall ? 600e3 : 2e6));
    if (n * f * f < small) return Pass3::single;
    if (saves) return Pass3::lines;
    const bool narrow = prec == 0 || (prec == 1 ? !wall || n > 1000000u : src && n > 4000000u);
    return narrow ? Pass3::columns : Pass3::lines;
}

// Whether a batch starts with the passes of its default shape rather than with
// single sweeps.  A tile of a pass costs the same however little of it is grid:
// 3.7 ns per step in FP32, 4.2 in FP16 (54 x 22 nodes), 4.1 in FP64 (58 x 10); a
// single sweep costs 13, 9 and 23 ps per node and about 0.7 ns per 256-node block.
// So a tile pays from 285, 465 or 180 nodes' worth of single sweeps on, and
// narrow or tiny instances do not fill that.  Up to two tiles per CU a launch
// costs more than the tiles.  us per step single sweeps / passes: 400 of 2 x 500
// FP32 6.1 / 35, FP64 11.0 / 85; 5000 of 8^2 7.1 / 17.2; 300 of 10 x 300 12.0 / 16.2; 4000 of
// 16^2 FP16 10.6 / 15.9, FP32 15.1 / 15.0; 1500 of 32^2 FP16 13.3 / 12.7; 64 of 4^2 3.8 / 1.7.
inline bool batch_passes_win(int prec, uint64_t nodes, uint64_t blocks, uint64_t tiles, uint64_t ncu) {
    const uint64_t tile_worth = prec == 0 ? 180 : (prec == 1 ? 285 : 465);
    return tiles <= 2 * ncu || tiles * tile_worth <= nodes + 50 * blocks;
}

}  // namespace lbm
