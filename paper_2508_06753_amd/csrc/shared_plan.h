// Launch shapes of the mid-M kernel that shares its rows (matmul_shared.hip): host code only, no HIP, so that a test can compile it
// by itself.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "midm_plan.h"

namespace w2 {

namespace shared {

// Launch shape: row tiles per wave, column blocks per wave, waves across the columns (the workgroup is cj * sh column blocks wide).
struct Plan { int rt, cj, sh; };                             // rt: 2 to 4

constexpr int BUFS = 4;                                      // buffers of a K range's chunks
constexpr int LDS = 160 * 1024;

// KiBs (eight rows x 128 bytes) that each wave of a range loads per chunk, and a buffer of them all
constexpr int loads(int rt, int sh) { return (2 * rt + sh - 1) / sh; }
constexpr int buf_bytes(int rt, int sh) { return loads(rt, sh) * sh * 1024; }
// bytes of local memory of one K range: its chunks, later its waves' partial results
constexpr int range_lds(int rt, int cj, int sh)
{
    return std::max(BUFS * buf_bytes(rt, sh), sh * midm::red_bytes(rt, cj));
}
// K ranges of a workgroup: as many as sixteen waves (at most 128 registers each) and the local memory allow.  Int8 rows, four row
// tiles x 2 blocks (three with groups of 64): more registers than that, twelve waves.
constexpr int k_ranges(int xt, int G, int rt, int cj, int sh)
{
    const int waves = xt == 0 && cj == 2 && rt + (G == 64) >= 4 ? 12 : 16;
    return std::min(waves / sh, (LDS - rt * 64) / range_lds(rt, cj, sh));
}

// Loads that may still be under way when a chunk is used, h its place among the ch chunks of a 256-k tile, nj a wave's loads per
// chunk.  It was asked for BUFS - 1 chunks ago, ahead of that chunk's arithmetic; since then BUFS - 2 chunks were and, behind a tile's
// last chunk, the weights and scales of another tile, one load of each per column block.
constexpr int under_way(int h, int ch, int nj, int cj)
{
    int tiles = 0;
    for (int e = 1; e < BUFS; ++e) tiles += (h - e + BUFS * ch) % ch == ch - 1;
    return (BUFS - 2) * nj + tiles * 2 * cj;
}

// The shapes that are built: column blocks per wave x waves across the columns, a width of every number of blocks that came out fastest
// on some grid (nine, eleven and thirteen never by more than a per cent).
constexpr int N_SHAPES = 12;
constexpr int SHAPES[N_SHAPES][2] = {{1, 2}, {1, 3}, {1, 4}, {1, 5}, {1, 6}, {1, 7}, {1, 8}, {2, 4}, {2, 5}, {2, 6}, {2, 7}, {2, 8}};

// (never the cheapest: two blocks for two row tiles of int8 rows)
constexpr bool built(int xt, int rt, int cj, int sh) { return rt >= 2 && !(xt == 0 && rt == 2 && cj * sh == 2); }

struct Ranges {
    int8_t n[2][2][3][N_SHAPES];                             // [activations][groups of 64][rt - 2][shape]
    constexpr Ranges() : n{}
    {
        for (int xt = 0; xt < 2; ++xt)
            for (int g = 0; g < 2; ++g)
                for (int rt = 2; rt <= 4; ++rt)
                    for (int s = 0; s < N_SHAPES; ++s) n[xt][g][rt - 2][s] = (int8_t)k_ranges(xt, g ? 64 : 128, rt, SHAPES[s][0], SHAPES[s][1]);
    }
};
constexpr Ranges RANGES;                                     // (at most eight)

// Where the kernel is offered: problems of the measurements below.  Up to sixteen rows (one row tile) the mid-M and the decode kernel
// are as fast: the fastest of both is 0.3 % faster than they are on 330 problems.
constexpr int64_t LEAST_ROWS = 17, MOST_ROWS = 144, LEAST_BLOCKS = 256, LEAST_TILES = 3, MOST_TILES = 80;
inline bool offered(int64_t M, int64_t n_cb, int64_t n_kt)
{
    return M >= LEAST_ROWS && M <= MOST_ROWS && n_cb >= LEAST_BLOCKS && n_kt >= LEAST_TILES && n_kt <= MOST_TILES;
}

// Price of a launch, linear in what it does; least-squares fits (us) to 15000 graph-timed launches on 1130 problems (K 768 to 20000,
// N 4096 to 57344, 17 to 150 rows, both group sizes, gated or not), a set for grids of one round and of more ([activations][rt - 2]
// [rounds > 1]): 5.3 % off in the root mean square near the fastest shape; the shapes chosen are 1.1 % slower than the fastest measured.
struct Coef {
    double launch, round, round_block,                       // fixed; per round, and times column blocks of a workgroup
           tile, tile_block, tile_block_g64,                 // per round and tile of K; times column blocks; more with groups of 64
           range_tile, range_block,                          // per round: per tile of a K range; per range and column block (the reduce)
           fill,                                             // tile_block again, by workgroups / 256: a full chip holds lower clocks
           stream, stream_band,                              // per tile of the projection: from memory, and once per band out of the L2s
           rows_mb;                                          // per MB of rows that all workgroups together read
};
constexpr Coef COEF[2][3][2] = {
    {{{2.457, 0, 0.04593, 0.01418, 0.02111, 0.0105, 0.2198, 0.05267, 0.006089, 8.156e-05, 0, 0.02242},
      {1.778, 0.01039, 0.0366, 0.04601, 0.02272, 0.007307, 0, 0.08942, 0, 8.545e-05, 4.241e-05, 0.02319}},
     {{2.351, 0, 0.0929, 0.03855, 0.02597, 0.01132, 0.217, 0.06765, 0.01111, 4.601e-05, 0, 0.01683},
      {1.606, 0.6568, 0.02418, 0.04947, 0.02205, 0.007497, 0.1766, 0.1037, 0.004363, 8.419e-05, 3.766e-05, 0.01046}},
     {{2.489, 0, 0.09684, 0, 0.02812, 0.0117, 0.4339, 0.08516, 0.01065, 6.476e-05, 0, 0.01143},
      {1.609, 1.076, 0.04674, 0, 0.02551, 0.01166, 0.3683, 0.09468, 0, 8.798e-05, 5.633e-05, 0.01592}}},
    {{{2.497, 0, 0.0687, 0.03736, 0.05069, 0.009496, 0.2698, 0.04188, 0.01511, 4.943e-05, 0, 0.01314},
      {1.966, 0, 0.0402, 0.03764, 0.05735, 0.007528, 0, 0.08147, 0.01231, 3.999e-05, 0, 0.01649}},
     {{2.271, 0, 0.07846, 0.03334, 0.0569, 0.009192, 0.3332, 0.08399, 0.01172, 6.009e-05, 0, 0.01797},
      {1.591, 0.2376, 0.07371, 0.09631, 0.05448, 0.008311, 0, 0.09976, 0.02291, 7.126e-05, 0, 0.01486}},
     {{2.364, 0, 0.108, 0.03584, 0.05818, 0.007654, 0.4674, 0.08793, 0.02124, 5.77e-05, 0, 0.01091},
      {2.574, 0.9403, 0.149, 0.001819, 0.07084, 0.008894, 0.3463, 0.03421, 0.01162, 3.578e-05, 0, 0.02487}}}};

// us: the price.  Row tiles per wave: as few bands as there can be, of equal height, or bands of two.
inline Plan plan(int xt, int64_t M64, int64_t n_cb64, int64_t n_kt64, bool gated, int G, double* us)
{
    const int M = (int)M64, n_cb = (int)n_cb64, n_kt = (int)n_kt64, row_tiles = (M + 15) / 16, fewest = (row_tiles + 3) / 4;
    const double tiles = (double)n_cb * n_kt, row_mb = (double)M * n_kt * (xt == 0 ? 256e-6 : 512e-6);
    Plan best = {2, 1, 3};
    *us = 1e30;
    // (this runs on every call in its range: the divisions once)
    int group_count[N_SHAPES], range_tiles[9];
    for (int s = 0; s < N_SHAPES; ++s) group_count[s] = (n_cb + SHAPES[s][0] * SHAPES[s][1] - 1) / (SHAPES[s][0] * SHAPES[s][1]);
    for (int k = 1; k <= 8; ++k) range_tiles[k] = (n_kt + k - 1) / k;
    for (int rt = (row_tiles + fewest - 1) / fewest;; rt = 2) {
        const int bands = (row_tiles + rt - 1) / rt;
        for (int s = 0; s < N_SHAPES; ++s) {
            const int cj = SHAPES[s][0], sh = SHAPES[s][1], width = cj * sh;
            if (!built(xt, rt, cj, sh) || (gated && (width & 1))) continue;  // (the gated epilogue pairs blocks of a workgroup)
            const int groups = group_count[s], wgs = groups * bands, rounds = (wgs + 255) >> 8;
            const int ks = std::min((int)RANGES.n[xt][G == 64][rt - 2][s], n_kt);
            const Coef& c = COEF[xt][rt - 2][rounds > 1];
            const double t = c.launch + rounds * (c.round + width * (c.round_block + c.range_block * ks) +
                                                  n_kt * (c.tile + width * (c.tile_block + (G == 64 ? c.tile_block_g64 : 0))) +
                                                  c.range_tile * range_tiles[ks]) +
                             c.fill * (1.0 / 256) * wgs * n_kt * width + tiles * (c.stream + c.stream_band * bands) + c.rows_mb * row_mb * groups;
            if (t < *us) { best = {rt, cj, sh}; *us = t; }
        }
        if (rt <= 2) break;
    }
    return best;
}

}  // namespace shared

}  // namespace w2
