// Launch shapes of the tiled kernels: host code only, no HIP, so that a test can compile it by itself.
//
// First, tile height and K ranges of the two kernels of 256-column workgroups (w2a8: matmul_a8_tiled128.hip, w2a16:
// matmul_a16_fold.hip).
//
// A workgroup (eight waves, one per CU) multiplies 16 ri rows, ri = 4 to 8, by 256 columns over one of `splits` near-equal
// ranges of K.  A taller tile shares an up-converted weight between more matrix instructions, but the workgroups run in
// rounds of 256 and a last round costs almost as much as a full one, and rows past M are multiplied like the others: 4096 x
// 28672 at M = 130 takes 33.5 us in two row tiles of 128 and 26.1 in two of 80; at M = 1000 130 us in 3.5 rounds of 128 rows
// and 121 in 3.94 rounds of 112.  So every (ri, splits) is priced and the cheapest wins.  The prices are linear in what a
// launch does, coefficients (us) fitted to graph-timed launches of every (ri, splits) on 280 (int8 rows, groups of 128), 100
// (groups of 64) and 392 (bf16 rows) problems, K 1024 to 28672, N 1024 to 57344, 40 to 4096 rows: they are 3.2, 2.4 and 3.2 %
// off in the root mean square, and the (ri, splits) that they choose are 0.2, 0.1 and 0.3 % slower than the fastest measured.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/w2mm.h"

namespace w2 {

namespace tiles {

enum Kind { A8_G128, A8_G64, A16 };

struct Shape {
    int ri, splits;
    double us;                                               // the price
};

constexpr int MAX_SPLITS = 8;
constexpr int64_t MAX_PART_BYTES = (int64_t)64 << 20;        // most bytes of partial results

// fp32 copies of the output in so many bytes (no product that a row count without limit could overflow to zero)
inline int64_t copies(int64_t bytes, int64_t M, int64_t N) { return bytes / 4 / M / N; }

struct Coef {
    double launch, wg,                  // fixed, and per workgroup / 256
           round, round_ri,             // first loads and epilogue, per round
           tile, tile_ri, tile_ri_wg,   // per 256 k and round; per workgroup / 256 (a full chip holds lower clocks)
           parts, part_value;           // the second launch, and per value of a partial result, written and read
};
constexpr Coef COEF[3] = {
    {2.957, 2.057, 0.0, 0.3544, 0.5388, 0.1307, 0.01674, 4.368, 0.7115e-6},
    {3.102, 2.146, 0.0, 0.3454, 0.5539, 0.1836, 0.01042, 4.137, 0.6599e-6},
    {2.500, 1.610, 1.146, 0.3411, 1.297, 0.1271, 0.07422, 3.773, 0.7268e-6}};

// wgs: workgroups, nk: 256-k tiles of the longest range
inline double price(const Coef& c, int64_t wgs, int64_t nk, int ri, int splits, double values)
{
    const double rounds = (double)((wgs + 255) >> 8), fill = (double)wgs / 256.0;
    double t = c.launch + c.wg * fill + rounds * (c.round + c.round_ri * ri) +
               (double)nk * (rounds * (c.tile + c.tile_ri * ri) + fill * c.tile_ri_wg * ri);
    if (splits > 1) t += c.parts + c.part_value * values * splits;
    return t;
}

// `cap`: fp32 copies of the output that the caller's workspace holds.  forced_ri, forced_splits: 0, or the only ones
// considered (splits: as many of them as fit).
inline Shape pick(Kind kind, int64_t M, int64_t N, int64_t n_kt, int64_t cap, int forced_ri = 0, int forced_splits = 0)
{
    Shape best = {8, 1, 1e30};
    int64_t most = std::min(std::min(n_kt / 2, cap), std::min((int64_t)MAX_SPLITS, copies(MAX_PART_BYTES, M, N)));
    int64_t least = 1;
    if (forced_splits > 0) least = most = std::max((int64_t)1, std::min((int64_t)forced_splits, std::min(cap, n_kt)));
    const double values = (double)M * (double)N;
    int64_t nk[17];                                          // (no more divisions than there have to be: this runs on every call)
    for (int64_t s = least; s == least || s <= most; ++s) nk[s] = (n_kt + s - 1) / s;
    for (int ri = forced_ri ? forced_ri : 4; ri <= (forced_ri ? forced_ri : 8); ++ri) {
        const int64_t wgs = (M + 16 * ri - 1) / (16 * ri) * ((N + 255) / 256);
        for (int64_t s = least; s == least || s <= most; ++s) {
            if (s > 1 && s > least && wgs * s > 768) break;  // (parts of a grid that is several rounds anyway never paid)
            const double t = price(COEF[kind], wgs * s, nk[s], ri, (int)s, values);
            if (t < best.us) best = {ri, (int)s, t};
        }
    }
    return best;
}

// ---- the same two kernels in workgroups of 128 columns: four waves, two workgroups to a CU, three of 64 and 80 rows.  Rounds are
// shorter, and the first loads and the store of one workgroup lie under the other's multiplication, but the activations are read by
// twice as many workgroups.  The fastest shape of 256 and of 128 columns (us): int8 rows, 4096 x 28672 gated at M = 1000 120 and 112,
// groups of 64 142 and 131; 8192 x 10240 at M = 2048 163 and 154; 8192 x 57344 gated at M = 2048 831 and 858; bf16 rows, 190 and 193,
// 263 and 273, 1408 and 1450.

constexpr unsigned slim_at_once(int ri) { return ri <= 5 ? 768 : 512; }

struct SlimCoef {
    double launch, wg,                                       // fixed, and per workgroup / 256
           tile, tile_ri,                                    // per 256 k and round; times row tiles
           tile_cu, tile_cu_ri,                              // per 256 k and workgroup of the busiest CU
           tile_wg, tile_wg_ri,                              // per 256 k and workgroup / 256 (a full chip holds lower clocks)
           parts, part_value;                                // the second launch, and per value of a partial result
};
// Fits to 13000 graph-timed launches (64 and 80 rows, 96 and more) on 1410 problems (K 1024 to 28672, N 1024 to 57344, 34 to 4096
// rows): 4.8 to 5.5 % off in the root mean square near the fastest; the shapes chosen are 0.6 to 0.8 % slower than the fastest measured.
constexpr SlimCoef SLIM_COEF[3][2] = {
    {{4.11, 1.042, 0.102, 0.04307, 0, 0.07706, 0, 0.01219, 2.851, 8.438e-07},
     {4.417, 1.773, 0, 0.04697, 0, 0.06986, 0.04931, 0.006411, 3.066, 6.93e-07}},
    {{4.486, 0.9412, 0.0173, 0.06897, 0.005868, 0.0973, 0, 0.01047, 2.793, 7.089e-07},
     {4.773, 1.671, 0, 0.06723, 0, 0.08206, 0, 0.0118, 2.903, 6.478e-07}},
    {{4.221, 0.9432, 0.2825, 0.04993, 0.02383, 0.1266, 0, 0.0438, 3.094, 6.252e-07},
     {5.203, 1.171, 0.03201, 0.0749, 0, 0.1009, 0, 0.05355, 2.704, 6.753e-07}}};

// The cheapest; parts as `pick` has them, and no grids of more than six workgroups to a CU in parts.
inline Shape slim(Kind kind, int64_t M, int64_t N, int64_t n_kt, int64_t cap)
{
    Shape best = {8, 1, 1e30};
    const int most = (int)std::min(std::min(n_kt / 2, cap), std::min((int64_t)MAX_SPLITS, copies(MAX_PART_BYTES, M, N)));
    int nk[MAX_SPLITS + 1];                                  // (this runs on every call: 32-bit divisions)
    nk[1] = (int)n_kt;
    for (int s = 2; s <= most; ++s) nk[s] = ((int)n_kt + s - 1) / s;
    const double values = (double)M * (double)N;
    const int64_t cols = (N + 127) / 128, row_tiles = (M + 15) / 16;
    for (int ri = 4; ri <= 8; ++ri) {
        const SlimCoef& c = SLIM_COEF[kind][ri > 5];
        const unsigned tiles = (unsigned)std::min((row_tiles + ri - 1) / ri * cols, (int64_t)1 << 30);
        for (int s = 1; s <= std::max(most, 1); ++s) {
            const unsigned wgs = tiles * s;
            if (s > 1 && (tiles > 1536 || wgs > 1536)) break;
            const double rounds = (wgs + slim_at_once(ri) - 1) / slim_at_once(ri), per_cu = (wgs + 255) >> 8, fill = wgs / 256.0;
            double t = c.launch + c.wg * fill +
                       nk[s] * (rounds * (c.tile + c.tile_ri * ri) + per_cu * (c.tile_cu + c.tile_cu_ri * ri) + fill * (c.tile_wg + c.tile_wg_ri * ri));
            if (s > 1) t += c.parts + c.part_value * values * s;
            if (t < best.us) best = {ri, s, t};
        }
    }
    return best;
}

// ---- the 64-row kernel of w2a8 (matmul_a8_tiled.hip)

// bn columns per workgroup, `kw` K ranges inside a workgroup (of bn / 32 waves each) times `splits` across workgroups.
struct Shape64 {
    int bn, kw, splits;
    double us;
};

// 256-column workgroups (two per CU): linear in the workgroups of the busiest CU and the rounds, 83 and 78 launches (groups of
// 128 and 64), 2.6 and 2.5 % off in the root mean square.
inline double price64_wide(int G, int64_t M, int64_t N, int64_t n_kt, int splits)
{
    const int64_t wgs = (M + 63) / 64 * ((N + 255) / 256) * splits;
    const double per_cu = (double)((wgs + 255) / 256), rounds = (double)((wgs + 511) / 512), fill = (double)wgs / 256.0;
    const double nk = (double)((n_kt + splits - 1) / splits);
    return G == 128 ? 5.121 + 1.922 * fill + nk * (0.6839 * per_cu + 0.2249 * rounds + 0.1988 * fill)
                    : 4.816 + 1.459 * fill + 0.4825 * rounds + nk * (0.7930 * per_cu + 0.2442 * rounds + 0.2361 * fill);
}

// Narrow workgroups; a CU holds one of four K ranges, two of two, four of one.  Fitted to every (bn, kw, splits) on 130
// problems for each group size that leave fewer than 400 workgroups of 256 columns: 4.2 and 3.8 % off; the choices are 0.7 and
// 0.2 % slower than the fastest measured (3.4 and 7.8 % with prices from the work of the busiest CU alone).
struct Coef64 {
    double launch, wg, round,                                // fixed, per workgroup / 256, per round
           tile_round, tile_cu, tile_wg;                     // per 256 k of a range: and round, busiest CU's workgroup, workgroup / 256
};
constexpr Coef64 COEF64[2][4] = {                            // 128 columns with 1, 2, 4 ranges; 64 columns
    {{3.683, 0.8661, 0.0, 0.8142, 0.1763, 0.0448}, {4.361, 1.641, 0.3831, 0.3615, 0.9383, 0.0696},
     {2.363, 0.7873, 3.827, 2.193, 0.0, 0.2682}, {5.479, 0.0, 0.0, 1.674, 0.0, 0.4263}},
    {{3.351, 1.172, 0.0, 1.317, 0.3121, 0.0963}, {4.812, 1.785, 0.0, 0.2825, 1.190, 0.0},
     {3.533, 1.848, 2.648, 3.240, 0.0, 0.3995}, {5.510, 0.0, 0.0, 1.933, 0.0, 0.3805}}};
constexpr double PARTS64[2][2] = {{2.249, 1.767e-6}, {2.231, 1.726e-6}};   // the second launch; per value of a partial result

inline double price64(int G, int64_t wgs, int64_t nk, int bn, int kw, int splits, double values)
{
    const Coef64& c = COEF64[G == 128 ? 0 : 1][bn == 64 ? 3 : kw >> 1];
    const int at_once = kw == 4 ? 8 : kw == 2 ? 9 : 10;      // log2 of the workgroups that run at a time
    const double rounds = (double)((wgs + (1 << at_once) - 1) >> at_once), per_cu = (double)((wgs + 255) >> 8), fill = (double)wgs / 256.0;
    double t = c.launch + c.wg * fill + c.round * rounds + (double)nk * (c.tile_round * rounds + c.tile_cu * per_cu + c.tile_wg * fill);
    if (splits > 1) t += PARTS64[G == 128 ? 0 : 1][0] + PARTS64[G == 128 ? 0 : 1][1] * values * splits;
    return t;
}

// The cheapest narrow launch that divides the tiles evenly.  forced_*: 0, or the only value considered (kw: or the next smaller
// one that divides the tiles).  64 columns: four ranges, one round, K not split across workgroups (on top of those they lost
// everywhere: 14336 x 4096 at M = 384 62 against 38 us).
inline Shape64 pick64(int G, int64_t M, int64_t N, int64_t n_kt, int64_t cap, int forced_bn = 0, int forced_kw = 0, int forced_splits = 0)
{
    const int bn = forced_bn == 64 ? 64 : 128;
    const int64_t room = std::max(cap, (int64_t)1), wgs = (M + 63) / 64 * ((N + bn - 1) / bn);
    int64_t least = 1, most = std::min(std::min((int64_t)16, room), std::max((int64_t)1, copies((int64_t)16 << 20, M, N)));
    if (forced_splits > 0) least = most = std::min((int64_t)forced_splits, std::min(room, n_kt));
    const double values = (double)M * (double)N;
    const int tiles = (int)n_kt;                             // (32-bit divisions: this runs on every call)
    Shape64 best = {bn, 1, (int)least, 1e30};
    for (int kw = 4; kw >= 1; kw >>= 1) {
        if (forced_kw && kw > forced_kw) continue;
        for (int64_t s = least; s <= most && s <= n_kt; ++s) {
            const int ranges = kw * (int)s;
            if (s > 1 && forced_splits <= 0 && (tiles < 2 * ranges || wgs * ranges > 1600)) break;
            const int nk = (tiles + ranges - 1) / ranges;
            if (kw > 1 && nk * ranges != tiles) continue;
            const double t = price64(G, wgs * s, nk, bn, kw, (int)s, values);
            if (t < best.us) best = {bn, kw, (int)s, t};
        }
        if (forced_kw && best.us < 1e30) break;
    }
    if (!forced_bn && forced_splits <= 1 && (forced_kw == 0 || forced_kw == 4) && n_kt % 4 == 0 && (M + 63) / 64 * ((N + 63) / 64) <= 256) {
        const double t = price64(G, (M + 63) / 64 * ((N + 63) / 64), n_kt / 4, 64, 4, 1, values);
        if (t < best.us) best = {64, 4, 1, t};
    }
    return best;
}

// 256 columns per workgroup: K split across workgroups only to fill the chip, in enough parts for about 1.5 workgroups per
// CU.  A part spans at least min_tiles 256-k tiles (below that the partial results and the second launch cost more than the
// idle CUs); at most 16 parts and 16 MiB of partial results (the second launch reads them all).
inline int splits64_wide(int64_t wgs, int64_t n_kt, int64_t min_tiles, int64_t M, int64_t N, int64_t cap)
{
    if (wgs >= 192 || cap < 2) return 1;
    int64_t s = (384 + wgs - 1) / wgs;
    s = std::min(std::min(s, n_kt / min_tiles), std::min((int64_t)16, cap));
    s = std::min(s, copies((int64_t)16 << 20, M, N));
    return s < 2 ? 1 : (int)s;
}

// 256 columns per workgroup unless that leaves the chip's 512 workgroup slots clearly underfilled.  Fewer than 400 tiles of
// 64 x 256: from a few dozen to a few hundred workgroups against 256 CUs, so K is cut both across and inside workgroups of
// 128 or 64 columns, by price.
inline Shape64 shape64(int G, int64_t M, int64_t N, int64_t n_kt, int64_t cap, const w2_tuning_t& tune)
{
    const int64_t wgs = (M + 63) / 64 * ((N + 255) / 256);
    const int bn = tune.tiled_bn;
    if (bn == 64 || bn == 128 || (bn != 256 && wgs < 400)) return pick64(G, M, N, n_kt, cap, bn, tune.tiled_kw, tune.splitk);
    const int splits = tune.splitk > 0 ? (int)std::min((int64_t)tune.splitk, std::min(std::max(cap, (int64_t)1), n_kt))
                                       : splits64_wide(wgs, n_kt, tune.splitk_min_tiles ? tune.splitk_min_tiles : 12, M, N, cap);
    return {256, 1, splits, price64_wide(G, M, N, n_kt, splits)};
}

// No launch of them is priced below: one 256-k tile in one workgroup.
constexpr double least(const Coef& c) { return c.launch + c.round + 4 * c.round_ri + c.tile + 4 * c.tile_ri; }
constexpr double least(const Coef64& c) { return c.launch + c.round + c.tile_round + c.tile_cu; }
constexpr double least_us(Kind kind)
{
    double t = least(COEF[kind]);
    if (kind != A16)
        for (const Coef64& c : COEF64[kind == A8_G128 ? 0 : 1]) t = least(c) < t ? least(c) : t;
    return t;
}
constexpr double LEAST_US[3] = {least_us(A8_G128), least_us(A8_G64), least_us(A16)};

// ---- w2a8: which of its two kernels, and its launch shape

struct A8Shape {
    int ri;                                                  // 16-row tiles per wave of the tall kernel (4 to 8); 0: the 64-row kernel
    int bn, kw, splits;                                      // columns per workgroup, K ranges inside and across workgroups
    double us;                                               // the price
};

inline A8Shape a8_shape(int G, int64_t M, int64_t N, int64_t n_kt, int64_t cap, const w2_tuning_t& tune)
{
    const Kind kind = G == 128 ? A8_G128 : A8_G64;
    if (tune.tiled_bm == 128) {                              // forced 128-row tiles (tuning and tests)
        const Shape t = pick(kind, M, N, n_kt, cap, 8, tune.splitk);
        const bool few = (M + 127) / 128 * ((N + 255) / 256) <= 128;
        const int bn = tune.tiled_bn == 128 || tune.tiled_bn == 256 ? tune.tiled_bn : few && t.splits < 2 ? 128 : 256;
        // (128 columns and groups of 64: a forced width keeps the whole K, as it did when no instantiation there split it; AUTO's
        // parts over 128 columns are `slim`'s)
        return {8, bn, 1, bn == 128 && G == 64 ? 1 : t.splits, t.us};
    }
    const Shape64 p = shape64(G, M, N, n_kt, cap, tune);
    const A8Shape low = {0, p.bn, p.kw, p.splits, p.us};
    // forced shapes that only the 64-row kernel has
    if (tune.tiled_bm == 64 || tune.tiled_bn == 64 || tune.tiled_bn == 128 || tune.tiled_kw || tune.tiled_wd) return low;
    const Shape t = pick(kind, M, N, n_kt, cap, 0, tune.splitk);
    // (256-column workgroups: the margins that leave the fewest of 380 measured problems slower than in these tiles.  Narrow ones
    // with groups of 64: over 120 problems near the line a share of 1.0 loses 1.0 %, 0.95 0.3 %; 27648 x 5440 at M = 506 without a
    // workspace 150 us in tall tiles, 137 in 64-row ones.  With groups of 128 1.0 is best: 0.2 %, 0.95 2.3 %.)
    const double share = p.bn < 256 ? (G == 128 ? 1.0 : 0.95) : G == 128 ? 0.985 : 0.965;
    const bool tall = t.us < p.us * share;
    return tall ? A8Shape{t.ri, 256, 1, t.splits, t.us} : low;
}

// ---- w2a16: the scale-folded kernel; forced 128-column workgroups keep 128 rows (tuning and tests)
inline Shape a16_shape(int64_t M, int64_t N, int64_t n_kt, int64_t cap, const w2_tuning_t& tune)
{
    return pick(A16, M, N, n_kt, cap, tune.tiled_bn == 128 ? 8 : 0, tune.splitk);
}

}  // namespace tiles

}  // namespace w2
