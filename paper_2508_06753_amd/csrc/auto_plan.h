// AUTO: which kernel a call goes to, and the launch shape of the kernels that have several.  Host code only, no HIP, so that a
// test can compile it by itself.  What is priced for the choice is launched as priced: a shape is found once per call.
#pragma once
#include <stdint.h>

#include "midm_plan.h"
#include "shared_plan.h"
#include "tile_plan.h"

namespace w2 {

namespace route {

// Most rows of each kernel.
constexpr int64_t DOT4_ROWS = 4, SMALL_ROWS = 16, GEMV_ROWS = 32, MIDM_ROWS = 256;

// The tiled kernels before the mid-M kernel where both take the rows: where their price (tile_plan.h) is under this share of its
// price (midm_plan.h).  By activations and by the shape that the mid-M kernel would run: eight K ranges and more to a workgroup are
// priced 3 to 9 % high on the deep K where the two meet, four and fewer are not.  Loss against the faster of the two, graph-timed on
// 1850 random problems of 33 to 250 rows around the line (K from 1024, N from 1024 up), in per cent by share:
//   int8 rows, fewer than eight ranges  0.86 3.9, 0.94 1.6, 1.0 1.0, 1.05 1.0     eight  0.84 0.54, 0.88 0.45, 0.94 0.6, 1.0 1.7
//   bf16 rows, fewer than eight ranges  0.93 1.5, 0.96 0.8, 1.0 0.3, 1.05 0.5     eight  0.90 1.8, 0.94 0.7, 0.96 0.6, 1.0 0.7
// With one share of 0.86 for all int8 and 0.93 for all bf16 rows 26880 x 9664 at M = 127 took 55 us instead of 47, 13312 x 6688
// with bf16 rows and groups of 64 at M = 226 57 instead of 51; 220 further problems whose kernel changed are 7 % faster.
constexpr double TILED_SHARE[2][2] = {{1.0, 0.88}, {1.0, 0.94}};
// (The int8 ones further by the kernel, whose price runs a few per cent low for the 64-row one on wide grids.  Fewer than eight
// ranges, loss by share: 64-row tiles 0.94 0.5, 1.0 1.0, taller ones 0.94 1.8, 1.0 1.0; 7680 x 33408 at M = 101 55 us against 51.)
constexpr double LOW_TILES_SHARE = 0.94;
inline double tiled_share(int a16, const midm::Plan& p, bool low_tiles)
{
    return low_tiles && p.ks < 8 ? LOW_TILES_SHARE : TILED_SHARE[a16][p.ks >= 8];
}

// The mid-M kernel that shares its rows (shared_plan.h) instead of what would run otherwise: where its price is under this share of
// that kernel's.  By what would run and by rows; loss or gain against never taking it, graph-timed on 1130 random problems of 17 to
// 150 rows (N from 4096, K from 768), time by share:
//   mid-M kernel, fewer than eight K ranges   to 32 rows   int8 0.96 0.985, 1.0 0.978, 1.06 0.970 (6 of 88 slower by over 3 %; 1 at 1.0)
//                                                          bf16 0.96 0.962, 0.98 0.953, 1.02 0.946 (4 of 77 slower; 1 at 0.98)
//                                             above        int8 1.0 0.909, 1.06 0.882;  bf16 1.0 0.886, 1.02 0.878, 1.06 0.879
//   eight K ranges: not offered.  Thirty of 2000 further problems, timed through these calls against never taking it: 33 to 64 rows
//                   1.0 1.012 (12544 x 15488 gated bf16 M = 46 29.6 -> 32.2 us), above 1.04 0.997 (18688 x 7168 int8 M = 73 21.8 -> 23.5)
//   64-row tiles 1.04 0.982;  tall tiles 0.92 0.990, 1.0 0.992 (2 of 26 slower);  w2a16 0.88 0.977, 1.0 0.986 (12 of 71 slower; 5 at 0.88)
constexpr double SHARED_SHARE_LOW = 1.04, SHARED_SHARE_TALL[2] = {0.92, 0.88};
inline double shared_share(int a16, int64_t M, const midm::Plan& p)
{
    if (p.ks >= 8) return 0.0;
    return M <= 32 ? (a16 ? 0.98 : 1.0) : a16 ? 1.02 : 1.06;
}

// The tiled kernels' 128-column workgroups (tiles::slim), from 33 rows on: where their price is under this share of that of the tiled
// shape that would run.  Graph-timed on random problems of 34 to 4096 rows, time by share against never taking them: 64-row tiles 0.92
// 0.928, 1.0 0.903 (2 of 135 slower by over 3 %), 1.06 0.901 (8); tall tiles of 256 columns, groups of 128 0.88 0.989 (7 of 157
// slower), 0.92 0.985 (15); groups of 64 0.90 0.973 (3 of 180), 0.94 0.971 (11); w2a16 0.90 0.966 (4 of 356), 0.94 0.965 (22).  Of
// 420 further problems near the lines, time by the quotient of the prices: groups of 128 0.88 to 0.90 0.942, to 0.92 0.983, to 0.94 0.987, to 0.96
// 1.008; groups of 64 0.90 to 0.92 0.981, to 0.94 0.983 (none slower by over 3 %), to 0.96 0.999; w2a16 0.90 to 0.92 0.985, to 0.94 1.010.
// (Part of what keeps the tall ones below 1: the prices of the 256-column tiles are from before their rows went straight to local
// memory and run about 8 % high.)  Where rows would be shared instead, 0.98.  Not offered where the mid-M kernel would run: 0.996 of its time over 414 problems.
constexpr double SLIM_SHARE = 0.98, SLIM_SHARE_LOW = 1.0, SLIM_SHARE_TALL[3] = {0.90, 0.94, 0.90};
constexpr int64_t SLIM_LEAST_ROWS = 33;

struct Problem {
    int64_t M, K, N;
    int64_t n_cb, n_kt;                                      // column blocks, 256-k tiles
    int G;
    bool gated;
    int64_t cap;                                             // fp32 copies of the output that the workspace holds
};

inline midm::Plan midm_shape(int a16, const Problem& p, const w2_tuning_t& tn, double* us = nullptr)
{
    return midm::plan(a16, p.M, p.n_cb, p.n_kt, p.gated, p.cap, tn, us, p.G);
}

// What takes the place of the kernel that would run, if anything does.
struct Instead {
    bool to_shared, to_slim;
    shared::Plan shared;
    tiles::Shape slim;
};

// `us`: price of the kernel that would run; the shares of it.  The two prices take a call up to 0.13 us on the host, of the 4.8 that a
// call of 17 to 144 rows takes there.  (Not where the caller says which rows the decode or the mid-M kernel
// gets, or what a launch shape is to be.)
inline Instead instead(int a16, const Problem& p, const w2_tuning_t& tn, double us, double shared_share, double slim_share)
{
    Instead r = {};
    if (tn.midm_min_m || tn.midm_max_m || tn.gemv_max_m || tn.midm_cbw || tn.splitk || tn.splitk_min_tiles || tn.tiled_bm || tn.tiled_bn ||
        tn.tiled_kw || tn.tiled_wd)
        return r;
    if (shared_share > 0 && shared::offered(p.M, p.n_cb, p.n_kt)) {
        double price;
        r.shared = shared::plan(a16, p.M, p.n_cb, p.n_kt, p.gated, p.G, &price);
        r.to_shared = price < us * shared_share;
        if (r.to_shared) { us = price; slim_share = slim_share > 0 ? SLIM_SHARE : 0; }
    }
    if (p.M >= SLIM_LEAST_ROWS && slim_share > 0) {
        r.slim = tiles::slim(a16 ? tiles::A16 : p.G == 128 ? tiles::A8_G128 : tiles::A8_G64, p.M, p.N, p.n_kt, p.cap);
        r.to_slim = r.slim.us < us * slim_share;
        if (r.to_slim) r.to_shared = false;
    }
    return r;
}

// ---- w2a8

struct A8 {
    int variant;                                             // (of the kernels that can be asked for by name)
    Instead instead;                                         // of it
    int fallback;                                            // where the decode kernel turns the rows down
    bool has_midm, has_tiled;                                // shapes found on the way
    midm::Plan midm;
    tiles::A8Shape tiled;
};

inline tiles::A8Shape a8_tiled_shape(const Problem& p, const w2_tuning_t& tn) { return tiles::a8_shape(p.G, p.M, p.N, p.n_kt, p.cap, tn); }

inline A8 a8(const Problem& p, const w2_tuning_t& tn)
{
    const int64_t M = p.M;
    A8 r = {};
    // Few rows: the decode kernel, which reads the weights once and keeps whole rows in local memory (the MFMA
    // form is at least as fast as dot4 from M = 1 on).  Then the mid-M kernel, then the tiled ones.
    // Where the mid-M kernel takes over (graph-timed, every launch with rows and weights of its own, us, what ran
    // before against the mid-M kernel): at M = 9 in general (4096 x 6144 5.3 against 5.2 at M = 16; 4096 x 28672 at
    // M = 8 / 9 9.2 / 10.1 against 9.6 / 9.7; 8192 x 10240 8.8 / 11.7 against 8.8 / 8.9).  At M = 5 where the decode
    // kernel has few workgroups and two pieces of a row per thread (decode / mid-M at M = 5 and 8, 192 to 512 column
    // blocks: K = 4096 0.91 .. 1.05, but 1.20 on 320 blocks; K = 5120 1.08 .. 1.24, 6144 1.03 .. 1.20, 7168 0.91 .. 1.10,
    // 8192 0.93 .. 1.01), on a deep K of few columns (17408 x 1024 1.19, x 2048 0.98), and below where it cannot hold the
    // rows in one round of workgroups (17408 x 5120 1.35, x 4096 0.94).  At 13 on 16384 columns and more with groups of
    // 64 (5120 x 34816 at M = 12 / 16 15.2 / 21.4 against 16.1 / 17.2).  At 17 where K near 8192 keeps its whole grid
    // busy in one round, 768 to 1024 column blocks (K = 8192 at M = 9 .. 16 0.91 .. 0.97, 7168 1.00 .. 1.05).
    const bool wide = p.n_cb >= 1024;
    const int midm_from = p.n_kt > 28 && p.n_kt <= 32 && p.n_cb >= 768 && p.n_cb <= 1024 ? 17
                        : wide                                                           ? (p.G == 128 ? 9 : 13)
                        : (p.n_kt > 64 && p.n_cb < 128) || (p.n_kt > 16 && p.n_kt <= 26 && p.n_cb <= 512) ? 5 : 9;
    const int midm_min = tn.midm_min_m ? tn.midm_min_m : midm_from;
    // Upper end, against the tiled kernels with a workspace: they win earlier the more columns there are to fill
    // the chip with (2048 x 57344 at M = 48 / 64 16.6 / 17.4 us against 15.3 / 18.5; 4096 x 28672 at M = 96 / 128
    // 24.3 / 25.2 against 20.4 / 24.9; 8192 x 10240 at M = 160 / 192 24.8 / 25.1 against 24.3 / 26.0; 5120 x 7168
    // at M = 192 / 256 17.4 / 17.5 against 14.1 / 17.7; 28672 x 5120 at M = 240 50.2 against 54.5).
    const int midm_max = tn.midm_max_m ? tn.midm_max_m
                       : p.n_cb >= 2560 ? 48 : p.n_cb >= 1536 ? 112 : p.n_cb > 448 ? 160 : p.G == 128 && p.n_kt > 104 && p.n_cb > 256 ? 192 : 240;
    // Below it, from 33 rows on, by price.
    bool tiled_first = false;
    double midm_us = 0;
    if (M > 32 && M >= midm_min && M <= midm_max && !tn.midm_max_m) {
        double& us = midm_us;
        r.midm = midm_shape(0, p, tn, &us);
        r.has_midm = true;
        if (us * tiled_share(0, r.midm, false) > tiles::LEAST_US[p.G == 128 ? tiles::A8_G128 : tiles::A8_G64]) {
            r.tiled = a8_tiled_shape(p, tn);
            r.has_tiled = true;
            tiled_first = r.tiled.us < us * tiled_share(0, r.midm, r.tiled.ri == 0);
        }
    }
    const bool midm_ok = M >= midm_min && M <= midm_max && !tiled_first && M <= MIDM_ROWS;
    // Rows of more than 72 KiB leave the decode kernel one workgroup per CU: then the grid must fit the chip in one
    // round (or K be moderate), else the mid-M kernel from M = 5 on there too.
    const int64_t row_bytes = M * (p.K + 32);
    int gcbw = 4;                                            // (the decode kernel's rule for five rows and more)
    while (gcbw > 1 && (p.n_cb / gcbw < 192 || (p.n_kt + 8 / gcbw - 1) / (8 / gcbw) > 16)) gcbw >>= 1;
    const int64_t gemv_wgs = (p.n_cb + gcbw - 1) / gcbw;
    const bool one_round = row_bytes <= 72 * 1024 || gemv_wgs <= 256 || p.n_kt <= 32;
    const int gemv_max = tn.gemv_max_m ? tn.gemv_max_m : one_round ? midm_from - 1 : 4;
    r.fallback = midm_ok || (!tn.midm_min_m && M >= 4 && M < midm_min && M <= midm_max) ? W2_VARIANT_MIDM
               : M <= SMALL_ROWS                                                        ? W2_VARIANT_SMALLM
                                                                                        : W2_VARIANT_TILED;
    r.variant = M <= tn.dot4_max_m && M <= DOT4_ROWS ? W2_VARIANT_DOT4
              : M <= gemv_max && M <= GEMV_ROWS      ? W2_VARIANT_GEMV
                                                     : r.fallback;
    if (r.variant == W2_VARIANT_MIDM && M >= shared::LEAST_ROWS) {
        if (!r.has_midm) { r.midm = midm_shape(0, p, tn, &midm_us); r.has_midm = true; }
        r.instead = instead(0, p, tn, midm_us, shared_share(0, M, r.midm), 0);
    } else if (r.variant == W2_VARIANT_TILED) {
        if (!r.has_tiled) { r.tiled = a8_tiled_shape(p, tn); r.has_tiled = true; }
        r.instead = instead(0, p, tn, r.tiled.us, r.tiled.ri ? SHARED_SHARE_TALL[0] : SHARED_SHARE_LOW, r.tiled.ri ? SLIM_SHARE_TALL[p.G == 64] : SLIM_SHARE_LOW);
    }
    return r;
}

// ---- w2a16

struct A16 {
    bool gemv_first;                                         // the decode kernel, where a workgroup can hold the rows
    Instead instead;                                         // of the mid-M or the tiled kernel
    bool to_midm;                                            // then the mid-M kernel, else the small-M or the tiled one
    bool has_midm, has_tiled;
    midm::Plan midm;
    tiles::Shape tiled;
};

inline tiles::Shape a16_tiled_shape(const Problem& p, const w2_tuning_t& tn) { return tiles::a16_shape(p.M, p.N, p.n_kt, p.cap, tn); }

inline bool a16_tiled_first(const Problem& p, const w2_tuning_t& tn, A16* r, double* midm_us)
{
    r->midm = midm_shape(1, p, tn, midm_us);
    r->has_midm = true;
    const double us = *midm_us * tiled_share(1, r->midm, false);
    if (us <= tiles::LEAST_US[tiles::A16]) return false;
    r->tiled = a16_tiled_shape(p, tn);
    r->has_tiled = true;
    return r->tiled.us < us;
}

inline A16 a16(const Problem& p, const w2_tuning_t& tn)
{
    const int64_t M = p.M;
    A16 r = {};
    // Few rows: the decode kernel wherever a workgroup can hold them, else the small-M kernel (both with the
    // zero-point construction); then the mid-M kernel; above, tiles of 64 to 128 rows.  Both of the latter fold the scale
    // into the weights: fewest vector instructions per matrix instruction.
    // Where the mid-M kernel takes over (graph-timed, every launch with rows and weights of its own, us, what ran
    // before against the mid-M kernel): at M = 3 for rows too long for a workgroup (17408 x 5120 16.5 against
    // 13.2), at M = 5 where K passes 4096 (5120 x 5120 8.2 against 5.8, 14336 x 4096 10.7 against 8.8, 8192 x 10240
    // 15.5 against 12.7) but for 768 to 1024 column blocks up to K = 8192, whose grid fills one round (decode / mid-M
    // at M = 5 and 8 0.85 .. 0.98; K = 9216 1.41 .. 1.53), at 8 on wide projections of K = 5120 (5120 x 34816 at M =
    // 6 / 8 19.1 / 24.3 against 20.4), and at 9 up to K = 4096 (4096 x 6144 at M = 8 / 9 5.9 / 7.1 against 5.7; 4096 x 28672 12.0 / 13.3
    // against 13.1), with groups of 64 and 16384 columns at 17 (at M = 16 / 24 13.9 / 22.0 against 14.7 / 17.6).
    const int midm_from = p.n_kt > 64                                  ? 3
                        : p.n_kt > 20 && p.n_kt <= 32 && p.n_cb >= 768 && p.n_cb <= 1024 ? 9
                        : p.n_kt > 20 || (p.n_kt > 16 && p.n_cb < 640) ? 5
                        : p.n_kt > 16                                  ? 8
                        : p.G == 128 || p.n_cb < 1024                  ? 9 : 17;
    const int midm_min = tn.midm_min_m ? tn.midm_min_m : midm_from;
    // Upper end, against the tiled kernel (8192 x 57344 at M = 64 / 96 95 / 101 us against 77 / 114; 4096 x 28672 at
    // M = 96 / 128 36.4 / 39.1 against 33.9 / 40.7; 4096 x 4096 at M = 256 22.9 against 12.3).  Below it, from 33 rows
    // on, by their prices (tile_plan.h, midm_plan.h).
    const int64_t midm_max = tn.midm_max_m                               ? tn.midm_max_m
                           : p.n_cb >= 2560                              ? 64
                           : p.n_cb >= 1024 || p.n_cb * p.n_kt > 40000   ? 96
                           : p.n_cb <= 448 && p.n_kt <= 56               ? 256 : 192;
    double midm_us = 0;
    const bool tiled_first = M > 32 && M >= midm_min && M <= midm_max && !tn.midm_max_m && a16_tiled_first(p, tn, &r, &midm_us);
    r.gemv_first = M < midm_min;
    // (from three rows on the mid-M kernel, not the small-M one, also takes what the decode kernel turns down)
    r.to_midm = (M >= midm_min || (!tn.midm_min_m && M >= 3)) && M <= midm_max && !tiled_first && M <= MIDM_ROWS;
    if (!r.gemv_first && r.to_midm && M >= shared::LEAST_ROWS) {
        if (!r.has_midm) { r.midm = midm_shape(1, p, tn, &midm_us); r.has_midm = true; }
        r.instead = instead(1, p, tn, midm_us, shared_share(1, M, r.midm), 0);
    } else if (!r.gemv_first && !r.to_midm && M > SMALL_ROWS) {
        if (!r.has_tiled) { r.tiled = a16_tiled_shape(p, tn); r.has_tiled = true; }
        r.instead = instead(1, p, tn, r.tiled.us, SHARED_SHARE_TALL[1], SLIM_SHARE_TALL[2]);
    }
    return r;
}

// Most parts that AUTO cuts K into across 128-column workgroups, given the room, with any epilogue (the gated one changes what the
// other kernels cost): what a workspace has to hold for that choice.
inline int slim_parts(int a16, Problem p, const w2_tuning_t& tn)
{
    int parts = 1;
    for (int gated = 0; gated <= (p.N % 32 == 0); ++gated) {
        p.gated = gated != 0;
        const Instead r = a16 ? route::a16(p, tn).instead : route::a8(p, tn).instead;
        if (r.to_slim && r.slim.splits > parts) parts = r.slim.splits;
    }
    return parts;
}

}  // namespace route

}  // namespace w2
