// The mid-M kernel's launch shape: host code only, no HIP, so that a test can compile it by itself.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/w2mm.h"

namespace w2 {

namespace midm {

constexpr int CHUNK_BYTES = 128;                             // bytes of a row in one staged chunk

constexpr int stage_bytes(int rt, int sh) { return rt * 16 * CHUNK_BYTES * (sh > 1 ? 2 : 1); }     // of one K range
constexpr int red_bytes(int rt, int cj) { return rt * 16 * (cj * 16 + 4) * 4; }                     // of one wave
// bytes of local memory of one K range (sh waves): its staged chunks, later its waves' partial results
constexpr int range_lds(int rt, int cj, int sh)
{
    return stage_bytes(rt, sh) > sh * red_bytes(rt, cj) ? stage_bytes(rt, sh) : sh * red_bytes(rt, cj);
}
// most waves of a workgroup: 16 where a wave's registers allow it (very deep and narrow projections), else 8
constexpr int max_waves(int rt, int cj) { return rt == 1 && cj <= 2 ? 16 : 8; }

// Launch shape: row tiles and column blocks per wave, K ranges per workgroup, waves that share a range, workgroups that
// K is split across (parts).
struct Plan { int rt, cj, ks, sh, sp; };

// Waves of each instantiation that a SIMD's registers hold (int8, bf16 rows; [rt - 1][cj: 1, 2, 4]).
constexpr int SIMD_WAVES[2][4][3] = {{{6, 5, 4}, {4, 3, 2}, {4, 3, 2}, {3, 2, 2}},
                                     {{6, 5, 4}, {4, 3, 2}, {3, 3, 2}, {4, 2, 2}}};

// The shapes of a workgroup: K ranges x waves that share one, and how many such workgroups a CU holds.
constexpr int FORMS[4][2] = {{16, 1}, {8, 1}, {4, 1}, {2, 2}};
constexpr int resident_of(int xt, int rt, int cj, int ks, int sh)
{
    const int by_lds = 160 * 1024 / (ks * range_lds(rt, cj, sh) + rt * 64);
    const int by_regs = 4 * SIMD_WAVES[xt][rt - 1][cj >> 1] / (ks * sh);
    const int r = by_lds < by_regs ? by_lds : by_regs;
    return r > 1 ? r : 1;
}
struct Resident {
    int8_t n[2][4][3][4];
    constexpr Resident() : n{}
    {
        for (int xt = 0; xt < 2; ++xt)
            for (int rt = 1; rt <= 4; ++rt)
                for (int cj = 1; cj <= 4; cj *= 2)
                    for (int f = 0; f < 4; ++f) n[xt][rt - 1][cj >> 1][f] = (int8_t)resident_of(xt, rt, cj, FORMS[f][0], FORMS[f][1]);
    }
};
constexpr Resident RESIDENT;

// Every candidate shape is priced with a linear model and the cheapest wins.  The terms are what the busiest CU has to
// do (nb workgroups, in rounds of as many as it holds at a time), the coefficients (us) a least-squares fit to 4400
// graph-timed launches: 20 projection shapes from 2048 x 2048 and 28672 x 1024 to 8192 x 57344, 4 to 192 rows.  On 70
// further shapes (K 2048 to 28672, N 1024 to 28672, 3 to 240 rows) its choices are on average 2.7 % (int8 rows) and
// 0.9 % (bf16 rows) slower than the fastest shape measured.
constexpr double COEF[2][13] = {
    {1.525, 0.1987e-2, 0.6254e-2, 1.419e-2, 1.127e-4, 0.3743e-4, 0.8993e-2, 0.4517e-1, 0.3403e-1, 0.6996, 0.6068e-1, 0.7275e-1, 0.3929e-3},
    {1.677, 1.494e-2, 0.3030e-2, 3.895e-2, 0.9297e-4, 0.9087e-4, 0.7657e-2, 0.0, 0.5634e-1, 0.4702, 0.9276e-1, 1.174e-1, 0.1319e-3}};

// Int8 rows: what all workgroups together read of the rows comes out of the L2s at about 12 MB a microsecond; on a deep K
// that is what a launch of narrow workgroups waits for, and the linear terms have no such limit.  Above 172 MB shapes of one
// or two column blocks per workgroup are left out, which leaves four, half the stream (28672 x 8192 at M = 32 / 48 / 144
// 23.2 / 29.5 / 66.8 -> 21.3 / 25.2 / 53.5 us, 8192 x 6144 at M = 128 11 % faster; 24576 x 5120 at M = 48, 188 MB, 16 %).
// The other side of the line: 17408 x 6144 at M = 48, 160 MB, takes 14.3 with two and 14.8 with four, 20480 x 4096 at M = 64,
// 168 MB, 21 % longer with four.  Over 1157 measured problems the choices are 2.8 % slow on average with the limit at 150 MB
// to 250 MB, and 27 to 30 % at worst.
constexpr int64_t ROW_BYTES_FROM_L2 = 172000000;

// K split across workgroups: a second launch adds the parts, which go to memory and back (us, and us per value of a part;
// fitted on 36 shapes from 8192 x 1024 to 28672 x 10240, int8 and bf16 rows), and it has to win by more than the model errs.
constexpr double PARTS_US[2] = {1.0, 2.0}, PARTS_US_PER_VALUE[2] = {3e-6, 2e-6}, PARTS_MARGIN = 1.04;

// `cap`: fp32 copies of the output that the workspace holds.  us: where the price goes, if wanted.
inline Plan plan(int xt, int64_t M64, int64_t n_cb64, int64_t n_kt64, bool gated, int64_t cap, const w2_tuning_t& tune,
                 double* us = nullptr)
{
    const double* c = COEF[xt];
    const int M = (int)M64, n_cb = (int)n_cb64, n_kt = (int)n_kt64;
    const double tiles = (double)n_cb * n_kt;
    const double part_us = PARTS_US_PER_VALUE[xt] * 16 * M * (double)n_cb;
    const int cbw = xt == 1 ? std::min(tune.midm_cbw, 4) : tune.midm_cbw;
    const int forced = tune.splitk > 1 ? (int)std::min<int64_t>(std::min(tune.splitk, n_kt), cap) : 0;
    Plan best = {1, 2, 1, 1, 1};
    double best_price = 1e30;
    // (this runs on every call of up to 256 rows: no division but by powers of two, where it can be had)
    auto price = [&](const Plan& p, int bands, int groups, int T, int resident) {
        const int wgs = groups * bands * p.sp, waves = p.ks * p.sh;
        const int nb = (wgs + 255) >> 8;
        const int rounds = nb <= resident ? 1 : (nb + resident - 1) / resident;
        const int rc = p.rt * p.cj;
        double t = c[0]
                 + (double)(nb * waves) * T * (c[1] * p.cj               // up-converts
                                               + c[2] * rc)             // matrix instructions and dequant
                 + c[3] * ((double)(nb * p.ks) * T * p.rt)               // activations through the L1
                 + tiles * (c[4] + c[5] * bands)                         // the weight stream; ... once per band out of L2
                 + c[6] * (nb * waves * rc)                              // reduce and store
                 + (double)rounds * T * (c[7] + c[8] * rc)               // latency per tile, multiply,
                 + rounds * (c[9] + c[10] * rc)                          // start and end of a wave
                 + c[11] * T
                 + c[12] * wgs;                                          // workgroups to launch
        if (p.sp > 1) t = PARTS_MARGIN * (t + PARTS_US[xt] + part_us * p.sp);
        return t;
    };
    const int row_tiles = std::min((M + 15) / 16, 4);
    for (int rt = 1; rt <= row_tiles; ++rt) {
        const int bands = (M + 16 * rt - 1) / (16 * rt);
        for (int lj = rt == 1 ? 0 : 1; lj <= 2; ++lj)
            for (int f = max_waves(rt, 1 << lj) == 16 ? 0 : 1; f < (xt == 0 ? 4 : 3); ++f) {
                const int cj = 1 << lj, sh = FORMS[f][1], lw = lj + (sh - 1);       // 1 << lw column blocks per workgroup
                if (gated && lw == 0) continue;                          // a workgroup pairs gate and up blocks
                if (cbw && 1 << lw != cbw) continue;
                const int groups = (n_cb + (1 << lw) - 1) >> lw;
                if (xt == 0 && lw <= 1 && !cbw && (int64_t)groups * M * n_kt * 256 > ROW_BYTES_FROM_L2) continue;
                const int resident = RESIDENT.n[xt][rt - 1][cj >> 1][f];
                auto offer = [&](int ks, int sp, int T, int res) {
                    const Plan p = {rt, cj, ks, sh, sp};
                    const double t = price(p, bands, groups, T, res);
                    if (t < best_price) { best = p; best_price = t; }
                };
                const int lk = 4 - f;                                    // FORMS[f][0] == 1 << lk
                if (forced > 1) {
                    const int ks = std::max(1, std::min(1 << lk, n_kt / forced));
                    offer(ks, forced, (n_kt + ks * forced - 1) / (ks * forced), resident);
                    continue;
                }
                if (n_kt >= 1 << lk) offer(1 << lk, 1, (n_kt + (1 << lk) - 1) >> lk, resident);
                else offer(n_kt, 1, 1, resident_of(xt, rt, cj, n_kt, sh));
                // Across workgroups: grids that leave half the chip idle, in as many parts as still run at once, one per CU, and
                // with bf16 rows (whose workgroups take longer) grids of one round in two per CU, where two fit; other
                // numbers of parts were hardly ever faster by more than 3 %.  From K = 8192 on, with int8 rows from 20480 (17408 x
                // 1024 at M = 5 7.1 us in parts, 5.6 in one piece).
                const int wgs = groups * bands;
                if (cap < 2 || n_kt < (xt == 0 ? 80 : 32) || lw == 0 || f == 0 || tune.splitk == 1) continue;
                const int at_once = wgs <= 128 ? 256 : xt == 1 && wgs <= 256 && resident >= 2 ? 512 : 0;
                const int sp = (int)std::min<int64_t>(std::min(at_once / wgs, n_kt >> (lk + 1)), std::min<int64_t>(8, cap));
                if (sp >= 2) offer(1 << lk, sp, (n_kt + (sp << lk) - 1) / (sp << lk), resident);
            }
    }
    if (us) *us = best_price;
    return best;
}

}  // namespace midm

}  // namespace w2
