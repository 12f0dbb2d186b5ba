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

constexpr int MAX_CJ = 5;
// Waves that a SIMD's registers hold at least ([kind of rows and groups][rt - 1][cj - 1]), over the instantiations that take the
// whole of K; pairs of waves, the exact dequant and two row tiles x 2 blocks with groups of 64 mostly hold one more, which the
// prices were fitted without.  A workgroup fewer than claimed costs a round: groups of 64 claimed five at one row tile x 2 blocks,
// and 1280 x 12896 took 8.3 us with 18 bf16 rows; with four 6.1 (22784 x 13184 at M = 8, claimed to hold parts in one round, 34.7
// -> 29.2).
enum Kind { INT8, BF16, BF16_G64, N_KINDS };                 // (int8 rows: both group sizes alike)
inline Kind kind_of(int xt, int G) { return xt == 0 ? INT8 : G == 64 ? BF16_G64 : BF16; }
constexpr int SIMD_WAVES[N_KINDS][4][MAX_CJ] = {{{6, 5, 4, 4, 3}, {4, 3, 3, 2, 2}, {4, 3, 2, 2, 2}, {3, 2, 2, 2, 1}},
                                                {{6, 5, 4, 4, 3}, {4, 3, 3, 2, 2}, {3, 3, 2, 2, 2}, {4, 2, 2, 2, 1}},
                                                {{6, 4, 4, 4, 3}, {4, 3, 3, 2, 2}, {3, 3, 2, 2, 2}, {4, 2, 2, 2, 1}}};
// The same where K is split across workgroups: two instantiations that store parts take more registers than the whole ones.
constexpr int simd_waves(int kind, int rt, int cj, bool parts)
{
    if (parts && kind != INT8 && rt == 1 && cj == 2) return 4;
    if (parts && kind == BF16_G64 && rt == 1 && cj == 4) return 3;
    return SIMD_WAVES[kind][rt - 1][cj - 1];
}

// The shapes of a workgroup: K ranges x waves that share one.
constexpr int N_FORMS = 5;
constexpr int FORMS[N_FORMS][2] = {{16, 1}, {8, 1}, {4, 1}, {2, 2}, {4, 2}};
constexpr int FORM_LOG[N_FORMS] = {4, 3, 2, 1, 2};           // FORMS[f][0] == 1 << FORM_LOG[f]
constexpr int resident_of(int kind, int rt, int cj, int ks, int sh, bool parts)
{
    const int by_lds = 160 * 1024 / (ks * range_lds(rt, cj, sh) + rt * 64);
    // A workgroup's waves go round the four SIMDs from the same one on, so of 5, 6, 9 or 10 waves it is the SIMD with the most that
    // fills up: 10 waves of one row tile x 2 blocks run one workgroup to a CU, not two, 6 of three row tiles x 2 blocks too.  Priced as
    // two 1536 x 8384 took 12.0 us with 71 bf16 rows, now 8.0 in another shape, 1280 x 6112 with 243 17.3 and 10.7, 2560 x 2112 with 79
    // int8 rows 6.1 and 4.6; 300 random problems whose shape changes 14 % less.
    const int waves = ks * sh, per_simd = simd_waves(kind, rt, cj, parts);
    const int by_regs = waves <= 4 ? 4 * per_simd / waves : per_simd / ((waves + 3) / 4);
    const int r = by_lds < by_regs ? by_lds : by_regs;
    return r > 1 ? r : 1;
}
struct Resident {
    int8_t n[N_KINDS][2][4][MAX_CJ][N_FORMS];                // workgroups that a CU holds; [1]: that store parts
    constexpr Resident() : n{}
    {
        for (int k = 0; k < N_KINDS; ++k)
            for (int parts = 0; parts < 2; ++parts)
                for (int rt = 1; rt <= 4; ++rt)
                    for (int cj = 1; cj <= MAX_CJ; ++cj)
                        for (int f = 0; f < N_FORMS; ++f)
                            n[k][parts][rt - 1][cj - 1][f] = (int8_t)resident_of(k, rt, cj, FORMS[f][0], FORMS[f][1], parts);
    }
};
constexpr Resident RESIDENT;

// Which shapes are built and offered.  Three and five column blocks per wave are there for the balance of wide grids, below.
constexpr bool built(int xt, int rt, int cj, int f)
{
    if (cj == 1) return rt == 1 && (f <= 2 || (f == 3 && xt == 0));
    if (f == 0) return rt == 1 && cj == 2;
    if (cj == 5 && rt == 4) return false;                    // more registers than there are
    if (f == 3) return cj == 3 || (xt == 0 && cj != 5);
    if (f == 4) return cj == 3 || cj == 5;
    return true;
}

struct Offered {
    int8_t n[2][2][4][MAX_CJ], f[2][2][4][MAX_CJ][N_FORMS];  // [activations][gated][rt - 1][cj - 1]: how many forms, and which
    constexpr Offered() : n{}, f{}
    {
        for (int xt = 0; xt < 2; ++xt)
            for (int gated = 0; gated < 2; ++gated)          // (the gated epilogue: a workgroup pairs gate and up blocks)
                for (int rt = 1; rt <= 4; ++rt)
                    for (int cj = 1; cj <= MAX_CJ; ++cj)
                        for (int k = 0; k < N_FORMS; ++k)
                            if (built(xt, rt, cj, k) && !(gated && (cj * FORMS[k][1]) & 1))
                                f[xt][gated][rt - 1][cj - 1][n[xt][gated][rt - 1][cj - 1]++] = (int8_t)k;
    }
};
constexpr Offered OFFERED;

// Every candidate shape is priced and the cheapest wins.  The price is linear in what the busiest CU has to do (in rounds of
// as many workgroups as it holds at a time); the coefficients (us) are least-squares fits to graph-timed launches.
//
// Up to 512 column blocks one set for all forms: 4400 launches, 20 projections, 4 to 192 rows; on 70 further shapes (K 2048 to
// 28672, 3 to 240 rows) its choices are 2.7 % (int8 rows) and 0.9 % (bf16 rows) slower than the fastest measured.
constexpr int NARROW_BLOCKS = 512;
constexpr double NARROW[2][13] = {
    {1.525, 0.1987e-2, 0.6254e-2, 1.419e-2, 1.127e-4, 0.3743e-4, 0.8993e-2, 0.4517e-1, 0.3403e-1, 0.6996, 0.6068e-1, 0.7275e-1, 0.3929e-3},
    {1.677, 1.494e-2, 0.3030e-2, 3.895e-2, 0.9297e-4, 0.9087e-4, 0.7657e-2, 0.0, 0.5634e-1, 0.4702, 0.9276e-1, 1.174e-1, 0.1319e-3}};

// Above, a set for every (column blocks per wave, form): 16000 launches, 33 projections from 1024 x 9728 to 23040 x 16736 and
// 8192 x 57344, 8 to 256 rows; on those the chosen shapes are 1.4 and 0.9 % slow (worst 15 %), where one set for all forms chose
// 3.5 and 2.5 % slow (worst 38 %), and their prices 4 % off in the root mean square.
struct Coef {
    double launch,
           tile, tile_rt, wg_rt,        // per workgroup of the busiest CU: a tile of its K range, times row tiles; reduce and store
           stream, stream_band,         // per tile of the projection: from memory, and once per band out of the L2s
           round_tile, round_tile_rt, round, round_rt,       // per round: latency of a tile; start and end of a wave
           range_tile,                  // per tile of a K range
           rows_mb;                     // per MB of rows that all workgroups together read
};
constexpr Coef COEF[2][MAX_CJ][N_FORMS] = {                  // int8, bf16 rows; cj 1 to 5; forms
    {
     {{2.431, 0, 0, 1.048, 0.0001273, 2.015e-06, 0.3426, 0, 0, 0, 0.3202, 0.0242},
      {2.163, 0, 0.09833, 0.2592, 0.000117, 3.393e-05, 0, 0, 0.1782, 0, 0.3913, 0.02309},
      {1.598, 0, 0, 0.1994, 0.0001609, 6.715e-05, 0, 0, 0, 0, 0.1526, 0.02484},
      {},
      {}},
     {{2.664, 0, 0, 1.128, 0.0001125, 1.338e-05, 0.4408, 0, 0, 0, 0.4218, 0.02653},
      {2.085, 0, 0.1529, 0.4011, 9.513e-05, 5.021e-05, 0, 0, 0, 0, 0.2687, 0.02794},
      {1.781, 0, 0.03083, 0.1981, 0.0001224, 3.459e-05, 0, 0.04539, 0.1191, 0, 0.2562, 0.0317},
      {2.197, 0.1084, 0.02598, 0.2066, 9.056e-05, 0, 0, 0.08755, 0, 0.1804, 0.1111, 0.02454},
      {}},
     {{},
      {1.894, 0.02003, 0.2264, 0.4611, 9.165e-05, 3.522e-05, 0, 0, 0.4704, 0.03959, 0.2737, 0.02961},
      {2.053, 0.07646, 0.05088, 0.2303, 0.0001018, 2.088e-05, 0, 0.05488, 0.2526, 0.08886, 0.1662, 0.03273},
      {2.132, 0.1999, 0.001542, 0.363, 7.641e-05, 0, 0.02526, 0.1406, 0.3148, 0.1909, 0.1545, 0.02994},
      {1.865, 0.3416, 0.04713, 0.5481, 5.089e-05, 3.261e-05, 0, 0.1352, 0.3251, 0.1703, 0.3333, 0.02748}},
     {{},
      {1.657, 0, 0.1718, 0.4612, 0.0001061, 4.125e-05, 0.1183, 0.05242, 0.5533, 0, 0.2812, 0.03284},
      {2.106, 0.0858, 0.05403, 0.2751, 9.8e-05, 3.066e-05, 0, 0.06871, 0.1138, 0.1826, 0.2346, 0.03084},
      {2.625, 0.1489, 0.04238, 0.4777, 8.78e-05, 0, 0, 0.1018, 0, 0.2283, 0.316, 0.03639},
      {}},
     {{},
      {2.486, 0, 0.2194, 0.8893, 7.169e-05, 4.504e-05, 0.3758, 0, 0.09598, 0, 0.1051, 0.03307},
      {2.979, 0.2958, 0.08543, 0.3727, 7.825e-05, 1.922e-06, 0.1439, 0.01192, 0, 0.167, 0.08797, 0.03184},
      {},
      {2.774, 0.8062, 0.2497, 1.225, 8.42e-05, 0, 0, 0, 0, 0, 0.248, 0.02686}},
    },
    {
     {{2.415, 0.1537, 0, 0.8938, 0.000125, 0.0001161, 0, 0, 0, 0, 0.9699, 0.02509},
      {2.07, 0, 0, 0.275, 0.0001237, 0.0001512, 0, 0, 0, 0, 0.7189, 0.02172},
      {1.524, 0.005756, 0, 0.2092, 0.0001979, 0.0001296, 0, 0, 0, 0, 0.2151, 0.01965},
      {},
      {}},
     {{2.353, 0, 0, 0.9682, 9.553e-05, 0.0001533, 0.09447, 0, 0, 0, 1.576, 0.02023},
      {2.235, 0, 0, 0, 9.657e-05, 0.000128, 0, 0.2732, 0.1739, 0.2768, 0.5055, 0.02159},
      {1.987, 0, 0.06387, 0.1528, 0.0001231, 8.57e-05, 0, 0.1168, 0.04058, 0, 0.3335, 0.0241},
      {},
      {}},
     {{},
      {2.124, 0.01793, 0.2754, 0.3611, 8.289e-05, 0.0001082, 0, 0.1328, 0.3913, 0, 0.3668, 0.02087},
      {2.319, 0.04381, 0.1128, 0.2272, 0.0001005, 8.079e-05, 0.06799, 0.07761, 0.02371, 0.01999, 0.3068, 0.02387},
      {2.767, 0.4085, 0.02473, 0.416, 6.769e-05, 0, 0, 0.1281, 0, 0.0613, 0.4312, 0.03212},
      {2.436, 0.7357, 0.3551, 0.5488, 5.968e-05, 7.868e-06, 0, 0, 0.08837, 0, 0.4526, 0.02128}},
     {{},
      {1.648, 0, 0.3189, 0.2526, 8.117e-05, 0.000116, 0.1001, 0.08021, 0.9146, 0, 0.5014, 0.02632},
      {2.123, 0.1475, 0.1689, 0.1968, 7.354e-05, 6.388e-05, 0.1357, 0.01849, 0.2683, 0.1653, 0.4311, 0.02372},
      {},
      {}},
     {{},
      {1.821, 0.6328, 0.445, 0, 6.619e-05, 0.0001025, 0, 0, 1.664, 0.4319, 0, 0.0224},
      {3.174, 0.3759, 0.2008, 0.3178, 6.152e-05, 4.659e-05, 0.2204, 0, 0, 0.1713, 0.2458, 0.02338},
      {},
      {3.012, 2.04, 0.3912, 1.104, 5.608e-05, 0, 0, 0, 0, 0, 0.199, 0.02283}},
    }};

// Three or five column blocks per wave: on more than 512 blocks, where no CU then has more of them to do than with any even
// number (fewer, where waves share a range): 5120 x 34816, 2176 blocks, takes 15.2 us with 16 int8 rows in 544 workgroups of four
// blocks, 12 on the busiest CU, and 13.5 in 726 of three, 9 on it; with 48 bf16 rows 32.9 and 27.4 (2 x 5 blocks); 8192 x 20480
// with 32 int8 rows 17.2 and 14.3.  Over 23 projections of 9216 to 57344 columns the fastest shapes gain 3 % (int8 rows) and 6 %
// (bf16 rows) by it.
// `groups`: workgroups across the columns, by their width in column blocks.
inline int busiest(const int* groups, int width, int bands) { return ((groups[width] * bands + 255) >> 8) * width; }
inline bool odd_balances(const int* groups, int cj, int sh, int bands)
{
    if (bands > 4) return false;
    const int odd = busiest(groups, cj * sh, bands), even = std::min(busiest(groups, 2 * sh, bands), busiest(groups, 4 * sh, bands));
    return sh == 1 ? odd <= even : odd < even;
}

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
                 double* us = nullptr, int G = 128)
{
    const int M = (int)M64, n_cb = (int)n_cb64, n_kt = (int)n_kt64;
    const double tiles = (double)n_cb * n_kt;
    const double part_us = PARTS_US_PER_VALUE[xt] * 16 * M * (double)n_cb;
    const int cbw = xt == 1 ? std::min(tune.midm_cbw, 4) : tune.midm_cbw;
    const int forced = tune.splitk > 1 ? (int)std::min<int64_t>(std::min(tune.splitk, n_kt), cap) : 0;
    Plan best = {1, 2, 1, 1, 1};
    double best_price = 1e30;
    // (this runs on every call of up to 256 rows: no division but by powers of two, where it can be had)
    const bool narrow = n_cb <= NARROW_BLOCKS;
    const Kind kind = kind_of(xt, G);
    const double row_mb = (double)M * n_kt * (xt == 0 ? 256e-6 : 512e-6);
    auto price = [&](const Plan& p, int f, int bands, int groups, int T, int resident) {
        const int nb = (groups * bands * p.sp + 255) >> 8;
        const int rounds = nb <= resident ? 1 : (nb + resident - 1) / resident;
        double t;
        if (narrow) {
            const double* c = NARROW[xt];
            const int waves = p.ks * p.sh, rc = p.rt * p.cj;
            t = c[0]
              + (double)(nb * waves) * T * (c[1] * p.cj                  // up-converts
                                          + c[2] * rc)                  // matrix instructions and dequant
              + c[3] * ((double)(nb * p.ks) * T * p.rt)                  // activations through the L1
              + tiles * (c[4] + c[5] * bands)                            // the weight stream; ... once per band out of L2
              + c[6] * (nb * waves * rc)                                 // reduce and store
              + (double)rounds * T * (c[7] + c[8] * rc)                  // latency per tile, multiply,
              + rounds * (c[9] + c[10] * rc)                             // start and end of a wave
              + c[11] * T
              + c[12] * (groups * bands * p.sp);                         // workgroups to launch
        } else {
            const Coef& c = COEF[xt][p.cj - 1][f];
            t = c.launch + nb * (T * (c.tile + c.tile_rt * p.rt) + c.wg_rt * p.rt) + tiles * (c.stream + c.stream_band * bands) +
                rounds * (T * (c.round_tile + c.round_tile_rt * p.rt) + c.round + c.round_rt * p.rt) + c.range_tile * T +
                c.rows_mb * row_mb * groups;
        }
        if (p.sp > 1) t = PARTS_MARGIN * (t + PARTS_US[xt] + part_us * p.sp);
        return t;
    };
    int group_count[2 * MAX_CJ + 1];
    for (int w : {1, 2, 3, 4, 5, 6, 8, 10}) group_count[w] = (n_cb + w - 1) / w;
    const int row_tiles = std::min((M + 15) / 16, 4);
    // (wide grids, one row tile per wave: up to four bands; beyond, every band streams and up-converts the weights again)
    for (int rt = M > 64 && !narrow ? 2 : 1; rt <= row_tiles; ++rt) {
        const int bands = (M + 16 * rt - 1) / (16 * rt);
        for (int cj = rt == 1 ? 1 : 2; cj <= MAX_CJ; ++cj) {
            const bool odd = cj == 3 || cj == 5;
            if (odd && narrow) continue;
            const int8_t n_forms = OFFERED.n[xt][gated][rt - 1][cj - 1], *forms = OFFERED.f[xt][gated][rt - 1][cj - 1];
            for (int i = 0; i < n_forms; ++i) {
                const int f = forms[i], sh = FORMS[f][1], width = cj * sh;   // column blocks per workgroup
                if (odd && !odd_balances(group_count, cj, sh, bands)) continue;
                if (!narrow && cj == 1 && sh == 2) continue;             // (not fitted there: four blocks per workgroup and more win)
                if (cbw && width != cbw) continue;
                const int groups = group_count[width];
                if (xt == 0 && width <= 2 && !cbw && (int64_t)groups * M * n_kt * 256 > ROW_BYTES_FROM_L2) continue;
                const int resident = RESIDENT.n[kind][0][rt - 1][cj - 1][f], resident_parts = RESIDENT.n[kind][1][rt - 1][cj - 1][f];
                auto offer = [&](int ks, int sp, int T, int res) {
                    const Plan p = {rt, cj, ks, sh, sp};
                    const double t = price(p, f, bands, groups, T, res);
                    if (t < best_price) { best = p; best_price = t; }
                };
                const int lk = FORM_LOG[f];
                if (forced > 1) {
                    if (odd) continue;
                    const int ks = std::max(1, std::min(1 << lk, n_kt / forced));
                    offer(ks, forced, (n_kt + ks * forced - 1) / (ks * forced), resident_parts);
                    continue;
                }
                if (n_kt >= 1 << lk) offer(1 << lk, 1, (n_kt + (1 << lk) - 1) >> lk, resident);
                else offer(n_kt, 1, 1, resident_of(kind, rt, cj, n_kt, sh, false));
                // Across workgroups: grids that leave half the chip idle, in as many parts as still run at once, one per CU, and
                // with bf16 rows (whose workgroups take longer) grids of one round in two per CU, where two fit; other
                // numbers of parts were hardly ever faster by more than 3 %.  From K = 8192 on, with int8 rows from 20480 (17408 x
                // 1024 at M = 5 7.1 us in parts, 5.6 in one piece).
                const int wgs = groups * bands;
                if (cap < 2 || n_kt < (xt == 0 ? 80 : 32) || cj == 1 || odd || f == 0 || tune.splitk == 1) continue;
                const int at_once = wgs <= 128 ? 256 : xt == 1 && wgs <= 256 && resident_parts >= 2 ? 512 : 0;
                const int sp = (int)std::min<int64_t>(std::min(at_once / wgs, n_kt >> (lk + 1)), std::min<int64_t>(8, cap));
                if (sp >= 2) offer(1 << lk, sp, (n_kt + (sp << lk) - 1) / (sp << lk), resident_parts);
            }
        }
    }
    if (us) *us = best_price;
    return best;
}

}  // namespace midm

}  // namespace w2
