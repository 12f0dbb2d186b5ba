// w2a8 for prefill, tiles of 64 to 128 rows: the compute-bound regime (Sec. III-C, GEMM
// results) on the int8 matrix cores.  Measured on MI355X, what limits this
// method there is vector-instruction issue: a SIMD issues one vector
// instruction, matrix ones included, about every four clocks, and per matrix
// instruction (16 clocks of matrix pipe) the method needs 256/G fmas to apply
// the group scales (Sec. II-D dequant, per group) plus 7/RI shift/mask
// instructions to up-convert (Sec. II-C), RI = row tiles that share a weight
// operand.  The 64-row kernel (RI = 4) runs at 5.2 vector instructions per
// matrix instruction; this one halves the up-convert share with 128-row wave
// tiles (RI = 8 x CJ = 2 column blocks of v_mfma_i32_16x16x64_i8) and spreads
// the remaining vector work evenly under the matrix instructions.  Lower tiles
// (RI = 4 .. 7) cost a tile 3.9 + RI parts of 12 instead of all twelve (K loop, G = 128)
// and are taken where 128 rows leave rows past M or a last round of workgroups
// mostly empty (tile_plan.h; 4096 x 28672 at M = 130 33.5 -> 26.1 us, 28672 x
// 8192 with groups of 64 at M = 242 to 277 30 to 45 % less):
//   - workgroup 16 RI rows x 256 columns (eight waves of 16 RI x 32, one workgroup
//     per CU) or x 128 (four waves, two workgroups per CU, three of RI = 4 and 5:
//     their loads, barriers and stores lie under one another's multiplication, which
//     grids of few rounds want; 4096 x 28672 gated at M = 1000, groups of 64, 142 ->
//     131 us, and tile_plan.h); a stage is 128 k = one group of G = 128, 32 matrix
//     instructions per wave;
//   - activations go from global to local memory directly, 16-byte pieces XORed by
//     row (conflict-free operand reads), six stages ahead in eight buffers
//     (eight-wave workgroups): the pair of stages (2S, 2S+1) reads stages 2S ..
//     2S+2 and asks for stages 2S+6 and 2S+7 in the buffers of the pair before, one
//     barrier per pair, so the waves of a workgroup may be a stage apart inside a
//     pair.  Four buffers (128 columns): one barrier per stage;
//   - the weights go from global memory to registers (the packed dword IS the
//     matrix operand), one 16-byte load per lane, column block and 256-k tile,
//     a tile ahead;
//   - buffers and weight registers are constants of a loop of four 256-k tiles: 3.0 vector
//     instructions per matrix instruction.  With activations through registers and
//     buffers numbered at run time, 3.4: 8192 x 57344 at M = 2048 887 -> 824 us, 4096 x
//     28672 at M = 1000 in tiles of 128 / 112 / 96 / 80 / 64 rows 135 / 128 / 146 / 149 /
//     159 -> 127 / 119 / 129 / 137 / 135 us, with groups of 64 159 / 151 / 162 / 176 /
//     182 -> 150 / 140 / 152 / 163 / 158;
//   - every wave is software-pipelined on its own: under a stage's matrix
//     instructions it reads the second k-step's operands and the next stage's
//     first ones, up-converts one operand ahead, and dequantises a finished
//     column block in two halves (16 fmas per eight matrix instructions);
//   - groups of 64 (G = 64): a k-step is a group, so every block of eight matrix
//     instructions leaves a finished group in one of two accumulator sets and
//     folds the other one in (32 fmas): 5.2 vector instructions per matrix
//     instruction against 6.1 in 64-row tiles (8192 x 57344 at M = 2048: 1118 ->
//     1051 us; 28672 x 8192 at M = 1024: 283 -> 256);
//   - dequant in ONE fma per accumulator: a group starts from BIAS = 2^21 (the
//     third MFMA operand), so acc = BIAS + 64*sum is positive and below 2^23 and
//     its bit pattern read as binary32 is the denormal acc * 2^-149:
//     y += as_float(acc) * (sw * 2^64); the bias term is taken out every 16
//     groups and at the end.  Requires fp32 denormals (the build keeps them and
//     the source refuses fast-math) and |sw| < 2^63.  (Starting from the bit
//     pattern of 1.5 * 2^23 instead, a normal number, is no faster -- denormal
//     operands cost the fma nothing here -- and carries six times the bias,
//     which costs the near-zero outputs their accuracy.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "tall_waits.h"
#include "w2_small_common.h"

#if defined(__HIP_DEVICE_COMPILE__) && defined(__FAST_MATH__)
#error "the one-fma dequant reads int32 accumulators as fp32 denormals: do not build with fast-math / flush-to-zero"
#endif

namespace w2 {

namespace t128 {

constexpr int CJ = 2;                              // 16-column blocks per wave
constexpr int BK = 128;
constexpr int CP_ROWS = 128;                       // most rows of a tile
constexpr int WN = 16 * CJ;
constexpr int A_ROW = BK;                          // bytes of a row in one stage: eight 16-byte pieces
// LDS buffers: 4 with a barrier after every stage; 8 with a barrier after every other stage (eight-wave
// workgroups, one per CU: the waves of a workgroup may then drift a stage apart inside a pair)
constexpr int nbuf_of(int bn) { return bn >= 256 ? 8 : 4; }
constexpr int E_STRIDE = WN * 2 + 16;              // epilogue: bytes per LDS row of a wave's result
constexpr int BIAS = 1 << 21;                      // > 64 * 127 * 2 * 128 = 2 080 768
constexpr float BIAS_F = 0x1p-128f;                // BIAS read as a float: 2^21 * 2^-149
constexpr int waves_of(int bn) { return bn / WN; }
constexpr int SX_BYTES = CP_ROWS * 4;                   // the tile's activation scales, parked for the epilogue
constexpr int P_STRIDE = WN * 4 + 16;              // partial results: bytes per LDS row
// KiBs of activations (eight rows) per wave and stage, and a stage of them
constexpr int loads(int bn, int ri) { return (2 * ri + waves_of(bn) - 1) / waves_of(bn); }
constexpr int a_buf(int bn, int ri) { return loads(bn, ri) * waves_of(bn) * 1024; }
constexpr int lds_bytes(int bn, int ri)
{
    return std::max(std::max(nbuf_of(bn) * a_buf(bn, ri), waves_of(bn) * 16 * ri * E_STRIDE), waves_of(bn) * 64 * P_STRIDE);
}
// waves per SIMD that the registers are held to: one eight-wave workgroup to a CU, three of four waves (80 rows and less), two
constexpr int simd_waves(int bn, int ri) { return bn >= 256 || ri > 5 ? 2 : 3; }

__device__ __forceinline__ v4i upconvert4(uint32_t w)
{
    v4i u;
    u[0] = (int)((w << 6) & 0xC0C0C0C0u);
    u[1] = (int)((w << 4) & 0xC0C0C0C0u);
    u[2] = (int)((w << 2) & 0xC0C0C0C0u);
    u[3] = (int)(w & 0xC0C0C0C0u);
    return u;
}

template <int G>
struct WTile {
    uint4 w[CJ];                                   // 16 bytes of codes per column block: dword t = k 64t .. 64t+63
    uint32_t s[CJ][G == 128 ? 1 : 2];              // the lane's column: 2 (G=128) or 4 (G=64) bf16 group scales
};

// SPLIT: K cut into gridDim.y near-equal ranges of whole 256-k tiles (c_lo tiles each, one more for the first
// c_rem ranges), one grid slice each; a range is entered by moving the base pointers, its fp32 results go to the
// workspace and a second launch sums them (Sec. II-D, K-splitting for the smaller shapes).  An instantiation of
// its own: the unsplit kernel is compiled exactly as before.
template <int G, bool DBG, int BN, bool SPLIT = false, int RI = 8>
__global__ void __launch_bounds__(64 * waves_of(BN), simd_waves(BN, DBG ? 8 : RI))
a8_tiled128_kernel(A8Args a, int tiles_m, int tiles_n, int group_m, int c_lo, int c_rem)
{
    constexpr int BM = 16 * RI;
    constexpr int WAVES = waves_of(BN);
    constexpr int GPT = TILE_K / G;
    constexpr int NBUF = nbuf_of(BN);
    constexpr bool PAIR = BN >= 256;               // a barrier after every other stage
    constexpr int AHEAD = tall::ahead(PAIR);       // stage it asks for the activations of stage it + AHEAD
    static_assert(AHEAD == (PAIR ? NBUF - 2 : NBUF - 1), "into the buffers that the barrier before freed");
    constexpr int NP = loads(BN, RI), A_BUF = a_buf(BN, RI);
    extern __shared__ __align__(16) int8_t smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wn = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, l16 = lane & 15;

    // workgroup -> tile: one contiguous chunk of ids per XCD (consecutive ids go to different XCDs),
    // bands of group_m row tiles inside, so that the workgroups resident on an XCD share activation rows
    // and weight columns through that XCD's L2
    const int64_t total = (int64_t)tiles_m * tiles_n;
    int64_t id = blockIdx.x;
    if (total % 8 == 0) id = (id & 7) * (total >> 3) + (id >> 3);
    const int64_t band = id / ((int64_t)group_m * tiles_n);
    const int64_t first_m = band * group_m;
    const int gm = (int)min((int64_t)group_m, tiles_m - first_m);
    const int64_t in_band = id - band * group_m * tiles_n;
    const int64_t tile_m = first_m + in_band % gm;
    const int64_t tile_n = in_band / gm;
    const int64_t m0 = tile_m * BM, n0 = tile_n * BN;

    const char* wb[CJ];
    const char* sb[CJ];
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
        int64_t c = tile_n * (BN / TILE_N) + wn * CJ + j;
        c = c < a.n_cb ? c : a.n_cb - 1;                     // clamp: loads stay in bounds
        wb[j] = reinterpret_cast<const char*>(a.codes + c * a.n_kt * 256);
        sb[j] = reinterpret_cast<const char*>(a.scales + c * a.n_kt * TILE_N * GPT);
    }
    uint32_t w_lane = (uint32_t)lane * 16u;
    uint32_t s_lane = (uint32_t)l16 * (GPT * 2u);
    int nkt = (int)a.n_kt;                                   // tiles this workgroup multiplies
    int kt0 = 0;                                             // the first of them
    if constexpr (SPLIT) {
        const int z = (int)blockIdx.y;
        kt0 = z * c_lo + min(z, c_rem);
        nkt = c_lo + (z < c_rem ? 1 : 0);
#pragma unroll
        for (int j = 0; j < CJ; ++j) {
            wb[j] += (int64_t)kt0 * 1024;
            sb[j] += (int64_t)kt0 * (TILE_N * GPT * 2);
        }
    }

    // The activations go from global to local memory directly, a KiB (eight rows x 128 bytes) per instruction.  A row's
    // 16-byte pieces stand there XORed by row mod 8 (operand reads without bank conflicts): the lanes fetch them in that
    // order.  Rows past M or past the tile lie past the resource's end; lane offsets stay below 128 * K <= 2^31.
    const int rows = (int)min((int64_t)BM, a.M - m0);
    const uint32_t stride = (uint32_t)a.K;
    const int8_t* const xbase = a.xq + m0 * a.K + (int64_t)kt0 * TILE_K;
    const uint32_t xbytes = (uint32_t)(rows - 1) * stride + (uint32_t)nkt * TILE_K;
    uint32_t xoff[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p)
        xoff[p] = (uint32_t)((wn + WAVES * p) * 8 + (lane >> 3)) * stride + (uint32_t)((lane & 7) ^ (lane >> 3)) * 16u;

    v4i acc[RI][CJ];
    float y[RI][CJ][4];
    float ssum[CJ] = {};                                     // sum of sw * 2^64 over the groups folded into y
    const v4i biasv = {BIAS, BIAS, BIAS, BIAS};
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < CJ; ++j) {
            acc[i][j] = biasv;
#pragma unroll
            for (int r = 0; r < 4; ++r) y[i][j][r] = 0.0f;
        }

    const int n_st = nkt * 2;                                // stages of 128 k
    // (past the range's end: nothing is read, but the instructions are there, for they are counted)
    auto load_a = [&](int st, int buf) {
        const __amdgpu_buffer_rsrc_t xr = make_rsrc(xbase, st < n_st ? xbytes : 0u);
#pragma unroll
        for (int p = 0; p < NP; ++p) load_to_lds(xr, smem + buf * A_BUF + (wn + WAVES * p) * 1024, xoff[p], (uint32_t)st * BK);
    };
    auto load_w = [&](int kt, WTile<G>& r) {
        kt = min(kt, nkt - 1);
        const int64_t w_off = (int64_t)kt * 1024;
        const int64_t s_off = (int64_t)kt * (TILE_N * GPT * 2);
        asm volatile("" : "+v"(w_lane), "+v"(s_lane));
#pragma unroll
        for (int j = 0; j < CJ; ++j) {
            r.w[j] = *reinterpret_cast<const uint4*>(wb[j] + w_off + w_lane);
            if constexpr (G == 128) {
                r.s[j][0] = *reinterpret_cast<const uint32_t*>(sb[j] + s_off + s_lane);
            } else {
                const uint2 v = *reinterpret_cast<const uint2*>(sb[j] + s_off + s_lane);
                r.s[j][0] = v.x;
                r.s[j][1] = v.y;
            }
        }
    };

    // the tile's activation scales, fetched now (unconditionally) and parked in LDS for the epilogue: loaded
    // there they would cost every workgroup a memory round trip with nothing to hide it
    float* sx_lds = reinterpret_cast<float*>(smem + lds_bytes(BN, RI));
    const float sx_mine = DBG ? 0.f : a.sx[min(m0 + (tid & (CP_ROWS - 1)), a.M - 1)];

    WTile<G> w0, w1;
    load_w(0, w0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) load_a(p, p);
    if (tid < CP_ROWS) sx_lds[tid] = sx_mine;                // (read after barriers that wait for local memory, in the epilogue)
    wait_loads<tall::at_start(PAIR, NP)>();       // stages 0, 1 (and 2) are there
    bare_barrier();

    // where a lane finds the operands of k-step 0 and 1 in buffers 0 .. 3 and, beyond the reach of an instruction's offset,
    // from 4 on
    const int a_e0 = l16 * A_ROW + (q ^ (l16 & 7)) * 16, a_e1 = l16 * A_ROW + ((4 + q) ^ (l16 & 7)) * 16;
    int a_f0 = a_e0 + 4 * A_BUF, a_f1 = a_e1 + 4 * A_BUF;
    asm volatile("" : "+v"(a_f0), "+v"(a_f1));

    // y += as_float(acc) * (sw * 2^64) for rows [i0, i0 + 4) of column block j
    constexpr int H0 = RI / 2;                               // row tiles of the first half
    auto dequant_half = [&](int j, int i0, float swS, int g) {
#pragma unroll
        for (int i = i0; i < (i0 ? RI : H0); ++i) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (DBG) {
                    const int64_t m = m0 + i * 16 + 4 * q + r;
                    const int64_t n = n0 + wn * WN + j * 16 + l16;
                    if (g >= 0 && m < a.M && n < a.N)
                        a.acc_out[(m * (a.K / G) + g) * a.N + n] = (acc[i][j][r] - BIAS) >> 6;
                }
                y[i][j][r] = fmaf(__int_as_float(acc[i][j][r]), swS, y[i][j][r]);
            }
        }
    };
    // G = 64: the group in accumulator set `set`, all rows, into column block j
    auto dequant_set = [&](int set, int j, float swS, int g) {
#pragma unroll
        for (int i = 0; i < RI; ++i) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (DBG) {
                    const int64_t m = m0 + i * 16 + 4 * q + r;
                    const int64_t n = n0 + wn * WN + j * 16 + l16;
                    if (g >= 0 && m < a.M && n < a.N)
                        a.acc_out[(m * (a.K / G) + g) * a.N + n] = (acc[i][set][r] - BIAS) >> 6;
                }
                y[i][j][r] = fmaf(__int_as_float(acc[i][set][r]), swS, y[i][j][r]);
            }
        }
        ssum[j] += swS;
    };
    auto scale_of = [&](const WTile<G>& w, int j, int h, int t) -> float {
        // G = 128: the stage's group is group h of the tile; G = 64: k-step t of stage h is group 2h + t
        const uint32_t pair = G == 128 ? w.s[j][0] : w.s[j][h];
        const int hi = G == 128 ? h : t;
        return __uint_as_float(hi ? (pair & 0xffff0000u) : (pair << 16)) * 0x1p64f;
    };
    auto dword_of = [&](const WTile<G>& w, int j, int h, int t) -> uint32_t {
        const int d = 2 * h + t;
        return d == 0 ? w.w[j].x : d == 1 ? w.w[j].y : d == 2 ? w.w[j].z : w.w[j].w;
    };

    v4i a0[RI], a1[RI];
#pragma unroll
    for (int i = 0; i < RI; ++i) a0[i] = *reinterpret_cast<const v4i*>(smem + a_e0 + i * 16 * A_ROW);
    v4i b_next = upconvert4(w0.w[0].x);                      // operand (k-step 0, column block 0) of the coming stage
    float pend_sw = 0.f;                                     // column block 1 of the previous stage: nothing yet
    int pend_g = -1;

    // One stage (G = 128: one group).  Order of the matrix instructions: column block 0, k-steps 0 and 1
    // (blocks A, B), then column block 1 (blocks C, D).  Vector work under them:
    //   A: second k-step's operands from LDS, up-convert (1,0), dequant the previous stage's column 1, rows 0..63
    //   B: up-convert (0,1), dequant the previous stage's column 1, rows 64..127
    //   C: up-convert (1,1), dequant this stage's column 0, rows 0..63
    //   D: next stage's first operands from LDS, up-convert its (0,0), dequant column 0, rows 64..127
    // sc: stage of the loop below, 0 .. 7, and its buffer (mod NBUF)
    auto stage = [&](int it, auto sc, const WTile<G>& wc, WTile<G>& wnx) {
        constexpr int h = decltype(sc)::value & 1, buf = decltype(sc)::value & (NBUF - 1), buf1 = (buf + 1) & (NBUF - 1);
        if constexpr (h == 0) load_w((it >> 1) + 1, wnx);
        __builtin_amdgcn_sched_barrier(0);
        load_a(it + AHEAD, (buf + AHEAD) & (NBUF - 1));
        __builtin_amdgcn_sched_barrier(0);                   // all loads are issued up here, unconditionally
        const int8_t* const ab = smem + (buf < 4 ? a_e1 : a_f1) + (buf & 3) * A_BUF;
        const int8_t* const abn = smem + (buf1 < 4 ? a_e0 : a_f0) + (buf1 & 3) * A_BUF;
        const WTile<G>& wn_tile = h == 1 ? wnx : wc;         // where the next stage finds its weights
        const float sw0 = scale_of(wc, 0, h, 0), sw1 = scale_of(wc, 1, h, 0);
        const int g = it;                                    // group index = stage index (G = 128)

        // before the next pair: stages up to its third have landed; what was asked for since, three more and a tile's weights,
        // may be under way.  (Four buffers: the next two stages; one more and, asked for in this stage, weights.)
        auto end_of_stage = [&]() {
            if constexpr (!PAIR || h == 1) {
                wait_loads<tall::behind(PAIR, h, NP, tall::weights(DBG, CJ))>();
                bare_barrier();
            }
        };
        const v4i b00 = b_next;
        // Each block is a scheduling region of its own (sched_barrier at its end): the vector work placed in a
        // block reads only accumulators finished at least one block (eight matrix instructions) earlier.  In one
        // region the scheduler pulled the fmas up to right behind the matrix instruction that produces their
        // operand, and every such pair stalls the wave until the matrix pipe has written the result (measured:
        // 2070 TOP/s; 4290 with the same fmas reading other registers).
        auto interleave = [&](bool with_lds, int rows) {     // per matrix instruction: [one LDS read] its share of the vector instructions
#pragma unroll
            for (int k = 0; k < RI; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (with_lds) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                if (rows == H0) __builtin_amdgcn_sched_group_barrier(0x002, (7 + 4 * H0 + RI - 1) / RI, 0);
                else if (rows == RI) __builtin_amdgcn_sched_group_barrier(0x002, (7 + 4 * RI + RI - 1) / RI, 0);
                else __builtin_amdgcn_sched_group_barrier(0x002, (7 + 4 * (RI - H0) + RI - 1) / RI, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        if constexpr (G == 64) {
            // A k-step is a group: every block leaves a whole group in one of two accumulator sets (acc[.][0] and
            // acc[.][1]), which the next block folds in row by row, eight matrix instructions behind.
            const float sw01 = scale_of(wc, 0, h, 1), sw11 = scale_of(wc, 1, h, 1);
#pragma unroll
            for (int i = 0; i < RI; ++i) a1[i] = *reinterpret_cast<const v4i*>(ab + i * 16 * A_ROW);
            const v4i b10 = upconvert4(dword_of(wc, 0, h, 1));
#pragma unroll
            for (int i = 0; i < RI; ++i) acc[i][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0[i], b00, biasv, 0, 0, 0);
            dequant_set(1, 1, pend_sw, pend_g);              // column 1's second group of the previous stage
            interleave(true, RI);
            const v4i b01 = upconvert4(dword_of(wc, 1, h, 0));
#pragma unroll
            for (int i = 0; i < RI; ++i) acc[i][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1[i], b10, biasv, 0, 0, 0);
            dequant_set(0, 0, sw0, 2 * g);
            interleave(false, RI);
            const v4i b11 = upconvert4(dword_of(wc, 1, h, 1));
#pragma unroll
            for (int i = 0; i < RI; ++i) acc[i][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0[i], b01, biasv, 0, 0, 0);
            dequant_set(1, 0, sw01, 2 * g + 1);
            interleave(false, RI);
#pragma unroll
            for (int i = 0; i < RI; ++i) a0[i] = *reinterpret_cast<const v4i*>(abn + i * 16 * A_ROW);
            b_next = upconvert4(dword_of(wn_tile, 0, h ^ 1, 0));
#pragma unroll
            for (int i = 0; i < RI; ++i) acc[i][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1[i], b11, biasv, 0, 0, 0);
            dequant_set(0, 1, sw1, 2 * g);
            pend_sw = DBG ? 1.0f : sw11;
            pend_g = 2 * g + 1;
            interleave(true, RI);
            end_of_stage();
            return;
        }
        // block A
#pragma unroll
        for (int i = 0; i < RI; ++i) a1[i] = *reinterpret_cast<const v4i*>(ab + i * 16 * A_ROW);
        const v4i b10 = upconvert4(dword_of(wc, 0, h, 1));
#pragma unroll
        for (int i = 0; i < RI; ++i) acc[i][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0[i], b00, biasv, 0, 0, 0);
        dequant_half(1, 0, pend_sw, pend_g);
        interleave(true, H0);
        // block B
        const v4i b01 = upconvert4(dword_of(wc, 1, h, 0));
#pragma unroll
        for (int i = 0; i < RI; ++i) acc[i][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1[i], b10, acc[i][0], 0, 0, 0);
        dequant_half(1, H0, pend_sw, pend_g);
        ssum[1] += pend_sw;
        interleave(false, RI - H0);
        // block C
        const v4i b11 = upconvert4(dword_of(wc, 1, h, 1));
#pragma unroll
        for (int i = 0; i < RI; ++i) acc[i][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0[i], b01, biasv, 0, 0, 0);
        dequant_half(0, 0, sw0, g);
        interleave(false, H0);
        // block D
#pragma unroll
        for (int i = 0; i < RI; ++i) a0[i] = *reinterpret_cast<const v4i*>(abn + i * 16 * A_ROW);
        b_next = upconvert4(dword_of(wn_tile, 0, h ^ 1, 0));
#pragma unroll
        for (int i = 0; i < RI; ++i) acc[i][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1[i], b11, acc[i][1], 0, 0, 0);
        dequant_half(0, H0, sw0, g);
        ssum[0] += sw0;
        pend_sw = DBG ? 1.0f : sw1;
        pend_g = g;
        interleave(true, RI - H0);
        end_of_stage();
    };

    auto tile = [&](int kt, auto oc, const WTile<G>& wc, WTile<G>& wnx) {
        constexpr int o = decltype(oc)::value;
        stage(kt * 2, std::integral_constant<int, o>{}, wc, wnx);
        stage(kt * 2 + 1, std::integral_constant<int, o + 1>{}, wc, wnx);
    };
    // four 256-k tiles (eight stages) per turn, so that buffers and the two sets of weight registers are constants
    for (int kt = 0; kt < nkt; kt += 4) {
        tile(kt, std::integral_constant<int, 0>{}, w0, w1);
        if (kt + 1 >= nkt) break;                            // uniform
        tile(kt + 1, std::integral_constant<int, 2>{}, w1, w0);
        if (kt + 2 >= nkt) break;
        tile(kt + 2, std::integral_constant<int, 4>{}, w0, w1);
        if (kt + 3 >= nkt) break;
        tile(kt + 3, std::integral_constant<int, 6>{}, w1, w0);
        if (G == 64 || (kt & 4)) {
            // take the accumulated bias term out every 16 groups, so that the running sums never carry
            // more than 16 groups of it (the rounding error stays near 2^-14 of the result, whatever K is)
#pragma unroll
            for (int j = 0; j < CJ; ++j) {
                // column 1 of the stage just finished is still pending: its scale is not in ssum[1] yet
                const float corr = ssum[j] * BIAS_F;
                ssum[j] = 0.f;
#pragma unroll
                for (int i = 0; i < RI; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) y[i][j][r] -= corr;
            }
        }
    }
    wait_loads<0>();                                         // (stages past the end still store zeros)
    __syncthreads();
    // the very last stage's column block 1
    if constexpr (G == 64) {
        dequant_set(1, 1, pend_sw, pend_g);
    } else {
        dequant_half(1, 0, pend_sw, pend_g);
        dequant_half(1, H0, pend_sw, pend_g);
        ssum[1] += pend_sw;
    }
    if constexpr (DBG) return;

    // y_true = (y - BIAS*2^-149 * ssum) * 2^(149-64) * 2^-6 * sx.  The wave's 128 x 32 result goes through
    // LDS (its own region; the barrier above freed the activation buffers) and
    // leaves as 16-byte stores.
    int8_t* ebase = smem + wn * (BM * E_STRIDE);
    uint16_t* eb = reinterpret_cast<uint16_t*>(ebase);
    const bool gated = a.epi.act == ACT_SILU_MUL;
    float bias[CJ];
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
        const int64_t n = n0 + wn * WN + j * 16 + l16;
        bias[j] = (a.epi.bias && n < a.N) ? bf16_to_f32(a.epi.bias[n]) : 0.f;
    }
    // (one copy of the loop per epilogue, picked here: a choice per element would have the compiler
    // evaluate the SiLU for every output and select afterwards)
    // (y - bias) * 2^79 in one fma (powers of two: exact products), then sx: in this order a row scale may be as large as
    // fp32 holds
    float cj[CJ];
#pragma unroll
    for (int j = 0; j < CJ; ++j) cj[j] = ssum[j] * -(BIAS_F * 0x1p79f);
    if constexpr (SPLIT) {
        // this range's results, dequantised, as fp32 rows of the workspace: the wave's 128 x 32 tile goes
        // through LDS 64 rows at a time (rows padded by 16 bytes: conflict-free both ways; the wave reads
        // back only what it wrote) and leaves as 16-byte stores in 128-byte runs
        float* dst = a.part + (int64_t)blockIdx.y * a.M * a.N;
        int8_t* pbase = smem + wn * (64 * P_STRIDE);
        const int prow = lane >> 3, pcol = (lane & 7) * 4;   // eight lanes per row piece
        const int64_t n = n0 + wn * WN + pcol;
#pragma unroll
        for (int h = 0; h < (RI + 3) / 4; ++h) {
#pragma unroll
            for (int i = 0; i < 4 && h * 4 + i < RI; ++i) {
                const float4 s4 = *reinterpret_cast<const float4*>(sx_lds + (h * 4 + i) * 16 + 4 * q);
                const float sr[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int j = 0; j < CJ; ++j)
                        *reinterpret_cast<float*>(pbase + (i * 16 + 4 * q + r) * P_STRIDE + (j * 16 + l16) * 4) =
                            fmaf(y[h * 4 + i][j][r], 0x1p79f, cj[j]) * sr[r];
            }
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const int row = p * 8 + prow;
                const int64_t m = m0 + h * 64 + row;
                const float4 v = *reinterpret_cast<const float4*>(pbase + row * P_STRIDE + pcol * 4);
                if (h * 64 + row < BM && m < a.M && n < a.N) *reinterpret_cast<float4*>(dst + m * a.N + n) = v;   // N % 8 == 0: all 4 or none
            }
        }
        return;
    }
    auto emit = [&](auto mode_c) {
        constexpr int MODE = decltype(mode_c)::value;        // ACT_NONE, ACT_SILU, ACT_SILU_MUL
#pragma unroll
        for (int i = 0; i < RI; ++i) {
            const float4 s4 = *reinterpret_cast<const float4*>(sx_lds + i * 16 + 4 * q);     // rows 4q .. 4q+3 of row tile i
            const float sr[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = i * 16 + 4 * q + r;
                float z[CJ];
#pragma unroll
                for (int j = 0; j < CJ; ++j) z[j] = fmaf(y[i][j][r], 0x1p79f, cj[j]) * sr[r] + bias[j];
                if constexpr (MODE == ACT_SILU_MUL) {
                    eb[row * (E_STRIDE / 2) + l16] = f32_to_bf16_rne(silu_f32(z[0]) * z[1]);
                } else {
                    static_assert(CJ == 2, "one packed conversion per row");
                    const uint32_t pk = MODE == ACT_SILU ? pack_bf16x2(silu_f32(z[0]), silu_f32(z[1])) : pack_bf16x2(z[0], z[1]);
                    eb[row * (E_STRIDE / 2) + l16] = (uint16_t)pk;
                    eb[row * (E_STRIDE / 2) + 16 + l16] = (uint16_t)(pk >> 16);
                }
            }
        }
    };
    if (gated) emit(std::integral_constant<int, ACT_SILU_MUL>{});
    else if (a.epi.act == ACT_SILU) emit(std::integral_constant<int, ACT_SILU>{});
    else emit(std::integral_constant<int, ACT_NONE>{});
    // the wave reads back only what it wrote itself: LDS operations of one wave complete in order
    const int wcols = gated ? WN / 2 : WN;                   // output columns of this wave
    const int lpr = wcols * 2 / 16;                          // lanes per row piece (16 bytes each): 4 or 2
    const int rpp = 64 / lpr;                                // rows per pass
    const int64_t ncol = (gated ? (n0 + wn * WN) / 2 : n0 + wn * WN) + (lane % lpr) * 8;   // first of this lane's 8 columns
    const int64_t n_out = gated ? a.N / 2 : a.N;
    for (int p = 0; p * rpp < BM; ++p) {
        const int row = p * rpp + lane / lpr;
        const int64_t m = m0 + row;
        const uint4 v = *reinterpret_cast<const uint4*>(ebase + row * E_STRIDE + (lane % lpr) * 16);
        if (row < BM && m < a.M && ncol < n_out) *reinterpret_cast<uint4*>(a.Y + m * a.ldy + ncol) = v;   // N % 8 == 0: all 8 or none
    }
}

template <int G, bool DBG, int BN, bool SPLIT = false, int RI = 8>
static int launch(const A8Args& a, int splits, hipStream_t stream)
{
    constexpr int WAVES = waves_of(BN), BM = 16 * RI;
    const int tiles_m = (int)((a.M + BM - 1) / BM);
    const int tiles_n = (int)((a.N + BN - 1) / BN);
    // Row tiles per band: the 32 workgroups resident on an XCD cover group_m row tiles x 32 / group_m column
    // tiles and fetch group_m MiB of activations and 16 / group_m MiB of weights per round at K = 8192: 4
    // moves the least through the XCD's L2 (measured as fast as 8 at M = 2048, 2 % faster at M = 4096).
    const int group_m = a.tune.tiled_group_m ? a.tune.tiled_group_m : 4;
    constexpr int lds = lds_bytes(BN, RI) + SX_BYTES;
    auto kern = a8_tiled128_kernel<G, DBG, BN, SPLIT, RI>;
    if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds, "w2_matmul_a8[tiled 128]")) return rc;
    const dim3 grid((unsigned)((int64_t)tiles_m * tiles_n), (unsigned)(SPLIT ? splits : 1)), block(64 * WAVES);
    hipLaunchKernelGGL(kern, grid, block, lds, stream, a, tiles_m, tiles_n, group_m, (int)(a.n_kt / (SPLIT ? splits : 1)),
                       (int)(a.n_kt % (SPLIT ? splits : 1)));
    int rc = check_launch("w2_matmul_a8[tiled 128]");
    if (rc || !SPLIT) return rc;
    return launch_splitk_reduce(a.part, splits, a.M, a.N, a.Y, a.ldy, a.epi, stream);
}

}  // namespace t128


template <int G, int BN, bool SPLIT>
static int launch_ri(const A8Args& a, const tiles::A8Shape& p, hipStream_t stream)
{
    switch (p.ri) {
    case 4: return t128::launch<G, false, BN, SPLIT, 4>(a, p.splits, stream);
    case 5: return t128::launch<G, false, BN, SPLIT, 5>(a, p.splits, stream);
    case 6: return t128::launch<G, false, BN, SPLIT, 6>(a, p.splits, stream);
    case 7: return t128::launch<G, false, BN, SPLIT, 7>(a, p.splits, stream);
    default: return t128::launch<G, false, BN, SPLIT>(a, p.splits, stream);
    }
}

template <int G>
static int launch_g(const A8Args& a, const tiles::A8Shape& p, hipStream_t stream)
{
    if (a.acc_out)                                           // (the test-only export has eight row tiles per wave)
        return p.bn == 128 ? t128::launch<G, true, 128>(a, 1, stream) : t128::launch<G, true, 256>(a, 1, stream);
    if (p.bn == 128) return p.splits >= 2 ? launch_ri<G, 128, true>(a, p, stream) : launch_ri<G, 128, false>(a, p, stream);
    return p.splits >= 2 ? launch_ri<G, 256, true>(a, p, stream) : launch_ri<G, 256, false>(a, p, stream);
}

int launch_a8_tiled128(const A8Args& a, const tiles::A8Shape& p, hipStream_t stream)
{
    return a.G == 128 ? launch_g<128>(a, p, stream) : launch_g<64>(a, p, stream);
}

}  // namespace w2
