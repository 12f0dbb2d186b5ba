// w2a16 for large M with the scale folded into the weights (Sec. II-D,
// "Alternative implementation": the 2-bit code and the 16-bit group scale are
// mixed into one 16-bit weight, which goes to a 16-bit matrix instruction with
// fp32 accumulation; nothing is dequantised afterwards).  With bf16 the four
// possible weights of a group and column, 0, +sw, -2 sw and -sw, are exact
// (sign flip, exponent + 1), so the matrix instruction sums exact products
// and ONE accumulator per output runs over the whole K: no zero-point term, no
// group sums of the activations, no per-group fma on the accumulators.
//
// Per lane and (group, column) the four weights sit in two registers, low
// bytes in one and high bytes in the other.  A dword of the packed tile holds
// 16 codes, four per byte; (w >> 2j) & 0x03030303 is four codes as four byte
// selectors, two v_perm_b32 look the low and the high bytes up, two more
// interleave them into pairs of adjacent k: 23 vector
// instructions per 16 weights.  They are amortised over a 128-row wave tile
// (RI = 8 row tiles x CJ = 2 column blocks of v_mfma_f32_16x16x32_bf16: 32
// matrix instructions per 64-k stage and wave), which is what makes this
// construction the faster one for prefill: it issues 1.66 vector
// instructions per matrix instruction where the zero-point kernel issues 5.9.
//
// Workgroup: 128 rows (lower tiles of 64 to 112 where those waste less: tile_plan.h;
// 4096 x 28672 at M = 300 95.7 -> 79.3 us) x (32 columns per wave: 256, or 128 in two workgroups per CU, three
// of 64 and 80 rows, where that is priced lower) x 64 k per stage; activations go
// to local memory by loads that write it directly, six stages ahead (eight
// buffers; four with 128 columns), 16-byte pieces XORed by row so that operands are
// read without bank conflicts; weights go from global memory to
// registers, one 16-byte load per lane, column block and 256-k tile, a whole
// tile ahead.  Each wave is software-pipelined on its own (next stage's weights
// are up-converted and its first operands read under this stage's matrix
// instructions).  Tried and slower: 256-row wave tiles at one wave per SIMD.
//
// What bounds it: the issue of vector instructions beside the matrix ones (every one per matrix instruction costs about
// a tenth of the matrix rate; the matrix pipe alone reaches 1745 TFLOP/s on such operands) and the local memory, which
// delivers a stage's operands in about the time that the matrix pipe takes.  So nothing but the up-convert is left on the
// vector pipe: activations that went through registers were written with four permutations and two address sums per 16
// bytes, and buffer indexes that were not constants cost two more sums a stage and 64-bit compares.  4096 x 28672 at M = 333,
// groups of 128 (us, tiles of 128 / 112 / 96 / 80 / 64 rows): 97.6 / 93.7 / 91.2 / 118.5 / 110.6 with activations through
// registers and 2.07 vector instructions per matrix instruction, 95.0 / 89.4 / 85.6 / 111.5 / 97.3 with direct loads (1.79),
// 90.0 / 83.9 / 79.1 / 102.7 / 91.0 with constant buffer indexes and 32-bit stage numbers (1.66).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "tall_waits.h"
#include "w2_small_common.h"

namespace w2 {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

namespace fold16 {

constexpr int CJ = 2;                              // 16-column blocks per wave
constexpr int BK = 64;
constexpr int WN = 16 * CJ;
constexpr int A_ROW = BK * 2;                      // bytes of a row in one stage: eight 16-byte pieces
// LDS buffers: 4 with a barrier after every stage; 8 with a barrier after every other stage (eight-wave
// workgroups, one per CU, where the LDS is there for it)
constexpr int nbuf_of(int bn) { return bn >= 256 ? 8 : 4; }
constexpr int E_STRIDE = WN * 2 + 16;              // epilogue: bytes per LDS row of a wave's result
constexpr int waves_of(int bn) { return bn / WN; }
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

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// The four weights of one (group, column): low bytes and high bytes, indexed by the raw code
// (00 -> 0, 01 -> +sw, 10 -> -2 sw, 11 -> -sw).
struct Lut { uint32_t lo4, hi4; };

__device__ __forceinline__ Lut make_lut(uint32_t s)          // s: bf16 bit pattern of the group scale
{
    const uint32_t neg = s ^ 0x8000u;
    // -2 sw: exponent + 1, or of a subnormal scale (a zero: -0) the mantissa twice
    const uint32_t neg2 = (s + min(s & 0x7fffu, 0x0080u)) ^ 0x8000u;
    const uint32_t a = s << 16;                              // [0, +sw]
    const uint32_t b = neg2 | (neg << 16);                   // [-2 sw, -sw]
    Lut l;
    l.lo4 = __builtin_amdgcn_perm(b, a, 0x06040200u);
    l.hi4 = __builtin_amdgcn_perm(b, a, 0x07050301u);
    return l;
}

// 16 codes of one dword -> b0 (k 8 .. 15 of the lane's 16-k block), b1 (k 0 .. 7): the upper half is multiplied first, so that
// sums over the same K ranges can be told from the mid-M kernel's
__device__ __forceinline__ void upconvert(uint32_t w, const Lut& l, v4i& b0, v4i& b1)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t t = (w >> (2 * j)) & 0x03030303u;     // the codes of k = 4j .. 4j+3 as byte selectors
        const uint32_t lo = __builtin_amdgcn_perm(0u, l.lo4, t);
        const uint32_t hi = __builtin_amdgcn_perm(0u, l.hi4, t);
        v4i& b = j < 2 ? b1 : b0;
        b[2 * (j & 1)] = (int)__builtin_amdgcn_perm(hi, lo, 0x05010400u);       // k = 4j, 4j+1
        b[2 * (j & 1) + 1] = (int)__builtin_amdgcn_perm(hi, lo, 0x07030602u);   // k = 4j+2, 4j+3
    }
}

__device__ __forceinline__ v4f mfma_bf16(const v4i& a, const v4i& b, const v4f& c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a),
                                                   __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

template <int G>
struct WTile {
    uint4 w[CJ];                                   // 16 bytes of codes per column block: dword t = k 64t .. 64t+63
    uint32_t s[CJ][G == 128 ? 1 : 2];              // the lane's column: 2 (G=128) or 4 (G=64) bf16 group scales
};

// RI: 16-row tiles per wave (the workgroup's rows: BM = 16 RI), 4 to 8
template <int G, int BN, int RI>
__global__ void __launch_bounds__(64 * waves_of(BN), simd_waves(BN, RI))
a16_fold_tiled_kernel(A16Args a, int tiles_m, int tiles_n, int group_m, int splits)
{
    constexpr int BM = 16 * RI;
    constexpr int WAVES = waves_of(BN);
    constexpr int GPT = TILE_K / G;
    constexpr int NBUF = nbuf_of(BN);
    constexpr bool PAIR = BN >= 256;                    // a barrier after every other stage
    constexpr int AHEAD = tall::ahead(PAIR);            // stage it asks for the activations of stage it + AHEAD
    static_assert(AHEAD == (PAIR ? NBUF - 2 : NBUF - 1), "into the buffers that the barrier before freed");
    constexpr int NP = loads(BN, RI), A_BUF = a_buf(BN, RI);
    extern __shared__ __align__(16) int8_t smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wn = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, l16 = lane & 15;

    // workgroup -> tile: one contiguous chunk of ids per XCD, bands of group_m row tiles inside
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

    // The activations go from global to local memory directly, a KiB (eight rows x 128 bytes) per instruction.  A row's
    // 16-byte pieces stand there XORed by row mod 8 (operand reads without bank conflicts), k-step e's piece of lane
    // quarter q, k 16q + 8 - 8e .. 16q + 15 - 8e, at slot (4e + q) ^ (row mod 8): the lanes fetch their pieces in that order.
    // Rows past M or past the tile lie past the resource's end; lane offsets stay below 2^32 (ldx <= 2^24).
    const int rows = (int)min((int64_t)BM, a.M - m0);
    const uint32_t stride = (uint32_t)a.ldx * 2u;
    const char* const xbase = reinterpret_cast<const char*>(a.X + m0 * a.ldx);
    // (128 rows of K = ldx = 2^24 are 2^32 bytes, one more than the resource counts; the last byte is no lane's offset)
    const uint32_t xbytes = (uint32_t)min((int64_t)(rows - 1) * stride + a.n_kt * (TILE_K * 2), (int64_t)0xffffffff);
    const int slot = (lane & 7) ^ (lane >> 3), piece = ((slot & 3) << 1) | (slot >> 2 ^ 1);
    uint32_t xoff[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) xoff[p] = (uint32_t)((wn + WAVES * p) * 8 + (lane >> 3)) * stride + (uint32_t)piece * 16u;

    v4f acc[RI][CJ];
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < CJ; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};

    // this workgroup's K range (split-K: blockIdx.y of `splits` near-equal ranges of whole tiles)
    const int kt_b = (int)(a.n_kt * blockIdx.y / splits), kt_e = (int)(a.n_kt * (blockIdx.y + 1) / splits);
    const int st_b = kt_b * 4, n_st = kt_e * 4;              // stages of 64 k: [st_b, n_st)
    // (past the range's end: nothing is read, but the instructions are there, for they are counted)
    auto load_a = [&](int st, int buf) {
        const __amdgpu_buffer_rsrc_t xr = make_rsrc(xbase, st < n_st ? xbytes : 0u);
#pragma unroll
        for (int p = 0; p < NP; ++p) load_to_lds(xr, smem + buf * A_BUF + (wn + WAVES * p) * 1024, xoff[p], (uint32_t)st * A_ROW);
    };
    auto load_w = [&](int kt, WTile<G>& r) {
        kt = min(kt, kt_e - 1);
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

    WTile<G> w0, w1;
    load_w(kt_b, w0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) load_a(st_b + p, p);
    wait_loads<tall::at_start(PAIR, NP)>();       // stages 0, 1 (and 2) are there
    bare_barrier();

    // (operands of k-step 0 and 1 in buffers 0 .. 3 and, beyond the reach of an instruction's offset, from 4 on)
    const int a_e0 = l16 * A_ROW + (q ^ (l16 & 7)) * 16, a_e1 = l16 * A_ROW + ((4 + q) ^ (l16 & 7)) * 16;
    int a_f0 = a_e0 + 4 * A_BUF, a_f1 = a_e1 + 4 * A_BUF;
    asm volatile("" : "+v"(a_f0), "+v"(a_f1));
    Lut lut[CJ];
    struct BSet { v4i b0[CJ], b1[CJ]; };

    // the weights of stage t of tile w, column block j (a group's look-up table is rebuilt where it begins)
    auto prep_b = [&](auto tc, const WTile<G>& w, int j, BSet& out) {
        constexpr int t = decltype(tc)::value;
        if constexpr (G == 64 || (t & 1) == 0) {
            const uint32_t pair = w.s[j][G == 128 ? 0 : t >> 1];
            const int g_in_pair = G == 128 ? t >> 1 : t & 1;
            lut[j] = make_lut(g_in_pair ? pair >> 16 : pair & 0xffffu);
        }
        const uint32_t wd = t == 0 ? w.w[j].x : t == 1 ? w.w[j].y : t == 2 ? w.w[j].z : w.w[j].w;
        upconvert(wd, lut[j], out.b0[j], out.b1[j]);
    };

    // Software pipeline.  A wave enters stage `it` with the stage's weights up-converted (bc) and its
    // first activation operands (a0) in registers.  Under the stage's 32 matrix instructions it
    // reads the second k-step's operands, up-converts the weights of stage it+1 (bn) and reads that stage's
    // first ones, so every wave keeps the matrix pipe and the vector pipe busy at the same
    // time whatever the other waves of the workgroup, which the barriers keep in step, are doing.
    // LDS: stage it reads buffers it and it+1.  Eight buffers: the pair of stages (2S, 2S+1) reads stages 2S .. 2S+2
    // and asks for stages 2S+6 and 2S+7 in the buffers of the pair before, which the barrier ahead of the pair freed;
    // that barrier follows every wave's wait for its loads up to stage 2S+2, two pairs old.  So waves of a workgroup
    // may be a stage apart inside a pair.  Four buffers: the same with a barrier after every stage.
    v4i a0[RI];
#pragma unroll
    for (int i = 0; i < RI; ++i) a0[i] = *reinterpret_cast<const v4i*>(smem + a_e0 + i * 16 * A_ROW);
    BSet bA, bB;
    prep_b(std::integral_constant<int, 0>{}, w0, 0, bA);
    prep_b(std::integral_constant<int, 0>{}, w0, 1, bA);
    constexpr int VPM = RI >= 6 ? 2 : 3;                     // vector instructions per matrix instruction
    // sc: stage of the loop below, 0 .. 7, and its buffer (mod NBUF)
    auto stage = [&](int it, auto sc, const WTile<G>& wc, WTile<G>& wnx, const BSet& bc, BSet& bn) {
        constexpr int t = decltype(sc)::value & 3, buf = decltype(sc)::value & (NBUF - 1);
        constexpr std::integral_constant<int, (t + 1) & 3> tn{};
        const WTile<G>& wn_tile = t == 3 ? wnx : wc;         // where stage it+1 finds its weights
        constexpr int buf1 = (buf + 1) & (NBUF - 1);
        if constexpr (t == 0) load_w((it >> 2) + 1, wnx);
        __builtin_amdgcn_sched_barrier(0);
        load_a(it + AHEAD, (buf + AHEAD) & (NBUF - 1));
        __builtin_amdgcn_sched_barrier(0);                   // all loads are issued up here, unconditionally
        const int8_t* const ab = smem + (buf < 4 ? a_e1 : a_f1) + (buf & 3) * A_BUF;
        const int8_t* const abn = smem + (buf1 < 4 ? a_e0 : a_f0) + (buf1 & 3) * A_BUF;
        v4i a1[RI];
#pragma unroll
        for (int i = 0; i < RI; ++i) a1[i] = *reinterpret_cast<const v4i*>(ab + i * 16 * A_ROW);
        prep_b(tn, wn_tile, 0, bn);
#pragma unroll
        for (int j = 0; j < CJ; ++j)
#pragma unroll
            for (int i = 0; i < RI; ++i) acc[i][j] = mfma_bf16(a0[i], bc.b0[j], acc[i][j]);
        prep_b(tn, wn_tile, 1, bn);
#pragma unroll
        for (int i = 0; i < RI; ++i) a0[i] = *reinterpret_cast<const v4i*>(abn + i * 16 * A_ROW);
#pragma unroll
        for (int j = 0; j < CJ; ++j)
#pragma unroll
            for (int i = 0; i < RI; ++i) acc[i][j] = mfma_bf16(a1[i], bc.b1[j], acc[i][j]);
        // issue order: one matrix instruction, then the LDS read and the two vector instructions it hides
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int k = 0; k < RI; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
            }
#pragma unroll
            for (int k = RI; k < RI * CJ; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, VPM, 0);
            }
        }
        // before the next pair: stages up to its third have landed; what was asked for since, three more, and a tile's
        // weights in its first stage, may be under way.  (Four buffers: the next two stages; one more.)
        if constexpr (!PAIR || (t & 1)) {
            wait_loads<tall::behind(PAIR, t, NP, tall::weights(false, CJ))>();
            bare_barrier();
        }
    };
    auto tile = [&](int kt, auto oc, const WTile<G>& wc, WTile<G>& wnx) {
        constexpr int o = decltype(oc)::value;
        stage(kt * 4, std::integral_constant<int, o>{}, wc, wnx, bA, bB);
        stage(kt * 4 + 1, std::integral_constant<int, o + 1>{}, wc, wnx, bB, bA);
        stage(kt * 4 + 2, std::integral_constant<int, o + 2>{}, wc, wnx, bA, bB);
        stage(kt * 4 + 3, std::integral_constant<int, o + 3>{}, wc, wnx, bB, bA);
    };
    for (int kt = kt_b; kt < kt_e; kt += 2) {
        tile(kt, std::integral_constant<int, 0>{}, w0, w1);
        if (kt + 1 < kt_e) tile(kt + 1, std::integral_constant<int, 4>{}, w1, w0);   // uniform
    }
    wait_loads<0>();                                         // (stages past the end still store zeros)
    __syncthreads();

    if (a.part) {
        // split-K: this range's fp32 partial results go to the workspace.  A lane holds single columns of
        // four rows per tile (4-byte stores in 64-byte runs: measured on the w2a8 kernel, 5 us of a 29 us
        // launch); the wave's tile goes through LDS, 64 rows at a time (a region of its own: the barrier at
        // the end of the last stage freed the activation buffers; rows padded by 16 bytes, conflict-free both
        // ways), and leaves as 16-byte stores in 128-byte runs.
        float* dst = a.part + (int64_t)blockIdx.y * a.M * a.N;
        int8_t* pbase = smem + wn * (64 * P_STRIDE);
        const int prow = lane >> 3, pcol = (lane & 7) * 4;   // eight lanes per row piece
        const int64_t n = n0 + wn * WN + pcol;
#pragma unroll
        for (int h = 0; h < (RI + 3) / 4; ++h) {
#pragma unroll
            for (int i = 0; i < 4 && h * 4 + i < RI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int j = 0; j < CJ; ++j)
                        *reinterpret_cast<float*>(pbase + (i * 16 + 4 * q + r) * P_STRIDE + (j * 16 + l16) * 4) = acc[h * 4 + i][j][r];
            // the wave reads back only what it wrote itself: LDS operations of one wave complete in order
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

    // The wave's 128 x 32 result goes through LDS (its own region; the barrier at the end of the last
    // stage freed the activation buffers) and leaves as 16-byte stores, four lanes per 64-byte row piece.
    int8_t* ebase = smem + wn * (BM * E_STRIDE);
    uint16_t* eb = reinterpret_cast<uint16_t*>(ebase);
    // Fused epilogue (Sec. II-D: bias and activation applied while the outputs are in registers).  The
    // gated form combines the wave's two column blocks, an even (gate) and an odd (up) one, into one.
    const bool gated = a.epi.act == ACT_SILU_MUL;
    float bias[CJ];
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
        const int64_t n = n0 + wn * WN + j * 16 + l16;
        bias[j] = (a.epi.bias && n < a.N) ? bf16_to_f32(a.epi.bias[n]) : 0.f;
    }
    // (one copy of the loop per epilogue, picked here: a choice per element would have the compiler
    // evaluate the SiLU for every output and select afterwards)
    auto emit = [&](auto mode_c) {
        constexpr int MODE = decltype(mode_c)::value;        // ACT_NONE, ACT_SILU, ACT_SILU_MUL
        static_assert(CJ == 2, "the epilogue pairs the wave's two column blocks");
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = i * 16 + 4 * q + r;
                const float z0 = acc[i][0][r] + bias[0], z1 = acc[i][1][r] + bias[1];
                if constexpr (MODE == ACT_SILU_MUL) {
                    eb[row * (E_STRIDE / 2) + l16] = f32_to_bf16_rne(silu_f32(z0) * z1);
                } else {
                    const uint32_t pk = MODE == ACT_SILU ? pack_bf16x2(silu_f32(z0), silu_f32(z1)) : pack_bf16x2(z0, z1);
                    eb[row * (E_STRIDE / 2) + l16] = (uint16_t)pk;
                    eb[row * (E_STRIDE / 2) + 16 + l16] = (uint16_t)(pk >> 16);
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

}  // namespace fold16

template <int G, int BN, int RI>
static int launch_fold_bn(const A16Args& a_in, int splits, hipStream_t stream)
{
    using namespace fold16;
    constexpr int BM = 16 * RI;
    A16Args a = a_in;
    if (splits < 2) a.part = nullptr;
    const int tiles_m = (int)((a.M + BM - 1) / BM);
    const int tiles_n = (int)((a.N + BN - 1) / BN);
    const int group_m = a.tune.tiled_group_m ? a.tune.tiled_group_m : 8;
    const dim3 grid((unsigned)((int64_t)tiles_m * tiles_n), (unsigned)(splits < 2 ? 1 : splits)), block(64 * waves_of(BN));
    constexpr int lds = lds_bytes(BN, RI);
    if (int rc = ensure_dynamic_lds(reinterpret_cast<const void*>(a16_fold_tiled_kernel<G, BN, RI>), lds,
                                    "w2_matmul_a16[scaled16 tiled]"))
        return rc;
    hipLaunchKernelGGL((a16_fold_tiled_kernel<G, BN, RI>), grid, block, lds, stream, a, tiles_m, tiles_n, group_m,
                       (int)grid.y);
    int rc = check_launch("w2_matmul_a16[scaled16 tiled]");
    if (rc || !a.part) return rc;
    return launch_splitk_reduce(a.part, splits, a.M, a.N, a.Y, a.ldy, a.epi, stream);
}

template <int G, int BN>
static int launch_fold_ri(const A16Args& a, const tiles::Shape& p, hipStream_t stream)
{
    switch (p.ri) {
    case 4: return launch_fold_bn<G, BN, 4>(a, p.splits, stream);
    case 5: return launch_fold_bn<G, BN, 5>(a, p.splits, stream);
    case 6: return launch_fold_bn<G, BN, 6>(a, p.splits, stream);
    case 7: return launch_fold_bn<G, BN, 7>(a, p.splits, stream);
    default: return launch_fold_bn<G, BN, 8>(a, p.splits, stream);
    }
}

int launch_a16_fold_tiled(const A16Args& a, const tiles::Shape& p, bool slim, hipStream_t stream)
{
    if (slim) return a.G == 128 ? launch_fold_ri<128, 128>(a, p, stream) : launch_fold_ri<64, 128>(a, p, stream);
    return a.G == 128 ? launch_fold_ri<128, 256>(a, p, stream) : launch_fold_ri<64, 256>(a, p, stream);
}

}  // namespace w2
