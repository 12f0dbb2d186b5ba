// Medium M (up to 256 rows), both activation types: between the memory-bound GEMV regime and the compute-bound GEMM
// regime of Sec. III-C.  The weight stream is read once per band of up to 64 rows, and every up-converted weight
// ("up-convert and compute", Sec. II-C) is multiplied into RT row tiles: v_mfma_i32_16x16x64_i8 for int8 rows,
// v_mfma_f32_16x16x32_bf16 for bf16 rows (Sec. II-D, "Alternative implementation"), on scale-folded weights from two row
// tiles per wave on, on the weights q and with a dequant per 64 k below.
//
// A wave owns RT row tiles x CJ column blocks x a contiguous run of k tiles; the waves of a workgroup split K (Sec.
// II-D, K-splitting for small shapes) and their partial results meet in local memory once, in a fixed order.  Where the
// column blocks are too few for the chip and K is deep, K is also split across workgroups, whose fp32 results go to the
// caller's workspace and are added by a second launch (28672 x 1024, 16 bf16 rows 13.6 -> 9.8 us, 28672 x 2048 18.4 ->
// 12.1; 28672 x 5120 at M = 64 33 -> 28).
//
// Why this shape.  What such a problem moves is the activations: every workgroup reads its rows over the whole K, 64
// bytes per clock and CU through the vector L1 whichever way they go.  With K split over the waves nothing that a wave
// reads is read by another wave of the workgroup, so the activations need no workgroup-wide staging and the main loop
// no barrier: a wave turns them around in a piece of local memory of its own.  It has to, because the matrix operand
// wants 16 rows per 16 bytes of k: loaded directly in that order the L1 delivers 16 B/clk (one cache line per lane),
// loaded as eight rows x 128 bytes per instruction 60 B/clk (measured, 256 CUs reading 64 rows of 4096..14336 bytes
// out of L2).  A chunk is 128 bytes of every row: loaded a chunk or two ahead into registers, written as it comes with
// the 16-byte pieces of row r XORed by r mod 8, read back as matrix operands without bank conflicts.  CJ column blocks
// share the operands that are read; RT row tiles share the up-converted weights (7 or 23 vector instructions per 16).
//
// SH = 2: pairs of waves take different column blocks of the same K range and share its chunks (two buffers, one
// barrier per chunk): half the activation traffic, for wide projections with int8 rows, and an even number of column blocks
// for the gated epilogue where a wave has three or five.
//
// Measured (graph-timed with weights out of memory, us; before = the kernels this one replaces, which shared 1024-k chunks
// of all rows between the waves of a workgroup with two barriers each, and split deep K across workgroups more often):
// int8 rows, M = 48: 4096 x 6144 9.7 -> 6.4, 4096 x 4096 9.4 -> 5.0, 14336 x 4096 17.3 -> 11.3, 17408 x 5120 18.9 ->
// 13.4, 3584 x 18944 24.5 -> 11.8, 4096 x 28672 17.1 -> 14.8; bf16 rows, M = 64: 4096 x 6144 16.4 -> 9.5, 14336 x 4096 27.3 ->
// 18.0, 4096 x 28672 33.6 -> 23.7, 28672 x 8192 54.9 -> 41.8.
//
// What bounds it (4096 x 28672, 64 int8 rows, 17.2 us; copies with parts taken out): without the activations 14.0,
// without the weight loads 12.9, without either 10.3, without the epilogue 14.8: a launch of this size is too short
// for its phases (first loads out of HBM, multiply, reduce) to overlap (counters over the whole launch: vector issue slots a
// third full, matrix pipe and local memory a fifth each, waves waiting a third of the time).  Deeper load windows, a second operand set read a chunk ahead, pinned interleaving
// of vector and matrix instructions and a start of K that differs per workgroup were measured and gave nothing.
#include <hip/hip_runtime.h>

#include "midm_common.h"

#if defined(__HIP_DEVICE_COMPILE__) && defined(__FAST_MATH__)
#error "the one-fma dequant reads int32 accumulators as fp32 denormals: do not build with fast-math / flush-to-zero"
#endif

namespace w2 {

namespace midm {

// XT 0: int8 rows (w2a8), 1: bf16 rows (w2a16)
// EX (int8 rows): every group's int32 sum is converted exactly before it is scaled; see the dequant below
// MODE: the product, a part of it (K split across workgroups), or
// the test-only export of the int32 group sums
constexpr int WHOLE = 0, PART = 1, GROUP_SUMS = 2;
template <int XT, int G, int RT, int CJ, int SH, bool EX, int MODE>
__global__ void __launch_bounds__(64 * max_waves(RT, CJ), max_waves(RT, CJ) / 4)
midm_kernel(const char* __restrict__ X, const char* __restrict__ codes, const char* __restrict__ scales, uint32_t stride, int M,
            int n_cb, int n_kt, int t_lo, int t_rem, Args a)
{
    constexpr bool DBG = MODE == GROUP_SUMS;
    constexpr int EB = XT == 0 ? 1 : 2;                      // bytes per activation
    constexpr int CH = TILE_K * EB / CHUNK_BYTES;            // chunks per tile: 2 or 4
    constexpr int GPT = TILE_K / G;
    constexpr bool FOLD = XT == 1 && RT > 1;                 // bf16 rows: the scale folded into the weights, or as they are
    constexpr int NJ = RT * 2 / SH;                          // 16-byte pieces per lane and chunk
    constexpr int D = 2;                                     // weight tiles in flight
    constexpr int SD = NJ <= 4 ? 2 : 1;                      // chunks in flight
    static_assert(D * CH % SD == 0, "register sets are picked at compile time");
    extern __shared__ __align__(16) int8_t smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = lane >> 4, l16 = lane & 15;
    const int m0 = blockIdx.y * (RT * 16);
    const int rows = min(RT * 16, M - m0);
    const int cg = wave % SH, kr = wave / SH;
    const int cb0 = (blockIdx.x * SH + cg) * CJ;
    // of the whole K (the dimensions of the workgroup come out of memory, and a 13th parameter would too: 0.2 us ahead of
    // the first loads, which only the parts of a deep K pay)
    const int range = MODE == PART ? blockIdx.z * ((blockDim.x >> 6) / SH) + kr : kr;
    const int t0 = range * t_lo + min(range, t_rem);
    const int T = t_lo + (range < t_rem ? 1 : 0);
    // waves that share chunks meet at barriers: the same count for all (past its run a wave reads zeros)
    const int T_all = SH > 1 ? t_lo + (t_rem > 0 ? 1 : 0) : T;
    const int nch = T * CH;
    int8_t* const my = smem + kr * range_lds(RT, CJ, SH);

    // the rows, from this run's first k on: rows past the last lie past the end of the resource, whose loads return
    // zeros and move nothing (the lane offset alone puts them there: (rows - 1) * stride + the run's bytes <= rows *
    // stride), and so does everything once there is no further chunk
    const char* xbase = X + (int64_t)m0 * stride + (int64_t)t0 * (TILE_K * EB);
    const uint32_t xbytes = (uint32_t)(rows - 1) * stride + (uint32_t)T * (TILE_K * EB);
    uint32_t xoff[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        xoff[j] = (uint32_t)((cg * NJ + j) * 8 + (lane >> 3)) * stride + (uint32_t)(lane & 7) * 16u;
    // local memory, per row 128 bytes: the 16-byte piece that k-step e gives to lane quarter q sits at slot
    // (4 e + q) ^ (row mod 8).  int8 rows: piece 4 e + q; bf16 rows (a lane's 16 k are two pieces): piece 2 q + e
    const int piece = lane & 7, f = XT == 0 ? piece : (piece >> 1) | ((piece & 1) << 2);
    const int st_off = (cg * NJ * 8 + (lane >> 3)) * CHUNK_BYTES + ((f ^ (lane >> 3)) * 16);
    const int rd0 = l16 * CHUNK_BYTES + ((q ^ (l16 & 7)) * 16);
    const int rd1 = l16 * CHUNK_BYTES + (((4 + q) ^ (l16 & 7)) * 16);

    // the run of each column block: loads past its end, or of a block past the last, return zeros and move nothing
    const char* wp[CJ];
    const char* sp[CJ];
    uint32_t wbytes[CJ], sbytes[CJ];
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
        const bool ok = cb0 + j < n_cb;
        const int64_t tile = (int64_t)(ok ? cb0 + j : cb0) * n_kt + t0;
        wp[j] = codes + tile * TILE_BYTES;
        sp[j] = scales + tile * (TILE_N * GPT * 2);
        wbytes[j] = ok ? (uint32_t)T * TILE_BYTES : 0u;
        sbytes[j] = ok ? (uint32_t)T * (TILE_N * GPT * 2) : 0u;
    }

    u32x4 stage[SD][NJ];
    auto load_x = [&](int c, int set) {
        const __amdgpu_buffer_rsrc_t xr = make_rsrc(xbase, c < nch ? xbytes : 0u);
#pragma unroll
        for (int j = 0; j < NJ; ++j) stage[set][j] = __builtin_amdgcn_raw_buffer_load_b128(xr, xoff[j], c * CHUNK_BYTES, 0);
    };
    u32x4 w[D][CJ];
    uint32_t sc[D][CJ][GPT / 2];
    auto load_w = [&](int i, int set) {
#pragma unroll
        for (int j = 0; j < CJ; ++j) {
            w[set][j] = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc(wp[j], wbytes[j]), lane * 16 + i * TILE_BYTES, 0, 0);
            const __amdgpu_buffer_rsrc_t sr = make_rsrc(sp[j], sbytes[j]);
            const int so = l16 * (GPT * 2) + i * (TILE_N * GPT * 2);
            if constexpr (G == 128) {
                sc[set][j][0] = __builtin_amdgcn_raw_buffer_load_b32(sr, so, 0, 0);
            } else {
                const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(sr, so, 0, 0);
                sc[set][j][0] = t[0];
                sc[set][j][1] = t[1];
            }
        }
    };

    // activations first, then the weights: vector memory returns in order
#pragma unroll
    for (int s = 0; s < SD; ++s) load_x(s, s);
#pragma unroll
    for (int i = 0; i < D; ++i) load_w(i, i);
    __builtin_amdgcn_sched_barrier(0);

    // Dequant of the int8 form above EXACT_ROWS in one fma: a group starts from BIAS = 2^21 (the third matrix operand), so
    // acc = BIAS + 64 * sum is positive and below 2^23 and its bit pattern read as binary32 is the denormal
    // acc * 2^-149: y += as_float(acc) * (sw * 2^64).  The bias, 2^-128 * (the sum of the scaled scales), is taken out
    // every four tiles and at the end.  Two accumulator sets alternate between groups; a finished group is dequantised
    // under the next one's matrix instructions.
    // EX: no bias; the sum is converted (one more instruction) and scaled as the decode kernel does it, which takes the
    // same row counts on other shapes: fp32 sums of exact products, any finite scale.
    constexpr int BIAS = EX ? 0 : 1 << 21;                   // > 64 * 127 * 2 * 128
    constexpr float SWS = EX ? 1.0f : 0x1p64f;
    const v4i biasv = {BIAS, BIAS, BIAS, BIAS};
    v4i acc[2][RT];
    v4f y[RT][CJ];
    float ssum[CJ];
    float pend_sw = 0.f;                                     // the finished group waiting in set 1: none yet
    int pend_g = 0;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        acc[0][rt] = biasv;
        acc[1][rt] = biasv;
#pragma unroll
        for (int j = 0; j < CJ; ++j) y[rt][j] = (v4f){0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int j = 0; j < CJ; ++j) ssum[j] = 0.f;

    auto dequant = [&](int b, int j) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (DBG) {
                    const int m = rt * 16 + 4 * q + r;
                    const int64_t n = (int64_t)(cb0 + j) * TILE_N + l16;
                    if (pend_sw != 0.f && n < a.N && m < rows)
                        a.acc_out[((int64_t)(m0 + m) * (n_kt * GPT) + pend_g) * a.N + n] = (acc[b][rt][r] - BIAS) >> 6;
                }
                y[rt][j][r] = fmaf(EX ? (float)acc[b][rt][r] : __int_as_float(acc[b][rt][r]), pend_sw, y[rt][j][r]);
            }
        if constexpr (!EX) ssum[j] += pend_sw;
    };
    v4f accf[2] = {(v4f){0.f, 0.f, 0.f, 0.f}, (v4f){0.f, 0.f, 0.f, 0.f}};      // bf16 rows, not folded: the same alternation
    auto dequant_f = [&](int b, int j) {
#pragma unroll
        for (int r = 0; r < 4; ++r) y[0][j][r] = fmaf(accf[b][r], pend_sw, y[0][j][r]);
    };
    auto settle = [&]() {
        if constexpr (EX) return;
#pragma unroll
        for (int j = 0; j < CJ; ++j) {
            const float corr = ssum[j] * 0x1p-128f;
            ssum[j] = 0.f;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int r = 0; r < 4; ++r) y[rt][j][r] -= corr;
        }
    };

    // up-converted operands of the coming block (a block: one column block of one chunk)
    v4i bn0, bn1;
    Lut lut[CJ];
    auto prepare_b = [&](const u32x4& wd, const uint32_t (&s)[GPT / 2], int h, int j) {
        if constexpr (XT == 0) {
            int u0[4], u1[4];
            upconvert(wd[2 * h], u0);
            upconvert(wd[2 * h + 1], u1);
            bn0 = (v4i){u0[0], u0[1], u0[2], u0[3]};
            bn1 = (v4i){u1[0], u1[1], u1[2], u1[3]};
        } else if constexpr (FOLD) {
            if (G == 64 || !(h & 1)) {                       // a group begins
                const uint32_t p = s[G == 128 ? 0 : h >> 1];
                const int hi = G == 128 ? h >> 1 : h & 1;
                lut[j] = make_lut(hi ? p >> 16 : p & 0xffffu);
            }
            upconvert16(wd[h], lut[j], bn0, bn1);
        } else {
            upconvert16(wd[h], Lut{0x80008000u, 0xbbbc3b00u}, bn0, bn1);     // 2^-8 * (0, 1, -2, -1)
        }
    };
    constexpr int SBUF = RT * 16 * CHUNK_BYTES;
    v4i f0[RT], f1[RT];                                      // matrix operands of the chunk's two k-steps
    // chunk c, in register set `set`: to local memory and back as matrix operands; chunk c + SD is requested.  Local
    // memory operations of one wave complete in order.
    auto turn_chunk = [&](int c, int set, int par) {
        int8_t* const buf = my + (SH > 1 ? par * SBUF : 0);
#pragma unroll
        for (int j = 0; j < NJ; ++j) *reinterpret_cast<u32x4*>(buf + st_off + j * 1024) = stage[set][j];
        load_x(c + SD, set);
        if constexpr (SH > 1) {
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            f0[rt] = *reinterpret_cast<const v4i*>(buf + rd0 + rt * 2048);
            f1[rt] = *reinterpret_cast<const v4i*>(buf + rd1 + rt * 2048);
        }
        __builtin_amdgcn_wave_barrier();
    };
    prepare_b(w[0][0], sc[0][0], 0, 0);

    for (int i0 = 0; i0 < T_all; i0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int i = i0 + u;
            if (i >= T_all) break;
#pragma unroll
            for (int h = 0; h < CH; ++h) {
                const int n = u * CH + h;                    // (constant after unrolling)
                turn_chunk(i * CH + h, n % SD, h & 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < CJ; ++j) {
                    const v4i b0 = bn0, b1 = bn1;
                    if (j + 1 < CJ) prepare_b(w[u][j + 1], sc[u][j + 1], h, j + 1);
                    else if (h + 1 < CH) prepare_b(w[u][0], sc[u][0], h + 1, 0);
                    else prepare_b(w[(u + 1) % D][0], sc[(u + 1) % D][0], 0, 0);
                    if constexpr (XT == 0) {
                        const int pj = (j + CJ - 1) % CJ;
                        const uint32_t p = sc[u][j][G == 128 ? 0 : h];
                        if constexpr (G == 128) {
                            const int b = (h * CJ + j) & 1;
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) acc[b][rt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f0[rt], b0, biasv, 0, 0, 0);
                            dequant(b ^ 1, pj);
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) acc[b][rt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f1[rt], b1, acc[b][rt], 0, 0, 0);
                            pend_sw = DBG ? 1.0f : __uint_as_float(h ? p & 0xffff0000u : p << 16) * SWS;
                            pend_g = (t0 + i) * GPT + h;
                        } else {
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) acc[0][rt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f0[rt], b0, biasv, 0, 0, 0);
                            dequant(1, pj);
                            pend_sw = DBG ? 1.0f : __uint_as_float(p << 16) * SWS;
                            pend_g = (t0 + i) * GPT + 2 * h;
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) acc[1][rt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f1[rt], b1, biasv, 0, 0, 0);
                            dequant(0, j);
                            pend_sw = DBG ? 1.0f : __uint_as_float(p & 0xffff0000u) * SWS;
                            pend_g = (t0 + i) * GPT + 2 * h + 1;
                        }
                    } else if constexpr (!FOLD) {
                        // One row tile (up to 16 rows): 2^-8 * sum x * q of every 64 k apart, then y += sw * sum: any
                        // finite scale, as in the decode kernel, which takes the same row counts on other shapes (the
                        // folded weight -2 sw does not exist from 2^127 on), and no finite row overflows a sum.  Four
                        // fmas per 64 k where the folded table takes ten instructions a group.
                        const uint32_t p = sc[u][j][G == 128 ? 0 : h >> 1];
                        const int b = (h * CJ + j) & 1;
                        accf[b] = mfma_bf16(f0[0], b0, (v4f){0.f, 0.f, 0.f, 0.f});
                        dequant_f(b ^ 1, (j + CJ - 1) % CJ);
                        accf[b] = mfma_bf16(f1[0], b1, accf[b]);
                        pend_sw = __uint_as_float((G == 128 ? h >> 1 : h & 1) ? p & 0xffff0000u : p << 16);
                    } else {
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) y[rt][j] = mfma_bf16(f0[rt], b0, y[rt][j]);
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) y[rt][j] = mfma_bf16(f1[rt], b1, y[rt][j]);
                    }
                }
            }
            if constexpr (XT == 0) {
                if ((i & 3) == 3) settle();
            }
            load_w(i + D, u);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (XT == 0) {
        dequant(1, CJ - 1);
        if constexpr (DBG) return;
        settle();
    } else if constexpr (!FOLD) {
        dequant_f(1, CJ - 1);
    }
    if constexpr (SH > 1) __syncthreads();                   // the staged chunks are read by the other wave too
    // (fetched under the reduction; read in the store loop it cost 0.1 us a launch)
    const float sx_mine = XT == 0 && !DBG ? a.sx[min(m0 + (int)(threadIdx.x & 63), M - 1)] : 0.f;
    constexpr int RS = CJ * 16 + 4;
    float* red = reinterpret_cast<float*>(my + cg * red_bytes(RT, CJ));
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int j = 0; j < CJ; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                red[(rt * 16 + 4 * q + r) * RS + j * 16 + l16] = y[rt][j][r];
    float* const sx_lds = reinterpret_cast<float*>(smem + (blockDim.x >> 6) / SH * range_lds(RT, CJ, SH));
    if constexpr (XT == 0) {
        if (threadIdx.x < RT * 16) sx_lds[threadIdx.x] = sx_mine;
    }
    __syncthreads();
    const int ks = (blockDim.x >> 6) / SH;
    constexpr int WC = SH * CJ;                              // column blocks of the workgroup
    const int wcb0 = blockIdx.x * WC;
    auto sum4 = [&](int row, int col) {
        v4f s = {0.f, 0.f, 0.f, 0.f};
        const int8_t* p = smem + (col / (CJ * 16)) * red_bytes(RT, CJ) + (row * RS + col % (CJ * 16)) * 4;
        // four ranges' loads ahead of the first addition: a loop over single ones waits for local memory each time (4096 x 28672,
        // four ranges, 64 bf16 rows 23.3 -> 22.9 us, int8 rows 17.9 -> 17.4)
        int k = 0;
        for (; k + 4 <= ks; k += 4) {
            v4f t[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = *reinterpret_cast<const v4f*>(p + (k + e) * range_lds(RT, CJ, SH));
#pragma unroll
            for (int e = 0; e < 4; ++e) s += t[e];
        }
        for (; k < ks; ++k) s += *reinterpret_cast<const v4f*>(p + k * range_lds(RT, CJ, SH));
        if constexpr (XT == 1 && !FOLD) s *= 256.0f;
        // 2^79 = 2^(149-64-6) (EX: 2^-6) on the sums, not on sx: a row scale may be as large as fp32 holds
        if constexpr (XT == 0) s = s * (EX ? 0x1p-6f : 0x1p79f) * sx_lds[row];
        return s;
    };
    auto add_bias = [&](v4f& v, int64_t n) {
        if (a.epi.bias) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += bf16_to_f32(a.epi.bias[n + e]);   // (the bias need not be aligned)
        }
    };
    auto put = [&](int row, int64_t n, const v4f& v) {
        *reinterpret_cast<uint2*>(a.Y + (int64_t)(m0 + row) * a.ldy + n) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
    };
    if constexpr (MODE == PART) {                            // the epilogue belongs to the launch that adds the parts
        float* dst = a.part + ((int64_t)blockIdx.z * M + m0) * a.N;
        for (int i = threadIdx.x; i < rows * WC * 4; i += blockDim.x) {
            const int row = i / (WC * 4), col = (i % (WC * 4)) * 4;
            const int64_t n = (int64_t)wcb0 * TILE_N + col;
            if (n < a.N) *reinterpret_cast<v4f*>(dst + row * a.N + n) = sum4(row, col);
        }
        return;
    }
    if (a.epi.act != ACT_SILU_MUL) {
        for (int i = threadIdx.x; i < rows * WC * 4; i += blockDim.x) {
            const int row = i / (WC * 4), col = (i % (WC * 4)) * 4;
            const int64_t n = (int64_t)wcb0 * TILE_N + col;
            if (n >= a.N) continue;
            v4f v = sum4(row, col);
            add_bias(v, n);
            if (a.epi.act == ACT_SILU) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = silu_f32(v[e]);
            }
            put(row, n, v);
        }
    } else if constexpr (WC >= 2) {
        for (int i = threadIdx.x; i < rows * WC * 2; i += blockDim.x) {
            const int row = i / (WC * 2), c = i % (WC * 2);
            const int gcol = (c >> 2) * 32 + (c & 3) * 4;
            const int64_t n = (int64_t)wcb0 * TILE_N + gcol;
            if (n >= a.N) continue;
            v4f g = sum4(row, gcol), v = sum4(row, gcol + 16);
            add_bias(g, n);
            add_bias(v, n + 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] *= silu_f32(g[e]);
            put(row, (int64_t)(wcb0 / 2 + (c >> 2)) * TILE_N + (c & 3) * 4, v);
        }
    }
}

template <int XT, int G, int RT, int CJ, int SH, bool EX, int MODE>
static int launch_t(const Head& h, const Args& a, const Plan& p, hipStream_t stream)
{
    if constexpr (MODE == WHOLE && CJ != 3 && CJ != 5) {     // (K is not split across workgroups where the columns fill the chip)
        if (p.sp > 1) return launch_t<XT, G, RT, CJ, SH, EX, PART>(h, a, p, stream);
    }
    const size_t lds = (size_t)p.ks * range_lds(RT, CJ, SH) + RT * 16 * sizeof(float);
    auto kern = midm_kernel<XT, G, RT, CJ, SH, EX, MODE>;
    if (int rc = ensure_dynamic_lds((const void*)kern, lds, "w2_matmul[midm]")) return rc;
    const dim3 grid((unsigned)((h.n_cb + CJ * SH - 1) / (CJ * SH)), (unsigned)((h.M + RT * 16 - 1) / (RT * 16)), (unsigned)p.sp),
               block(64 * p.ks * SH);
    const int ranges = p.ks * p.sp;
    hipLaunchKernelGGL(kern, grid, block, lds, stream, h.X, h.codes, h.scales, h.stride, h.M, h.n_cb, h.n_kt,
                       h.n_kt / ranges, h.n_kt % ranges, a);
    const int rc = check_launch("w2_matmul[midm]");
    if (rc || MODE != PART) return rc;
    return launch_splitk_reduce(a.part, p.sp, h.M, a.N, a.Y, a.ldy, a.epi, stream);
}

template <int XT, int G, int RT, int CJ>
static int launch_sh(const Head& h, const Args& a, const Plan& p, hipStream_t stream)
{
    constexpr bool PAIRS = built(XT, RT, CJ, 3) || built(XT, RT, CJ, 4);
    if constexpr (XT == 0 && RT <= 2) {
        if (h.M <= EXACT_ROWS) {
            if constexpr (PAIRS) {
                if (p.sh == 2) return launch_t<XT, G, RT, CJ, 2, true, WHOLE>(h, a, p, stream);
            }
            return launch_t<XT, G, RT, CJ, 1, true, WHOLE>(h, a, p, stream);
        }
    }
    if constexpr (PAIRS) {
        if (p.sh == 2) return launch_t<XT, G, RT, CJ, 2, false, WHOLE>(h, a, p, stream);
    }
    return launch_t<XT, G, RT, CJ, 1, false, WHOLE>(h, a, p, stream);
}

template <int XT, int G>
static int launch_g(const Head& h, const Args& a, const Plan& p, hipStream_t stream)
{
    if (a.acc_out) {                                         // the test-only export of the int32 accumulators: one width
        if constexpr (XT == 0) {
            const Plan d = {p.rt, 2, (int)min((int64_t)8, (int64_t)h.n_kt), 1, 1};
            switch (p.rt) {
            case 1: return launch_t<0, G, 1, 2, 1, true, GROUP_SUMS>(h, a, d, stream);
            case 2: return launch_t<0, G, 2, 2, 1, true, GROUP_SUMS>(h, a, d, stream);
            case 3: return launch_t<0, G, 3, 2, 1, false, GROUP_SUMS>(h, a, d, stream);
            default: return launch_t<0, G, 4, 2, 1, false, GROUP_SUMS>(h, a, d, stream);
            }
        }
    }
    switch (p.rt * 8 + p.cj) {
    case 8 + 1: return launch_sh<XT, G, 1, 1>(h, a, p, stream);
    case 8 + 2: return launch_sh<XT, G, 1, 2>(h, a, p, stream);
    case 8 + 3: return launch_sh<XT, G, 1, 3>(h, a, p, stream);
    case 8 + 4: return launch_sh<XT, G, 1, 4>(h, a, p, stream);
    case 8 + 5: return launch_sh<XT, G, 1, 5>(h, a, p, stream);
    case 16 + 2: return launch_sh<XT, G, 2, 2>(h, a, p, stream);
    case 16 + 3: return launch_sh<XT, G, 2, 3>(h, a, p, stream);
    case 16 + 4: return launch_sh<XT, G, 2, 4>(h, a, p, stream);
    case 16 + 5: return launch_sh<XT, G, 2, 5>(h, a, p, stream);
    case 24 + 2: return launch_sh<XT, G, 3, 2>(h, a, p, stream);
    case 24 + 3: return launch_sh<XT, G, 3, 3>(h, a, p, stream);
    case 24 + 4: return launch_sh<XT, G, 3, 4>(h, a, p, stream);
    case 24 + 5: return launch_sh<XT, G, 3, 5>(h, a, p, stream);
    case 32 + 2: return launch_sh<XT, G, 4, 2>(h, a, p, stream);
    case 32 + 3: return launch_sh<XT, G, 4, 3>(h, a, p, stream);
    default: return launch_sh<XT, G, 4, 4>(h, a, p, stream);
    }
}

}  // namespace midm

// (beyond 256 rows the tiled kernels' reuse of the weights wins everywhere)

bool a8_midm_supports(const A8Args& a) { return a.M >= 1 && a.M <= 256; }
bool a16_midm_supports(const A16Args& a) { return a.M >= 1 && a.M <= 256; }

// What w2_workspace_size adds for this range on a deep K (K > 13312): fp32 copies of the output, 2..16 of them, as many
// parts as about 64 workgroups across the columns need for one workgroup per CU.
size_t midm_room_bytes(int64_t M, int64_t N, int64_t n_cb, int64_t n_kt)
{
    const int64_t chunks = (n_kt + 3) / 4;                   // of 1024 k
    if (chunks < 14) return 0;
    const int64_t cbw = n_cb >= 8 * 64 ? 8 : n_cb >= 4 * 64 ? 4 : 2;
    const int64_t wgs = (n_cb + cbw - 1) / cbw * ((M + 63) / 64);
    const int64_t s = min(min((256 + wgs / 2) / wgs, chunks / 3), (int64_t)16);
    return s < 2 ? 0 : (size_t)s * M * N * sizeof(float);
}

int launch_a8_midm(const A8Args& a, const midm::Plan& p, hipStream_t stream)
{
    const midm::Head h = {(const char*)a.xq, (const char*)a.codes, (const char*)a.scales, (uint32_t)a.K, (int)a.M, (int)a.n_cb, (int)a.n_kt};
    const midm::Args k = {a.sx, a.Y, a.acc_out, a.acc_out ? nullptr : a.part, a.N, a.ldy, a.epi};
    return a.G == 128 ? midm::launch_g<0, 128>(h, k, p, stream) : midm::launch_g<0, 64>(h, k, p, stream);
}

int launch_a16_midm(const A16Args& a, const midm::Plan& p, hipStream_t stream)
{
    const midm::Head h = {(const char*)a.X, (const char*)a.codes, (const char*)a.scales, (uint32_t)(a.ldx * 2), (int)a.M, (int)a.n_cb, (int)a.n_kt};
    const midm::Args k = {nullptr, a.Y, nullptr, a.part, a.N, a.ldy, a.epi};
    return a.G == 128 ? midm::launch_g<1, 128>(h, k, p, stream) : midm::launch_g<1, 64>(h, k, p, stream);
}

}  // namespace w2
