// Medium M on grids of several column blocks per CU, both activation types: the mid-M kernel (matmul_midm.hip) with its rows shared by
// the whole workgroup.
//
// Why.  A workgroup reads its rows over the whole K, and what the CUs together read of rows and weights adds up in the L2s: on 4096
// x 28672 with 48 int8 rows the rows alone (448 workgroups of four blocks: 88 MB) take 4.0 us, the weights (31 MB out of memory) 4.1,
// both 8.0, also where different waves or different CUs read them, however far ahead.  So a workgroup is a CU's share of the columns
// wide, SH waves x CJ column blocks, and its K ranges (as many as sixteen waves allow) read every row once: 224 workgroups of eight
// blocks, 44 MB.  Widths of two to eight blocks, ten, twelve, fourteen and sixteen: 5120 x 34816, 2176 blocks, is one round of 218
// workgroups of ten.
//
// The rows go straight to local memory, 128 bytes of each at a time (a chunk), four buffers a range, three chunks under way; 16-byte
// pieces XORED by row.  A barrier per chunk, behind every wave's counted wait for its own loads.  No registers hold rows on their way,
// which is what leaves room for sixteen waves: four per SIMD, whose matrix and vector instructions cover each other's waits.  Weights,
// up-convert, dequant and the meeting of the ranges are the other kernel's.
//
// Measured (graph-timed through the public calls with weights out of memory, us; matmul_midm.hip's best shape -> this kernel, where AUTO
// takes it): 4096 x 28672 int8 M = 48 / 64 16.2 / 18.3 -> 13.7 / 15.5, bf16 M = 64 24.2 -> 22.0; gated int8 M = 48 15.1 -> 12.3, bf16
// M = 64 23.0 -> 20.5; 5120 x 34816 gated int8 M = 24 / 32 / 48 / 64 17.9 / 19.3 / 20.2 / 23.9 -> 15.8 / 16.3 / 18.5 / 21.1, bf16 M = 32 /
// 48 / 64 25.3 / 27.9 / 36.6 -> 23.4 / 26.6 / 30.3; 8192 x 57344 gated int8 M = 48 39.6 -> 33.8.  Counters (4096 x 28672 gated): vector
// issue 39 % of the launch, matrix pipe 18 % (48 int8 rows) and 29 % (64 bf16 rows), waves wait half their time.  What bounds it (4096 x 28672, 48 int8 rows, copies with parts taken out, of 13.5): loads alone 11.6, without any 9.8,
// launch and epilogue 3.5; with 64 bf16 rows, of 20.9: 13.9, 16.0, matrix instructions alone 11.0.
#include <hip/hip_runtime.h>

#include "midm_common.h"
#include "shared_plan.h"

#if defined(__HIP_DEVICE_COMPILE__) && defined(__FAST_MATH__)
#error "the one-fma dequant reads int32 accumulators as fp32 denormals: do not build with fast-math / flush-to-zero"
#endif

namespace w2 {

namespace shared {

using namespace midm;
using shared::Plan;
using shared::built;
using shared::range_lds;

// XT 0: int8 rows (w2a8), 1: bf16 rows (w2a16).  EX (int8 rows): every group's sum is converted exactly before it is scaled.
template <int XT, int G, int RT, int CJ, int SH, bool EX>
__global__ void __launch_bounds__(64 * SH * k_ranges(XT, G, RT, CJ, SH), (SH * k_ranges(XT, G, RT, CJ, SH) + 3) / 4)
shared_kernel(const char* __restrict__ X, const char* __restrict__ codes, const char* __restrict__ scales, uint32_t stride, int M,
            int n_cb, int n_kt, int t_lo, int t_rem, Args a)
{
    constexpr int EB = XT == 0 ? 1 : 2;                      // bytes per activation
    constexpr int CH = TILE_K * EB / CHUNK_BYTES;            // chunks per tile: 2 or 4
    constexpr int GPT = TILE_K / G;
    static_assert(RT >= 2, "bf16 rows: the scale folded into the weights");
    constexpr int NJ = loads(RT, SH);                        // 16-byte pieces per lane and chunk
    constexpr int CB = buf_bytes(RT, SH), RANGE = range_lds(RT, CJ, SH);
    constexpr int D = 2;                                     // weight tiles in flight
    static_assert(D * CH % BUFS == 0, "buffers are constants of the unrolled loop");
    extern __shared__ __align__(16) int8_t smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = lane >> 4, l16 = lane & 15;
    const int m0 = blockIdx.y * (RT * 16);
    const int rows = min(RT * 16, M - m0);
    const int cg = wave % SH, kr = wave / SH;
    const int cb0 = (blockIdx.x * SH + cg) * CJ;
    const int t0 = kr * t_lo + min(kr, t_rem);
    const int T = t_lo + (kr < t_rem ? 1 : 0);
    // the waves meet at barriers: the same count for all (past its run a wave reads zeros)
    const int T_all = t_lo + (t_rem > 0 ? 1 : 0);
    const int nch = T * CH;
    int8_t* const my = smem + kr * RANGE;

    // the rows, from this run's first k on: rows past the last lie past the end of the resource, whose loads return
    // zeros and move nothing (the lane offset alone puts them there: (rows - 1) * stride + the run's bytes <= rows *
    // stride), and so does everything once there is no further chunk
    const char* xbase = X + (int64_t)m0 * stride + (int64_t)t0 * (TILE_K * EB);
    const uint32_t xbytes = (uint32_t)(rows - 1) * stride + (uint32_t)T * (TILE_K * EB);
    // (a buffer has room for every load of every wave: those past the last row store zeros behind the rows)
    // local memory, per row 128 bytes: the 16-byte piece that k-step e gives to lane quarter q sits at slot
    // (4 e + q) ^ (row mod 8).  int8 rows: piece 4 e + q; bf16 rows (a lane's 16 k are two pieces): piece 2 q + e
    const int slot = (lane & 7) ^ (lane >> 3), piece = XT == 0 ? slot : ((slot & 3) << 1) | (slot >> 2);
    uint32_t xoff[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        xoff[j] = (uint32_t)((cg * NJ + j) * 8 + (lane >> 3)) * stride + (uint32_t)piece * 16u;
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

    auto load_x = [&](int c, int buf) {
        const __amdgpu_buffer_rsrc_t xr = make_rsrc(xbase, c < nch ? xbytes : 0u);
#pragma unroll
        for (int j = 0; j < NJ; ++j) load_to_lds(xr, my + buf * CB + (cg * NJ + j) * 1024, xoff[j], (uint32_t)c * CHUNK_BYTES);
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
    for (int s = 0; s < BUFS - 1; ++s) load_x(s, s);
#pragma unroll
    for (int i = 0; i < D; ++i) load_w(i, i);
    __builtin_amdgcn_sched_barrier(0);

    // dequant as in matmul_midm.hip: one fma on the bit pattern of BIAS + 64 * sum, or (EX) an exact conversion ahead of it
    constexpr int BIAS = EX ? 0 : 1 << 21;                   // > 64 * 127 * 2 * 128
    constexpr float SWS = EX ? 1.0f : 0x1p64f;
    const v4i biasv = {BIAS, BIAS, BIAS, BIAS};
    v4i acc[2][RT];
    v4f y[RT][CJ];
    float ssum[CJ];
    float pend_sw = 0.f;                                     // the finished group waiting in set 1: none yet
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
                y[rt][j][r] = fmaf(EX ? (float)acc[b][rt][r] : __int_as_float(acc[b][rt][r]), pend_sw, y[rt][j][r]);
            }
        if constexpr (!EX) ssum[j] += pend_sw;
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
        } else {
            if (G == 64 || !(h & 1)) {                       // a group begins
                const uint32_t p = s[G == 128 ? 0 : h >> 1];
                const int hi = G == 128 ? h >> 1 : h & 1;
                lut[j] = make_lut(hi ? p >> 16 : p & 0xffffu);
            }
            upconvert16(wd[h], lut[j], bn0, bn1);
        }
    };
    v4i f0[RT], f1[RT];                                      // matrix operands of the chunk's two k-steps
    // Behind the barrier every wave's part of the chunk is there, and nobody reads the chunk before any more: its matrix
    // instructions have been issued, so its operands have been read.
    auto wait_chunk = [&](int h) {
        if (h == 0) wait_loads<under_way(0, CH, NJ, CJ)>();
        else if (h == 1) wait_loads<under_way(1, CH, NJ, CJ)>();
        else if (h == 2) wait_loads<under_way(2, CH, NJ, CJ)>();
        else wait_loads<under_way(3, CH, NJ, CJ)>();
    };
    auto turn_chunk = [&](int c, int buf, int h) {
        wait_chunk(h);
        bare_barrier();
        load_x(c + BUFS - 1, (buf + BUFS - 1) % BUFS);
        __builtin_amdgcn_sched_barrier(0);
        const int8_t* const b = my + buf * CB;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            f0[rt] = *reinterpret_cast<const v4i*>(b + rd0 + rt * 2048);
            f1[rt] = *reinterpret_cast<const v4i*>(b + rd1 + rt * 2048);
        }
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
                turn_chunk(i * CH + h, n % BUFS, h);
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
                            pend_sw = __uint_as_float(h ? p & 0xffff0000u : p << 16) * SWS;
                        } else {
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) acc[0][rt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f0[rt], b0, biasv, 0, 0, 0);
                            dequant(1, pj);
                            pend_sw = __uint_as_float(p << 16) * SWS;
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) acc[1][rt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f1[rt], b1, biasv, 0, 0, 0);
                            dequant(0, j);
                            pend_sw = __uint_as_float(p & 0xffff0000u) * SWS;
                        }
                    } else {
                        // (the upper k-step first: another order of additions than matmul_midm.hip's, so that the results of the
                        // two can be told apart)
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) y[rt][j] = mfma_bf16(f1[rt], b1, y[rt][j]);
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) y[rt][j] = mfma_bf16(f0[rt], b0, y[rt][j]);
                    }
                }
            }
            if constexpr (XT == 0) {
                if ((i & 3) == 1) settle();              // (every four tiles; not after the same ones as in matmul_midm.hip)
            }
            load_w(i + D, u);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (XT == 0) {
        dequant(1, CJ - 1);
        settle();
    }
    wait_loads<0>();                                         // (chunks past the run's end still store zeros)
    __syncthreads();
    // (fetched under the reduction; read in the store loop it cost 0.1 us a launch)
    const float sx_mine = XT == 0 ? a.sx[min(m0 + (int)(threadIdx.x & 63), M - 1)] : 0.f;
    constexpr int RS = CJ * 16 + 4;
    float* red = reinterpret_cast<float*>(my + cg * red_bytes(RT, CJ));
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int j = 0; j < CJ; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                red[(rt * 16 + 4 * q + r) * RS + j * 16 + l16] = y[rt][j][r];
    float* const sx_lds = reinterpret_cast<float*>(smem + (blockDim.x >> 6) / SH * RANGE);
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
        // (four ranges' loads ahead of the first addition)
        int k = 0;
        for (; k + 4 <= ks; k += 4) {
            v4f t[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = *reinterpret_cast<const v4f*>(p + (k + e) * RANGE);
#pragma unroll
            for (int e = 0; e < 4; ++e) s += t[e];
        }
        for (; k < ks; ++k) s += *reinterpret_cast<const v4f*>(p + k * RANGE);
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
    } else if constexpr (WC % 2 == 0) {                      // (gate and up blocks in pairs: even widths only)
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

template <int XT, int G, int RT, int CJ, int SH, bool EX>
static int launch_t(const Head& h, const Args& a, hipStream_t stream)
{
    const int ks = min(k_ranges(XT, G, RT, CJ, SH), h.n_kt);
    const size_t lds = (size_t)ks * range_lds(RT, CJ, SH) + RT * 16 * sizeof(float);
    auto kern = shared_kernel<XT, G, RT, CJ, SH, EX>;
    if (int rc = ensure_dynamic_lds((const void*)kern, lds, "w2_matmul[mid-M, shared rows]")) return rc;
    const dim3 grid((unsigned)((h.n_cb + CJ * SH - 1) / (CJ * SH)), (unsigned)((h.M + RT * 16 - 1) / (RT * 16))), block(64 * ks * SH);
    hipLaunchKernelGGL(kern, grid, block, lds, stream, h.X, h.codes, h.scales, h.stride, h.M, h.n_cb, h.n_kt, h.n_kt / ks, h.n_kt % ks, a);
    return check_launch("w2_matmul[mid-M, shared rows]");
}

template <int XT, int G, int RT, int CJ, int SH>
static int launch_sh(const Head& h, const Args& a, hipStream_t stream)
{
    if constexpr (!built(XT, RT, CJ, SH)) {
        set_error("w2_matmul[mid-M, shared rows]: %d x %d blocks not built for %d row tiles", CJ, SH, RT);
        return W2_ERR_UNSUPPORTED_SHAPE;
    } else {
        if constexpr (XT == 0 && RT <= 2) {
            if (h.M <= EXACT_ROWS) return launch_t<XT, G, RT, CJ, SH, true>(h, a, stream);
        }
        return launch_t<XT, G, RT, CJ, SH, false>(h, a, stream);
    }
}

template <int XT, int G, int RT>
static int launch_rt(const Head& h, const Args& a, const Plan& p, hipStream_t stream)
{
    switch (p.cj * 16 + p.sh) {
    case 16 + 2: return launch_sh<XT, G, RT, 1, 2>(h, a, stream);
    case 16 + 3: return launch_sh<XT, G, RT, 1, 3>(h, a, stream);
    case 16 + 4: return launch_sh<XT, G, RT, 1, 4>(h, a, stream);
    case 16 + 5: return launch_sh<XT, G, RT, 1, 5>(h, a, stream);
    case 16 + 6: return launch_sh<XT, G, RT, 1, 6>(h, a, stream);
    case 16 + 7: return launch_sh<XT, G, RT, 1, 7>(h, a, stream);
    case 16 + 8: return launch_sh<XT, G, RT, 1, 8>(h, a, stream);
    case 32 + 4: return launch_sh<XT, G, RT, 2, 4>(h, a, stream);
    case 32 + 5: return launch_sh<XT, G, RT, 2, 5>(h, a, stream);
    case 32 + 6: return launch_sh<XT, G, RT, 2, 6>(h, a, stream);
    case 32 + 7: return launch_sh<XT, G, RT, 2, 7>(h, a, stream);
    default: return launch_sh<XT, G, RT, 2, 8>(h, a, stream);
    }
}

template <int XT, int G>
static int launch_g(const Head& h, const Args& a, const Plan& p, hipStream_t stream)
{
    switch (p.rt) {
    case 2: return launch_rt<XT, G, 2>(h, a, p, stream);
    case 3: return launch_rt<XT, G, 3>(h, a, p, stream);
    default: return launch_rt<XT, G, 4>(h, a, p, stream);
    }
}

}  // namespace shared

int launch_a8_shared(const A8Args& a, const shared::Plan& p, hipStream_t stream)
{
    const midm::Head h = {(const char*)a.xq, (const char*)a.codes, (const char*)a.scales, (uint32_t)a.K, (int)a.M, (int)a.n_cb, (int)a.n_kt};
    const midm::Args k = {a.sx, a.Y, nullptr, nullptr, a.N, a.ldy, a.epi};
    return a.G == 128 ? shared::launch_g<0, 128>(h, k, p, stream) : shared::launch_g<0, 64>(h, k, p, stream);
}

int launch_a16_shared(const A16Args& a, const shared::Plan& p, hipStream_t stream)
{
    const midm::Head h = {(const char*)a.X, (const char*)a.codes, (const char*)a.scales, (uint32_t)(a.ldx * 2), (int)a.M, (int)a.n_cb, (int)a.n_kt};
    const midm::Args k = {nullptr, a.Y, nullptr, nullptr, a.N, a.ldy, a.epi};
    return a.G == 128 ? shared::launch_g<1, 128>(h, k, p, stream) : shared::launch_g<1, 64>(h, k, p, stream);
}

}  // namespace w2
