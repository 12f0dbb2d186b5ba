// Off-line weight pre-formatting (Sec. II-B: the 2-bit tensor is re-laid-out
// ahead of time because inference weights are frozen) and its inverse, used
// by the round-trip test.
#include <hip/hip_runtime.h>

#include "w2_internal.h"

namespace w2 {

// A workgroup converts 16 column blocks x one k tile (256 k): bound by memory, one byte read per weight and a quarter
// written.  A thread reads a column block's 16 codes of 16 consecutive rows, 16 bytes a row with all loads in flight
// (16 lanes cover 256 contiguous bytes), packs four codes at a time where they lie, transposes 4 x 4 bytes per four
// columns and leaves 16 dwords in local memory (column blocks 260 dwords apart: no bank conflicts), from where every
// tile goes out as one contiguous KiB.  The block's scales move in the same launch.  4096 x 28672: 139 -> 32 us by
// the caller's clock, the rate of a copy (one thread per dword with 16 byte loads each, and a second launch for the scales, before).
constexpr int PP_CB = 16;                                    // column blocks per workgroup
constexpr int PP_STRIDE = 260;                               // dwords between column blocks in local memory

// 16 codes at p; ALIGN: what the address is known to be a multiple of
template <int ALIGN>
__device__ __forceinline__ uint4 load_codes16(const uint8_t* p)
{
    if constexpr (ALIGN == 16) return *reinterpret_cast<const uint4*>(p);
    uint4 v;
    if constexpr (ALIGN == 8) {
        const uint2 a = *reinterpret_cast<const uint2*>(p), b = *reinterpret_cast<const uint2*>(p + 8);
        v = make_uint4(a.x, a.y, b.x, b.y);
    } else {
        __builtin_memcpy(&v, p, 16);
    }
    return v;
}

template <int ALIGN>
__device__ __forceinline__ uint2 load_codes8(const uint8_t* p)
{
    uint2 v;
    if constexpr (ALIGN >= 8) v = *reinterpret_cast<const uint2*>(p);
    else __builtin_memcpy(&v, p, 8);
    return v;
}

template <int ALIGN, bool TERNARY>
__global__ void __launch_bounds__(256)
prepack_kernel(const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scales, int64_t N, int64_t n_cb,
               int64_t n_kt, int gpt, int64_t groups_x, uint32_t* __restrict__ out, uint16_t* __restrict__ out_scales,
               int32_t* __restrict__ bad_codes)
{
    __shared__ __align__(16) uint32_t tile[PP_CB * PP_STRIDE];
    constexpr uint32_t ZERO = TERNARY ? 0x01010101u : 0x02020202u;      // the codes of value 0
    const int64_t kt = blockIdx.x / groups_x;
    const int64_t cb0 = (blockIdx.x - kt * groups_x) * PP_CB;
    const int tid = threadIdx.x;
    const int c = tid & 15, t = (tid >> 4) & 3, q = tid >> 6;
    const int64_t cb = cb0 + c, n0 = cb * TILE_N;
    uint32_t v[16][4];
    if (n0 + TILE_N <= N) {
        const uint8_t* src = codes + (kt * TILE_K + t * 64 + q * 16) * N + n0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint4 x = load_codes16<ALIGN>(src + r * N);
            v[r][0] = x.x; v[r][1] = x.y; v[r][2] = x.z; v[r][3] = x.w;
        }
    } else {
        // N % 8 == 0: eight columns of the last block, or none; the missing ones are value 0
        const bool half = n0 < N;
        const uint8_t* src = codes + (kt * TILE_K + t * 64 + q * 16) * N + (half ? n0 : 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            uint2 x = load_codes8<ALIGN>(src + r * N);
            if (!half) x = make_uint2(ZERO, ZERO);
            v[r][0] = x.x; v[r][1] = x.y; v[r][2] = ZERO; v[r][3] = ZERO;
        }
    }
    // codes outside the alphabet (none, in a sound checkpoint): counted, and stored as value 0
    uint32_t ill = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) ill |= (v[r][e] & 0xfcfcfcfcu) | (TERNARY ? v[r][e] & (v[r][e] >> 1) & 0x01010101u : 0u);
    if (ill) {
        int bad = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t x = v[r][e];
                const uint32_t b = (x & 0xfcfcfcfcu) | (TERNARY ? x & (x >> 1) & 0x01010101u : 0u);
                const uint32_t top = (((b & 0x7f7f7f7fu) + 0x7f7f7f7fu) | b) & 0x80808080u;      // a bit per non-zero byte
                const uint32_t mask = (top >> 7) * 0xffu;
                bad += __popc(top);
                v[r][e] = (x & ~mask) | (ZERO & mask);
            }
        if (bad_codes) atomicAdd(bad_codes, bad);
    }
    uint32_t* mine = tile + c * PP_STRIDE + q * 64 + t;      // dword (lane, t) at 4 * lane + t, lane = 16 q + column
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t p[4];                                       // p[b]: bits 2j of byte i = row 4 j + b of column 4 e + i
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            p[b] = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t x = v[4 * j + b][e];          // code c -> the two's complement of its value
                p[b] |= (TERNARY ? (x + 0x03030303u) & 0x03030303u : x ^ 0x02020202u) << (2 * j);
            }
        }
        // 4 x 4 bytes transposed: column 4 e + i takes byte i of p[0..3]
        const uint32_t lo01 = __builtin_amdgcn_perm(p[1], p[0], 0x05010400u), hi01 = __builtin_amdgcn_perm(p[1], p[0], 0x07030602u);
        const uint32_t lo23 = __builtin_amdgcn_perm(p[3], p[2], 0x05010400u), hi23 = __builtin_amdgcn_perm(p[3], p[2], 0x07030602u);
        mine[(4 * e + 0) * 4] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
        mine[(4 * e + 1) * 4] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
        mine[(4 * e + 2) * 4] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
        mine[(4 * e + 3) * 4] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
    }
    // the scales of one column per thread
    const int64_t n = cb0 * TILE_N + tid;
    if (cb0 + (tid >> 4) < n_cb) {
        uint16_t* dst = out_scales + (((cb0 + (tid >> 4)) * n_kt + kt) * TILE_N + (tid & 15)) * gpt;
        for (int g = 0; g < gpt; ++g) dst[g] = n < N ? scales[(kt * gpt + g) * N + n] : 0;
    }
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int i = 0; i < PP_CB / 4; ++i) {
        const int cl = i * 4 + wave;
        if (cb0 + cl < n_cb)
            *reinterpret_cast<uint4*>(out + ((cb0 + cl) * n_kt + kt) * 256 + lane * 4) = *reinterpret_cast<const uint4*>(tile + cl * PP_STRIDE + lane * 4);
    }
}

// Inverse: one thread per canonical code.
__global__ void __launch_bounds__(256)
unpack_codes_kernel(const uint32_t* __restrict__ packed, int64_t K, int64_t N, int64_t n_kt,
                    int codec, uint8_t* __restrict__ codes)
{
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= K * N) return;
    const int64_t k = id / N, n = id % N;
    const int64_t cb = n / TILE_N, kt = k / TILE_K;
    const int kk = (int)(k % TILE_K);
    const int t = kk / 64, qb = (kk % 64) / 16, j = (kk % 16) / 4, b = kk % 4;
    const int lane = qb * 16 + (int)(n % TILE_N);
    const uint32_t w = packed[((cb * n_kt + kt) * 64 + lane) * 4 + t];
    int x = (w >> (8 * b + 2 * j)) & 3;
    int q = x >= 2 ? x - 4 : x;
    codes[id] = (uint8_t)(q + (codec == 0 ? 2 : 1));
}

__global__ void __launch_bounds__(256)
unpack_scales_kernel(const uint16_t* __restrict__ pscales, int64_t K, int64_t N, int G,
                     int64_t n_kt, int gpt, uint16_t* __restrict__ scales)
{
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t Kg = K / G;
    if (id >= Kg * N) return;
    const int64_t g = id / N, n = id % N;
    const int64_t cb = n / TILE_N, kt = g / gpt;
    scales[id] = pscales[((cb * n_kt + kt) * TILE_N + (n % TILE_N)) * gpt + (g % gpt)];
}

int launch_prepack(const uint8_t* codes, const uint16_t* scales, const Layout& L, int codec,
                   void* packed, int32_t* bad_codes, hipStream_t stream)
{
    const int64_t groups_x = (L.n_cb + PP_CB - 1) / PP_CB;
    const dim3 grid((unsigned)(groups_x * L.n_kt)), block(256);
    uint16_t* out_scales = (uint16_t*)((char*)packed + L.codes_bytes);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, 0, stream, codes, scales, L.N, L.n_cb, L.n_kt, L.gpt, groups_x,
                           (uint32_t*)packed, out_scales, bad_codes);
        return check_launch("w2_prepack");
    };
    // how the caller's rows are aligned: start and length (a multiple of 8)
    const uintptr_t a = (uintptr_t)codes | (uintptr_t)L.N;
    const bool tern = codec != 0;
    if (a % 16 == 0) return tern ? go(prepack_kernel<16, true>) : go(prepack_kernel<16, false>);
    if (a % 8 == 0) return tern ? go(prepack_kernel<8, true>) : go(prepack_kernel<8, false>);
    return tern ? go(prepack_kernel<1, true>) : go(prepack_kernel<1, false>);
}

int launch_unpack(const void* packed, const Layout& L, int codec, uint8_t* codes,
                  uint16_t* scales, hipStream_t stream)
{
    const int64_t n_codes = L.K * L.N;
    const int64_t n_scales = (L.K / L.G) * L.N;
    hipLaunchKernelGGL(unpack_codes_kernel, dim3((unsigned)((n_codes + 255) / 256)), dim3(256), 0,
                       stream, (const uint32_t*)packed, L.K, L.N, L.n_kt, codec, codes);
    hipLaunchKernelGGL(unpack_scales_kernel, dim3((unsigned)((n_scales + 255) / 256)), dim3(256), 0,
                       stream, (const uint16_t*)((const char*)packed + L.codes_bytes), L.K, L.N,
                       L.G, L.n_kt, L.gpt, scales);
    return check_launch("w2_debug_unpack");
}

}  // namespace w2
