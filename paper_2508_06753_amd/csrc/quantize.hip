// Per-token int8 quantisation of the activations (Sec. II-B; Sec. II-D: the
// abs-max of the quantisation granularity gives the scale, entries are
// multiplied by the inverse of the scale and converted to int8).  One scale
// per row.  Every operation is a single IEEE binary32 operation (correctly
// rounded divide, one multiply, round-half-even), so the int8 codes are
// reproducible bit for bit.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "w2_internal.h"

namespace w2 {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The definition's rounding and clamp, bits 0..7 of the result the int8 code: t = x * inv (one rounded multiply),
// clamped to +-127, rounded half to even by adding 1.5 * 2^23 (|t| < 2^22: one more rounding).
__device__ __forceinline__ uint32_t quant_bits(float x, float inv)
{
#pragma clang fp contract(off)
    const float t = __builtin_amdgcn_fmed3f(x * inv, -127.0f, 127.0f);
    return __float_as_uint(t + 12582912.0f);
}

// low bytes of a, b, c, d -> one dword
__device__ __forceinline__ uint32_t pack4(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    return __builtin_amdgcn_perm(b, a, 0x0c0c0400u) | __builtin_amdgcn_perm(d, c, 0x04000c0cu);
}

// One workgroup per row.  A few rows (decode) are a chain of latencies: the row arrives (a cold miss), its abs-max is
// reduced inside the waves (DPP) and across them (one trip through local memory, one barrier), one division, out; many
// rows are bound by memory.  The row stays in registers, NV 16-byte vectors per thread, all in flight before the first
// is used (range-checked loads: slots past the end of the row read zeros and move nothing), so it is read once; only
// rows beyond eight vectors per thread are read a second time.  Measured (replayed graph, rows of its own per launch, us;
// before: generic lane shuffles, two barriers, four predicated vectors per thread whatever the row, seven instructions
// to round and clamp a value): bf16 48 x 4096 2.76 -> 2.32, 48 x 14336 3.68 -> 2.89, 200 x 14336 5.7 -> 3.9,
// 2048 x 8192 12.5 -> 9.7 (5.2 TB/s); fp32 8 x 4096 2.65 -> 2.29, 200 x 14336 10.2 -> 4.8, 2048 x 8192 18.3 -> 15.6.
template <bool BF16, int NV, bool GSUM>
__global__ void __launch_bounds__(1024)
quantize_rows_kernel(const void* __restrict__ X, int64_t ldx, int8_t* __restrict__ xq, int64_t K, float* __restrict__ sx,
                     int32_t* __restrict__ gsum, int G)
{
    constexpr int EPT = BF16 ? 8 : 4;                        // elements per vector
    constexpr int EB = BF16 ? 2 : 4;
    const int64_t m = blockIdx.x;
    const char* row = reinterpret_cast<const char*>(X) + m * ldx * EB;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n_waves = blockDim.x >> 6;
    const int step = blockDim.x * 16;                        // bytes between a thread's vectors
    const int64_t row_bytes = K * EB;
    __shared__ float s_red[16];

    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(row), 0,
                                                                             (int)min(row_bytes, (int64_t)1 << 30), 0x00020000);
    u32x4 v[NV];
#pragma unroll
    for (int c = 0; c < NV; ++c) v[c] = __builtin_amdgcn_raw_buffer_load_b128(rr, (int)threadIdx.x * 16 + c * step, 0, 0);

    auto value = [&](const u32x4& d, int e) -> float {
        if constexpr (BF16) return __uint_as_float(e & 1 ? d[e >> 1] & 0xffff0000u : d[e >> 1] << 16);
        else return __uint_as_float(d[e]);
    };
    float amax = 0.0f;
#pragma unroll
    for (int c = 0; c < NV; ++c)
#pragma unroll
        for (int e = 0; e < EPT; ++e) amax = fmaxf(amax, fabsf(value(v[c], e)));
    if constexpr (NV == 8) {
        for (int64_t o = (int64_t)threadIdx.x * 16 + NV * step; o < row_bytes; o += step) {
            const u32x4 d = *reinterpret_cast<const u32x4*>(row + o);
#pragma unroll
            for (int e = 0; e < EPT; ++e) amax = fmaxf(amax, fabsf(value(d, e)));
        }
    }
    amax = wave_max_f32(amax);
    if (n_waves > 1) {
        if (lane == 0) s_red[wave] = amax;
        __syncthreads();
        amax = wave_max_f32((lane & 15) < n_waves ? s_red[lane & 15] : 0.0f);    // every wave reduces the partial maxima itself
    }
    const float inv = amax > 0.0f ? __fdiv_rn(127.0f, amax) : 0.0f;

    auto emit = [&](const u32x4& d, int64_t o) {
        const int64_t k = o / EB;
        uint32_t b[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) b[e] = quant_bits(value(d, e), inv);
        const uint32_t p0 = pack4(b[0], b[1], b[2], b[3]);
        if constexpr (BF16) *reinterpret_cast<uint2*>(xq + m * K + k) = make_uint2(p0, pack4(b[4], b[5], b[6], b[7]));
        else *reinterpret_cast<uint32_t*>(xq + m * K + k) = p0;
        if constexpr (GSUM) {
            // Each group occupies G / EPT (8 to 32) consecutive, aligned lanes, and K % 256 == 0 makes the active lanes
            // of a wave a whole number of such runs (a bf16 row of 256 values fills half a wave: lanes 0..31): a lane
            // only ever reads lanes of its own, fully active, run.
            int sum = 0;
#pragma unroll
            for (int e = 0; e < EPT; ++e) sum += (int)(int8_t)(b[e] & 0xffu);
            const int run = G / EPT;
            for (int off = 1; off < run; off <<= 1) sum += __shfl_xor(sum, off);
            if ((lane & (run - 1)) == 0) gsum[m * (K / G) + k / G] = sum;
        }
    };
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const int o = (int)threadIdx.x * 16 + c * step;
        if (o < row_bytes) emit(v[c], o);                    // whole groups of lanes (K % 256 == 0)
    }
    if constexpr (NV == 8) {
        for (int64_t o = (int64_t)threadIdx.x * 16 + NV * step; o < row_bytes; o += step)
            emit(*reinterpret_cast<const u32x4*>(row + o), o);
    }
    if (threadIdx.x == 0) sx[m] = amax > 0.0f ? __fdiv_rn(amax, 127.0f) : 0.0f;
}

int launch_quantize(const void* X, int x_is_bf16, int64_t M, int64_t K, int64_t ldx, int G,
                    int8_t* xq, float* sx, int32_t* gsum, hipStream_t stream)
{
    if (M == 0) return 0;
    // Few rows (decode): one wide workgroup per row to shorten the serial chain.
    // Many rows (prefill): 256 threads, several rows per CU, unless a thread would hold more than eight vectors.
    const int64_t vecs = K / (x_is_bf16 ? 8 : 4);            // 16-byte vectors of a row: a multiple of 32
    int threads = M <= 64 ? 512 : 256;
    while (threads < 1024 && vecs > (int64_t)8 * threads) threads <<= 1;
    while (threads > 64 && threads > vecs) threads >>= 1;
    const int64_t nv = (vecs + threads - 1) / threads;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)M), dim3(threads), 0, stream, X, ldx, xq, K, sx, gsum, G);
        return check_launch("w2_quantize_rows");
    };
    auto by_type = [&](auto nv_c) {
        constexpr int NV = decltype(nv_c)::value;
        if (gsum) return x_is_bf16 ? go(quantize_rows_kernel<true, NV, true>) : go(quantize_rows_kernel<false, NV, true>);
        return x_is_bf16 ? go(quantize_rows_kernel<true, NV, false>) : go(quantize_rows_kernel<false, NV, false>);
    };
    if (nv <= 1) return by_type(std::integral_constant<int, 1>{});
    if (nv <= 2) return by_type(std::integral_constant<int, 2>{});
    if (nv <= 4) return by_type(std::integral_constant<int, 4>{});
    return by_type(std::integral_constant<int, 8>{});
}

}  // namespace w2
