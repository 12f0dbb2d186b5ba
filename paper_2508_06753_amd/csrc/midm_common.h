// What the two mid-M kernels (matmul_midm.hip: a wave's rows in a piece of local memory of its own; matmul_shared.hip: rows shared by
// the workgroup) have in common: arguments, weights for the bf16 matrix instruction, where the dequant is exact.
#pragma once
#include <hip/hip_runtime.h>

#include "midm_plan.h"
#include "w2_small_common.h"

namespace w2 {

namespace midm {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct Args {                                                // what is needed after the first loads
    const float* sx;
    uint16_t* Y;
    int32_t* acc_out;
    float* part;                                             // K split across workgroups too: [blockIdx.z][M][N] fp32
    int64_t N, ldy;
    Epilogue epi;
};

// the head of the arguments: scalar kernel parameters, which a wave finds in registers at its launch
struct Head {
    const char* X;                                           // int8 or bf16 rows
    const char* codes;
    const char* scales;
    uint32_t stride;                                         // bytes between rows
    int M, n_cb, n_kt;                                       // (and t_lo, t_rem: tiles per K range, one more for the first t_rem)
};

// The four weights of one (group, column), low bytes and high bytes, indexed by the raw code
// (00 -> 0, 01 -> +sw, 10 -> -2 sw: sign flipped and exponent + 1, 11 -> -sw).
struct Lut { uint32_t lo4, hi4; };

__device__ __forceinline__ Lut make_lut(uint32_t s)          // s: bf16 bit pattern of the group scale
{
    const uint32_t neg = s ^ 0x8000u;
    // -2 sw: exponent + 1, or of a subnormal scale (a zero: -0) the mantissa twice
    const uint32_t neg2 = (s + min(s & 0x7fffu, 0x0080u)) ^ 0x8000u;
    const uint32_t a = s << 16;
    const uint32_t b = neg2 | (neg << 16);
    Lut l;
    l.lo4 = __builtin_amdgcn_perm(b, a, 0x06040200u);
    l.hi4 = __builtin_amdgcn_perm(b, a, 0x07050301u);
    return l;
}

// 16 codes of one dword -> b0 (k 0..7 of the lane's 16-k block), b1 (k 8..15)
__device__ __forceinline__ void upconvert16(uint32_t w, const Lut& l, v4i& b0, v4i& b1)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t t = (w >> (2 * j)) & 0x03030303u;
        const uint32_t lo = __builtin_amdgcn_perm(0u, l.lo4, t);
        const uint32_t hi = __builtin_amdgcn_perm(0u, l.hi4, t);
        const int d0 = (int)__builtin_amdgcn_perm(hi, lo, 0x05010400u);
        const int d1 = (int)__builtin_amdgcn_perm(hi, lo, 0x07030602u);
        if (j < 2) { b0[2 * j] = d0; b0[2 * j + 1] = d1; }
        else { b1[2 * j - 4] = d0; b1[2 * j - 3] = d1; }
    }
}

__device__ __forceinline__ v4f mfma_bf16(const v4i& a, const v4i& b, const v4f& c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

// Int8 rows: up to 32 rows the decode kernel takes every group's sum exactly, and so does this kernel, whichever of the
// two a shape goes to (the conversion costs 1 % on average over 2048 x 2048 .. 28672 x 8192, 4096 x 6144 at M = 16
// 5.10 -> 5.13 us, 3584 x 18944 with groups of 64 7.9 -> 8.5 at worst); above, the prefill kernels' one-fma form.
constexpr int64_t EXACT_ROWS = 32;

}  // namespace midm

}  // namespace w2
