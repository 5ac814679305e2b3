// FP32 operands as three bf16 parts (see conv_split.hip), shared by the split-operand kernels.
#pragma once

#include "common.h"

namespace mnb {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int POSB = 48;              // LDS bytes of eight staged terms: 3 parts x 8 x 2
constexpr int STEPB = 3 * 64 * 16;    // bytes of one reduction step of a 16-filter fragment

// Values from here on take the branch of split8: some would round up to an infinity.
constexpr float SPLIT_BIG = 3.3895e38f;
__device__ __forceinline__ float max8(const float* x) {
    float big = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) big = fmaxf(big, fabsf(x[i]));
    return big;
}

// Eight floats into three bf16 octets, each part the nearest to what the parts before it leave, so
// that the products left out have no sign in common (cut off instead, they pull every sum towards
// zero by 4e-8, which thousands of rows do not average out).  Values that would round up to an
// infinity are cut off.  An infinity is a third part alone: it meets the first part of a weight, whose
// sign is the weight's, and not the others.  NaN is NaN in every part.  ANY = false: without the branch
// these take, for finite values below SPLIT_BIG (and NaN).
template <bool ANY = true>
__device__ __forceinline__ void split8(const float* x, uintx4& h, uintx4& m, uintx4& l) {
    const float big = ANY ? max8(x) : 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const floatx2 v = {x[2 * i], x[2 * i + 1]};
        unsigned p = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
        if (big >= SPLIT_BIG) {
            const unsigned t0 = fabsf(v[0]) == INFINITY ? 0u : __float_as_uint(v[0]) >> 16;
            const unsigned t1 = fabsf(v[1]) == INFINITY ? 0u : __float_as_uint(v[1]) & 0xffff0000u;
            if (fabsf(v[0]) >= SPLIT_BIG) p = (p & 0xffff0000u) | t0;
            if (fabsf(v[1]) >= SPLIT_BIG) p = (p & 0xffffu) | t1;
        }
        const floatx2 r = {v[0] - __uint_as_float(p << 16), v[1] - __uint_as_float(p & 0xffff0000u)};
        unsigned q = __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf16x2));
        if (big >= SPLIT_BIG) {
            if (fabsf(r[0]) == INFINITY) q &= 0xffff0000u;
            if (fabsf(r[1]) == INFINITY) q &= 0xffffu;
        }
        const floatx2 t = {r[0] - __uint_as_float(q << 16), r[1] - __uint_as_float(q & 0xffff0000u)};
        h[i] = p;
        m[i] = q;
        l[i] = __builtin_bit_cast(unsigned, __builtin_convertvector(t, bf16x2));
    }
}

// The parts of a filter weight, each the nearest to what the parts before it leave, to dst, dst + 512 and
// dst + 1024.  The first part of a nonzero weight is never zero (the smallest bf16 number instead, which the
// second then takes back), so that an infinite operand gives the infinity an FP32 product gives and no
// 0 x inf.  The matrix instruction keeps denormal parts; what a weight below 2^-110 has under 2^-133, the
// smallest bf16 number, is rounded away.
__device__ __forceinline__ void split_weight(float w, unsigned short* dst) {
    float r = w;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        unsigned h = __float_as_uint(r) >> 16;
        if (fabsf(r) < SPLIT_BIG) h = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{r, 0.f}, bf16x2)) & 0xffffu;
        if (s == 0 && w != 0.f) h |= (h & 0x7fff) == 0;
        r -= __uint_as_float(h << 16);
        dst[s * 512] = (unsigned short)h;
    }
}

// The six part products of filter fragments W[FN][3] (rows of the result) and one fragment R[3] of the
// other operand (its columns), the leading one into hi[j][i], the others into low[j][i].
#define MNB_SPLIT_MM(FN_, W, R, hi, low, i)                                                            \
    {                                                                                                 \
        _Pragma("unroll") for (int j_ = 0; j_ < FN_; ++j_)                                            \
            low[j_][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[j_][2], R[0], low[j_][i], 0, 0, 0); \
        _Pragma("unroll") for (int j_ = 0; j_ < FN_; ++j_)                                            \
            hi[j_][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[j_][0], R[0], hi[j_][i], 0, 0, 0);   \
        _Pragma("unroll") for (int j_ = 0; j_ < FN_; ++j_)                                            \
            low[j_][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[j_][1], R[1], low[j_][i], 0, 0, 0); \
        _Pragma("unroll") for (int j_ = 0; j_ < FN_; ++j_)                                            \
            low[j_][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[j_][0], R[2], low[j_][i], 0, 0, 0); \
        _Pragma("unroll") for (int j_ = 0; j_ < FN_; ++j_)                                            \
            low[j_][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[j_][1], R[0], low[j_][i], 0, 0, 0); \
        _Pragma("unroll") for (int j_ = 0; j_ < FN_; ++j_)                                            \
            low[j_][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[j_][0], R[1], low[j_][i], 0, 0, 0); \
    }

}  // namespace mnb
