// Device pieces of the convolutions that contract on the matrix cores (tern_conv_matrix.hip has the
// reasons): widening of 2-bit codes to 4-bit floats, the matrix instruction, the cut points of Eq. 6 as
// floats and their decisions on accumulators.
#pragma once
#include "tern_internal.h"

namespace tern {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// (mask, sign) word of 32 channels -> two words whose 4-bit field i holds, for two channels each,
// the sign in bits 3 / 2 and the mask in bits 1 / 0: channels 4 i + 1 / 4 i in the first, 4 i + 3 /
// 4 i + 2 in the second.
__device__ __forceinline__ v2u interleave(uint32_t m, uint32_t s, uint32_t m33)
{
    v2u w;
    w.x = __builtin_amdgcn_bitop3_b32(m33, m, s << 2, 0xca);   // m33 ? m : s << 2
    w.y = __builtin_amdgcn_bitop3_b32(m33, m >> 2, s, 0xca);
    return w;
}

// Two interleaved words -> 32 four-bit floats (E2M1: +1 = 0010, -1 = 1010, 0 = x000).
__device__ __forceinline__ v4i expand(v2u w, uint32_t maa)
{
    v4i o;
    o.x = (int)((w.x << 1) & maa);
    o.y = (int)(w.x & maa);
    o.z = (int)((w.y << 1) & maa);
    o.w = (int)(w.y & maa);
    return o;
}

// 32 filters x 32 voxels x 64 channels; 4-bit operands occupy the first four of the eight operand
// registers, and constant zero scale operands select the instruction without block scales.
__device__ __forceinline__ v16f multiply(v4i a, v4i b, v16f c)
{
    const v8i a8 = __builtin_shufflevector(a, a, 0, 1, 2, 3, -1, -1, -1, -1);
    const v8i b8 = __builtin_shufflevector(b, b, 0, 1, 2, 3, -1, -1, -1, -1);
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, c, 4, 4, 0, 0, 0, 0);
}

// Cut points as what the accumulators start from, -(hi + 1/2), and what turns acc - hi - 1/2 into
// acc - lo + 1/2.  Sums stay within 2^21 (the launchers see to it), so clamping to 2^21 + 1 changes no
// decision and every intermediate is a multiple of 1/2 below 2^23: exact.  Filters that do not exist
// (live false) get code 0.
constexpr int kMatrixSumLimit = 1 << 21;
struct Cut {
    float start, width;
};
__device__ __forceinline__ Cut cut_of(int lo, int hi, bool live)
{
    constexpr int L = kMatrixSumLimit + 1;
    lo = live ? max(-L, min(L, lo)) : -L;
    hi = live ? max(-L, min(L, hi)) : L;
    const Cut c = {-(float)hi - 0.5f, (float)(hi - lo + 1)};
    return c;
}

// Appends to pos / neg the signs of acc - hi - 1/2 (set: not above hi) and of acc - lo + 1/2 (set: below
// lo): one vector instruction and two.  BITS = 5 leaves a gap of four (undefined) bits behind them.
template <int BITS>
__device__ __forceinline__ void decide(uint32_t& pos, uint32_t& neg, float acc, float width)
{
    pos = __builtin_amdgcn_alignbit(pos, __float_as_uint(acc), 32 - BITS);
    neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc + width), 32 - BITS);
}

// The decisions of a 32 x 32 block (K = 4) or of its first 8 K rows, register v = filter 8 (v / 4) + 4 g + v % 4:
// widths come four at a time from LDS (for the lane's own half g), highest filter first, so that filter
// 8 k + 4 g + j ends up at bit 8 k + j.
template <int K>
__device__ __forceinline__ void decide_rows(uint32_t& pos, uint32_t& neg, const v16f& acc, const float* widths)
{
    pos = neg = 0u;
#pragma unroll
    for (int k = K - 1; k >= 0; --k) {
        const float4 w = *reinterpret_cast<const float4*>(widths + 8 * k);
        decide<1>(pos, neg, acc[4 * k + 3], w.w);
        decide<1>(pos, neg, acc[4 * k + 2], w.z);
        decide<1>(pos, neg, acc[4 * k + 1], w.y);
        if (k > 0) decide<5>(pos, neg, acc[4 * k], w.x);
        else decide<1>(pos, neg, acc[4 * k], w.x);
    }
}
__device__ __forceinline__ void decide_block(uint32_t& pos, uint32_t& neg, const v16f& acc, const float* widths)
{
    decide_rows<4>(pos, neg, acc, widths);
}

// pos / neg as decide_block leaves them to packed words, lane = voxel l % 32: lanes 0-31 get the voxels'
// mask words, lanes 32-63 their sign words (+1 wins where both decisions hold).
template <uint32_t MASK>
__device__ __forceinline__ uint32_t word_of(uint32_t pos, uint32_t neg)
{
    const uint32_t m = __builtin_amdgcn_bitop3_b32(pos, neg, MASK, 0x8a);          // (~pos | neg) & mask
    const uint32_t s = __builtin_amdgcn_bitop3_b32(pos, neg, MASK, 0x80);          // pos & neg & mask
    const auto sw = __builtin_amdgcn_permlane32_swap(m, s, false, false);
    return sw[0] | (sw[1] << 4);                                                   // both halves' filters
}
__device__ __forceinline__ uint32_t block_word(uint32_t pos, uint32_t neg) { return word_of<0x0f0f0f0fu>(pos, neg); }
__device__ __forceinline__ uint32_t half_block_word(uint32_t pos, uint32_t neg) { return word_of<0x00000f0fu>(pos, neg); }

}  // namespace
}  // namespace tern
