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

__device__ __forceinline__ void decide_block(uint32_t& pos, uint32_t& neg, const v16f& acc, const float* widths)
{
    decide_rows<4>(pos, neg, acc, widths);
}

// The same decisions with fewer vector instructions, for kernels whose time they are.  A SIMD takes 4.1 cycles for a
// shift-in and 2.1 for an addition (register-only loops), 10.3 for a sum's three instructions above; one
// v_cvt_scalef32_2xpk16_fp6_f32 turns 32 floats into 6-bit ones, signs and all, in 66, and the additions are one
// matrix instruction.  The 6-bit floats lie in a row, a sum's two decisions next to each other, six bits apart over
// six words, so that two selections by bits collect them, in an order that is the filters': row r of a block is
// filter row_filter(r).
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef uint32_t v6u __attribute__((ext_vector_type(6)));

// Register i of the lanes of half g holds row 8 (i / 4) + 4 g + i % 4; its first decision ends up at bit 5 + 12 i
// modulo 32 (one lower from i = 8 on), the second six higher, and half 1 goes two higher, into the gaps.
__device__ __forceinline__ int row_filter(int row)
{
    const int i = 4 * (row >> 3) + (row & 3), g = (row >> 2) & 1;
    return ((5 + 12 * (i & 7)) & 31) - (i >> 3) + 2 * g;
}
__device__ __forceinline__ int filter_row(int filter)
{
    const int g = (filter >> 1) & 1, high = ~filter & 1, m = filter >> 2;
    const int i = ((3 * m + 5) & 7) + 8 * high;
    return 8 * (i >> 2) + 4 * g + (i & 3);
}

struct Decider {
    uint32_t first, third, odd;      // bits that hold decisions in words 0 and 2 (of three), odd bits
    v8bf ones;
};
__device__ __forceinline__ Decider decider()
{
    Decider d = {0x20820820u, 0x82082082u, 0xaaaaaaaau, {}};
    v4u one = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    asm volatile("" : "+v"(d.first), "+v"(d.third), "+v"(d.odd), "+v"(one));
    d.ones = __builtin_bit_cast(v8bf, one);
    return d;
}
// A row's width as three bf16 numbers (at most 23 bits: exactly), the rows' operand of the additions.
__device__ __forceinline__ v8bf width_operand(float w, bool lower_half)
{
    const uint32_t hi = __float_as_uint(w) & 0xffff0000u;
    const float rest = w - __uint_as_float(hi);
    const uint32_t mid = __float_as_uint(rest) & 0xffff0000u;
    const uint32_t low = __float_as_uint(rest - __uint_as_float(mid));
    const v4u o = {lower_half ? (hi >> 16) | mid : 0u, lower_half ? low >> 16 : 0u, 0u, 0u};
    return __builtin_bit_cast(v8bf, o);
}
// acc as for decide(): a block's packed words, lane = voxel l % 32, mask words in lanes 0-31, sign words in 32-63.
__device__ __forceinline__ uint32_t decided_word(const v16f& acc, v8bf widths, const Decider& d)
{
    const v16f below = __builtin_amdgcn_mfma_f32_32x32x16_bf16(widths, d.ones, acc, 0, 0, 0);
    // Sums are halves and never 0: a 6-bit float keeps the sign.  (The instruction writes before it has read all.)
    v6u c = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(acc, below, 1.0f);
    asm volatile("" : "+v"(c) : "v"(acc), "v"(below));
    const uint32_t a = __builtin_amdgcn_bitop3_b32(d.third, c[2], __builtin_amdgcn_bitop3_b32(d.first, c[0], c[1], 0xca), 0xca);
    const uint32_t b = __builtin_amdgcn_bitop3_b32(d.third, c[5], __builtin_amdgcn_bitop3_b32(d.first, c[3], c[4], 0xca), 0xca);
    const uint32_t z = __builtin_amdgcn_bitop3_b32(d.odd, a, b >> 1, 0xca);
    const uint32_t neg = __builtin_amdgcn_alignbit(z, z, 6);
    const uint32_t m = __builtin_amdgcn_bitop3_b32(z, neg, 0x33333333u, 0x8a);
    const uint32_t s = __builtin_amdgcn_bitop3_b32(z, neg, 0x33333333u, 0x80);
    const auto sw = __builtin_amdgcn_permlane32_swap(m, s, false, false);
    return sw[0] | (sw[1] << 2);
}

}  // namespace
}  // namespace tern
