// Pointwise ternary convolution for gfx950: a 1x1x1 kernel with unit stride and no padding
// (paper section 2, Eq. 9; the 1x1 rows of Table 1).
//
// An output voxel depends on one input voxel only, so there is no halo, no LDS and no barrier: the volume
// is a flat list of voxels.  A wave holds the filters of 32 NB channels in registers, widened to 4-bit
// floats once, and their cut points; it walks blocks of 32 voxels, each fetched from global memory straight
// into the matrix instruction's lanes (a block's records are one contiguous run: lanes 0-31 take the mask
// words of a voxel's word pair, lanes 32-63 the sign words, and one half-wave swap sorts them), four
// blocks ahead of their use (two blocks ahead, cut points in registers instead of LDS and accumulators that
// the compiler put into accumulation registers: 21 us where this takes 12).  Bound by memory where the
// output is int32, by the decisions on the sums where it is packed (through 6-bit floats in large launches: with three
// vector instructions to a sum 64 -> 64 channels on 96^3 took 11.1 us, now 9.8).  Measured
// against one lane per voxel with bit counts: 64 -> 64 channels on 96^3 24.5 -> 9.8 us packed (28 MB,
// 2.9 TB/s) and 39.0 -> 36.9 us int32 (6.5 TB/s), 128 -> 128 on 64^3 22.0 -> 8.9, 256 -> 256 on 609
// voxels 9.2 -> 2.9, 32 -> 32 on 64^3 4.7 -> 3.9.
#include <type_traits>

#include "tern_internal.h"
#include "tern_matrix_common.h"
#include "tern_point_choice.h"

namespace tern {
namespace {

constexpr int kPointThreads = 64 * kPointWaves;

struct PointParams {
    const uint32_t* in;      // packed [voxels][2][wd] (batch items folded for packed output)
    const uint32_t* wgt;     // filter bank [words or pairs][co_pad][2][wc]; binary: [..][co_pad][wc]
    const int32_t* lo;
    const int32_t* hi;
    int32_t* out_acc;        // [n][c_out][voxels] or null
    uint32_t* out_packed;    // [voxels][2][wd_out] or null
    int32_t voxels;          // per grid.z slice
    int32_t blocks_per_wave;
    int32_t c_out, wd_out, co_pad;
};

// S: steps of 64 channels (word pairs); ODD: an odd number of words per voxel (the last pair is half
// empty, bank and records are read word by word); BIN: sign-only filters; OUT: int32 sums, packed codes shifted
// in one by one, or packed codes through 6-bit floats.
enum { kSums = 0, kShifted = 1, kSix = 2 };
template <int S, int NB, int OUT, bool BIN, bool ODD>
__global__ __launch_bounds__(kPointThreads) __attribute__((amdgpu_waves_per_eu(3))) void conv_point_kernel(PointParams p)
{
    constexpr bool PACKED = OUT != kSums, SIX = OUT == kSix;
    constexpr int WD = ODD ? 2 * S - 1 : 2 * S;
    constexpr int REC = 2 * WD;                          // words of a voxel record
    const int lane = threadIdx.x & 63, i32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int blocks = (int)(((uint32_t)p.voxels + 31u) >> 5);
    const int c0 = blockIdx.y * (32 * NB);
    const uint32_t* in_n = p.in + (size_t)blockIdx.z * (size_t)p.voxels * REC;
    // cut points of the workgroup's filters: start values, then widths
    __shared__ __align__(16) float cuts[PACKED ? 64 * NB : 4];
    if constexpr (PACKED) {
        if (threadIdx.x < 32 * NB) {
            const int co = c0 + (int)threadIdx.x;
            const bool live = co < p.c_out;
            const Cut c = cut_of(live ? p.lo[co] : 0, live ? p.hi[co] : 0, live);
            const int at = SIX ? ((int)threadIdx.x & ~31) + filter_row((int)threadIdx.x & 31) : (int)threadIdx.x;
            cuts[at] = c.start;
            cuts[32 * NB + at] = c.width;
        }
    }
    const int64_t first64 = ((int64_t)blockIdx.x * (kPointThreads / 64) + wave) * p.blocks_per_wave;
    const int first = (int)min(first64, (int64_t)blocks);
    const int last = min(blocks, first + p.blocks_per_wave) - 1;   // before first: nothing to do

    uint32_t m33 = 0x33333333u, maa = 0xaaaaaaaau;
    asm volatile("" : "+v"(m33), "+v"(maa));

    // One block's words, (mask, sign) per step once sorted.  Voxels past the end repeat the last one.
    auto fetch = [&](v2u (&x)[S], int b) {
        const int v0 = b * 32;
        const uint32_t lane_v = (uint32_t)min(i32, p.voxels - 1 - v0);
        const uint32_t* src = in_n + (size_t)v0 * REC + lane_v * REC;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if constexpr (!ODD) {
                x[s] = *reinterpret_cast<const v2u*>(src + g * WD + 2 * s);
            } else {
                const bool live = 2 * s + 1 < WD || g == 0;
                const int q = live ? 2 * s + g : 2 * s;
                x[s].x = src[q];
                x[s].y = src[WD + q];
                if (!live) x[s].x = x[s].y = 0u;
            }
        }
    };
    // Past the end of a wave's run the last block is fetched again, except word by word (three, five and seven
    // words): there each load touches 32 lines, and short runs spent their time on repeats (7 words -> 256
    // channels on 14 208 voxels 12.5 -> 6.7 us).  Elsewhere the branch costs more than the loads (1 word -> 256
    // channels on 196 608 voxels 10.6 us, 12.6 with it; 8 words on 53 350 12.0 and 13.0).
    constexpr int AHEAD = 4;
    auto fetch_within = [&](v2u (&x)[S], int b) {
        if constexpr (!ODD || S == 1) fetch(x, max(0, min(b, last)));
        else if (b <= last) fetch(x, b);
    };
    v2u x[AHEAD][S];
#pragma unroll
    for (int k = 0; k < AHEAD; ++k)
        fetch_within(x[k], first + k);

    // ---- filters and cut points ----------------------------------------------------------------
    v4i F[NB][S];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int co = c0 + nb * 32 + (SIX ? row_filter(i32) : i32);   // below co_pad: whole blocks of 32 exist
#pragma unroll
        for (int s = 0; s < S; ++s) {
            v2u w;
            if constexpr (!ODD) {
                const uint32_t* row = p.wgt + (size_t)s * p.co_pad * (BIN ? 2 : 4);
                if constexpr (BIN) {
                    w.y = row[co * 2 + g];
                } else {
                    const v2u r = *reinterpret_cast<const v2u*>(row + co * 4 + 2 * g);
                    const auto sw = __builtin_amdgcn_permlane32_swap(r.x, r.y, false, false);
                    w.x = sw[0]; w.y = sw[1];
                }
            } else {
                const int q = min(2 * s + g, WD - 1);     // (past the end: any word, the voxel's is zero)
                if constexpr (BIN) w.y = p.wgt[((size_t)q * p.co_pad + co)];
                else w = *reinterpret_cast<const v2u*>(p.wgt + ((size_t)q * p.co_pad + co) * 2);
            }
            if constexpr (BIN) w.x = 0xffffffffu;
            F[nb][s] = expand(interleave(w.x, w.y, m33), maa);
        }
    }
    if constexpr (PACKED) __syncthreads();
    if (first > last) return;
    v16f start[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float4 h = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if constexpr (PACKED) h = *reinterpret_cast<const float4*>(cuts + nb * 32 + 8 * k + 4 * g);
            start[nb][4 * k] = h.x; start[nb][4 * k + 1] = h.y; start[nb][4 * k + 2] = h.z; start[nb][4 * k + 3] = h.w;
        }

    Decider d;
    v8bf widths[NB];
    if constexpr (SIX) {
        d = decider();
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) widths[nb] = width_operand(cuts[32 * NB + nb * 32 + i32], g == 0);
    }

    // ---- blocks of 32 voxels -------------------------------------------------------------------
    auto block = [&](v2u (&x)[S], int b) {
        v4i V[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if constexpr (ODD) {
                V[s] = expand(interleave(x[s].x, x[s].y, m33), maa);
            } else {
                const auto sw = __builtin_amdgcn_permlane32_swap(x[s].x, x[s].y, false, false);
                V[s] = expand(interleave(sw[0], sw[1], m33), maa);
            }
        }
        fetch_within(x, b + AHEAD);
        v16f acc[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            acc[nb] = multiply(F[nb][0], V[0], start[nb]);
#pragma unroll
            for (int s = 1; s < S; ++s) acc[nb] = multiply(F[nb][s], V[s], acc[nb]);
        }
        const int vox = b * 32 + i32;
        if constexpr (PACKED) {
            uint32_t word[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if constexpr (SIX) {
                    word[nb] = decided_word(acc[nb], widths[nb], d);
                } else {
                    uint32_t pos, neg;
                    decide_block(pos, neg, acc[nb], cuts + 32 * NB + nb * 32 + 4 * g);
                    word[nb] = block_word(pos, neg);
                }
            }
            if (vox < p.voxels) {
                uint32_t* o = p.out_packed + ((size_t)(b * 32) * 2u + (uint32_t)(i32 * 2)) * p.wd_out + g * p.wd_out + (c0 >> 5);
                if (NB == 2 && (p.wd_out & 1) == 0) {
                    *reinterpret_cast<v2u*>(o) = v2u{word[0], word[NB - 1]};
                } else {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        if (c0 + nb * 32 < p.c_out) o[nb] = word[nb];
                }
            }
        } else {
            if (vox < p.voxels) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int cb = c0 + nb * 32 + 4 * g;
                    int32_t* o = p.out_acc + ((size_t)blockIdx.z * p.c_out + cb) * (size_t)p.voxels + vox;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int dc = (v >> 2) * 8 + (v & 3);
                        if (cb + dc < p.c_out) o[(size_t)dc * p.voxels] = (int32_t)acc[nb][v];
                    }
                }
            }
        }
    };
    for (int b = first; b <= last; b += AHEAD) {
#pragma unroll
        for (int k = 0; k < AHEAD; ++k)
            if (b + k <= last) block(x[k], b + k);
    }
}

template <int S, int NB, bool ODD>
void launch_blocks(const PointParams& p, int out, bool binary, dim3 grid, hipStream_t s)
{
    const auto go = [&](auto o, auto bin) {
        hipLaunchKernelGGL((conv_point_kernel<S, NB, decltype(o)::value, decltype(bin)::value, ODD>), grid, dim3(kPointThreads), 0, s, p);
    };
    const auto with = [&](auto o) { binary ? go(o, std::true_type{}) : go(o, std::false_type{}); };
    if (out == kSums) return with(std::integral_constant<int, kSums>{});
    if (out == kSix) return with(std::integral_constant<int, kSix>{});
    with(std::integral_constant<int, kShifted>{});
}

template <int S, bool ODD>
void launch_steps(const PointParams& p, int out, bool binary, int nb, dim3 grid, hipStream_t s)
{
    if constexpr (S <= 2)                                // (two filter blocks to a wave: up to four words)
        if (nb == 2) return launch_blocks<S, 2, ODD>(p, out, binary, grid, s);
    launch_blocks<S, 1, ODD>(p, out, binary, grid, s);
}

}  // namespace

// Up to eight words per voxel (the filters of a wave stay in registers) and, with several taps' worth of
// channels packed into a word (c_in <= 16), never: a single tap has a plain bank.  int32 output has a grid
// layer per batch item: batches beyond the grid's 65535 layers go through the tiled kernel.
bool conv_point_applies(const ConvParams& p)
{
    if (!p.out_packed && p.n > 65535) return false;
    if (p.kd * p.kh * p.kw != 1) return false;
    if (p.sd != 1 || p.sh != 1 || p.sw != 1 || p.pd != 0 || p.ph != 0 || p.pw != 0) return false;
    return p.tp_slots == 0 && p.wd_in <= 8;
}

int launch_conv_point(const ConvParams& c, hipStream_t s)
{
    const bool packed = c.out_packed != nullptr;
    PointParams p;
    p.in = c.in; p.wgt = c.wgt; p.lo = c.lo; p.hi = c.hi;
    p.out_acc = c.out_acc; p.out_packed = c.out_packed;
    // packed output: batch items are just more voxels; int32 output keeps them apart (grid.z)
    const int64_t voxels = (int64_t)c.d * c.h * c.w * (packed ? c.n : 1);
    const int gz = packed ? 1 : c.n;
    p.voxels = (int32_t)voxels;                          // at most 2^31 - 1 per tensor
    p.c_out = c.c_out; p.wd_out = c.wd_out; p.co_pad = c.co_pad;
    const PointLaunch l = point_launch(voxels, gz, c.c_out, c.wd_in, packed);
    if (l.groups > 65535) return TERN_ESHAPE;
    p.blocks_per_wave = l.blocks_per_wave;
    const dim3 grid((unsigned)l.gx, (unsigned)l.groups, (unsigned)gz);
    const int out = !packed ? kSums : l.six ? kSix : kShifted;
    switch (c.wd_in) {
        case 1: launch_steps<1, true>(p, out, c.binary != 0, l.nb, grid, s); break;
        case 2: launch_steps<1, false>(p, out, c.binary != 0, l.nb, grid, s); break;
        case 3: launch_steps<2, true>(p, out, c.binary != 0, l.nb, grid, s); break;
        case 4: launch_steps<2, false>(p, out, c.binary != 0, l.nb, grid, s); break;
        case 5: launch_steps<3, true>(p, out, c.binary != 0, l.nb, grid, s); break;
        case 6: launch_steps<3, false>(p, out, c.binary != 0, l.nb, grid, s); break;
        case 7: launch_steps<4, true>(p, out, c.binary != 0, l.nb, grid, s); break;
        default: launch_steps<4, false>(p, out, c.binary != 0, l.nb, grid, s); break;
    }
    TERN_HIP_CHECK(hipGetLastError());
    return TERN_OK;
}

}  // namespace tern
