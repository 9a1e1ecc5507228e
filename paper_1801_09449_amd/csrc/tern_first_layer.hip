// First layer of a network on a scalar volume: Eq. 6 on the intensities and the layer's convolution, activation
// and re-packing in one launch, with the products on the matrix cores.
//
// A workgroup turns the intensities of a box of columns (x, y) into 4-bit codes, PLANES of a column to a record in
// LDS, and a record is an operand as it is: the codes of a column's planes are consecutive products of
// v_mfma_f32_32x32x64_f8f6f4, and the filter operand has the weights of the tap column at the planes that an
// output needs and zeros at the others.  Shallow kernels (KD = 1, 3): seven planes to a 32-bit record, nine tap
// columns in 63 of a step's 64 products, 8 - KD output planes from the same voxel operand with as many filter
// operands.  Stacks (KD = 15): sixteen planes to a record, four tap columns to a step, three steps.
// In-plane strides, dilations and paddings only move the columns that a lane reads.  Where taps lie so far apart that
// the box between them holds more columns than they read, each of three taps has a band of its own in LDS (FAR).
//
// What bounds it: intensities in, words out, and the decisions (three vector instructions per sum); gathering
// the taps bit by bit, as the vector units needed them, took most of the time of the kernels before.  Measured
// against those: 3x3x3 to 16 channels on 128 x 128 x 64 16.3 -> 9.9 us, 15x3x3 to 32 channels on one stack of
// 15 x 236 x 172 10.1 -> 6.4, on sixteen (gathered to memory, then convolved) 28.1 -> 16.  Far taps, in a box or
// gathered before: 3x3x3 to 64 channels with dilation 19 on 79 x 170 x 278 140 -> 53, 15x3x3 to 16 with dilation 19 on two
// stacks of 18 x 243 x 55 21.5 -> 8.7 (the kernel that gathered and convolved in one launch: 96 and 9.1).
#include <type_traits>

#include "tern_internal.h"
#include "tern_matrix_choice.h"
#include "tern_matrix_common.h"

namespace tern {
namespace {

constexpr int kFirstThreads = 256;       // four waves: two along x, two over rows
constexpr int kTileX = 64;               // output columns of a workgroup along x, 32 to a wave

struct FirstPlan {
    int32_t hx, cols;                    // columns along x and in all
    int32_t rows;                        // output rows of a wave
    Divisor tiles_x, tiles_y, tiles_z, hx_div;
    int32_t weights, cuts;               // LDS byte offsets: operands' parts and cut points
    // (FAR) an axis of the columns: extent of a tap's band (of all taps in one: more than there are), voxels between
    // neighbours in it, columns between neighbouring outputs and between neighbouring taps
    struct Axis {
        int32_t band, step, lane, tap;
    } x, y;
};

// FEW: at most 16 filters, the lower half of a block's rows.
// TOGETHER: all of a tile's planes without a branch between them, so that one's products run under another's decisions.
template <int KD, bool FEW, bool FAR, bool TOGETHER>
__global__ __launch_bounds__(kFirstThreads) void first_conv_kernel(FirstConvParams p, FirstPlan t)
{
    extern __shared__ __align__(16) uint8_t lds8[];
    constexpr bool STACK = KD > 7;
    constexpr int PLANES = STACK ? KD : 7;                 // input planes of a record
    constexpr int TZ = STACK ? 1 : 8 - KD;                 // output planes of a tile
    constexpr int TAPS = KD * 9, WORDS = (TAPS + 31) / 32;
    const int tid = threadIdx.x, lane = tid & 63, i32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int bid = blockIdx.x;
    {   // contiguous runs of tiles per XCD
        const int per_xcd = gridDim.x >> 3;
        if (bid < (per_xcd << 3)) bid = (bid & 7) * per_xcd + (bid >> 3);
    }
    const int row = quotient(bid, t.tiles_x), tix = bid - row * t.tiles_x.d;
    const int layer = quotient(row, t.tiles_y), tiy = row - layer * t.tiles_y.d;
    const int n = quotient(layer, t.tiles_z), tiz = layer - n * t.tiles_z.d;
    const int ox0 = tix * kTileX, oy0 = tiy * (2 * t.rows), oz0 = tiz * TZ;
    const int gx0 = ox0 * p.sw - p.pw, gy0 = oy0 * p.sh - p.ph, gz0 = oz0 - p.pd;

    // ---- this thread's share of the filters: tap column `col` of filter f, nibble a = tap plane a -------
    const int f = tid & 31;
    int fb = blockIdx.y;
    uint32_t wm[WORDS], ws[WORDS];
    int cut_lo, cut_hi;
    auto fetch_filters = [&]() {
#pragma unroll
        for (int q = 0; q < WORDS; ++q) {
            const v2u w = *reinterpret_cast<const v2u*>(p.wgt + ((size_t)q * p.co_pad + fb * 32 + f) * 2);
            wm[q] = w.x; ws[q] = w.y;
        }
        const int co = min(fb * 32 + f, p.c_out - 1);
        cut_lo = p.lo[co]; cut_hi = p.hi[co];
    };
    fetch_filters();
    const float lo = p.in_lo[0], hi = p.in_hi[0];

    // ---- intensities -> codes ---------------------------------------------------------------------------
    const size_t plane = (size_t)p.h * p.w;
    const float* src_n = p.src + (size_t)n * p.d * plane;
    constexpr int U = 2;                                   // columns that a thread has in flight (a stack's one: 6.4 us for 6.2)
    auto fill = [&](int base) {
        float v[U][PLANES];
        bool in_plane[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = min(base + u * kFirstThreads + tid, t.cols - 1);
            const int cy = quotient(e, t.hx_div), cx = e - cy * t.hx;
            int iy = gy0 + cy, ix = gx0 + cx;
            if constexpr (FAR) {
                const int by = (cy >= t.y.band) + (cy >= 2 * t.y.band), bx = (cx >= t.x.band) + (cx >= 2 * t.x.band);
                iy = gy0 + by * p.dh + (cy - by * t.y.band) * t.y.step;
                ix = gx0 + bx * p.dw + (cx - bx * t.x.band) * t.x.step;
            }
            in_plane[u] = (uint32_t)iy < (uint32_t)p.h && (uint32_t)ix < (uint32_t)p.w;
            const int off = in_plane[u] ? iy * p.w + ix : 0;
#pragma unroll
            for (int j = 0; j < PLANES; ++j) {
                const int iz = gz0 + j;                    // (planes outside the volume read plane 0)
                v[u][j] = src_n[((uint32_t)iz < (uint32_t)p.d ? (size_t)iz : 0) * plane + off];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = base + u * kFirstThreads + tid;
            uint32_t code[STACK ? 2 : 1];
#pragma unroll
            for (int k = 0; k < (STACK ? 2 : 1); ++k) code[k] = 0u;
#pragma unroll
            for (int j = PLANES - 1; j >= 0; --j) {
                uint32_t q = v[u][j] < lo ? 0xau : 0u;     // (false for NaN)
                q = v[u][j] > hi ? 0x2u : q;               // +1 wins should the cut points be crossed
                q = (uint32_t)(gz0 + j) < (uint32_t)p.d ? q : 0u;
                code[j >> 3] = (code[j >> 3] << 4) | q;
            }
            if (e < t.cols) {
                if constexpr (STACK) *reinterpret_cast<v2u*>(lds8 + e * 8) = in_plane[u] ? v2u{code[0], code[1]} : v2u{0u, 0u};
                else *reinterpret_cast<uint32_t*>(lds8 + e * 4) = in_plane[u] ? code[0] : 0u;
            }
        }
    };
    fill(0);

    // ---- filters and cut points -> LDS --------------------------------------------------------------------
    float* cuts = reinterpret_cast<float*>(lds8 + t.cuts);
    auto stage_filters = [&]() {
        // Column records: shallow [9][32] of 32 bits, stacks [12][32] of 64 bits (columns 9 .. 11 are zero).
        for (int col = tid >> 5; col < (STACK ? 12 : 9); col += kFirstThreads / 32) {
            uint32_t r[2] = {0u, 0u};
            if (col < 9) {
#pragma unroll
                for (int a = 0; a < KD; ++a) {
                    constexpr int kBits = 9;
                    const int q = (a * kBits) >> 5, sh = (a * kBits) & 31;
                    const uint32_t m = __builtin_amdgcn_alignbit(q + 1 < WORDS ? wm[q + 1 < WORDS ? q + 1 : q] : 0u, wm[q], sh) >> col;
                    const uint32_t s = __builtin_amdgcn_alignbit(q + 1 < WORDS ? ws[q + 1 < WORDS ? q + 1 : q] : 0u, ws[q], sh) >> col;
                    r[a >> 3] |= ((m & 1u) << 1 | (s & m & 1u) << 3) << (4 * (a & 7));
                }
            }
            if constexpr (STACK) *reinterpret_cast<v2u*>(lds8 + t.weights + (col * 32 + f) * 8) = v2u{r[0], r[1]};
            else *reinterpret_cast<uint32_t*>(lds8 + t.weights + (col * 32 + f) * 4) = r[0];
        }
        if (tid < 32) {
            const Cut cut = cut_of(cut_lo, cut_hi, fb * 32 + tid < p.c_out);
            cuts[tid] = cut.start;
            cuts[32 + tid] = cut.width;
        }
    };
    stage_filters();
    for (int base = U * kFirstThreads; base < t.cols; base += U * kFirstThreads) fill(base);
    __syncthreads();

    const bool active = ox0 + 32 * (wave & 1) < p.ow;
    const int x = 32 * (wave & 1) + i32, ox = ox0 + x;
    const int col_x = FAR ? min(x, p.ow - 1 - ox0) : x;    // (a narrow volume has no more columns)
    const int lane_x = FAR ? t.x.lane : p.sw, lane_y = FAR ? t.y.lane : p.sh, tap_x = FAR ? t.x.tap : p.dw, tap_y = FAR ? t.y.tap : p.dh;
    auto contract = [&]() {
        // ---- operands of the filters, start values ---------------------------------------------------------------
        constexpr int STEPS = STACK ? 3 : 1;
        v4i A[STACK ? STEPS : TZ];
        if constexpr (STACK) {
#pragma unroll
            for (int q = 0; q < STEPS; ++q) {
                const v2u a = *reinterpret_cast<const v2u*>(lds8 + t.weights + ((4 * q + 2 * g) * 32 + i32) * 8);
                const v2u b = *reinterpret_cast<const v2u*>(lds8 + t.weights + ((4 * q + 2 * g + 1) * 32 + i32) * 8);
                A[q] = v4i{(int)a.x, (int)a.y, (int)b.x, (int)b.y};
            }
        } else {
            // lanes 0-31: tap columns 0 .. 3 and, above their seven planes, planes 0 .. 3 of column 4; lanes 32-63:
            // columns 5 .. 8 and planes 4 .. 6 of column 4
            const uint32_t* w = reinterpret_cast<const uint32_t*>(lds8 + t.weights) + i32;
            const uint32_t w4 = w[4 * 32];
            uint32_t wc[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) wc[j] = w[(5 * g + j) * 32];
#pragma unroll
            for (int z = 0; z < TZ; ++z)
#pragma unroll
                for (int j = 0; j < 4; ++j) A[z][j] = (int)((wc[j] << (4 * z)) | (((w4 << (4 * z)) >> (4 * j + 16 * g)) << 28));
        }
        v16f start;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float4 h = *reinterpret_cast<const float4*>(cuts + 8 * k + 4 * g);
            start[4 * k] = h.x; start[4 * k + 1] = h.y; start[4 * k + 2] = h.z; start[4 * k + 3] = h.w;
        }
        const float* widths = cuts + 32 + 4 * g;

        // (a row of output can be more than 2^32 words)
        const size_t line = (size_t)p.ow * (2u * p.wd_out), slab = p.oh * line;
        auto decided = [&](const v16f& acc) {
            uint32_t pos, neg;
            decide_rows<FEW ? 2 : 4>(pos, neg, acc, widths);
            return FEW ? half_block_word(pos, neg) : block_word(pos, neg);
        };
        uint32_t* out = p.out_packed + ((size_t)n * p.od + oz0) * slab + (size_t)(oy0 + (wave >> 1) * t.rows) * line +
                        (size_t)ox * (2u * p.wd_out) + g * p.wd_out + fb;
        // columns of this lane's taps, LDS bytes from that of tap (0, 0)
        constexpr int REC = STACK ? 8 : 4;
        auto tap_col = [&](int col) { return ((col / 3) * tap_y * t.hx + (col % 3) * tap_x) * REC; };
        for (int r = 0; r < t.rows; ++r, out += line) {
            const int y = (wave >> 1) * t.rows + r, oy = oy0 + y;
            if (oy >= p.oh) break;
            const uint8_t* at = lds8 + (y * lane_y * t.hx + col_x * lane_x) * REC;
            if constexpr (STACK) {
                v16f acc = start;
#pragma unroll
                for (int q = 0; q < STEPS; ++q) {
                    // (columns past the ninth have zero weights: any codes do)
                    const int c0 = g ? min(4 * q + 2, 8) : 4 * q, c1 = g ? min(4 * q + 3, 8) : min(4 * q + 1, 8);
                    const v2u a = *reinterpret_cast<const v2u*>(at + tap_col(c0)), b = *reinterpret_cast<const v2u*>(at + tap_col(c1));
                    acc = multiply(A[q], v4i{(int)a.x, (int)a.y, (int)b.x, (int)b.y}, acc);
                }
                const uint32_t word = decided(acc);
                if (ox < p.ow) *out = word;
            } else {
                const uint32_t mid = *reinterpret_cast<const uint32_t*>(at + tap_col(4));
                v4i B;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t col = *reinterpret_cast<const uint32_t*>(at + (g ? tap_col(5 + j) : tap_col(j)));
                    B[j] = (int)(col | ((mid >> (4 * j + 16 * g)) << 28));
                }
                uint32_t* o = out;
                if (TOGETHER && oz0 + TZ <= p.od) {
                    uint32_t word[TZ];
#pragma unroll
                    for (int z = 0; z < TZ; ++z) word[z] = decided(multiply(A[z], B, start));
                    if (ox < p.ow) {
#pragma unroll
                        for (int z = 0; z < TZ; ++z, o += slab) *o = word[z];
                    }
                } else {
#pragma unroll
                    for (int z = 0; z < TZ; ++z, o += slab)
                        if (oz0 + z < p.od) {
                            const uint32_t word = decided(multiply(A[z], B, start));
                            if (ox < p.ow) *o = word;
                        }
                }
            }
        }
    };
    if constexpr (FAR && !FEW) {
        // all filters on the columns that are there, where the launch has tiles enough
        for (;;) {
            if (active) contract();
            fb += gridDim.y;
            if (fb * 32 >= p.c_out) break;
            fetch_filters();
            __syncthreads();
            stage_filters();
            __syncthreads();
        }
    } else {
        if (active) contract();
    }
}

// Columns of one axis: all between the first tap of the first output and the last of the last, or (far) three bands of
// one column to an output.
inline int64_t box_of(int outputs, int stride, int dil) { return (int64_t)(outputs - 1) * stride + 2 * (int64_t)dil + 1; }
inline int64_t axis_of(int outputs, int stride, int dil, bool far, FirstPlan::Axis& a)
{
    a.band = far ? outputs : 1 << 20;
    a.step = far ? stride : 1;
    a.lane = far ? 1 : stride;
    a.tap = far ? outputs : dil;
    return far ? 3 * outputs : box_of(outputs, stride, dil);
}

template <int KD>
void plan_first(const FirstConvParams& p, FirstPlan& t, bool& far, dim3& grid, size_t& lds)
{
    constexpr bool STACK = KD > 7;
    constexpr int TZ = STACK ? 1 : 8 - KD, REC = STACK ? 8 : 4;
    const int64_t tx = cdiv(p.ow, kTileX), tz = cdiv(p.od, TZ);
    // Bands where they are fewer by a quarter: a box's lines come whole, and bands read them up to three times (a stack
    // with steps of three and dilation 3: 196 columns in a box, 192 in bands, 17 and 21 us).  At most 256 columns in a row and
    // eight rows to a row of outputs, so that four outputs' records, or two's, are within 16 KB (stacks: 32).
    const int wide = p.ow < kTileX ? p.ow : kTileX;
    const bool far_x = box_of(wide, p.sw, p.dw) > 4 * wide;
    int64_t hx, hy, tiles;
    for (t.rows = 4;; t.rows >>= 1) {
        const bool far_y = box_of(2 * t.rows, p.sh, p.dh) > 8 * t.rows;
        far = box_of(kTileX, p.sw, p.dw) > 4 * kTileX || far_y;
        hx = axis_of(far ? wide : kTileX, p.sw, p.dw, far && far_x, t.x);
        hy = axis_of(2 * t.rows, p.sh, p.dh, far_y, t.y);
        tiles = tx * cdiv(p.oh, 2 * t.rows) * tz * p.n;    // at most the voxels
        // two workgroups per compute unit
        if (t.rows == 1 || (hx * hy <= 4096 && tiles >= 512)) break;
    }
    t.hx = (int32_t)hx;
    t.cols = (int32_t)(hx * hy);
    t.hx_div = divisor(t.hx);
    t.tiles_x = divisor((int32_t)tx);
    t.tiles_y = divisor(cdiv(p.oh, 2 * t.rows));
    t.tiles_z = divisor((int32_t)tz);
    t.weights = (t.cols * REC + 15) & ~15;
    t.cuts = t.weights + (STACK ? 12 * 32 * 8 : 9 * 32 * 4);
    lds = (size_t)t.cuts + 64 * sizeof(float);
    grid = dim3((unsigned)tiles, far && tiles >= 512 ? 1u : (unsigned)cdiv(p.c_out, 32));
}

template <int KD>
void launch_first(const FirstConvParams& p, hipStream_t s)
{
    FirstPlan t;
    bool far;
    dim3 grid;
    size_t lds;
    plan_first<KD>(p, t, far, grid, lds);
    const auto go = [&](auto few, auto apart, auto together) {
        hipLaunchKernelGGL((first_conv_kernel<KD, decltype(few)::value, decltype(apart)::value, decltype(together)::value>), grid, dim3(kFirstThreads), lds, s, p, t);
    };
    const std::true_type yes;
    const std::false_type no;
    const auto apart = [&](auto few, auto together) { far ? go(few, yes, together) : go(few, no, together); };
    if constexpr (KD == 15) {
        p.c_out <= 16 ? apart(yes, no) : apart(no, no);
    } else {
        // A tile's planes together take the registers of a fifth wave of a SIMD (3x3x3: 104 to 112 of them, 92 to 96 without; single
        // planes have four waves either way; far taps with more than 16 filters up to 1.15 times as long together).  So they are
        // where the launch takes no more rounds of four workgroups per compute unit than of five, and, beyond one
        // round, with up to three words of filters, whose stores come that close together: 3x3x3 to 256 channels on
        // 4 x 30 x 55 x 16 19.2 us by planes and 20.8 together, to 128 on 2 x 40 x 57 x 67 19.9 and 21.8; to 64 on 56 x 155 x 165 25.1
        // and 22.7, to 32 on 2 x 33 x 29 x 22 6.4 and 6.1.
        const int64_t wgs = (int64_t)grid.x * grid.y;
        const bool together = KD == 1 || wgs <= 1024 || (p.wd_out <= 3 && (wgs + 1023) / 1024 == (wgs + 1279) / 1280);
        const std::bool_constant<KD == 1> by_planes;           // (no such form of single planes)
        if (p.c_out <= 16) together ? apart(yes, yes) : apart(yes, by_planes);
        else if (far) go(no, yes, no);
        else together ? go(no, no, yes) : go(no, no, by_planes);
    }
}

}  // namespace

// One-channel input, 3 x 3 in the plane by 1, 3 or 15 planes, unit depth stride and dilation.  (The further limits
// decide between workspace layouts of tern_fcn_forward and tern_net_forward.)
bool first_conv_applies(int32_t c_in, const tern_conv_geom& g, const tern_dims& out)
{
    if (c_in != 1 || g.k[1] != 3 || g.k[2] != 3 || g.stride[0] != 1 || g.dil[0] != 1) return false;
    if (g.k[0] != 1 && g.k[0] != 3 && g.k[0] != 15) return false;
    const int planes = g.k[0] == 15 ? 1 : 8;
    return (int64_t)cdiv(out.d, planes) * out.n <= 65535 && cdiv(out.h, 4) <= 65535;
}

int launch_first_conv(const FirstConvParams& p, hipStream_t s)
{
    if (p.kd == 1) launch_first<1>(p, s);
    else if (p.kd == 3) launch_first<3>(p, s);
    else launch_first<15>(p, s);
    TERN_HIP_CHECK(hipGetLastError());
    return TERN_OK;
}

}  // namespace tern
