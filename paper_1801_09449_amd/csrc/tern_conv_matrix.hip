// Tiled ternary convolution with the inner product taken by the matrix instructions.  Same packed
// activations, same filter banks, same halo tiles in LDS and the same integers as the bit-count kernels
// (tern_conv_tiled.hip); what differs is the unit that contracts.  A ternary code is the 4-bit float
// +1 = 0010, -1 = 1010 or 0 = x000, and v_mfma_f32_32x32x64_f8f6f4 takes 32 filters x 32 voxels x 64
// channels of them in 32 cycles of a SIMD: 32 products per lane and cycle, against 32 per four vector
// instructions (12 cycles at best) of the masked-Hamming step.  Sums are floats and exact: every partial
// sum is an integer, or an integer and a half, far below 2^23.
//
// Rows of the product are filters, columns are voxels, so that in the result a lane holds 16 filters of
// one voxel and re-packing is shifts within the lane.  A wave owns VB blocks of 32 voxels (a box of the
// output) x NB blocks of 32 filters and walks the kernel taps and channel words in bank order, 64
// channels per step: lanes 0-31 hold the step's first word (or, where a voxel has an odd number of
// words, its first (tap, word) entry), lanes 32-63 its second.
//
// What bounds it: beside a matrix instruction a SIMD has room for about four vector instructions (a
// register-only loop: 32.7 cycles per matrix instruction with none, 33.8 with four, 42 with eight, 53
// with twelve), so the 2-bit codes must not be widened where they are used most.  Voxels are widened once,
// on their way into LDS (16 bytes per word and voxel, a 16-byte read per operand; with 8-byte records
// widened behind the read the same launches took 6-14 % longer).  Filter words come from the bank as bits
// and are widened per wave and step, ten instructions for a block that VB matrix instructions use; VB = 4
// with NB = 2 leaves three vector instructions per matrix instruction and uses all registers (two waves
// per SIMD).  Small launches, where a wave's chain of steps is what takes the time, split a tile's steps
// over two to eight waves that add their sums in LDS (exact, so in any order): 512 -> 256 channels 3 x 3 on
// 52 x 36 13.0 -> 8.7 us, 256 -> 256 on 16^3 17.7 -> 10.1, 32 -> 32 on 24^3 7.2 -> 5.9.  Under full load the
// clock falls to 1.9 GHz, where 32 cycles are 8 000 TFLOP/s for the chip.
// A step is to be its loads, its widening and its matrix instructions and nothing else: tap offsets lie ready in a
// register's lanes, bank rows come through a descriptor whose end stands for the last row's absent partner, and no branch
// stands around a load.  With a scalar walk over taps and words, its branches, clamped row numbers and bank words two steps
// ahead a small wave's step took 470 cycles, now 230 (32 -> 32 on 24^3: 5.0 -> 4.3 us; 96 -> 70 stride 2 on 2 x 45 x 53 x 37
// 12.6 -> 11.1; a six-layer encoder 39.1 -> 35.6).
// What stands in front of the first matrix instruction counts for a launch of 5 to 9 us: workgroup and wave numbers
// are divided by multiplication (ten integer divisions were 250 instructions before the first load), cut points
// and halo items are fetched at once, and halo voxels go through a buffer descriptor that returns zeros outside the
// volume.  Together: 32 -> 32 on 24^3 5.46 -> 4.99 us, 96 -> 70 stride 2 on 2 x 45 x 53 x 37 13.9 -> 12.5, 64 -> 64
// on 96^3 with dilation 2 53.8 -> 51.5, a U-Net's eighteen launches 125.6 -> 113.3.  A wave by itself issues an instruction,
// scalar or vector, every 2.4 ns, and the halo voxels arrive 0.1 to 0.4 us after the last of their loads, which 250
// instructions stood in front of: strides and counts come ready from the host, and bank rows, cut points and operands' places
// are fetched and computed behind those loads.  64 -> 64 3 x 3 on 232 x 168 4.71 -> 4.49 us, on sixteen planes
// 17.3 -> 16.5, a U-Net on one stack 81.0 -> 78.9.  (Coordinates stepped with carries instead of divisions, records of up to
// four words to a load: shorter per voxel, longer in front of the first, 32 -> 32 on 24^3 4.23 -> 4.69 us.)
// Measured, fused output, bit-count kernels before: 64 -> 64 channels on 64^3: 88 -> 13.2 us, on 96^3 with
// dilation 2: 276 -> 43 us; 256 -> 256 on 2 x 32^3: 321 -> 42 us (5 500 TFLOP/s: loop 38, fill 3, epilogue 1 us);
// 64 -> 64 3 x 3 on 16 planes of 232 x 168: 83 -> 15.7 us.
#include <type_traits>

#include "tern_internal.h"
#include "tern_matrix_choice.h"
#include "tern_matrix_common.h"

namespace tern {
namespace {

// Where a tile's words come from when the input lies in two tensors (ConvPair): byte offsets from the first
// of the two in memory.
struct PairPlan {
    const uint32_t* base;
    uint32_t reach;                  // bytes from there to the end of both
    uint32_t start[2], item[2];      // first byte, bytes per batch item
    uint32_t line[2], rec[2];        // bytes per row and per voxel
    int32_t h[2];
    int32_t up[2][3], first[2][3];
    int32_t nch0;                    // word pairs of source 0
};

struct MatrixPlan {
    int32_t lxb, lyb;                // a wave's voxels: 2^lxb x 2^lyb x the rest
    int32_t lwy, lwz, nwc;           // waves of a workgroup along y and z (log2) and over filter groups
    int32_t lks;                     // waves that share a tile's steps and add up their sums in LDS (log2)
    int32_t hx, hy, hz;              // halo extents in voxels
    Divisor tiles_x, tiles_y, tiles_z;
    int32_t threads, tiles;          // of a workgroup, of the launch
    uint32_t reach;                  // bytes of input, or of its part from a tile's first plane to its last (FAR: its rows of a plane)
    int32_t whole;                   // all of the input
    uint32_t rec, line, slice, item; // input bytes of a voxel, a row, a plane, a batch item (item: if whole)
    int32_t nch;                     // words (or word pairs) per voxel
    int32_t rows, row_bytes;         // of the filter bank
    int32_t plane, items;            // voxels of a plane of the halo tile, units of its fill
    int32_t pl;                      // LDS bytes of one word plane
    int32_t zero_off;                // LDS byte offset of a zero record (odd word counts)
    int32_t tp_log;                  // tap-packed bank: log2 of the taps per row
    int32_t cut_off;                 // LDS byte offset of the staged cut points
    Reciprocal r_hx, r_pl, r_ch, r_kw, r_kh, r_nch, r_nwc;
    PairPlan pair;                   // (kPair)
};

// What the words are: ternary or binary (sign-only) filter banks, two-digit activations, or the tap-packed
// bank of up to 16 input channels (several taps share a filter word; here each tap is a word of its own), or
// ternary banks with the activations in two tensors (an upsampled one and a cropped one behind it: joining
// them in memory first took a launch of 4 us at 15 to 90 thousand voxels and 12 to 13 us at sixteen times as many).
enum { kTernary = 0, kBinary = 1, kDigits = 2, kTapPacked = 3, kPair = 4 };


// Two balanced-ternary digits per value (low + 3 high, -4 .. 4) to the E2M1 code of the value
// (magnitudes 1, 2, 3, 4 = 0010, 0100, 0101, 0110), channels in the order of expand().
__device__ __forceinline__ v4i expand_digits(uint32_t lm, uint32_t hm, uint32_t ls, uint32_t hs)
{
    const uint32_t b3 = (hm & hs) | (lm & ls & ~hm);
    const uint32_t b2 = hm;
    const uint32_t b1 = lm & ~(hm & (ls ^ hs));
    const uint32_t b0 = hm & ~lm;
    v4i o;
    o.x = (int)((b0 & 0x11111111u) | ((b1 << 1) & 0x22222222u) | ((b2 << 2) & 0x44444444u) | ((b3 << 3) & 0x88888888u));
    o.y = (int)(((b0 >> 1) & 0x11111111u) | (b1 & 0x22222222u) | ((b2 << 1) & 0x44444444u) | ((b3 << 2) & 0x88888888u));
    o.z = (int)(((b0 >> 2) & 0x11111111u) | ((b1 >> 1) & 0x22222222u) | (b2 & 0x44444444u) | ((b3 << 1) & 0x88888888u));
    o.w = (int)(((b0 >> 3) & 0x11111111u) | ((b1 >> 2) & 0x22222222u) | ((b2 >> 1) & 0x44444444u) | (b3 & 0x88888888u));
    return o;
}

// FAR: a tile's planes together, or the filter bank, span more than 4 GB: a buffer descriptor takes the tile's rows of one plane
// at a time, and bank rows are read by 64-bit addresses.
template <int VB, int NB, bool PACKED, int KIND, bool ODD, bool SPLIT, bool FAR>
__global__ __launch_bounds__(512) void conv_matrix_kernel(ConvParams p, MatrixPlan t)
{
    extern __shared__ __align__(16) uint8_t lds8[];
    const int tid = threadIdx.x;
    const int nthreads = t.threads;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int bid = blockIdx.x;
    {   // contiguous runs of tiles per XCD (workgroups go to the 8 XCDs round-robin)
        const int per_xcd = t.tiles >> 3;
        if (bid < (per_xcd << 3)) bid = (bid & 7) * per_xcd + (bid >> 3);
    }
    const int row = quotient(bid, t.tiles_x), tix = bid - row * t.tiles_x.d;
    const int layer = quotient(row, t.tiles_y), tiy = row - layer * t.tiles_y.d;
    const int n = quotient(layer, t.tiles_z), tiz = layer - n * t.tiles_z.d;
    const int X = 1 << t.lxb, Y = 1 << t.lyb, Z = (32 * VB) >> (t.lxb + t.lyb);
    const int ox0 = tix << t.lxb, oy0 = tiy << (t.lyb + t.lwy), oz0 = tiz * (Z << t.lwz);
    const int lks = SPLIT ? t.lks : 0, nks = 1 << lks;
    const int ks = wave & (nks - 1), wtile = wave >> lks;
    const int wsp = (int)quotient((uint32_t)wtile, t.r_nwc), wc = wtile - wsp * t.nwc;
    const int wy = wsp & ((1 << t.lwy) - 1), wz = wsp >> t.lwy;
    const int cb = (blockIdx.y * t.nwc + wc) * (32 * NB);   // first filter of this wave
    const bool active = cb < p.c_out;

    const int i32 = lane & 31, g = lane >> 5;
    constexpr int REC = 16;                                 // LDS bytes per word and voxel: 32 four-bit floats
    static_assert(KIND != kTapPacked || ODD, "one word per voxel");
    constexpr bool ROWS = (ODD || KIND == kDigits) && KIND != kTapPacked;           // the lane groups read different bank rows
    const int plane = t.plane;

    // ---- filter words ------------------------------------------------------------------------
    constexpr int FW = KIND == kDigits ? 4 : KIND == kBinary ? (ODD ? 1 : 2) : (ODD ? 2 : 4);  // words per filter and row
    const int row_bytes = t.row_bytes;
    const int entries = p.kd * p.kh * p.kw * (KIND == kDigits && !ODD ? t.nch >> 1 : t.nch);     // (tap, word or pair of words)
    const int all_steps = ODD ? (entries + 1) >> 1 : entries;
    // this wave's steps: first .. first + steps - 1
    const int first = (all_steps * ks) >> lks;
    const int steps = ((all_steps * (ks + 1)) >> lks) - first;
    // (odd numbers of entries) a last entry without a partner, under one's filters unless those can be zeros
    const bool half_last = ODD && (KIND == kBinary || FAR) && ks == nks - 1 && (entries & 1) != 0;
    // Which way the sums are decided: through the 6-bit floats where the instructions count, shifted in one by one in
    // the small waves of short launches, where only a wave's own time does (a U-Net's fifteen launches on one stack
    // 86.3 us, through the 6-bit floats 87.6).
    constexpr bool SIX = PACKED && VB == 4;
    uint32_t lane_f = (uint32_t)((SIX ? row_filter(i32) : i32) * FW * 4);
    if constexpr (ROWS) lane_f += (uint32_t)(g * row_bytes);
    else if constexpr (KIND != kTapPacked) lane_f += (uint32_t)(KIND == kBinary ? 4 * g : 8 * g);
    // Steps whose words are under way at once.  Their loads stand between those of the halo tile and its words, and take
    // registers: six steps of one filter block leave a small wave 80, six waves to a SIMD (two-tensor inputs: 82, five).  With
    // eight there were five of most forms, and launches that need the sixth took up to 1.16 times as long: 256 -> 96 on
    // 12 x 62 x 62 24.4 -> 20.6 us, 128 -> 96 stride 2 on 4 x 80 x 16 x 70 16.0 -> 13.4; with four, int32 sums of few steps up to
    // 1.07.  Two-digit rows take two loads to a step, and those of six steps were 4 to 13 % of small launches: 128 -> 128, 2 x 2,
    // on sixteen planes of 37 x 44 4.7 -> 3.9 us, 256 -> 257 on 49 x 7 x 32 14.3 -> 13.3.
    constexpr int AHEAD = VB == 4 || KIND == kDigits ? 2 : NB == 1 ? 6 : 4;
    v2u f[AHEAD][NB];
    // The words of a step's bank rows, in turn, through a buffer descriptor that ends with the wave's last row and reads as
    // zeros from there on.  FAR, where the bank may be of any size: a step's, or the last step's again.
    constexpr int AT_ONCE = ROWS ? 2 : 1;
    const int last_row = min(t.rows, KIND == kTapPacked ? t.rows : AT_ONCE * (first + steps));
    const __amdgpu_buffer_rsrc_t bank_src =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p.wgt), 0, (int)((uint32_t)last_row * (uint32_t)row_bytes), 0x00020000);
    const uint32_t* bank = p.wgt + (size_t)(active ? cb : 0) * FW;
    uint32_t next = lane_f + (uint32_t)((active ? cb : 0) * FW * 4) + (uint32_t)(KIND == kTapPacked ? 0 : AT_ONCE * first) * (uint32_t)row_bytes;
    auto fetch_f = [&](v2u (&to)[NB], int step) {
        if constexpr (!FAR) {
            const uint32_t o = KIND == kTapPacked ? next + (uint32_t)((2 * (first + step)) >> t.tp_log) * (uint32_t)row_bytes : next;
            if constexpr (KIND != kTapPacked) next += (uint32_t)(AT_ONCE * row_bytes);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if constexpr (KIND == kBinary) {
                    to[nb].x = __builtin_amdgcn_raw_buffer_load_b32(bank_src, o + nb * 32 * FW * 4, 0, 0);
                } else if constexpr (KIND == kDigits) {
                    to[nb].x = __builtin_amdgcn_raw_buffer_load_b32(bank_src, o + nb * 32 * FW * 4, 0, 0);
                    to[nb].y = __builtin_amdgcn_raw_buffer_load_b32(bank_src, o + nb * 32 * FW * 4 + 8, 0, 0);
                } else {
                    to[nb] = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(bank_src, o + nb * 32 * FW * 4, 0, 0));
                }
            }
        } else {
            const int s = first + min(step, steps - 1), row = KIND == kTapPacked ? (2 * s) >> t.tp_log : AT_ONCE * s;
            const uint8_t* b = reinterpret_cast<const uint8_t*>(bank) + (size_t)row * (size_t)row_bytes;
            uint32_t o = lane_f;
            if constexpr (ROWS && ODD) {
                if (half_last && s == all_steps - 1 && g) o -= (uint32_t)row_bytes;   // any row: its activations are zero
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const uint32_t* w = reinterpret_cast<const uint32_t*>(b + o) + nb * 32 * FW;
                if constexpr (KIND == kBinary) to[nb].x = w[0];
                else if constexpr (KIND == kDigits) to[nb].x = w[0], to[nb].y = w[2];
                else to[nb] = *reinterpret_cast<const v2u*>(w);
            }
        }
    };
    // Cut points of the workgroup's filters, thread j those of filter j (a workgroup has at least as many
    // threads).  Staged behind the halo tile: fetched there they cost another round trip in front of the barrier
    // (0.4 to 0.9 us of a launch of 5 to 9).
    const int wg_filters = t.nwc * 32 * NB;
    int cut_lo = 0, cut_hi = 0;

    // ---- operands' places in LDS -------------------------------------------------------------------
    int lane_v[VB];
    auto tap_off = [&](int tap) {
        const int r = (int)quotient((uint32_t)tap, t.r_kw), a = (int)quotient((uint32_t)r, t.r_kh);
        return (((a * p.dd * t.hy) + (r - a * p.kh) * p.dh) * t.hx + (tap - r * p.kw) * p.dw) * REC;
    };
    const int nch = KIND == kDigits && !ODD ? t.nch >> 1 : t.nch;
    const int inc_ch = ODD ? t.pl : 2 * t.pl;
    // The entries' LDS offsets lie in the lanes of a register, so that a step is a readlane: lanes 48 and up those of the
    // first two steps, lanes 0 to 47 those of the next, in turn.
    int table, entry = 48, entry0 = (ODD ? 2 : 1) * first;
    auto tabulate = [&]() {
        const int e = min(entry0 + (lane < 48 ? lane + (ODD ? 4 : 2) : lane - 48), entries - 1);   // (the last again past the end)
        const int tap = (int)quotient((uint32_t)e, t.r_nch);
        table = tap_off(tap) + (e - tap * nch) * inc_ch;
    };
    // All that has time until the halo tile's first words arrive.
    auto meanwhile = [&]() {
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) fetch_f(f[k], k);
        if constexpr (PACKED) {
            const int co = min((int)blockIdx.y * wg_filters + min(tid, wg_filters - 1), p.c_out - 1);
            cut_lo = p.lo[co];
            cut_hi = p.hi[co];
        }
#pragma unroll
        for (int vb = 0; vb < VB; ++vb) {
            const int vi = vb * 32 + i32;
            const int x = vi & (X - 1), y = (vi >> t.lxb) & (Y - 1), z = vi >> (t.lxb + t.lyb);
            const int v = ((wz * Z + z) * p.sd * t.hy + (wy * Y + y) * p.sh) * t.hx + x * p.sw;
            lane_v[vb] = v * REC + (ODD ? 0 : g * t.pl);
        }
        tabulate();
    };

    uint32_t m33 = 0x33333333u, maa = 0xaaaaaaaau;
    asm volatile("" : "+v"(m33), "+v"(maa));

    // ---- halo tile -> LDS ----------------------------------------------------------------------
    const int gx0 = ox0 * p.sw - p.pw, gy0 = oy0 * p.sh - p.ph, gz0 = oz0 * p.sd - p.pd;
    {
        // Offsets are in bytes and modulo 2^32; voxels outside the volume get one past the end, which reads as zeros.
        const uint32_t* from = KIND == kPair ? t.pair.base : p.in;
        uint32_t origin = (uint32_t)gz0 * t.slice + (uint32_t)gy0 * t.line + (uint32_t)gx0 * t.rec;
        if constexpr (KIND != kPair && !FAR) {
            if (t.whole) {
                origin += (uint32_t)n * t.item;
            } else {
                const int zb = max(gz0, 0);
                from += ((size_t)n * p.d + zb) * (size_t)(t.slice >> 2);
                origin -= (uint32_t)zb * t.slice;
            }
        }
        __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(from), 0, t.reach, 0x00020000);
        uint32_t pair0 = 0, pair1 = 0;                      // the batch item's first bytes; word pair c of source 1 is pair c - nch0 there
        if constexpr (KIND == kPair) {
            pair0 = t.pair.start[0] + (uint32_t)n * t.pair.item[0];
            pair1 = t.pair.start[1] + (uint32_t)n * t.pair.item[1] - 8u * (uint32_t)t.pair.nch0;
        }
        constexpr uint32_t OUTSIDE = 0xfffffff0u;
        int items = t.items;
        constexpr bool PAIRS = !ODD || KIND == kDigits;     // two words per plane and item
        // Items a thread keeps in flight (single words: more would cost a wave per SIMD).  Eight where the registers are
        // there anyway: 64 channels on 8 x 8 x 8 with dilation 2 are 6.75 items to a thread, and the second round trip
        // for the rest was 2.5 % of the launch (96^3: 49.4 -> 48.2 us).
        constexpr int FILL = PAIRS ? (VB == 4 ? 8 : 6) : 3;
        auto round = [&](int base, auto first_one) {
            uint32_t r[FILL][4];
            int dst[FILL];
#pragma unroll
            for (int k = 0; k < FILL; ++k) {
                if (k > 0 && base + k * nthreads >= items) break;   // (the same for every thread)
                const uint32_t e = (uint32_t)(base + k * nthreads + tid);
                const uint32_t v = quotient(e, t.r_ch);
                const uint32_t c = e - __umul24(v, (uint32_t)t.nch);
                const uint32_t hz = quotient(v, t.r_pl);
                const uint32_t q = v - __umul24(hz, (uint32_t)plane);
                const uint32_t hy = quotient(q, t.r_hx);
                const uint32_t hx = q - __umul24(hy, (uint32_t)t.hx);
                const bool live = e < (uint32_t)items;
                dst[k] = live ? (int)(__umul24(c, (uint32_t)(PAIRS && KIND != kDigits ? 2 * t.pl : t.pl)) + v * REC) : -1;
                const bool inside = live & ((uint32_t)(gz0 + (int)hz) < (uint32_t)p.d) & ((uint32_t)(gy0 + (int)hy) < (uint32_t)p.h) &
                                    ((uint32_t)(gx0 + (int)hx) < (uint32_t)p.w);
                if constexpr (KIND == kPair) {
                    const PairPlan& u = t.pair;
                    const bool a = c < (uint32_t)u.nch0;
                    const int iz = gz0 + (int)hz, iy = gy0 + (int)hy, ix = gx0 + (int)hx;
                    const int z = a ? (iz + u.first[0][0]) >> u.up[0][0] : (iz + u.first[1][0]) >> u.up[1][0];
                    const int y = a ? (iy + u.first[0][1]) >> u.up[0][1] : (iy + u.first[1][1]) >> u.up[1][1];
                    const int x = a ? (ix + u.first[0][2]) >> u.up[0][2] : (ix + u.first[1][2]) >> u.up[1][2];
                    const uint32_t plane_row = __umul24((uint32_t)z, (uint32_t)(a ? u.h[0] : u.h[1])) + (uint32_t)y;
                    const uint32_t vrec = a ? u.rec[0] : u.rec[1];
                    uint32_t o = (a ? pair0 : pair1) + __umul24(plane_row, a ? u.line[0] : u.line[1]) + __umul24((uint32_t)x, vrec) + 8u * c;
                    o = inside ? o : OUTSIDE;
                    const v2u m = __builtin_amdgcn_raw_buffer_load_b64(src, o, 0, 0);
                    const v2u sg = __builtin_amdgcn_raw_buffer_load_b64(src, inside ? o + (vrec >> 1) : OUTSIDE, 0, 0);
                    r[k][0] = m.x; r[k][1] = m.y; r[k][2] = sg.x; r[k][3] = sg.y;
                    continue;
                }
                uint32_t o = origin + hz * t.slice + hy * t.line + __umul24(hx, t.rec) + (PAIRS ? 8u : 4u) * c;
                o = inside ? o : OUTSIDE;
                if constexpr (PAIRS) {
                    const v2u a = __builtin_amdgcn_raw_buffer_load_b64(src, o, 0, 0);
                    const v2u b = __builtin_amdgcn_raw_buffer_load_b64(src, o, t.rec >> 1, 0);
                    r[k][0] = a.x; r[k][1] = a.y; r[k][2] = b.x; r[k][3] = b.y;
                } else {
                    r[k][0] = __builtin_amdgcn_raw_buffer_load_b32(src, o, 0, 0);
                    r[k][2] = __builtin_amdgcn_raw_buffer_load_b32(src, o, t.rec >> 1, 0);
                }
            }
            if constexpr (decltype(first_one)::value) meanwhile();
#pragma unroll
            for (int k = 0; k < FILL; ++k) {
                if (k > 0 && base + k * nthreads >= items) break;
                if (dst[k] >= 0) {
                    uint8_t* d = lds8 + dst[k];
                    if constexpr (KIND == kDigits) {
                        *reinterpret_cast<v4i*>(d) = expand_digits(r[k][0], r[k][1], r[k][2], r[k][3]);
                    } else if constexpr (PAIRS) {
                        *reinterpret_cast<v4i*>(d) = expand(interleave(r[k][0], r[k][2], m33), maa);
                        *reinterpret_cast<v4i*>(d + t.pl) = expand(interleave(r[k][1], r[k][3], m33), maa);
                    } else {
                        *reinterpret_cast<v4i*>(d) = expand(interleave(r[k][0], r[k][2], m33), maa);
                    }
                }
            }
        };
        // The first round by itself: in front of a loop the compiler waits for every load that is under way.
        if constexpr (!FAR) {
            round(0, std::true_type{});
            for (int base = FILL * nthreads; base < items; base += FILL * nthreads) round(base, std::false_type{});
        } else {
            meanwhile();
            const int yb = max(gy0, 0);
            for (int hz = 0, base = 0; hz < t.hz; ++hz) {
                const int z = min(max(gz0 + hz, 0), p.d - 1);   // (a plane outside the volume reads nothing)
                from = p.in + (((size_t)n * p.d + z) * p.h + yb) * (size_t)(t.line >> 2);
                src = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(from), 0, t.reach, 0x00020000);
                origin = (uint32_t)(gy0 - yb) * t.line + (uint32_t)gx0 * t.rec - (uint32_t)hz * t.slice;
                items = (hz + 1) * plane * t.nch;
                for (; base < items; base += FILL * nthreads) round(base, std::false_type{});
                base = items;
            }
        }
        if (ODD && (KIND == kBinary || FAR) && tid < 4) reinterpret_cast<uint32_t*>(lds8 + t.zero_off)[tid] = 0u;
    }
    // Cut points in LDS: start values, then widths.
    float* cuts = reinterpret_cast<float*>(lds8 + t.cut_off);
    if constexpr (PACKED) {
        if (tid < wg_filters) {
            const Cut cut = cut_of(cut_lo, cut_hi, (int)blockIdx.y * wg_filters + tid < p.c_out);
            const int at = SIX ? (tid & ~31) + filter_row(tid & 31) : tid;
            cuts[at] = cut.start;
            cuts[wg_filters + at] = cut.width;
        }
    }
    __syncthreads();
    if (!SPLIT && !active) return;

    // ---- contraction ---------------------------------------------------------------------------
    auto next_entry = [&]() { return __builtin_amdgcn_readlane(table, entry++); };
    auto next_table = [&]() {                                  // (after a whole number of rounds of either loop)
        if (__builtin_expect(entry == 48, 0)) {
            entry = 0;
            entry0 += 48;
            tabulate();
        }
    };
    auto fetch_v = [&](v4i (&x)[VB], int step) {
        if constexpr (ODD) {
            const int o0 = next_entry(), o1 = next_entry();
            const int o = g ? o1 : o0;
            const bool dead = half_last && step == steps - 1;
#pragma unroll
            for (int vb = 0; vb < VB; ++vb) {
                int a = lane_v[vb] + o;
                if (dead) a = g ? t.zero_off : a;
                x[vb] = *reinterpret_cast<const v4i*>(lds8 + a);
            }
        } else {
            const int o = next_entry();
#pragma unroll
            for (int vb = 0; vb < VB; ++vb) x[vb] = *reinterpret_cast<const v4i*>(lds8 + lane_v[vb] + o);
        }
    };
    v16f acc[VB][NB], start[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
        for (int v = 0; v < 16; ++v) start[nb][v] = 0.0f;
        if constexpr (PACKED) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 h = *reinterpret_cast<const float4*>(cuts + (wc * NB + nb) * 32 + 8 * k + 4 * g);
                start[nb][4 * k] = h.x; start[nb][4 * k + 1] = h.y; start[nb][4 * k + 2] = h.z; start[nb][4 * k + 3] = h.w;
            }
            if (ks > 0) {                                      // once per sum
#pragma unroll
                for (int v = 0; v < 16; ++v) start[nb][v] = 0.0f;
            }
        }
    }

    auto widen_block = [&](v4i (&F)[NB], const v2u (&f)[NB], int step, int nb) {
        if constexpr (KIND == kBinary) {
            v2u u;
            u.x = (f[nb].x << 2) | m33;
            u.y = f[nb].x | m33;
            F[nb] = expand(u, maa);
        } else if constexpr (KIND == kTapPacked) {
            const uint32_t sh = (uint32_t)(((2 * (first + step) + g) & ((1 << t.tp_log) - 1)) * p.tp_shift);
            F[nb] = expand(interleave(f[nb].x >> sh, f[nb].y >> sh, m33), maa);
        } else if constexpr (!ROWS) {
            // lanes 0-31 hold both mask words, lanes 32-63 both sign words of a filter
            const auto sw = __builtin_amdgcn_permlane32_swap(f[nb].x, f[nb].y, false, false);
            F[nb] = expand(interleave(sw[0], sw[1], m33), maa);
        } else {
            F[nb] = expand(interleave(f[nb].x, f[nb].y, m33), maa);
        }
    };
    auto widen = [&](v4i (&F)[NB], const v2u (&f)[NB], int step) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) widen_block(F, f, step, nb);
    };
    auto contract = [&](const v4i (&F)[NB], const v4i (&x)[VB], auto first) {
#pragma unroll
        for (int vb = 0; vb < VB; ++vb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                acc[vb][nb] = multiply(F[nb], x[vb], decltype(first)::value ? start[nb] : acc[vb][nb]);
    };

    v4i x0[VB], x1[VB];
    v4i F0[NB], F1[NB];
    fetch_v(x0, 0);
    fetch_v(x1, 1);
    entry = 0;
    if constexpr (VB == 4) {
        // Operands of step i + 1 are fetched and widened between step i's matrix instructions, filter words two steps further
        // ahead.  In front of all of them, both waves of a SIMD do that at the same time, with the matrix cores idle: the same steps
        // so ordered take 46.1 us for 44.5 on 64 -> 64 channels, 96^3 with dilation 2, and 45.6 for 42.1 on 256 -> 256, 2 x 32^3 (with
        // a wave priority for that part 47.2 and 41.3).  The scalar walk before them, which had that order, took 47.6 and 42.8.
        // (The barriers hold the order; a load moved above the last use of its registers has the compiler copy them and wait.)
        auto column = [&](const v4i (&F)[NB], const v4i (&x)[VB], int vb) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[vb][nb] = multiply(F[nb], x[vb], acc[vb][nb]);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto step_of = [&](const v4i (&F)[NB], const v4i (&x)[VB], v4i (&F_next)[NB], v2u (&words)[NB], v4i (&x_next)[VB], int next) {
            column(F, x, 0);
            fetch_v(x_next, next);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int vb = 1; vb < VB; ++vb) {
                column(F, x, vb);
                if (vb <= NB) widen_block(F_next, words, next, vb - 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            fetch_f(words, next + 2);
            __builtin_amdgcn_sched_barrier(0);
        };
        widen(F0, f[0], 0);
        fetch_f(f[0], 2);
        widen(F1, f[1], 1);
        fetch_f(f[1], 3);
        __builtin_amdgcn_sched_barrier(0);
        contract(F0, x0, std::true_type{});
        int i = 1;
        for (; i + 2 <= steps; i += 2) {
            next_table();
            step_of(F1, x1, F0, f[0], x0, i + 1);
            step_of(F0, x0, F1, f[1], x1, i + 2);
        }
        if (i < steps) contract(F1, x1, std::false_type{});
    } else {
        // Voxels of the next two steps and filter words of the next AHEAD are under way, with no branch around their
        // loads: behind one the compiler waits for all that may be.
#pragma unroll
        for (int vb = 0; vb < VB; ++vb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[vb][nb] = start[nb];
        [&]() __attribute__((always_inline)) {
            for (int done = 0;; done += AHEAD) {
                next_table();
#pragma unroll
                for (int k = 0; k < AHEAD; ++k) {
                    v4i (&x)[VB] = k & 1 ? x1 : x0;
                    widen(F0, f[k], done + k);
                    fetch_f(f[k], done + k + AHEAD);
                    contract(F0, x, std::false_type{});
                    if (done + k + 1 >= steps) return;
                    fetch_v(x, done + k + 2);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }();
    }

    // ---- partial sums ------------------------------------------------------------------------------
    // A tile's sums go through LDS in quads, four registers of a wave (a byte of 32 voxels' words), and each of its waves
    // adds up and finishes as many: quads ks * Q .. ks * Q + Q - 1.  (Whole blocks left four or six of eight waves without
    // any and the others with seven round trips to LDS: 1.0 to 2.6 us of a launch, now 0.8 to 1.7.)
    constexpr int QUADS = VB * NB * 4;
    if constexpr (SPLIT) {
        __syncthreads();                                       // everyone is done with the halo tile
        float* mine = reinterpret_cast<float*>(lds8) + (size_t)wave * (QUADS * 256) + lane * 4;
#pragma unroll
        for (int u = 0; u < QUADS; ++u) {
            const v16f& a = acc[u / 4 / NB][u / 4 % NB];
            const int k = 4 * (u & 3);
            *reinterpret_cast<float4*>(mine + u * 256) = make_float4(a[k], a[k + 1], a[k + 2], a[k + 3]);
        }
        __syncthreads();
        if (!active) return;
    }

    // ---- epilogue: lane = voxel l % 32 of a block, register v = filter 8 (v / 4) + 4 g + v % 4 -----
    // A block's voxels differ from block 0's by the same box offset in every lane.  Voxel numbers are below 2^31: in 64 bits
    // the steps from block to block took 19 scalar instructions each (64 -> 64 3 x 3 on sixteen planes of 232 x 168 16.5 -> 15.7
    // us, 64 -> 64 on 64^3 13.5 -> 13.2; as arguments from the host, which come through a load of their own, 16.5 and 13.6).
    const int lx = i32 & (X - 1), ly = (i32 >> t.lxb) & (Y - 1), lz = i32 >> (t.lxb + t.lyb);
    const int bx = ox0, by = oy0 + wy * Y, bz = oz0 + wz * Z;
    auto inside = [&](int vb, uint32_t& step) {                // step: voxels from block 0
        const int dx = (vb * 32) & (X - 1), dy = ((vb * 32) >> t.lxb) & (Y - 1), dz = (vb * 32) >> (t.lxb + t.lyb);
        step = (uint32_t)((dz * p.oh + dy) * p.ow + dx);
        return lx < p.ow - bx - dx && ly < p.oh - by - dy && lz < p.od - bz - dz;
    };
    const uint32_t vox0 = (((uint32_t)n * p.od + bz) * p.oh + by) * p.ow + bx + ((uint32_t)(lz * p.oh) + ly) * p.ow + lx;
    // int32 sums of rows 8 k + j, j < 4, of quads k from a block's filter c0 on (c0 with the lane's 4 g)
    const size_t cs = (size_t)p.od * p.oh * p.ow;
    auto sums_at = [&](int c0, uint32_t step) { return p.out_acc + ((size_t)n * p.c_out + c0) * cs + (vox0 + step - (uint32_t)n * (uint32_t)cs); };
    auto store_quads = [&](int32_t* o, int c0, auto quads, auto&& value) {
        constexpr int N = decltype(quads)::value;
        const bool all = (c0 & ~7) + 8 * N <= p.c_out;      // (the same for every lane)
#pragma unroll
        for (int v = 0; v < 4 * N; ++v) {
            if (all || c0 + (v >> 2) * 8 + (v & 3) < p.c_out) *o = (int32_t)value(v);
            o += (v & 3) == 3 ? 5 * cs : cs;
        }
    };
    if constexpr (SPLIT) {
        auto finish = [&](auto log2_waves) {
            constexpr int LKS = decltype(log2_waves)::value, Q = QUADS >> LKS, QB = Q < 4 ? Q : 4;   // (quads of one block)
            const float* theirs = reinterpret_cast<const float*>(lds8) + ((size_t)(wtile << LKS) * QUADS + ks * Q) * 256 + lane * 4;
            float4 sum[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                float4 part[1 << LKS];
#pragma unroll
                for (int o = 0; o < 1 << LKS; ++o) part[o] = *reinterpret_cast<const float4*>(theirs + (o * QUADS + q) * 256);
                sum[q] = part[0];
#pragma unroll
                for (int o = 1; o < 1 << LKS; ++o) {
                    sum[q].x += part[o].x; sum[q].y += part[o].y; sum[q].z += part[o].z; sum[q].w += part[o].w;
                }
            }
#pragma unroll
            for (int q0 = 0; q0 < Q; q0 += QB) {
                const int u = ks * Q + q0, vb = u / 4 / NB, nb = u / 4 % NB, k0 = u & 3;
                uint32_t step;
                if (!inside(vb, step)) continue;
                if constexpr (PACKED) {
                    const float* widths = cuts + wg_filters + (wc * NB + nb) * 32 + 8 * k0 + 4 * g;
                    uint32_t pos = 0u, neg = 0u;
#pragma unroll
                    for (int q = QB - 1; q >= 0; --q) {
                        const float4 w = *reinterpret_cast<const float4*>(widths + 8 * q);
                        const float4 a = sum[q0 + q];
                        decide<1>(pos, neg, a.w, w.w);
                        decide<1>(pos, neg, a.z, w.z);
                        decide<1>(pos, neg, a.y, w.y);
                        if (q > 0) decide<5>(pos, neg, a.x, w.x);
                        else decide<1>(pos, neg, a.x, w.x);
                    }
                    const uint32_t word = block_word(pos, neg);
                    uint32_t* o = p.out_packed + (size_t)(vox0 + step) * (2u * p.wd_out) + g * p.wd_out + (cb >> 5) + nb;
                    if constexpr (QB == 4) *o = word;
                    else if constexpr (QB == 2) reinterpret_cast<uint16_t*>(o)[k0 >> 1] = (uint16_t)word;
                    else reinterpret_cast<uint8_t*>(o)[k0] = (uint8_t)word;
                } else {
                    const int c0 = cb + nb * 32 + 8 * k0 + 4 * g;
                    store_quads(sums_at(c0, step), c0, std::integral_constant<int, QB>{}, [&](int v) {
                        const float4& a = sum[q0 + (v >> 2)];
                        return (v & 3) == 0 ? a.x : (v & 3) == 1 ? a.y : (v & 3) == 2 ? a.z : a.w;
                    });
                }
            }
        };
        if (lks == 1) finish(std::integral_constant<int, 1>{});
        else if (lks == 2) finish(std::integral_constant<int, 2>{});
        else finish(std::integral_constant<int, 3>{});
        return;
    }
    if constexpr (PACKED) {
        uint32_t* out = p.out_packed + (size_t)vox0 * (2u * p.wd_out) + g * p.wd_out + (cb >> 5);
        Decider d;
        v8bf widths[NB];
        if constexpr (SIX) {
            d = decider();
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) widths[nb] = width_operand(cuts[wg_filters + (wc * NB + nb) * 32 + i32], g == 0);
        }
#pragma unroll
        for (int vb = 0; vb < VB; ++vb) {
            uint32_t word[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if constexpr (SIX) {
                    word[nb] = decided_word(acc[vb][nb], widths[nb], d);
                } else {
                    uint32_t pos, neg;
                    decide_block(pos, neg, acc[vb][nb], cuts + wg_filters + (wc * NB + nb) * 32 + 4 * g);
                    word[nb] = block_word(pos, neg);
                }
            }
            uint32_t step;
            if (inside(vb, step)) {
                uint32_t* o = out + (size_t)step * (2u * p.wd_out);
                // (two blocks of filters come where there is an even number of blocks: all words exist)
                if constexpr (NB == 2) *reinterpret_cast<v2u*>(o) = v2u{word[0], word[1]};
                else *o = word[0];
            }
        }
    } else {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int c0 = cb + nb * 32 + 4 * g;
#pragma unroll
            for (int vb = 0; vb < VB; ++vb) {
                uint32_t step;
                if (inside(vb, step)) store_quads(sums_at(c0, step), c0, std::integral_constant<int, 4>{}, [&](int v) { return acc[vb][nb][v]; });
            }
        }
    }
}

template <int VB, int NB, bool PACKED, int KIND, bool ODD, bool SPLIT, bool FAR>
int launch_variant(const ConvParams& p, const MatrixPlan& t, size_t lds_bytes, dim3 grid, int threads, hipStream_t s)
{
    auto kern = conv_matrix_kernel<VB, NB, PACKED, KIND, ODD, SPLIT, FAR>;
    if (lds_bytes > 64 * 1024) {
        static thread_local int raised_on_device = -1;
        int dev = 0;
        TERN_HIP_CHECK(hipGetDevice(&dev));
        if (raised_on_device != dev) {
            TERN_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               lds_limit_for_current_device()));
            raised_on_device = dev;
        }
    }
    hipLaunchKernelGGL(kern, grid, dim3(threads), lds_bytes, s, p, t);
    TERN_HIP_CHECK(hipGetLastError());
    return TERN_OK;
}

template <int VB, int NB, bool PACKED, bool SPLIT, bool FAR>
int launch_kind(const ConvParams& p, const MatrixPlan& t, bool odd, size_t lds, dim3 grid, int threads, hipStream_t s)
{
    if constexpr (PACKED && !FAR)
        if (t.pair.base) return launch_variant<VB, NB, PACKED, kPair, false, SPLIT, FAR>(p, t, lds, grid, threads, s);
    if (p.tp_slots) return launch_variant<VB, NB, PACKED, kTapPacked, true, SPLIT, FAR>(p, t, lds, grid, threads, s);
    if (p.digits)
        return odd ? launch_variant<VB, NB, PACKED, kDigits, true, SPLIT, FAR>(p, t, lds, grid, threads, s)
                   : launch_variant<VB, NB, PACKED, kDigits, false, SPLIT, FAR>(p, t, lds, grid, threads, s);
    if (p.binary)
        return odd ? launch_variant<VB, NB, PACKED, kBinary, true, SPLIT, FAR>(p, t, lds, grid, threads, s)
                   : launch_variant<VB, NB, PACKED, kBinary, false, SPLIT, FAR>(p, t, lds, grid, threads, s);
    return odd ? launch_variant<VB, NB, PACKED, kTernary, true, SPLIT, FAR>(p, t, lds, grid, threads, s)
               : launch_variant<VB, NB, PACKED, kTernary, false, SPLIT, FAR>(p, t, lds, grid, threads, s);
}

}  // namespace

// Two tensors as one buffer: both within 4 GB, rows and row numbers within the kernel's 24-bit products.
static bool pair_plan(const ConvPair& pair, int32_t n, PairPlan& u)
{
    const bool both = pair.s[1].wd > 0;
    const uintptr_t a = (uintptr_t)pair.s[0].p, b = both ? (uintptr_t)pair.s[1].p : a, base = a < b ? a : b;
    uint64_t end = 0;
    for (int i = 0; i < 2; ++i) {
        const PairSource& q = pair.s[i];
        const bool there = i == 0 || both;
        const int64_t rec = 8 * (int64_t)q.wd, line = there ? q.w * rec : 0, rows = there ? (int64_t)q.d * q.h : 0;
        if (line >= 1 << 24 || rows >= 1 << 24 || q.d >= 1 << 24) return false;
        const uint64_t start = (i == 0 ? a : b) - base, bytes = (uint64_t)n * (uint64_t)(rows * line);
        if (start > 0xffff0000u || bytes > 0xffff0000u || start + bytes > 0xffff0000u) return false;
        if (start + bytes > end) end = start + bytes;
        u.start[i] = (uint32_t)start;
        u.item[i] = (uint32_t)(rows * line);
        u.line[i] = (uint32_t)line;
        u.rec[i] = (uint32_t)rec;
        u.h[i] = q.h;
        for (int k = 0; k < 3; ++k) { u.up[i][k] = q.up_log[k]; u.first[i][k] = q.first[k]; }
    }
    u.base = (const uint32_t*)base;
    u.reach = (uint32_t)end;
    u.nch0 = pair.s[0].wd / 2;
    return true;
}

// Every convolution goes this way except those that one of the limits below sends to the bit-count
// kernels: more than 128 taps (the bound of the reciprocals of kernel extents, and as far as it was measured), sums that could pass
// 2^21 (the epilogue works with halves; LDS runs out first, so far), halo tiles that do not fit in LDS, and tiles
// whose rows of a plane span more than 4 GB.
// A tile holds all words of its voxels: 3 x 3 x 3 kernels fit up to 47 words (1504 channels) at stride 1, 19 with
// dilation 2, 10 with 3, 14 at stride 2, 7 and 4 with dilation 2 and 3; from the next word on they take three
// to eight times as long as their neighbours.
// Slower here than with bit counts, and left so: one and two channels (16 or 32 taps to a filter word there) to
// at most 16 filters under 64 to 128 taps, 0.8 to 1.35 times with no rule of sizes that tells them apart (1 -> 16
// channels, 5^3: 15.6 and 17.9 us on 48^3, 56^3 to 80^3 0.91 to 1.0 times); at most 8 filters with dilated kernels
// on 256 channels, where 16-byte records take a second round of workgroups (256 -> 8, dilation 3, 88 x 66 x 2: 14.7
// and 17.4 us); int32 sums of some twenty voxels whose tile the bit-count kernel could not hold and left to the
// direct one (6.7 and 8.4 us).
bool launch_conv_matrix(const ConvParams& p, const ConvPair* pair, hipStream_t s, int* rc)
{
    MatrixPlan t;
    t.pair.base = nullptr;
    if (pair && !pair_plan(*pair, p.n, t.pair)) return false;
    const int64_t taps = (int64_t)p.kd * p.kh * p.kw;
    if (taps > 128 || taps * p.c_in * (p.digits ? 2 : 1) > kMatrixSumLimit) return false;
    const int64_t lds_limit = lds_limit_for_current_device();
    if (lds_limit <= 0) { *rc = TERN_EHIP; return true; }
    const int words = p.digits ? p.wd_in / 2 : p.wd_in;
    const bool odd = (words & 1) != 0, packed = p.out_packed != nullptr;
    const MatrixShape shape = {p.n, p.c_out, p.od, p.oh, p.ow, p.kd, p.kh, p.kw, p.sd, p.sh, p.sw, p.dd, p.dh, p.dw,
                               words, p.digits, packed ? 1 : 0, (int32_t)lds_limit};
    Choice c, settled;
    Tile q;
    if (!choose_cached(shape, c, &settled)) return false;
    if (!p.tp_slots || c.vb == 4) c = settled;
    if (!tile_of(shape, c, q)) return false;
    // A tile's planes within 4 GB (a volume's may be more), or else its rows of each: then with waves of 128 voxels on 32
    // filters (64 -> 64 channels, 3 x 3, on a plane of 16 400 x 16 400 6.9 ms; half of it, which one descriptor reaches, 3.4,
    // with bit counts 17.6).
    const int64_t line_bytes = 8 * (int64_t)p.wd_in * p.w, plane_bytes = line_bytes * p.h;
    bool whole;
    int64_t reach = input_reach(p.n, p.d, plane_bytes, q.hz, whole);
    if (pair) reach = t.pair.reach;
    // The filter bank within 4 GB, or else the launch as chosen, without a split (2^19 filters of 1152 channels, 3 x 3 x 3, on
    // 4 x 6 x 9 3.8 ms, with bit counts 122; of 256, 11 x 11, on 90 x 100 53 ms, with waves of 128 voxels on 32 filters 69).
    const int64_t bank_rows = bank_rows_of(taps, p.wd_in, p.wc, p.tp_slots), row_bytes = (int64_t)p.co_pad * p.wc * (p.binary ? 4 : 8);
    const bool far_input = reach > kReach, far = far_input || !bank_in_reach(bank_rows, row_bytes);
    if (far && pair) return false;
    if (far_input) {
        const bool flat = p.od == 1, deep = p.od > 1 && p.kd > 1;
        const int8_t* sh = kWaveShape[1][flat][0];
        c = {4, 1, sh[0], sh[1], 1, 1, 1, 1};
        while (c.nwc < 4 && 2 * c.nwc <= cdiv(p.c_out, 32)) c.nwc *= 2;
        (deep ? c.nwz : c.nwy) = 4 / c.nwc;
        if (!tile_of(shape, c, q)) {
            c.nwy = c.nwz = 1;
            if (!tile_of(shape, c, q)) return false;
        }
    } else if (far) {
        c.nks = 1;
        if (!tile_of(shape, c, q)) return false;
    }
    if (far) {
        reach = line_bytes * (q.hy < p.h ? q.hy : p.h);
        if (reach > kReach) return false;
    }
    const int X = 1 << c.lxb, Y = 1 << c.lyb, Z = (32 * c.vb) >> (c.lxb + c.lyb);
    const int64_t gy = q.wgs / q.tiles;
    if (q.tiles > 0x7fffffff || gy > 65535) return false;
    t.lxb = c.lxb; t.lyb = c.lyb; t.lwy = log2_up(c.nwy); t.lwz = log2_up(c.nwz); t.nwc = c.nwc;
    t.hx = (int32_t)q.hx; t.hy = (int32_t)q.hy; t.hz = (int32_t)q.hz;
    t.tiles_x = divisor(cdiv(p.ow, X)); t.tiles_y = divisor(cdiv(p.oh, Y * c.nwy)); t.tiles_z = divisor(cdiv(p.od, Z * c.nwz));
    t.reach = (uint32_t)reach;
    t.whole = whole;
    t.rec = 8u * (uint32_t)p.wd_in; t.line = (uint32_t)line_bytes; t.slice = (uint32_t)plane_bytes;
    t.item = (uint32_t)(plane_bytes * p.d);
    t.nch = p.digits || odd ? words : words / 2;
    t.rows = (int32_t)bank_rows;
    t.row_bytes = (int32_t)row_bytes;
    t.plane = t.hx * t.hy;
    t.items = (int32_t)q.items;
    t.pl = (int32_t)(q.hx * q.hy * q.hz * 16);
    t.zero_off = words * t.pl;
    t.cut_off = (int32_t)q.cuts;
    t.lks = log2_up(c.nks);
    const int threads = 64 * c.nwy * c.nwz * c.nwc * c.nks;
    t.threads = threads; t.tiles = (int32_t)q.tiles;
    t.r_nwc = reciprocal((uint32_t)c.nwc, 8);
    const uint32_t emax = (uint32_t)q.items;
    t.r_hx = reciprocal((uint32_t)t.hx, emax);
    t.r_pl = reciprocal((uint32_t)(t.hx * t.hy), emax);
    t.r_ch = reciprocal((uint32_t)t.nch, emax);
    const int per_tap = p.digits && !odd ? words / 2 : t.nch;    // entries or steps of a tap
    t.r_nch = reciprocal((uint32_t)per_tap, (uint32_t)(taps * per_tap + 2));
    t.r_kw = reciprocal((uint32_t)p.kw, 128);
    t.r_kh = reciprocal((uint32_t)p.kh, 128);
    t.tp_log = 0;
    if (p.tp_slots)
        while ((p.tp_shift << t.tp_log) < 32) ++t.tp_log;
    const dim3 grid((unsigned)q.tiles, (unsigned)gy);
    const size_t lds = (size_t)q.lds;
    note_launch(TERN_KERNEL_TILED, c.vb / 2, 32 * c.nb, c.nks, threads, grid.x, grid.y, lds);
    const auto kind = [&](auto vb, auto nb, auto split, auto beyond) {
        constexpr int VB = decltype(vb)::value, NB = decltype(nb)::value;
        constexpr bool SPLIT = decltype(split)::value, FAR = decltype(beyond)::value;
        return packed ? launch_kind<VB, NB, true, SPLIT, FAR>(p, t, odd, lds, grid, threads, s)
                      : launch_kind<VB, NB, false, SPLIT, FAR>(p, t, odd, lds, grid, threads, s);
    };
    const std::integral_constant<int, 1> one;
    const std::integral_constant<int, 2> two;
    const std::integral_constant<int, 4> four;
    const std::true_type yes;
    const std::false_type no;
    const auto unsplit = [&](auto beyond) {
        if (c.vb == 4) return c.nb == 2 ? kind(four, two, no, beyond) : kind(four, one, no, beyond);
        return c.nb == 2 ? kind(two, two, no, beyond) : kind(two, one, no, beyond);
    };
    if (far) *rc = unsplit(yes);
    else if (c.nks > 1) *rc = c.nb == 2 ? kind(two, two, yes, no) : kind(two, one, yes, no);
    else *rc = unsplit(no);
    return true;
}

}  // namespace tern
