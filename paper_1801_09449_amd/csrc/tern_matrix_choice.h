// The launch of a tiled convolution on the matrix cores (tern_conv_matrix.hip): what a wave and a workgroup
// take, chosen from sizes alone.  Host code without HIP, so that a test can compile it by itself.
//
// A program whose extents are new on every call pays for the choice on every call, so it has to cost little
// beside a launch: 2.4 us on average over random geometries and 4.0 us for 256 -> 256 channels on 32^3 (an EPYC core;
// a Xeon at 2.7 GHz 4.6 and 6.9), the second look at small launches in it: 0.1 on average, 0.4 of the 2.4 us of 512 -> 256,
// 3 x 3, on 52 x 36.  Every candidate's whole estimate, two powers among them, would take twice as long.
#pragma once
#include <stdint.h>
#include <string.h>

#include <cmath>
#include <memory>
#include <new>

#include "tern_division.h"

namespace tern {
namespace {

// All that a choice depends on.
struct MatrixShape {
    int32_t n, c_out, od, oh, ow;
    int32_t kd, kh, kw, sd, sh, sw, dd, dh, dw;
    int32_t words;                   // words per plane that are contracted (two-digit input: pairs)
    int32_t digits, packed;
    int32_t lds_limit;               // bytes a workgroup may use
};

// What a launch is made of, apart from the kernel's own arguments.
struct Choice {
    int32_t vb, nb;                  // 32-voxel and 32-filter blocks of a wave
    int32_t lxb, lyb, nwy, nwz, nwc;
    int32_t nks;
};

// Extents that follow from a choice.
struct Tile {
    int64_t hx, hy, hz, tiles, wgs, lds, items;
    int64_t cuts;                    // LDS offset of the cut points: behind the halo tile and the partial sums
};

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int32_t cdiv(int32_t a, int32_t b) { return (a + b - 1) / b; }

constexpr int64_t kMaxHalo = 20480, kMaxItems = 32768;   // voxels of a halo tile, units of its fill

// The halo tile of nwy x nwz waves; false if it does not fit.
inline bool halo_of(const MatrixShape& s, int vb, int lxb, int lyb, int nwy, int nwz, Tile& t)
{
    const int64_t x = (int64_t)1 << lxb, y = (int64_t)nwy << lyb, z = (int64_t)nwz * ((32 * vb) >> (lxb + lyb));
    t.hx = (x - 1) * s.sw + (int64_t)(s.kw - 1) * s.dw + 1;
    t.hy = (y - 1) * s.sh + (int64_t)(s.kh - 1) * s.dh + 1;
    t.hz = (z - 1) * s.sd + (int64_t)(s.kd - 1) * s.dd + 1;
    if (t.hx > kMaxHalo || t.hy > kMaxHalo || t.hz > kMaxHalo || t.hx * t.hy * t.hz > kMaxHalo) return false;
    const int64_t voxels = t.hx * t.hy * t.hz;
    const bool odd = (s.words & 1) != 0;
    t.items = voxels * (s.digits || odd ? s.words : s.words / 2);
    t.lds = s.words * voxels * 16 + (odd ? 16 : 0);
    return t.lds <= s.lds_limit && t.items <= kMaxItems;
}

// LDS with partial sums and cut points; false if that does not fit.
inline bool lds_of(const MatrixShape& s, const Choice& c, Tile& t)
{
    const int64_t sums = (int64_t)(c.nwy * c.nwz * c.nwc * c.nks) * (c.vb * c.nb * 4096);
    if (c.nks > 1 && t.lds < sums) t.lds = sums;
    t.cuts = t.lds;
    if (s.packed) t.lds += (int64_t)c.nwc * c.nb * 32 * 8;
    return t.lds <= s.lds_limit;
}

inline bool tile_of(const MatrixShape& s, const Choice& c, Tile& t)
{
    if (!halo_of(s, c.vb, c.lxb, c.lyb, c.nwy, c.nwz, t) || !lds_of(s, c, t)) return false;
    const int z = c.nwz * ((32 * c.vb) >> (c.lxb + c.lyb));
    t.tiles = cdiv((int64_t)s.ow, (int64_t)1 << c.lxb) * cdiv((int64_t)s.oh, (int64_t)c.nwy << c.lyb) * cdiv((int64_t)s.od, (int64_t)z) * s.n;
    t.wgs = t.tiles * cdiv(cdiv(s.c_out, 32 * c.nb), c.nwc);
    return true;
}

// What the kernel reads through buffer descriptors has to lie within reach of their 32-bit offsets.
constexpr int64_t kReach = 0xffff0000ll;
// Bytes that the input's descriptor spans: all of the input, or a tile's planes in it.
inline int64_t input_reach(int32_t n, int32_t d, int64_t plane_bytes, int64_t hz, bool& whole)
{
    whole = plane_bytes * d * n <= kReach;
    return whole ? plane_bytes * d * n : plane_bytes * (hz < d ? hz : d);
}
inline int64_t bank_rows_of(int64_t taps, int32_t wd_in, int32_t wc, int32_t tp_slots)
{
    return tp_slots ? cdiv(taps, (int64_t)tp_slots) : taps * (wd_in / wc);
}
// Rows past the end of the filter bank have to read as zeros (the absent partner of the last row) or are fetched and not used
// (up to twelve, those of the six steps under way): a row is at most 8 MB (2^19 filters), and 256 MB are left for them.
inline bool bank_in_reach(int64_t rows, int64_t row_bytes) { return (rows + 1) * row_bytes <= 0xf0000000ll; }

// Estimated time of a launch in clock cycles, the 1.73-norm of two parts.  Throughput (busy): the fullest
// compute unit's share of matrix instructions (32 cycles each) and of vector instructions (a wave's fixed
// part, per 64 halo items, per step and its operands, per accumulator block of the epilogue).  Latency: as
// many rounds of workgroups as registers and LDS leave no room for at once, each as long as one wave takes by
// itself.  The weights are a fit to 1400 launches on 54 shapes, from the 2-D layers of a U-Net to 96-cubed volumes
// (workgroups of powers of two only; the search looks at more), of kernels whose small waves took twice as long
// for a step as now and which added partial sums by whole blocks.  Of 1868 launches of the kernels as they are on those shapes, the choice, with the
// second look and the rows of int32 sums below, takes 2.3 % longer than the best one in the geometric mean and 19 % at the most.
// A choice looks at some two hundred launches, so no candidate of this search costs an integer division (the second look
// divides: it has at most forty).
inline int32_t steps_of(const MatrixShape& s, int lks)             // of a wave, the longest
{
    return (int32_t)(((int64_t)s.kd * s.kh * s.kw * s.words + ((int64_t)2 << lks)) >> (lks + 1));
}
constexpr double kShare[9] = {0, 1.0, 0.5, 0, 0.25, 0, 0, 0, 0.125};                  // of nks waves
constexpr uint32_t kPer64[9] = {0, 1u << 26, 1u << 25, 22369622, 1u << 24, 13421773, 11184811, 9586981, 1u << 23};   // 2^32 / (64 waves), up
// Resident workgroups of a compute unit by their waves (one to eight): 8, 12, 16 and 24 waves of 4 x 2, 4 x 1, 2 x 2 and
// 2 x 1 blocks of 32 voxels and 32 filters.  Registers leave room for those, and for 16 waves where 12 are counted: so counted
// the choice was as good in the mean (0.998 over 779 launches) and 8 to 15 % longer for five of them.
constexpr uint8_t kFit[4][9] = {{8, 8, 4, 2, 2, 1, 1, 1, 1}, {12, 12, 6, 4, 3, 2, 2, 1, 1}, {16, 16, 8, 5, 4, 3, 2, 2, 2}, {24, 24, 12, 8, 6, 4, 4, 3, 3}};
constexpr double kInverse[25] = {0, 1.0, 1.0 / 2, 1.0 / 3, 1.0 / 4, 1.0 / 5, 1.0 / 6, 1.0 / 7, 1.0 / 8, 1.0 / 9, 1.0 / 10, 1.0 / 11, 1.0 / 12,
                                 1.0 / 13, 1.0 / 14, 1.0 / 15, 1.0 / 16, 1.0 / 17, 1.0 / 18, 1.0 / 19, 1.0 / 20, 1.0 / 21, 1.0 / 22, 1.0 / 23, 1.0 / 24};

inline int waves_of(const Choice& c) { return c.nwy * c.nwz * c.nwc * c.nks; }        // at most 8
// Halo items per wave in units of 64, rounded up (the sum stays below 2^16).
inline int rounds64_of(int waves, int64_t items) { return (int)(((uint64_t)(items + 64 * waves - 1) * kPer64[waves]) >> 32); }
// (helpers: waves beyond the filter groups, which only help to fill the halo tile)
inline double busy_of(const MatrixShape& s, const Choice& c, int64_t per_cu, int helpers, int32_t steps, int rounds64)
{
    const double blocks = c.vb * c.nb;
    const double vector = 730.0 + 280.0 * rounds64 + steps * (3.0 + c.vb + 38.0 * c.nb) + blocks * (s.packed ? 94.0 : 390.0) * kShare[c.nks] +
                          (c.nks > 1 ? 200.0 + 15.0 * blocks : 0.0);
    return (double)per_cu * 0.25 * ((waves_of(c) - helpers) * (0.8 * 32.0 * steps * blocks + vector) + helpers * (100.0 + 280.0 * rounds64));
}
inline double latency_of(const Choice& c, int64_t per_cu, int64_t lds, int32_t steps, int rounds64)
{
    const int blocks = c.vb * c.nb;
    int fit = kFit[blocks >= 8 ? 0 : c.vb == 4 ? 1 : c.nb == 2 ? 2 : 3][waves_of(c)];
    const int by_lds = (int)(163840.0f / (float)(int32_t)lds);     // (exact: no quotient is that close below a whole number)
    if (by_lds < fit) fit = by_lds < 1 ? 1 : by_lds;
    const double alone = 4400.0 + 2280.0 * ((rounds64 + 5) / 6) + steps * (129.0 + 32.0 * blocks) + 111.0 * blocks * kShare[c.nks] +
                         (c.nks > 1 ? 28.0 + 174.0 * blocks : 0.0);
    const int64_t rounds = (int64_t)((double)(per_cu + fit - 1) * kInverse[fit] + 1.0 / 64);
    return (double)rounds * alone;
}
inline double norm_cost(double busy, double latency) { return std::pow(busy, 1.73) + std::pow(latency, 1.73); }

// The norm of (1, r) for r in 0 .. 1, from below: a bound of the norm without a power.
struct NormTable {
    double v[65];
    NormTable()
    {
        for (int i = 0; i <= 64; ++i) v[i] = std::pow(1.0 + std::pow(i / 64.0, 1.73), 1.0 / 1.73) * (1.0 - 1e-12);
    }
};
inline double norm_bound(double a, double b)
{
    static const NormTable table;
    const double hi = a > b ? a : b, lo = a > b ? b : a;
    return hi * table.v[(int)(lo / hi * 64.0)];
}

// Shapes of a wave's voxels (log2 of x and y extent), 64 and 128 voxels, volumes and single planes.
constexpr int8_t kWaveShape[2][2][6][2] = {{{{3, 3}, {3, 2}, {2, 3}, {2, 2}, {4, 2}, {4, 1}}, {{3, 3}, {4, 2}, {2, 4}, {5, 1}}},
                                           {{{3, 3}, {3, 4}, {4, 3}, {3, 2}, {4, 2}, {2, 2}}, {{3, 4}, {4, 3}, {5, 2}, {2, 5}}}};
constexpr int kWaveShapes[2] = {6, 4};

// The launch of least estimated time; false if no halo tile fits in LDS.  Between equals the one that comes
// first by (vb, nb, nwc, waves in space, nks, shape).  Candidates that share a halo tile are looked at
// together, and put aside by bounds without divisions (no split makes a tile's `busy` less).
inline bool choose(const MatrixShape& s, Choice& best)
{
    const int fb = cdiv(s.c_out, 32);
    const int flat = s.od == 1;
    const bool deep = s.od > 1 && s.kd > 1;
    const int64_t all_steps = ((int64_t)s.kd * s.kh * s.kw * s.words + 1) / 2;
    // Two filter blocks per wave: the bank holds whole blocks of 32 filters.  Not for int32 sums of two-digit input
    // after two to eight steps, where they were slower than the bit counts (128 channels -> 232, single taps on
    // 26 675 voxels 22.3 us, with one block 17.6, bit counts 19.3).
    const int most_nb = (fb & 1) || (s.digits && !s.packed && all_steps > 1 && all_steps <= 8) ? 1 : 2;
    int deepest = 0;                                 // log2 of the deepest split
    while (deepest < 3 && all_steps >= 8 << deepest) ++deepest;
    double cost = 1e300, root = 1e300;               // of the best so far, and its norm
    int order = 0;
    int32_t steps[4];
    for (int lks = 0; lks < 4; ++lks) steps[lks] = steps_of(s, lks);
    // Waves over filter groups: powers of two, or all groups at once.  Beyond those they only help to fill the
    // halo tile: with the smallest waves, where that takes one wave's round trips more than once, a compute unit
    // has one workgroup and the steps are split as far as they go.  One wave that fills a wide tile alone is slow: 96 -> 19 channels,
    // 3 x 1 x 1 with stride 2 and dilation 3 on 2 x (1, 4, 1), 12.6 us alone and 5.6 with seven helpers; over 160
    // small launches the geometric mean falls by 8 %, and 15 of 16 that had been slower than the bit-count
    // kernels no longer are.  With two steps a wave instead of four, splits of eight took 15 % longer than splits of four.
    struct Groups {
        int n, nwc[8], per_tile[8];
    } groups[3];
    for (int nb = 1; nb <= 2; ++nb) {
        Groups& g = groups[nb];
        const int all = fb / nb;
        g.n = 0;
        for (int nwc = 1; nwc <= 8; ++nwc)
            if (!(nwc & (nwc - 1)) || nwc == all) {
                g.nwc[g.n] = nwc;
                g.per_tile[g.n++] = cdiv(all, nwc);
            }
    }
    auto over = [](int64_t extent, int log2) { return (extent + ((int64_t)1 << log2) - 1) >> log2; };
    for (int vb = 4; vb >= 2; vb -= 2) {
        double wave[3][4], alone[3][4];              // bounds from below: no halo items, one round of workgroups
        for (int nb = 1; nb <= 2; ++nb)
            for (int lks = 0; lks < 4; ++lks) {
                const Choice one = {vb, nb, 0, 0, 1, 1, 1, 1 << lks};
                wave[nb][lks] = busy_of(s, one, 1, 0, steps[lks], 0) * kShare[1 << lks] * (1.0 - 1e-9);
                alone[nb][lks] = latency_of(one, 1, 1, steps[lks], 1) * (1.0 - 1e-9);
            }
        for (int k = 0; k < kWaveShapes[flat]; ++k)
            // waves are stacked along z, where neighbours share halo planes, else along y
            for (int lws = 0; lws < 4; ++lws) {
                const int nws = 1 << lws;
                const int8_t* sh = kWaveShape[vb == 4][flat][k];
                Choice c = {vb, 0, sh[0], sh[1], deep ? 1 : nws, deep ? nws : 1, 0, 0};
                Tile halo;
                if (!halo_of(s, vb, c.lxb, c.lyb, c.nwy, c.nwz, halo)) break;
                const int lzb = (vb == 4 ? 7 : 6) - c.lxb - c.lyb + (deep ? lws : 0);
                halo.tiles = over(s.ow, c.lxb) * over(s.oh, c.lyb + (deep ? 0 : lws)) * over(s.od, lzb) * s.n;
                const double fill = (double)(halo.tiles * halo.items) * (280.0 / 64.0 / 1024.0);
                for (c.nb = 1; c.nb <= most_nb; ++c.nb) {
                    const Groups& g = groups[c.nb];
                    if ((double)(halo.tiles * nws * (fb / c.nb)) * (1.0 / 256.0) * wave[c.nb][0] + fill > root) continue;
                    for (int i = 0; i < g.n && g.nwc[i] * nws <= 8; ++i) {
                        c.nwc = g.nwc[i];
                        halo.wgs = halo.tiles * g.per_tile[i];
                        const int beyond = c.nwc > fb / c.nb ? nws * (c.nwc - fb / c.nb) : 0;
                        if (beyond && (vb > 2 || c.nb > 1 || halo.items <= 64 * nws * (fb / c.nb) || halo.wgs > 256)) break;
                        // a split leaves each wave at least four steps; only the smaller waves have one
                        for (int lks = beyond ? deepest : 0; lks < 4; ++lks) {
                            c.nks = 1 << lks;
                            if (c.nks * nws * c.nwc > 8 || (lks > 0 && (vb > 2 || lks > deepest))) break;
                            const int helpers = beyond << lks;
                            const int64_t per_cu = (halo.wgs + 255) >> 8;
                            const int waves = nws * c.nwc << lks;
                            if ((double)(per_cu * (waves - helpers)) * wave[c.nb][lks] > root || alone[c.nb][lks] > root) continue;
                            Tile t = halo;
                            if (!lds_of(s, c, t)) continue;
                            const int r = rounds64_of(waves, t.items);
                            const double busy = busy_of(s, c, per_cu, helpers, steps[lks], r);
                            if (busy > root) continue;
                            const double latency = latency_of(c, per_cu, t.lds, steps[lks], r);
                            if (norm_bound(busy, latency) > root) continue;
                            const double x = norm_cost(busy, latency);
                            const int o = ((((vb * 4 + c.nb) * 16 + c.nwc) * 4 + lws) * 4 + lks) * 8 + k;
                            if (x > cost || (x == cost && o > order)) continue;
                            cost = x;
                            root = std::pow(x, 1.0 / 1.73) * (1.0 + 1e-12);
                            order = o;
                            best = c;
                        }
                    }
                }
            }
    }
    return cost < 1e300;
}

// A second look at launches of the small waves, which a wave's own time decides: how its waves are shared out between
// space, filters and steps, in tiles of the same shape.  The estimate above takes up to six halo items a lane for one round
// trip; they are instructions, a wave by itself issues one every 2.4 ns, and waves that share a halo tile fill it together.
// Its time here, in ns: a wave's own as long as launches come in whole rounds, and what the waves of a SIMD take together, the
// norm of both.  The weights are a fit to launches on 252 shapes of up to 20 GMAC, planes and volumes; another launch is
// taken where it is 4 % shorter, on 40 of them, by 6 % in the geometric mean (2 % longer to 20 % shorter): 128 -> 128 channels
// 3 x 3 on 113 x 81 5.2 -> 4.5 us, 512 -> 256 on 52 x 36 6.9 -> 6.3, 64 -> 64 on 232 x 168 4.5 -> 4.1.  Not from 6 us on, where
// rates decide (216 -> 32, 3 x 3, on sixteen of 43 x 197 13.6 and 14.7); and the caller leaves tap-packed filters out, whose
// shifts make a step longer than it is here (5 -> 26 on 2 x 30 x 56 x 14 4.9 and 5.4).  The fit is to one-digit input; an item
// of two digits takes longer to widen and counts half as much again (counted like the others, 64 -> 37,
// 2 x 2 x 2 with stride 2, on 4 x 78 x 6 x 66 went to half the waves, 5.5 -> 6.7 us, and 128 -> 64, 2 x 2 x 2, on 2 x 6 x 78 x 20 5.8 -> 6.5).
inline double small_cost(const MatrixShape& s, const Choice& c, const Tile& t, int lks)
{
    const int waves = waves_of(c), groups = cdiv(s.c_out, 32) / c.nb, active = c.nwc > groups ? waves / c.nwc * groups : waves;
    const double rounds64 = (s.digits ? 1.5 : 1.0) * rounds64_of(waves, t.items), steps = steps_of(s, lks);
    const double blocks = c.nb, two = c.nb - 1, split = c.nks > 1 ? 1.0 : 0.0;
    const int64_t per_cu = (t.wgs + 255) >> 8;
    const double wave = 560.0 + 83.0 * rounds64 + (20.0 + 35.0 * two) * steps + blocks * ((s.packed ? 270.0 : 400.0) * kShare[c.nks] + 380.0 * split);
    const double busy = (double)per_cu * 0.25 * (active * wave + (waves - active) * (500.0 + 83.0 * rounds64));
    int fit = kFit[c.nb == 2 ? 2 : 3][waves];
    const int by_lds = (int)(163840.0f / (float)(int32_t)t.lds);
    if (by_lds < fit) fit = by_lds < 1 ? 1 : by_lds;
    const double alone = 840.0 + 147.0 * rounds64 + (98.0 + 75.0 * two) * steps + blocks * (s.packed ? 150.0 : 1600.0) * kShare[c.nks] +
                         split * (420.0 + 330.0 * two);
    const double latency = (double)((per_cu + fit - 1) / fit) * alone;
    return std::sqrt(busy * busy + latency * latency);
}
// int32 sums of the large waves: a store writes a row of the wave's voxels, and rows of 4 or 8 are an eighth or a quarter of a
// 128-byte line, whose parts reach memory one by one once the waves of a chip hold more of them than its caches.  Waves of 16
// voxels along x instead, where the stores count beside the products and few more tiles are needed: 24 -> 128 channels on
// 4 x 26 x 87 x 76 171 -> 95 us, 32 -> 128 on 76 x 72 x 43 61 -> 36, 64 -> 160, 3 x 3, on eight planes of 200 x 167 44 -> 35.  The lines
// are drawn on 499 launches: with more entries, or more tiles than that, up to 1.7 times as long.
inline void lengthen_rows(const MatrixShape& s, Choice& c)
{
    if (c.vb != 4 || s.packed || c.lxb >= 4) return;
    const int64_t entries = (int64_t)s.kd * s.kh * s.kw * s.words;
    const bool much = 4.0 * s.n * s.c_out * ((double)s.od * s.oh * s.ow) >= 80e6;
    const int sixteenths = entries <= 32 ? (much ? 20 : 17) : entries <= 54 && much ? 17 : 0;
    Choice x = c;
    x.lxb = 4;
    x.lyb = s.od == 1 ? 3 : 2;
    Tile from, to;
    if (tile_of(s, c, from) && tile_of(s, x, to) && to.tiles * 16 <= from.tiles * sixteenths) c = x;
}
inline void settle(const MatrixShape& s, Choice& c)
{
    if (c.vb != 2) return lengthen_rows(s, c);
    const Choice from = c;
    Tile t;
    if (!tile_of(s, from, t)) return;
    const int fb = cdiv(s.c_out, 32);
    const bool deep = s.od > 1 && s.kd > 1;
    const int64_t all_steps = ((int64_t)s.kd * s.kh * s.kw * s.words + 1) / 2;
    double least = small_cost(s, from, t, log2_up(from.nks));
    if (least > 6000.0) return;
    least *= 0.96;
    for (int nws = 1; nws <= 8; nws *= 2) {
        const int nwy = deep ? 1 : nws, nwz = deep ? nws : 1;
        Tile halo;
        if (!halo_of(s, 2, from.lxb, from.lyb, nwy, nwz, halo)) break;
        for (int nb = 1; nb <= from.nb; ++nb)                      // (two blocks of filters only where they were allowed)
            for (int nwc = 1; nwc * nws <= 8 && nwc <= fb / nb; ++nwc) {
                if ((nwc & (nwc - 1)) && nwc != fb / nb) continue;
                // (a split leaves each wave at least four steps)
                for (int lks = 0; lks < 4 && nwc * nws << lks <= 8 && (lks == 0 || all_steps >= 4 << lks); ++lks) {
                    const Choice x = {2, nb, from.lxb, from.lyb, nwy, nwz, nwc, 1 << lks};
                    if (!tile_of(s, x, t)) continue;
                    const double cost = small_cost(s, x, t, lks);
                    if (cost < least) { least = cost; c = x; }
                }
            }
    }
}

// Each thread keeps the choices of the geometries it met last, by hash, two to a place (a found one takes
// 13 ns).  A network has about a dozen: of 64 kept in the order of their making, those of six image sizes
// pushed each other out.  `settled`: the same after the second look.
inline bool choose_cached(const MatrixShape& s, Choice& c, Choice* settled = nullptr)
{
    struct Entry {
        MatrixShape shape;
        Choice c, settled;
        int32_t ok;
    };
    const auto make = [](const MatrixShape& shape, Choice& a, Choice& b) {
        const bool ok = choose(shape, a);
        b = a;
        if (ok) settle(shape, b);
        return ok;
    };
    Choice other;
    Choice& b = settled ? *settled : other;
    constexpr int kPlaces = 256;
    static thread_local std::unique_ptr<Entry[]> table;
    if (!table) {
        table.reset(new (std::nothrow) Entry[2 * kPlaces]);
        if (!table) return make(s, c, b);
        memset(static_cast<void*>(table.get()), 0, sizeof(Entry) * 2 * kPlaces);   // (no shape has zero words)
    }
    uint64_t h = 0;
    int32_t v[sizeof s / 4];
    memcpy(v, &s, sizeof s);
    for (int32_t x : v) h = (h ^ (uint32_t)x) * 0x9e3779b97f4a7c15u, h ^= h >> 29;
    Entry* e = &table[2 * (h >> 32) % (2 * kPlaces)];
    for (int i = 0; i < 2; ++i)
        if (memcmp(&e[i].shape, &s, sizeof s) == 0) { c = e[i].c; b = e[i].settled; return e[i].ok != 0; }
    e[1] = e[0];
    e[0].shape = s;
    e[0].ok = make(s, e[0].c, e[0].settled);
    c = e[0].c;
    b = e[0].settled;
    return e[0].ok != 0;
}

}  // namespace
}  // namespace tern
