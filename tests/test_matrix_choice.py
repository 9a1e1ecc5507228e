"""The launch chooser of the tiled matrix kernel (csrc/tern_matrix_choice.h, host code): against a plain search
over every launch with the estimate written out in ordinary divisions, over random geometries."""
import os
import re
import shutil
import subprocess
import tempfile

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1801_09449_amd", "csrc")

SOURCE = r"""
#include "tern_matrix_choice.h"
#include <chrono>
#include <cstdio>
#include <random>
#include <vector>
using namespace tern;

static double up(double x) { return std::ceil(x); }

static double plain_cost(const MatrixShape& s, const Choice& c, const Tile& t)
{
    const double steps = up(((double)s.kd * s.kh * s.kw * s.words + 1.0) / 2.0 / c.nks);
    const int waves = c.nwy * c.nwz * c.nwc * c.nks, groups = (s.c_out + 31) / 32 / c.nb;
    const int active = waves / c.nwc * (c.nwc < groups ? c.nwc : groups);
    const double blocks = c.vb * c.nb, split = c.nks > 1 ? 1.0 : 0.0;
    const double per_cu = up((double)t.wgs / 256.0), rounds = up((double)t.items / (64.0 * waves));
    const double vector = 730.0 + 280.0 * rounds + steps * (3.0 + c.vb + 38.0 * c.nb) + blocks * (s.packed ? 94.0 : 390.0) / c.nks +
                          split * (200.0 + 15.0 * blocks);
    const double busy = per_cu / 4.0 * (active * (25.6 * steps * blocks + vector) + (waves - active) * (100.0 + 280.0 * rounds));
    double fit = std::floor(4.0 * (blocks >= 8 ? 2 : c.vb == 4 ? 3 : c.nb == 2 ? 4 : 6) / waves);
    fit = std::fmax(1.0, std::fmin(fit, std::floor(163840.0 / (double)t.lds)));
    const double alone = 4400.0 + 2280.0 * up(rounds / 6.0) + steps * (129.0 + 32.0 * blocks) + 111.0 * blocks / c.nks +
                         split * (28.0 + 174.0 * blocks);
    return std::pow(busy, 1.73) + std::pow(up(per_cu / fit) * alone, 1.73);
}

// Every launch in the order that decides between equals.
static bool search(const MatrixShape& s, Choice& best, double& cost)
{
    static const int volume[2][6][2] = {{{3, 3}, {3, 2}, {2, 3}, {2, 2}, {4, 2}, {4, 1}}, {{3, 3}, {3, 4}, {4, 3}, {3, 2}, {4, 2}, {2, 2}}};
    static const int plane[2][6][2] = {{{3, 3}, {4, 2}, {2, 4}, {5, 1}}, {{3, 4}, {4, 3}, {5, 2}, {2, 5}}};
    const int fb = (s.c_out + 31) / 32, all_steps = (s.kd * s.kh * s.kw * s.words + 1) / 2;
    const bool deep = s.od > 1 && s.kd > 1;
    cost = 1e300;
    for (int vb = 2; vb <= 4; vb += 2)
        for (int nb = 1; nb <= 2; ++nb)
            for (int nwc = 1; nwc <= 8; ++nwc)
                for (int nws = 1; nws <= 8; nws *= 2)
                    for (int nks = 1; nks <= 8; nks *= 2)
                        for (int k = 0; k < (s.od == 1 ? 4 : 6); ++k) {
                            const int* sh = (s.od == 1 ? plane : volume)[vb == 4][k];
                            const int groups = fb / nb;
                            if (nb == 2 && ((fb & 1) || (s.digits && !s.packed && all_steps > 1 && all_steps <= 8))) continue;
                            if ((nwc & (nwc - 1)) && nwc != groups) continue;
                            if (nks * nws * nwc > 8 || (nks > 1 && (vb > 2 || all_steps < 4 * nks))) continue;
                            const Choice c = {vb, nb, sh[0], sh[1], deep ? 1 : nws, deep ? nws : 1, nwc, nks};
                            Tile t;
                            if (!tile_of(s, c, t)) continue;
                            // waves that only help to fill
                            if (nwc > groups && (vb > 2 || nb > 1 || t.wgs > 256 || t.items <= 64 * nws * groups || (nks < 8 && all_steps >= 8 * nks))) continue;
                            const double x = plain_cost(s, c, t);
                            if (x < cost) { cost = x; best = c; }
                        }
    return cost < 1e300;
}

int main()
{
    std::mt19937_64 r(1);
    auto log_int = [&](double a, double b) { return (int)std::lround(std::exp(std::uniform_real_distribution<>(std::log(a), std::log(b))(r))); };
    auto pick = [&](std::initializer_list<int> l) { return *(l.begin() + r() % l.size()); };
    std::vector<MatrixShape> all;
    for (int i = 0; i < 20000; ++i) {
        MatrixShape s = {pick({1, 1, 2, 4, 16, log_int(1, 100000)}), pick({32, 64, 128, 256, 512, log_int(1, 3000)}), log_int(1, 300), log_int(1, 300),
                         log_int(1, 300), pick({1, 1, 2, 3, 3, 3, 5}), pick({1, 2, 3, 3, 5}), pick({1, 2, 3, 3, 5}), pick({1, 1, 2}),
                         pick({1, 1, 2, 4}), pick({1, 1, 2}), pick({1, 1, 2, 3}), pick({1, 1, 2, 3}), pick({1, 1, 2, 3}),
                         pick({1, 2, 3, 4, 8, log_int(1, 60)}), pick({0, 0, 1}), pick({0, 1}), 160 * 1024};
        if (r() % 3 == 0) s.od = s.kd = 1;
        if (r() % 9 == 0) s.lds_limit = 64 * 1024;
        all.push_back(s);
    }
    const auto now = [] { return std::chrono::steady_clock::now(); };
    std::vector<Choice> a(all.size()), b(all.size());
    std::vector<double> cost(all.size());
    std::vector<char> ok(all.size());
    const auto t0 = now();
    for (size_t i = 0; i < all.size(); ++i) ok[i] = search(all[i], a[i], cost[i]);
    const auto t1 = now();
    long differ = 0, none = 0, kept = 0;
    for (size_t i = 0; i < all.size(); ++i) differ += choose(all[i], b[i]) != (bool)ok[i];
    const auto t2 = now();
    for (size_t i = 0; i < all.size(); ++i) {
        if (!ok[i]) { ++none; continue; }
        Tile t;
        if (!tile_of(all[i], b[i], t) || !(plain_cost(all[i], b[i], t) <= cost[i] * (1 + 1e-12))) ++differ;
        if (b[i].nwy * b[i].nwz * b[i].nwc * b[i].nks > 8 || t.lds > all[i].lds_limit) ++differ;
    }
    for (int round = 0; round < 2; ++round)                 // first made, then found or made again
        for (size_t i = 0; i < 1500; ++i)
            for (int twice = 0; twice < 2; ++twice) {
                Choice c;
                if (choose_cached(all[i], c) != (bool)ok[i] || (ok[i] && memcmp(&c, &b[i], sizeof c) != 0)) ++kept;
            }
    printf("differ %ld kept %ld none %ld of %zu ratio %.3f\n", differ, kept, none, all.size(), (double)(t2 - t1).count() / (t1 - t0).count());
}
"""


WAVES = r"""
#include "tern_matrix_choice.h"
#include <cstdio>
int main()
{
    // n, c_out, output extents, kernel, stride, dilation, words, digits, packed
    const tern::MatrixShape s[] = {{2, 19, 1, 2, 1, 3, 1, 1, 2, 2, 2, 3, 3, 3, 3, 0, 1, 163840}, {2, 2, 48, 1, 2, 1, 1, 1, 2, 2, 2, 1, 1, 1, 9, 1, 1, 163840},
                                   {1, 32, 67, 1, 42, 1, 1, 1, 1, 2, 2, 1, 1, 1, 5, 1, 0, 163840}, {1, 8, 41, 5, 7, 2, 2, 2, 2, 2, 2, 3, 3, 3, 1, 0, 0, 163840},
                                   {2, 8, 3, 37, 5, 3, 3, 3, 1, 2, 2, 3, 3, 3, 1, 0, 1, 163840}, {1, 64, 64, 64, 64, 3, 3, 3, 1, 1, 1, 1, 1, 1, 2, 0, 1, 163840}};
    for (const auto& x : s) {
        tern::Choice c;
        tern::Tile t;
        if (!tern::choose(x, c) || !tern::tile_of(x, c, t)) return 1;
        const int waves = c.nwy * c.nwz * c.nwc * c.nks;
        printf("%d %d %d\n", waves, (int)((t.items + 64 * waves - 1) / (64 * waves)), c.nwc * c.nb * 32 <= (x.c_out + 31) / 32 * 32);
    }
}
"""


SETTLED = r"""
#include "tern_matrix_choice.h"
#include <cstdio>
#include <random>
using namespace tern;
int main()
{
    std::mt19937_64 r(3);
    auto pick = [&](std::initializer_list<int> l) { return *(l.begin() + r() % l.size()); };
    long changed = 0, wrong = 0;
    for (int i = 0; i < 6000; ++i) {
        const bool flat = r() % 2;
        MatrixShape s = {pick({1, 1, 2, 4}), pick({8, 32, 64, 70, 128, 256, 512}), flat ? 1 : 2 + (int)(r() % 40), 2 + (int)(r() % 200), 2 + (int)(r() % 200),
                         flat ? 1 : pick({2, 3}), pick({1, 2, 3, 5}), pick({1, 2, 3, 5}), 1, pick({1, 2}), pick({1, 2}), 1, pick({1, 3}), pick({1, 3}),
                         pick({1, 2, 3, 4, 7, 8, 16}), pick({0, 0, 1}), pick({0, 1}), pick({65536, 163840})};
        Choice a, b, c;
        Tile ta, tb;
        if (!choose_cached(s, a, &b)) continue;
        if (!tile_of(s, a, ta) || !tile_of(s, b, tb)) { ++wrong; continue; }
        const int steps = (s.kd * s.kh * s.kw * s.words + 1) / 2, groups = (s.c_out + 31) / 32;
        if (memcmp(&a, &b, sizeof a) == 0) continue;
        ++changed;
        if (a.vb == 4) {
            // int32 sums in rows of 16, in workgroups and with steps as before, and up to a quarter more tiles
            if (s.packed || a.lxb > 3 || b.lxb != 4 || b.vb != 4 || a.nb != b.nb || a.nwy != b.nwy || a.nwz != b.nwz || a.nwc != b.nwc || b.nks != 1) ++wrong;
            if (tb.tiles * 16 > ta.tiles * 20 || tb.lds > s.lds_limit || tb.items > kMaxItems || s.kd * s.kh * s.kw * s.words > 54) ++wrong;
            continue;
        }
        // same tile of a wave, small waves only; within a workgroup, its LDS and the steps; an even number of filter blocks for pairs
        if (a.vb != 2 || b.vb != 2 || a.lxb != b.lxb || a.lyb != b.lyb || b.nb > a.nb || (b.nb == 2 && groups % 2)) ++wrong;
        if (b.nwy * b.nwz * b.nwc * b.nks > 8 || tb.lds > s.lds_limit || tb.items > kMaxItems || b.nwc > groups / b.nb) ++wrong;
        if (b.nks > 1 && steps < 4 * b.nks) ++wrong;
        if (small_cost(s, b, tb, log2_up(b.nks)) > 0.96 * small_cost(s, a, ta, log2_up(a.nks)) || small_cost(s, a, ta, log2_up(a.nks)) > 6000.0) ++wrong;
        Choice again;
        if (!choose_cached(s, c, &again) || memcmp(&again, &b, sizeof b) || memcmp(&c, &a, sizeof a)) ++wrong;
    }
    printf("%ld %ld\n", changed, wrong);
}
"""


RESIDENT = r"""
#include "tern_matrix_choice.h"
#include <cstdio>
using namespace tern;
int main()
{
    // (n, c_out, output, kernel, stride, dilation, words, digits, packed, LDS limit); workgroups of eight waves
    const MatrixShape s = {1, 64, 1, 64, 64, 1, 3, 3, 1, 1, 1, 1, 1, 1, 2, 0, 1, 163840};
    for (int nb = 1; nb <= 2; ++nb) {
        const Choice c = {2, nb, 3, 3, 8, 1, 1, 1};
        auto square = [&](int per_cu) {
            const Tile t = {0, 0, 0, 0, 256 * per_cu, 8192, 512, 0};
            const double x = small_cost(s, c, t, 0);
            return x * x;
        };
        // per_cu^2 of the waves' common time and rounds^2 of one workgroup's, which two leave at one round
        const double common = (square(2) - square(1)) / 3.0, alone = square(1) - common;
        int fit = 2;
        while (square(fit + 1) - (fit + 1) * (fit + 1) * common < 1.5 * alone) ++fit;
        printf("%d ", fit);
    }
}
"""


DIGITS = r"""
#include "tern_matrix_choice.h"
#include <cstdio>
using namespace tern;
int main()
{
    // (n, c_out, output, kernel, stride, dilation, words, digits, packed, LDS limit): two-digit input, a tile's fill against its steps
    // (planes of a batch are planes of one volume)
    const MatrixShape s[] = {{4, 37, 40, 4, 34, 2, 2, 2, 2, 2, 2, 1, 1, 1, 2, 1, 1, 163840}, {1, 64, 16, 24, 64, 1, 3, 3, 1, 2, 2, 1, 1, 1, 3, 1, 1, 163840},
                             {2, 64, 7, 79, 21, 2, 2, 2, 1, 1, 1, 1, 1, 1, 4, 1, 1, 163840}, {1, 32, 4, 107, 97, 1, 2, 2, 1, 1, 1, 1, 1, 1, 4, 1, 1, 163840}};
    for (const MatrixShape& x : s) {
        Choice a, b;
        Tile ta, tb;
        if (!choose_cached(x, a, &b) || !tile_of(x, a, ta) || !tile_of(x, b, tb)) return 1;
        printf("%d ", rounds64_of(waves_of(b), tb.items) <= rounds64_of(waves_of(a), ta.items));
    }
}
"""


REACH = r"""
#include "tern_matrix_choice.h"
#include <cstdio>
using namespace tern;
int main()
{
    int wrong = 0;
    bool whole;
    // input: all of it, a tile's planes of it, more than there are, planes that do not fit
    wrong += input_reach(2, 8, 1 << 28, 4, whole) != (1ll << 30) || whole;
    wrong += input_reach(1, 15, 1 << 28, 4, whole) != 15ll << 28 || !whole;
    wrong += input_reach(1, 16, 1 << 28, 4, whole) != (1ll << 30) || whole;
    wrong += input_reach(7, 2, 1 << 29, 4, whole) != (1ll << 30) || whole;
    wrong += input_reach(1, 65535, 65536, 3, whole) != kReach || !whole;
    wrong += input_reach(1, 65536, 65536, 3, whole) != 3 * 65536 || whole;
    wrong += input_reach(1, 3, 1ll << 31, 3, whole) != 3ll << 31 || whole;
    // bank: (taps, words of the input, words of a row, taps to a word) -> rows; plain even and odd, digits, tap-packed
    wrong += bank_rows_of(27, 36, 2, 0) != 486 || bank_rows_of(27, 37, 1, 0) != 999 || bank_rows_of(9, 4, 2, 0) != 18;
    wrong += bank_rows_of(27, 1, 1, 2) != 14 || bank_rows_of(9, 1, 1, 32) != 1 || bank_rows_of(128, 1, 1, 4) != 32;
    // the most filters: rows of 8 and 4 MB (ternary, even and odd words), 4 and 2 MB (binary); the last row that fits and the next
    const int64_t co = 1 << 19;
    const int64_t bytes[4] = {co * 16, co * 8, co * 8, co * 4};
    for (int64_t b : bytes) {
        const int64_t rows = 0xf0000000ll / b - 1;
        wrong += !bank_in_reach(rows, b) || bank_in_reach(rows + 1, b);
        // the bank with the twelve rows fetched past its end, two words of 32 bits and two blocks of filters on
        wrong += (rows + 13) * b + 1024 > kReach;
    }
    printf("%d", wrong);
}
"""


ROWS = r"""
#include "tern_matrix_choice.h"
#include <cstdio>
using namespace tern;
int main()
{
    // (n, c_out, output, kernel, stride, dilation, words, digits, packed, LDS limit)
    const MatrixShape volume = {1, 128, 76, 72, 43, 3, 3, 3, 1, 1, 1, 1, 1, 1, 1, 0, 0, 163840}, planes = {8, 160, 1, 198, 165, 1, 3, 3, 1, 1, 1, 1, 1, 1, 2, 0, 0, 163840};
    auto row = [](MatrixShape s, int lxb, int lyb) {
        Choice c = {4, 1, lxb, lyb, 1, 1, 1, 1};
        settle(s, c);
        printf("%d%d ", c.lxb, c.lyb);
    };
    row(volume, 3, 2); row(volume, 2, 2); row(volume, 4, 3); row(planes, 3, 4); row(planes, 2, 5); row(planes, 5, 2);
    MatrixShape s = volume;
    s.packed = 1; row(s, 3, 2);                              // packed words
    s = volume; s.words = 2; row(s, 3, 2);                   // 54 entries, as many tiles
    s.ow = 35; row(s, 3, 2);                                 // a fifth more
    s = volume; s.words = 3; row(s, 3, 2);                   // 81 entries
    s = volume; s.c_out = 80; row(s, 3, 2);                  // 75 MB, as many tiles
    s.ow = 35; row(s, 3, 2);                                 // a fifth more
    s = volume; s.ow = 35; row(s, 3, 2);                     // 98 MB, a fifth more
    s.ow = 18; s.c_out = 256; row(s, 3, 2);                  // a third more
}
"""


DIVISIONS = r"""
#include "tern_matrix_choice.h"
#include <cstdio>
#include <random>
int main()
{
    long wrong = 0;
    std::mt19937_64 r(2);
    const auto quotient = [](uint32_t e, tern::Divisor d) { return (uint32_t)(((uint64_t)e * d.m) >> d.s); };
    for (int i = 0; i < 400000; ++i) {
        const int32_t d = i < 2000 ? i + 1 : i < 2100 ? 0x7fffffff - (i - 2000) : (int32_t)(r() % 0x7fffffff >> (r() % 31)) + 1;
        const tern::Divisor q = tern::divisor(d);
        const uint32_t last = 0x7fffffffu / (uint32_t)d * (uint32_t)d;        // the largest multiple
        for (uint32_t e : {0u, (uint32_t)d - 1, (uint32_t)d, last - 1, last, 0x7fffffffu, (uint32_t)(r() & 0x7fffffffu)})
            wrong += quotient(e, q) != e / (uint32_t)d;
    }
    for (uint32_t d = 1; d <= 8; ++d)                                          // waves of a workgroup over filter groups
        for (uint32_t e = 0; e < 8; ++e) wrong += (e * tern::reciprocal(d, 8).m) >> tern::reciprocal(d, 8).s != e / d;
    for (uint32_t d = 1; d < 600; ++d) {
        const tern::Reciprocal q = tern::reciprocal(d, 32768);
        for (uint32_t e = 0; e < 32768; ++e) wrong += (e * q.m) >> q.s != e / d;
    }
    printf("%ld\n", wrong);
}
"""


def build_and_run(tmp_path, source):
    (tmp_path / "t.cpp").write_text(source)
    subprocess.run(["g++", "-O3", "-std=c++17", "-I", CSRC, str(tmp_path / "t.cpp"), "-o", str(tmp_path / "t")], check=True)
    return subprocess.run([str(tmp_path / "t")], check=True, capture_output=True, text=True).stdout


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_no_wave_fills_a_wide_halo_tile_alone(tmp_path):
    """Launches of few workgroups and few steps, where a split leaves waves idle: these fill too, at most
    eight items a lane here (single waves had 15 to 63).  Large launches have no such waves."""
    rows = [tuple(map(int, l.split())) for l in build_and_run(tmp_path, WAVES).splitlines()]
    assert all(waves >= 4 and items <= 8 for waves, items, _ in rows[:5]), rows
    assert rows[5][2] == 1, rows


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_cheap_choice_is_the_choice_of_a_plain_search(tmp_path):
    """Same estimated time for every geometry (bounds put nothing better aside, no division was rounded wrongly),
    what is kept is found again, and a choice costs a fraction of the search."""
    out = build_and_run(tmp_path, SOURCE).split()
    got = dict(zip(out[::2], out[1::2]))
    print(out)
    assert got["differ"] == "0" and got["kept"] == "0"
    assert 0 < int(got["none"]) < 4000
    assert float(out[out.index("ratio") + 1]) < 0.6


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_divisions_by_multiplication(tmp_path):
    """The launch's reciprocals give the quotients of the integers, at multiples and beside them up to 2^31."""
    assert build_and_run(tmp_path, DIVISIONS).strip() == "0"


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_second_look_keeps_to_what_a_launch_may_be(tmp_path):
    """The launches that the second look puts in place of small waves' first choice: same tiles, within the limits of a
    workgroup, shorter by its estimate, and found again with the first choice."""
    changed, wrong = map(int, build_and_run(tmp_path, SETTLED).split())
    assert changed > 100 and wrong == 0


READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def kernels_of(lib):
    """name -> (vector registers, bytes of scratch) of the library's kernels, from the notes of its code objects."""
    with open(lib, "rb") as f:
        data = f.read()
    out = {}
    for part in data.split(b"__CLANG_OFFLOAD_BUNDLE__")[1:]:
        at = part.find(b"\x7fELF")
        if at < 0:
            continue
        with tempfile.NamedTemporaryFile(suffix=".elf") as t:
            t.write(part[at:])
            t.flush()
            notes = subprocess.run([READELF, "--notes", t.name], stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True).stdout
        for k in notes.split("  - .agpr_count:")[1:]:
            value = lambda key: re.search(r"\.%s:\s+(\S+)" % key, k).group(1)
            out[value("name")] = int(value("vgpr_count")), int(value("private_segment_fixed_size"))
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs llvm-readelf")
def test_resident_waves_of_the_matrix_kernels():
    """The launch choice counts 24, 16 and 8 waves of a compute unit resident; a kernel's registers, in eights of a SIMD's
    512, have to leave room for them."""
    from paper_1801_09449_amd import build
    if not os.path.exists(build.LIB):
        pytest.skip("needs the built library")
    found = 0
    for name, (registers, scratch) in kernels_of(build.LIB).items():
        m = re.search(r"conv_matrix_kernelILi(\d)ELi(\d)ELb[01]ELi(\d)E", name)
        if not m:
            continue
        found += 1
        vb, nb, kind = map(int, m.groups())
        waves = 4 * (512 // (-(-registers // 8) * 8))
        least = 8 if vb * nb == 8 else 16 if vb * nb == 4 else 24
        if (vb, nb, kind) == (2, 1, 4):        # input in two tensors
            least = 20
        assert waves >= least and scratch == 0, (name, registers, scratch)
    assert found == 146


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs llvm-readelf")
def test_resident_waves_of_the_first_layer_kernels():
    """Of a volume's kernels the ones that take a tile's planes one by one leave room for five waves of a SIMD, the ones that
    take them together for four, which the launch counts on; the far ones of more than 16 filters have four."""
    from paper_1801_09449_amd import build
    if not os.path.exists(build.LIB):
        pytest.skip("needs the built library")
    found = 0
    for name, (registers, scratch) in kernels_of(build.LIB).items():
        m = re.search(r"first_conv_kernelILi3ELb([01])ELb([01])ELb([01])E", name)
        if not m:
            continue
        found += 1
        few, far, together = (x == "1" for x in m.groups())
        waves = 512 // (-(-registers // 8) * 8)
        assert waves >= (4 if together or (far and not few) else 5) and scratch == 0, (name, registers, scratch)
    assert found == 7


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_second_look_counts_the_same_resident_waves(tmp_path):
    """24 and 16 waves of a compute unit, three and two workgroups of eight, in the second look as in the first."""
    assert build_and_run(tmp_path, RESIDENT).split() == ["3", "2"]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_rows_of_int32_sums(tmp_path):
    """Which launches of the large waves get rows of 16 voxels (log2 extents along x and y)."""
    assert build_and_run(tmp_path, ROWS).split() == ["42", "42", "43", "43", "43", "52", "32", "42", "32", "32", "42", "32", "42", "32"]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_second_look_counts_the_fill_of_two_digit_input(tmp_path):
    """Launches that took 1.06 to 1.22 times as long with their steps split over fewer waves, which fill the tile alone."""
    assert build_and_run(tmp_path, DIGITS).split() == ["1"] * 4


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_reach_of_the_buffer_descriptors(tmp_path):
    """Which inputs and filter banks the kernel's ordinary form takes, on both sides of the limits."""
    assert build_and_run(tmp_path, REACH) == "0"
