// The launch of a pointwise convolution (tern_conv_point.hip): filters and blocks of 32 voxels to a wave, and
// workgroups, chosen from sizes alone.  Host code without HIP, so that a test can compile it by itself.
#pragma once
#include <stdint.h>

namespace tern {
namespace {

constexpr int kPointWaves = 4;           // waves of a workgroup

struct PointLaunch {
    int32_t nb, groups;                  // 32-filter blocks of a wave, waves that share a run of voxels
    int32_t six;                         // packed codes through 6-bit floats
    int32_t blocks_per_wave;
    int64_t gx;                          // workgroups along the voxels
};

// voxels: of a grid layer, of which there are `layers` (int32 output: one per batch item).
inline PointLaunch point_launch(int64_t voxels, int32_t layers, int32_t c_out, int32_t words, bool packed)
{
    PointLaunch l;
    const int32_t fb = (c_out + 31) / 32;
    const int64_t blocks = (voxels + 31) / 32;
    // Two filter blocks per wave where they come in pairs, fit the registers (up to four words) and the
    // launch still has a wave per SIMD.
    l.nb = fb % 2 == 0 && words <= 4 && blocks * layers * (fb / 2) >= 1024 ? 2 : 1;
    l.groups = fb / l.nb;
    const int64_t work = blocks * layers * l.groups;
    // Decisions through 6-bit floats once waves have a second block (one filter block: a third; from five words on, whose
    // products hide part of the shifts, a fifth), which pays for the operands that they set up; with fewer they are
    // shifted in.  Shifted and through the floats: 128 -> 28 channels on 100 thousand voxels 3.1 and 3.2 us, 256 -> 28 on
    // 17 thousand 3.13 and 3.35, 256 -> 256 on 38 thousand 6.1 and 6.6; 256 -> 8 on 1.1 million 15.8 and 15.0.
    l.six = packed && work > (words > 4 ? 16384 : fb == 1 ? 8192 : 3072);
    // Blocks per wave: as many as leave all waves resident, since setting a wave up (filters, cut points) costs as much as
    // two blocks and one that waits for another's end comes late.  Four waves to a SIMD, three where the floats' registers
    // hold no more (two filter blocks of three and four words): 128 -> 64 channels on 130 thousand voxels 4.3 us shifted
    // with four waves, 4.8 through the floats with four and 3.8 with three; 96 -> 64 on 130 thousand 4.6 and 4.0; 128 -> 64
    // on 885 thousand 11.4 and 10.8.  Three also rather than four of one block each (64 -> 64 on 130 thousand 3.8 and 3.4).
    // int32: eight where several groups write sums from up to three words: a block's stores take longer than the setting up
    // (32 -> 256 channels on 2 x 26 675 voxels 16.4 us with four, 12.4; one group of few filters 3.9 and 4.3, eight
    // words -> 128 channels 19.7 and 22.0).
    const bool three = l.six && words <= 4 && ((l.nb == 2 && words > 2) || work <= 4096);
    const int64_t wanted = three ? 3072 : !packed && l.groups > 1 && words <= 3 ? 8192 : 4096;
    // Groups write neighbouring words of the same voxels.  Workgroups go to the eight XCDs in turn, so with a multiple of
    // eight to a group those of the same voxels share an L2, where their words make whole lines (the workgroups that
    // fill up find nothing to do): 96 -> 128 channels on 262 112 voxels, six blocks to a wave, 342 workgroups to a group
    // 10.7 us, 344 9.0; 64 -> 256 on 270 thousand, nine blocks, 17.8 and 11.2.  int32 sums are whole lines already
    // (32 -> 256 channels on 11 550 voxels 5.1 us, filled up 5.4).
    const bool fill_up = packed && l.groups > 1 && words <= 4;
    // (128 -> 512 on 846 thousand: at most 64 blocks 86 us, 69 blocks, one round of waves, 68)
    const int64_t most = l.six ? 256 : 64;
    int64_t per = (work + wanted - 1) / wanted;
    if (per > most) per = most;
    for (;; ++per) {
        l.gx = (blocks + kPointWaves * per - 1) / (kPointWaves * per);
        if (!fill_up) break;
        l.gx = (l.gx + 7) / 8 * 8;
        // (waves beyond those that are resident would come after the others)
        if (!l.six || per >= most || l.gx == 8 || l.gx * l.groups * kPointWaves <= wanted) break;
    }
    l.blocks_per_wave = (int32_t)per;
    return l;
}

}  // namespace
}  // namespace tern
