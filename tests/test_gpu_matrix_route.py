"""The default tiled convolution (inner products on the matrix cores) at the edges of its tiles, words and
limits, against the oracle, and against the bit-count kernels over random geometries.  Everything is
integers: equality is exact."""
import numpy as np
import pytest

import oracle
import synth
from oracle import ConvGeom

pytestmark = pytest.mark.gpu

CO_BLOCK = 3     # a tuning override: the thread gets the bit-count kernels


@pytest.fixture(scope="module")
def G():
    import torch
    import paper_1801_09449_amd as T
    from tests import gpu_util
    T.lib()
    assert torch.cuda.is_available()
    return gpu_util


def check(G, c):
    acc, packed = G.run_case(c)
    want = oracle.conv3d(c.act, c.wgt, ConvGeom(c.k, c.stride, c.pad, c.dil))
    np.testing.assert_array_equal(acc, want)
    np.testing.assert_array_equal(packed, oracle.pack(oracle.threshold(want, c.lo, c.hi)))


EDGES = [
    # name, n, c_in, c_out, vol, k, stride, pad, dil
    ("one_voxel",       1,  64,  64, (1, 1, 1),    3, 1, 1, 1),
    ("tile_minus_one",  1,  64,  64, (7, 7, 15),   3, 1, 1, 1),
    ("tile_plus_one",   2,  64,  33, (9, 9, 17),   3, 1, 1, 1),
    ("one_filter",      1,  64,   1, (8, 8, 8),    3, 1, 1, 1),
    ("three_blocks",    1,  64,  65, (8, 8, 8),    3, 1, 1, 1),
    ("odd_words",       1,  96, 128, (6, 9, 10),   3, 1, 1, 1),
    ("odd_entries",     1,  96,  32, (5, 5, 5),    1, 2, 0, 1),
    ("even_entries",    1,  32,  32, (5, 8, 9),    (2, 3, 3), 1, 1, 1),
    ("five_words",      1, 130,  64, (4, 9, 8),    3, 1, 1, 1),
    ("taps_64",         1,  33,  32, (6, 6, 6),    4, 1, 0, 1),
    ("taps_65",         1,  33,  32, (7, 6, 15),   (1, 5, 13), 1, 0, 1),
    ("taps_125",        1,  64,  32, (7, 8, 9),    5, 1, 2, 1),
    ("taps_128",        1,  64,  32, (4, 9, 10),   (2, 8, 8), 1, 0, 1),
    ("taps_129",        1,  64,  32, (4, 5, 45),   (1, 3, 43), 1, 0, 1),
    ("c1",              1,   1,  32, (9, 9, 9),    3, 1, 1, 1),
    ("c2_even_taps",    1,   2,  40, (5, 9, 8),    (1, 2, 2), 1, 0, 1),
    ("c5",              1,   5,  32, (6, 8, 9),    3, 2, 1, 1),
    ("c16",             2,  16,  64, (6, 8, 9),    3, 1, 2, 2),
    ("many_waves",      1,  32, 256, (6, 24, 24),  3, 1, 1, 1),
    ("large_waves",     1,  64, 128, (20, 40, 44), 3, 1, 1, 1),
    ("plane",           1, 128, 128, (1, 65, 33),  (1, 3, 3), 1, (0, 1, 1), 1),
    ("planes",          7,  64,  64, (1, 33, 31),  (1, 3, 3), 1, 0, 1),
    ("wide_halo",       1, 256,  32, (10, 11, 12), 3, 2, 3, 3),
]


@pytest.mark.parametrize("spec", EDGES, ids=[s[0] for s in EDGES])
def test_edges_of_tiles_words_and_taps(G, spec):
    name, n, ci, co, vol, k, s, p, d = spec
    check(G, synth.conv_case("mx_" + name, n, ci, co, vol, k, s, p, d, p0_w=0.5, p0_a=0.4, seed=801))


@pytest.mark.parametrize("sign", [1, -1])
def test_largest_sums_and_cut_points_around_them(G, sign):
    """All codes equal: every product is +1 (or -1) and the sums are the largest a shape can give; cut
    points one below, at and one above them, and the ends of the int32 range."""
    c = synth.conv_case("mx_sums", 1, 1024, 40, (4, 5, 6), seed=802)
    c.act[:] = 1
    c.wgt[:] = sign
    top = sign * 27 * 1024
    i32 = np.iinfo(np.int32)
    pairs = [(top - 1, top - 1), (top, top), (top + 1, top + 1), (top, top - 1), (i32.min, i32.max),
             (i32.max, i32.max), (i32.min, i32.min), (-(1 << 21) - 5, (1 << 21) + 5)]
    c.lo = np.array([pairs[i % 8][0] for i in range(40)], np.int32)
    c.hi = np.array([pairs[i % 8][1] for i in range(40)], np.int32)
    check(G, c)


@pytest.mark.parametrize("ci,co,vol,k", [(256, 256, (4, 8, 9), 3), (512, 32, (1, 9, 17), (1, 3, 3)), (96, 70, (6, 7, 8), 3),
                                         (32, 32, (9, 8, 8), 3), (16, 40, (8, 9, 8), 3), (160, 64, (5, 6, 7), (3, 3, 2)),
                                         (64, 128, (8, 8, 8), 5)])
def test_steps_split_over_waves(G, ci, co, vol, k):
    """Small launches share a tile's steps among waves that add their sums in LDS: every output is written
    (the buffer starts as garbage) and right, for even, odd and tap-packed word layouts and a batch."""
    import torch
    import paper_1801_09449_amd as T
    c = synth.conv_case("mx_split", 2, ci, co, vol, k, 1, 1, 1, seed=820 + ci, p0_a=0.4)
    act, bank = T.tern_pack(G.dev(c.act)), T.tern_pack_filters(G.dev(c.wgt))
    want = oracle.conv3d(c.act, c.wgt, ConvGeom(c.k, c.stride, c.pad, c.dil))
    g = dict(k=c.k, stride=c.stride, pad=c.pad, dil=c.dil)
    acc = torch.full(want.shape, 12345, dtype=torch.int32, device="cuda")
    T.tern_conv3d(act, ci, bank, co, out=acc, **g)
    assert T.tern_last_launch()["tap_split"] > 1
    packed = torch.full((2,) + want.shape[2:] + (2, T.tern_words(co)), -3,
                        dtype=torch.int32, device="cuda")
    T.tern_conv3d(act, ci, bank, co, thr_lo=G.dev(c.lo), thr_hi=G.dev(c.hi), out=packed, **g)
    assert T.tern_last_launch()["tap_split"] > 1
    np.testing.assert_array_equal(acc.cpu().numpy(), want)
    np.testing.assert_array_equal(G.words(packed), oracle.pack(oracle.threshold(want, c.lo, c.hi)))


ONE_SIDED = [  # n, c_in, c_out, vol, k, pad: split, tiled in small and in large waves, pointwise with even and odd words
    (1, 256, 64, (4, 8, 9), 3, 1), (1, 16, 40, (8, 9, 8), 3, 1), (2, 128, 64, (24, 40, 41), 3, 1), (1, 33, 32, (30, 33, 31), 3, 1),
    (1, 64, 128, (20, 40, 44), 3, 1), (2, 64, 64, (5, 9, 31), 1, 0), (1, 160, 40, (5, 9, 31), 1, 0), (1, 300, 40, (5, 9, 31), 1, 0)]


@pytest.mark.parametrize("kind", ["ternary", "binary", "digits"])
@pytest.mark.parametrize("n,ci,co,vol,k,pad", ONE_SIDED)
def test_one_cut_point_out_of_reach_and_the_other_among_the_sums(G, kind, n, ci, co, vol, k, pad):
    """The sums start from the upper cut point, clamped beyond every sum: with that one at the end of its range
    and the lower one among the sums, codes are right only if no product added to a start of 2^21 loses its
    last bit (and the other way round)."""
    import torch
    import paper_1801_09449_amd as T
    c = synth.conv_case("mx_one", n, ci, co, vol, k, 1, pad, 1, seed=850 + ci, p0_a=0.4)
    w = np.where(c.wgt < 0, -1, 1).astype(np.int8) if kind == "binary" else c.wgt
    act, g = T.tern_pack(G.dev(c.act)), dict(k=c.k, stride=c.stride, pad=c.pad, dil=c.dil)
    if kind == "binary":
        call = lambda **kw: T.tern_conv3d(act, ci, T.tern_pack_filters_binary(G.dev(w)), co, binary=True, **g, **kw)
    elif kind == "digits":
        pooled, c2 = T.tern_pool_digits(act, ci, (1, 1, 1))
        call = lambda **kw: T.tern_conv3d(pooled, c2, T.tern_pack_filters(G.dev(T.tern_digits_weights(w))), co, digits=True, **g, **kw)
    else:
        call = lambda **kw: T.tern_conv3d(act, ci, T.tern_pack_filters(G.dev(w)), co, **g, **kw)
    want = oracle.conv3d(c.act, w, ConvGeom(c.k, c.stride, c.pad, c.dil))
    i32 = np.iinfo(np.int32)
    mid = np.median(want.transpose(1, 0, 2, 3, 4).reshape(co, -1), axis=1).astype(np.int32) + np.arange(co, dtype=np.int32) % 3 - 1
    ends = [(mid, i32.max), (mid, (1 << 21) + 1), (mid, (1 << 21) - 1), (i32.min, mid), (-(1 << 21) - 1, mid), (mid, mid), (mid + 1, mid)]
    for lo, hi in ends:
        lo, hi = (np.broadcast_to(np.asarray(v, np.int32), (co,)).copy() for v in (lo, hi))
        got = call(thr_lo=G.dev(lo), thr_hi=G.dev(hi))
        torch.cuda.synchronize()
        np.testing.assert_array_equal(G.words(got), oracle.pack(oracle.threshold(want, lo, hi)), err_msg=str((lo[:3], hi[:3])))


def reference(act, w, pad):
    """Cross-correlation at stride 1 by one float32 product per tap (sums below 2^24: exact), int32 on the GPU."""
    import torch
    a, wt = act.float(), w.float()
    x = torch.nn.functional.pad(a, (pad[2], pad[2], pad[1], pad[1], pad[0], pad[0]))
    o = [x.shape[2 + i] - w.shape[2 + i] + 1 for i in range(3)]
    out = torch.zeros((act.shape[0], w.shape[0], o[0] * o[1] * o[2]), device="cuda")
    for z in range(w.shape[2]):
        for y in range(w.shape[3]):
            for v in range(w.shape[4]):
                tap = wt[:, :, z, y, v].contiguous()
                for i in range(act.shape[0]):
                    out[i] += tap @ x[i, :, z:z + o[0], y:y + o[1], v:v + o[2]].reshape(w.shape[1], -1)
    return out.view(act.shape[0], w.shape[0], *o).int()


TABLES = [
    # A wave holds the offsets of its first two steps (one entry each, or two where words are odd in number) and of the next 48
    # entries: entries on both sides of the first and second renewal.  (small or large waves, filters of a wave, waves that
    # share the steps, renewals): n, c_in, c_out, output, kernel
    ((1, 32, 1, 0), 4, 32, 32, (1, 160, 197), (1, 4, 13)), ((1, 32, 1, 1), 4, 32, 32, (1, 160, 197), (1, 1, 53)),
    ((1, 32, 1, 2), 4, 32, 32, (1, 300, 337), (1, 1, 101)), ((1, 32, 1, 0), 1, 64, 32, (1, 400, 437), (1, 1, 49)),
    ((1, 32, 1, 1), 1, 64, 32, (1, 400, 437), (1, 3, 17)), ((1, 32, 1, 1), 1, 64, 32, (1, 400, 437), (1, 7, 14)),
    ((1, 32, 1, 2), 1, 64, 32, (1, 400, 437), (1, 9, 11)), ((1, 32, 4, 2), 1, 480, 32, (20, 40, 43), (3, 3, 3)),
    ((1, 32, 2, 1), 1, 512, 64, (20, 40, 43), (2, 3, 3)), ((1, 64, 1, 1), 1, 224, 256, (20, 40, 43), (1, 3, 3)),
    ((1, 64, 1, 2), 1, 768, 256, (20, 40, 43), (1, 3, 3)), ((1, 64, 2, 2), 2, 480, 256, (12, 24, 27), (2, 3, 3)),
    ((1, 32, 1, 0), 4, 16, 32, (1, 160, 197), (1, 4, 13)), ((1, 32, 1, 1), 4, 16, 32, (1, 160, 197), (1, 1, 53)),
    ((1, 32, 1, 2), 4, 16, 32, (1, 300, 337), (1, 1, 101)),
    ((2, 32, 1, 0), 4, 32, 32, (1, 240, 277), (1, 4, 13)), ((2, 32, 1, 1), 4, 32, 32, (1, 240, 277), (1, 1, 53)),
    ((2, 32, 1, 1), 4, 32, 32, (1, 240, 277), (1, 10, 10)), ((2, 32, 1, 2), 4, 32, 32, (1, 240, 277), (1, 1, 101)),
    ((2, 64, 1, 1), 4, 32, 64, (1, 300, 337), (1, 1, 53)), ((2, 64, 1, 2), 4, 32, 64, (1, 300, 337), (1, 8, 13)),
    ((2, 32, 1, 0), 4, 64, 32, (1, 240, 277), (1, 5, 10)), ((2, 32, 1, 1), 4, 64, 32, (1, 240, 277), (1, 3, 17)),
    ((2, 32, 1, 2), 4, 64, 32, (1, 240, 277), (1, 9, 11)), ((2, 64, 1, 1), 4, 64, 64, (1, 300, 337), (1, 7, 14)),
    ((2, 64, 1, 2), 4, 64, 64, (1, 300, 337), (1, 1, 101)), ((2, 32, 1, 1), 4, 16, 32, (1, 240, 277), (1, 1, 53)),
    ((2, 32, 1, 2), 4, 16, 32, (1, 240, 277), (1, 1, 101)),
    ("digits", (1, 32, 1, 2), 1, 480, 256, (20, 40, 43), (1, 3, 3)), ("digits", (1, 32, 1, 2), 1, 256, 256, (20, 40, 43), (3, 3, 3)),
    ("digits", (2, 64, 1, 2), 1, 256, 256, (30, 60, 63), (3, 3, 3))]


@pytest.mark.parametrize("case", TABLES, ids=lambda c: "-".join(map(str, c)).replace(" ", ""))
def test_entries_of_a_wave_and_its_tables(G, case):
    import torch
    import paper_1801_09449_amd as T
    digits = case[0] == "digits"
    form, n, ci, co, out, k = case[-6:]
    gen = torch.Generator("cuda").manual_seed(817)
    vol = tuple(o + a - 1 for o, a in zip(out, k))
    act = torch.randint(-1, 2, (n, ci) + vol, generator=gen, device="cuda", dtype=torch.int8)
    w = torch.randint(-1, 2, (co, ci) + k, generator=gen, device="cuda", dtype=torch.int8)
    words = T.tern_words(ci)
    entries = k[0] * k[1] * k[2] * words // (1 if words % 2 else 2)
    lo, hi = torch.full((co,), -9, dtype=torch.int32, device="cuda"), torch.arange(co, device="cuda", dtype=torch.int32) % 21
    for binary in (False,) if digits else (False, True):
        wt = torch.where(w < 0, w, torch.ones_like(w)) if binary else w
        a, c2 = T.tern_pack(act), ci
        if digits:
            a, c2 = T.tern_pool_digits(a, ci, (1, 1, 1))
            bank = T.tern_pack_filters(G.dev(T.tern_digits_weights(wt.cpu().numpy())))
        else:
            bank = T.tern_pack_filters_binary(wt) if binary else T.tern_pack_filters(wt)
        want = reference(act, wt, (0, 0, 0))
        for kw in ({}, dict(thr_lo=lo, thr_hi=hi)):
            got = T.tern_conv3d(a, c2, bank, co, k=k, pad=0, binary=binary, digits=digits, **kw)
            plan = T.tern_last_launch()
            renewals = (entries // plan["tap_split"] - (5 if words % 2 else 3)) // 48
            if not kw and not binary:
                assert (plan["voxels_per_lane"], plan["channels_per_pass"], plan["tap_split"], renewals) == form
            assert bool(renewals) == bool(form[3])
            assert torch.equal(got, T.tern_threshold_pack(want, lo, hi) if kw else want), (binary, bool(kw))


@pytest.mark.parametrize("binary", [False, True])
@pytest.mark.parametrize("n,ci,co,vol,k", [
    (1, 64, 32, (8, 9, 10), (5, 5, 6)), (1, 96, 70, (7, 20, 21), (5, 5, 6)), (1, 64, 70, (24, 40, 40), (3, 5, 9)), (2, 64, 128, (20, 40, 40), (3, 5, 9)),
    (1, 64, 64, (64, 64, 64), (1, 3, 43)), (1, 32, 128, (48, 64, 72), (3, 5, 9)), (1, 32, 20, (64, 64, 72), (3, 5, 9)),
    (1, 1, 32, (16, 16, 16), (5, 5, 6)), (1, 4, 70, (40, 40, 40), (5, 5, 6)), (1, 16, 128, (64, 64, 64), (5, 5, 6)), (20, 64, 64, (1, 90, 84), (1, 12, 12))])
def test_bit_count_plans_where_the_matrix_kernel_does_not_go(G, n, ci, co, vol, k, binary):
    """More than 128 taps, without an override: the plans that the bit-count kernels choose by themselves for
    small, middling and large launches, whole and ragged filter counts, one word, several and several taps to
    a word, volumes and stacks of planes."""
    import torch
    import paper_1801_09449_amd as T
    gen = torch.Generator("cuda").manual_seed(860 + ci)
    act = torch.randint(-1, 2, (n, ci) + vol, generator=gen, device="cuda", dtype=torch.int8)
    w = torch.randint(-1, 2, (co, ci) + k, generator=gen, device="cuda", dtype=torch.int8)
    if binary:
        w = torch.where(w < 0, w, torch.ones_like(w))
    pad = tuple(x // 2 for x in k)
    want = reference(act, w, pad)
    a, bank = T.tern_pack(act), T.tern_pack_filters_binary(w) if binary else T.tern_pack_filters(w)
    got = T.tern_conv3d(a, ci, bank, co, k=k, pad=pad, binary=binary)
    assert T.tern_last_launch()["kernel"] == T.KERNEL_TILED
    assert torch.equal(got, want)
    lo, hi = torch.full((co,), -3, dtype=torch.int32, device="cuda"), torch.arange(co, device="cuda", dtype=torch.int32) % 7
    packed = T.tern_conv3d(a, ci, bank, co, k=k, pad=pad, thr_lo=lo, thr_hi=hi, binary=binary)
    v = (1, -1, 1, 1, 1)
    codes = (want > hi.view(v)).to(torch.int8) - ((want < lo.view(v)) & ~(want > hi.view(v))).to(torch.int8)
    assert torch.equal(packed, T.tern_pack(codes))


@pytest.mark.parametrize("n,ci,co,vol,k", [
    (1, 24, 64, (60, 80, 70), (3, 3, 3)), (2, 32, 70, (41, 53, 75), (3, 3, 3)), (1, 64, 33, (75, 81, 113), (3, 3, 3)), (16, 8, 40, (1, 181, 203), (1, 3, 3)),
    (8, 16, 64, (1, 150, 171), (1, 3, 3)), (3, 96, 160, (1, 190, 171), (1, 3, 3))])
def test_int32_sums_in_rows_of_16_voxels(G, n, ci, co, vol, k):
    """Large int32 results, whose waves are turned along x, with remainders along every axis and in the filters."""
    import torch
    import paper_1801_09449_amd as T
    gen = torch.Generator("cuda").manual_seed(870 + ci)
    act = torch.randint(-1, 2, (n, ci) + vol, generator=gen, device="cuda", dtype=torch.int8)
    w = torch.randint(-1, 2, (co, ci) + k, generator=gen, device="cuda", dtype=torch.int8)
    pad = tuple(x // 2 for x in k)
    want = reference(act, w, pad)
    got = T.tern_conv3d(T.tern_pack(act), ci, T.tern_pack_filters(w), co, k=k, pad=pad, out=torch.full_like(want, 12345))
    assert T.tern_last_launch()["voxels_per_lane"] == 2
    assert torch.equal(got, want)
    wb = torch.where(w < 0, w, torch.ones_like(w))
    got = T.tern_conv3d_binary(T.tern_pack(act), ci, T.tern_pack_filters_binary(wb), co, k, 1, pad, 1)
    assert torch.equal(got, reference(act, wb, pad))


@pytest.mark.parametrize("n,ci,co,vol,k,s,p,d,digits", [
    (5, 96, 8, (2, 3, 2), (3, 1, 1), 2, (3, 0, 0), 3, False), (2, 96, 19, (1, 4, 1), (3, 1, 1), 2, (3, 0, 0), 3, False),
    (2, 288, 2, (96, 2, 3), 1, 2, 0, 1, True), (1, 160, 32, (67, 2, 83), 1, (1, 2, 2), 0, 1, True),
    (1, 32, 8, (79, 6, 11), 2, 2, 3, 3, False), (2, 32, 8, (1, 69, 5), 3, (1, 2, 2), 3, 3, False),
    (1, 330, 14, (3, 48, 4), 1, (1, 2, 2), 0, 1, False), (1, 287, 70, (2, 1, 7), (3, 1, 1), 2, (1, 0, 0), 1, False)])
def test_waves_that_only_help_to_fill(G, n, ci, co, vol, k, s, p, d, digits):
    """Small launches with a wide halo tile have more waves than filter groups and splits: the others take part
    in the fill and in the barriers and write nothing (int32 and packed output into buffers of garbage)."""
    import torch
    import paper_1801_09449_amd as T
    c = synth.conv_case("mx_help", n, ci, co, vol, k, s, p, d, seed=840 + ci, p0_a=0.4)
    g = dict(k=c.k, stride=c.stride, pad=c.pad, dil=c.dil)
    act = T.tern_pack(G.dev(c.act))
    if digits:
        act, c2 = T.tern_pool_digits(act, ci, (1, 1, 1))
        bank = T.tern_pack_filters(G.dev(T.tern_digits_weights(c.wgt)))
        call = lambda **kw: T.tern_conv3d(act, c2, bank, co, digits=True, **g, **kw)
    else:
        bank = T.tern_pack_filters(G.dev(c.wgt))
        call = lambda **kw: T.tern_conv3d(act, ci, bank, co, **g, **kw)
    want = oracle.conv3d(c.act, c.wgt, ConvGeom(c.k, c.stride, c.pad, c.dil))
    acc = torch.full(want.shape, 12345, dtype=torch.int32, device="cuda")
    call(out=acc)
    plan = T.tern_last_launch()
    assert plan["kernel"] == T.KERNEL_TILED
    assert plan["threads"] // 64 > plan["tap_split"] * -(-co // plan["channels_per_pass"]), plan
    packed = torch.full((n,) + want.shape[2:] + (2, T.tern_words(co)), -3, dtype=torch.int32, device="cuda")
    call(thr_lo=G.dev(c.lo), thr_hi=G.dev(c.hi), out=packed)
    np.testing.assert_array_equal(acc.cpu().numpy(), want)
    np.testing.assert_array_equal(G.words(packed), oracle.pack(oracle.threshold(want, c.lo, c.hi)))


def random_form(i):
    u = synth.uniform_int(16, 0, 10 ** 6, 12000 + i, 11)
    pick = lambda j, lo, hi: int(lo + u[j] % (hi - lo + 1))
    c_in = [1, 4, 16, 31, 32, 64, 65, 96, 128, 256, 512][pick(0, 0, 10)]
    k = tuple(pick(1 + a, 1, 4) for a in range(3))
    dil = tuple(pick(4 + a, 1, 3) for a in range(3))
    pad = tuple(pick(7 + a, 0, 3) for a in range(3))
    vol = tuple(max(pick(10 + a, 1, 26), dil[a] * (k[a] - 1) + 1 - 2 * pad[a]) for a in range(3))
    return synth.conv_case("mx_rnd%d" % i, pick(13, 1, 3), c_in, [8, 32, 33, 64, 70, 128, 160, 256][pick(14, 0, 7)], vol, k,
                           tuple(1 + (pick(15, 0, 7) >> a & 1) for a in range(3)), pad, dil, seed=803 + i, p0_a=0.4)


@pytest.mark.parametrize("block", range(4))
def test_same_integers_as_the_bit_count_kernels(G, block):
    """Ternary and binary filters, int32 and packed output, over random geometries: the default launch
    against the one that an override sends to the bit-count kernels."""
    import torch
    import paper_1801_09449_amd as T
    for i in range(20 * block, 20 * block + 20):
        c = random_form(i)
        act, w = T.tern_pack(G.dev(c.act)), G.dev(c.wgt)
        ci, co = c.act.shape[1], c.wgt.shape[0]
        g = dict(k=c.k, stride=c.stride, pad=c.pad, dil=c.dil)
        wb = torch.where(w < 0, w, torch.ones_like(w))
        calls = []
        for fn, bank in ((T.tern_conv3d, T.tern_pack_filters(w)), (T.tern_conv3d_binary, T.tern_pack_filters_binary(wb))):
            calls.append(lambda fn=fn, bank=bank: fn(act, ci, bank, co, **g))
            calls.append(lambda fn=fn, bank=bank: fn(act, ci, bank, co, thr_lo=G.dev(c.lo), thr_hi=G.dev(c.hi), **g))
        for j, call in enumerate(calls):
            here = call()
            T.tern_set_option(CO_BLOCK, 16)
            try:
                there = call()
            finally:
                T.tern_set_option(CO_BLOCK, 0)
            assert torch.equal(here, there), (i, j, c.act.shape, c.wgt.shape, g)


@pytest.mark.parametrize("words", range(1, 10))
@pytest.mark.parametrize("vox", [(1, 1, 1), (1, 1, 31), (1, 3, 11), (5, 16, 27)], ids=["1", "31", "33", "2160"])
def test_pointwise_blocks_and_words(G, words, vox):
    """Single-tap convolutions: every word count the pointwise kernel takes (and the first it does not),
    blocks of 32 voxels with and without a remainder, a batch (folded for packed output), filter counts
    with one block, two and a remainder, ternary and binary filters."""
    import torch
    import paper_1801_09449_amd as T
    for co, n in ((1, 1), (33, 2), (64, 3), (200, 1)):
        c = synth.conv_case("px", n, 32 * words - (words & 3), co, vox, k=1, pad=0, seed=830 + words, p0_a=0.4)
        check(G, c)
        assert (T.tern_last_launch()["kernel"] == T.KERNEL_POINTWISE) == (words <= 8)
        w = np.where(c.wgt < 0, -1, 1).astype(np.int8)
        got = T.tern_conv3d_binary(T.tern_pack(G.dev(c.act)), c.act.shape[1], T.tern_pack_filters_binary(G.dev(w)), co, 1, 1, 0, 1)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy(), oracle.conv3d(c.act, w, ConvGeom(c.k, c.stride, c.pad, c.dil)))


def test_pointwise_many_blocks_per_wave(G):
    """More blocks than waves: a wave walks several, the last one fewer and a part of one."""
    check(G, synth.conv_case("px_many", 1, 64, 64, (64, 65, 67), k=1, pad=0, seed=829, p0_a=0.4))


@pytest.mark.parametrize("ci,co", [(32, 100), (96, 64), (130, 200), (224, 129), (256, 96)])
@pytest.mark.parametrize("vol", [(1, 41, 99), (19, 50, 53)], ids=["one_or_two_blocks", "several"])
def test_pointwise_runs_shorter_and_longer_than_the_fetch_is_ahead(G, ci, co, vol):
    """Waves with fewer blocks than are fetched ahead, and with more and a remainder."""
    check(G, synth.conv_case("px_runs", 2, ci, co, vol, k=1, pad=0, seed=832 + ci, p0_a=0.4))


@pytest.mark.parametrize("ci,co,vox", [
    (32, 32, 270001), (64, 64, 100001), (40, 96, 60001), (96, 128, 50001), (96, 40, 262113), (128, 64, 98305),    # through 6-bit floats
    (100, 200, 20011), (128, 70, 33333), (160, 64, 270001), (256, 300, 60001), (224, 8, 530001),
    (64, 100, 4099), (128, 256, 9001), (256, 256, 33001)])                                                        # shifted in
def test_pointwise_packed_large_and_filled_up(G, ci, co, vox):
    """Packed codes at the edges of the launch's rules: 6-bit floats and shifts, one and two filter blocks to a wave,
    groups whose workgroups are filled up to a multiple of eight; a part block at the end."""
    import torch
    import paper_1801_09449_amd as T
    g = torch.Generator(device="cuda").manual_seed(ci + co)
    act = torch.randint(-1, 2, (1, ci, 1, 1, vox), generator=g, device="cuda", dtype=torch.int8)
    w = torch.randint(-1, 2, (co, ci, 1, 1, 1), generator=g, device="cuda", dtype=torch.int8)
    lo = torch.randint(-9, 3, (co,), generator=g, device="cuda", dtype=torch.int32)
    hi = lo + torch.randint(-2, 12, (co,), generator=g, device="cuda", dtype=torch.int32)
    a = T.tern_pack(act)
    for binary in (False, True):
        wb = torch.where(w < 0, w, torch.ones_like(w)) if binary else w
        acc = reference(act, wb, (0, 0, 0))
        want = T.tern_threshold_pack(acc, lo, hi)
        fn, pack = (T.tern_conv3d_binary, T.tern_pack_filters_binary) if binary else (T.tern_conv3d, T.tern_pack_filters)
        assert torch.equal(fn(a, ci, pack(wb), co, 1, 1, 0, 1, thr_lo=lo, thr_hi=hi), want)
        assert T.tern_last_launch()["kernel"] == T.KERNEL_POINTWISE


@pytest.mark.parametrize("ci", [32, 192])
def test_pointwise_batches_beyond_the_grid(G, ci):
    """More batch items than a grid has layers, int32 and packed output, binary and ternary filters."""
    import torch
    import paper_1801_09449_amd as T
    c = synth.conv_case("px_batch", 65539, ci, 3, (1, 1, 2), k=1, pad=0, seed=831, p0_a=0.4)
    check(G, c)
    w = np.where(c.wgt < 0, -1, 1).astype(np.int8)
    got = T.tern_conv3d_binary(T.tern_pack(G.dev(c.act)), ci, T.tern_pack_filters_binary(G.dev(w)), 3, 1, 1, 0, 1)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got.cpu().numpy(), oracle.conv3d(c.act, w, ConvGeom(c.k, c.stride, c.pad, c.dil)))


@pytest.mark.parametrize("ci,co,vol,k,stride,binary", [
    (64, 64, (1, 16400, 16400), (1, 3, 3), 1, False),       # one plane of 4.3 GB
    (40, 70, (4, 9000, 8500), (3, 3, 3), 1, False),         # 1.2 GB each, four to a tile; a last word part empty
    (96, 20, (4, 9400, 9800), (2, 3, 3), 2, True),          # odd word count, strided, binary filters
])
def test_planes_of_a_tile_beyond_four_gigabytes(G, ci, co, vol, k, stride, binary):
    """Tiles whose planes together span more than 4 GB stay on the matrix cores.  Against the same convolution of boxes
    cut out of the volume: its corners and its middle."""
    import torch
    import paper_1801_09449_amd as T
    d, h, w = vol
    g = torch.Generator(device="cuda").manual_seed(ci)
    act = torch.randint(-2**31, 2**31 - 1, (1, d, h, w, 2, T.tern_words(ci)), generator=g, device="cuda", dtype=torch.int32)
    if ci % 32:
        act[..., -1] &= (1 << ci % 32) - 1
    act[:, :, :, :, 1] &= act[:, :, :, :, 0]
    wgt = torch.randint(-1, 2, (co, ci) + k, generator=g, device="cuda", dtype=torch.int8)
    bank = T.tern_pack_filters_binary(torch.where(wgt < 0, wgt, torch.ones_like(wgt))) if binary else T.tern_pack_filters(wgt)
    lo, hi = (torch.full((co,), v, device="cuda", dtype=torch.int32) for v in (-8, 9))
    pad = tuple(min(1, a - 1) for a in k)
    st = (1 if d == 1 else stride, stride, stride)
    conv = lambda a, p: T.tern_conv3d(a, ci, bank, co, k, st, p, 1, thr_lo=lo, thr_hi=hi, binary=binary)
    got = conv(act, pad)
    plan = T.tern_last_launch()
    assert plan["kernel"] == T.KERNEL_TILED and (plan["voxels_per_lane"], plan["channels_per_pass"]) == (2, 32)
    for cy, cx in ((0, 0), (0, w - 300), (h - 300, 0), (h - 300, w - 300), (h // 2, w // 2)):
        y0, x0 = cy // stride * stride, cx // stride * stride
        box = act[:, :, y0:y0 + 300, x0:x0 + 300].contiguous()
        want = conv(box, pad)
        oy, ox = y0 // stride, x0 // stride
        n, m = want.shape[2], want.shape[3]
        # outputs whose taps are all in the box, or beyond the volume's own edge
        ys, ye = (0 if y0 == 0 else 2), (n if y0 + 300 >= h else n - 2)
        xs, xe = (0 if x0 == 0 else 2), (m if x0 + 300 >= w else m - 2)
        assert torch.equal(got[:, :, oy + ys:oy + ye, ox + xs:ox + xe], want[:, :, ys:ye, xs:xe]), (cy, cx)
    del act, got
    torch.cuda.empty_cache()


@pytest.mark.parametrize("ci,vol,k,co,form", [
    # even and odd words: rows of pairs; single words, an odd number of them
    (256, (1, 4, 9), (1, 11, 11), 1 << 19, (1, 64)), (288, (1, 4, 9), (1, 11, 11), 1 << 19, (1, 64)), (288, (1, 4, 9), (1, 11, 11), (1 << 19) - 32, (1, 32)),
    (1152, (2, 3, 5), (3, 3, 3), 1 << 19, (1, 64)), (1184, (2, 3, 5), (3, 3, 3), 1 << 19, (1, 64)), (1184, (2, 3, 5), (3, 3, 3), (1 << 19) - 40, (1, 32)),
    (256, (1, 90, 100), (1, 11, 11), 1 << 19, (2, 64)), (576, (8, 12, 14), (3, 3, 6), (1 << 19) - 32, (2, 32))])   # (waves of 128 voxels)
def test_filter_bank_beyond_four_gigabytes(G, ci, vol, k, co, form):
    """A bank that no buffer descriptor reaches, and the row past its end, against the same convolution with some of its filters."""
    import torch
    import paper_1801_09449_amd as T
    part, pad, cp = 2048, tuple(a // 2 for a in k), (co + 31) // 32 * 32
    gen = torch.Generator("cuda").manual_seed(ci)
    act = T.tern_pack(torch.randint(-1, 2, (1, ci) + vol, generator=gen, device="cuda", dtype=torch.int8))
    words = ci // 32
    wc = 1 + (words + 1) % 2
    bank = torch.randint(-2**31, 2**31 - 1, (k[0] * k[1] * k[2] * words // wc, cp, 2, wc), generator=gen, device="cuda", dtype=torch.int32)
    bank[:, :, 1] &= bank[:, :, 0]
    assert (bank.shape[0] + 1) * cp * 8 * wc > 0xf0000000
    lo, hi = torch.full((co,), -40, device="cuda", dtype=torch.int32), torch.arange(co, device="cuda", dtype=torch.int32) % 60
    small = vol[1] < 50
    acc = T.tern_conv3d(act, ci, bank.view(-1), co, k, 1, pad) if small else None
    packed = T.tern_conv3d(act, ci, bank.view(-1), co, k, 1, pad, thr_lo=lo, thr_hi=hi)
    plan = T.tern_last_launch()
    assert plan["kernel"] == T.KERNEL_TILED and (plan["voxels_per_lane"], plan["channels_per_pass"], plan["tap_split"]) == form + (1,)
    for a in (0, cp // 64 * 32 - part // 2, cp - part):
        few, n = bank[:, a:a + part].contiguous().view(-1), min(part, co - a)
        want = T.tern_conv3d(act, ci, few, n, k, 1, pad)
        if small:
            assert torch.equal(acc[:, a:a + n], want)
        assert torch.equal(packed[..., a // 32:(a + part) // 32], T.tern_threshold_pack(want, lo[a:a + n].contiguous(), hi[a:a + n].contiguous()))
    del bank, acc, packed, want
    torch.cuda.empty_cache()
