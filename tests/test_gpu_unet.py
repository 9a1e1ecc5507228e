"""GPU parity for the U-Net pieces around the ternary convolution: gather/concat on packed
tensors, 2-D (single-plane) convolutions, average pooling folded into the next convolution, the
real-weight prediction layer, and the whole Table 1 network, each against the CPU oracle on the
same seeded inputs.  Integer and bit results must match exactly; the float prediction layer
within the bound its summation order implies."""
import numpy as np
import pytest

import oracle
import synth
from oracle import ConvGeom

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    import paper_1801_09449_amd as T
    from tests import gpu_util
    T.lib()
    assert torch.cuda.is_available()
    return gpu_util


def tern(shape, seed, p0=0.35, tid=synth.T_ACT):
    return synth.ternary(shape, p0, seed, tid)


def gpu_pack(G, x):
    import paper_1801_09449_amd as T
    return T.tern_pack(G.dev(x))


# ---- tern_concat --------------------------------------------------------------------------------
@pytest.mark.parametrize("c,vol,up", [(5, (2, 3, 4), (1, 2, 2)), (33, (1, 5, 7), (1, 2, 2)), (64, (3, 4, 5), (2, 1, 3)),
                                      (70, (2, 2, 2), (3, 3, 3))])
def test_upsample_nearest(G, c, vol, up):
    import paper_1801_09449_amd as T
    x = tern((2, c) + vol, 5)
    got = T.tern_concat([(gpu_pack(G, x), c, up)])
    np.testing.assert_array_equal(G.words(got), oracle.pack(oracle.upsample_nearest(x, up)))


def test_centre_crop(G):
    import paper_1801_09449_amd as T
    x = tern((2, 40, 3, 9, 12), 6)
    want = oracle.centre_crop(x, (2, 4, 7))
    got = T.tern_concat([(gpu_pack(G, x), 40, 1, (0, 2, 2))], out_spatial=(2, 4, 7))
    np.testing.assert_array_equal(G.words(got), oracle.pack(np.ascontiguousarray(want)))


@pytest.mark.parametrize("chans", [(32, 32), (64, 64), (20, 50), (1, 1), (31, 33, 7), (96, 5, 40, 3), (7,) * 8])
def test_concat_any_channel_counts(G, chans):
    """Word-aligned and unaligned channel counts, up to the maximum number of sources."""
    import paper_1801_09449_amd as T
    parts = [tern((2, c, 2, 5, 6), 10 + i) for i, c in enumerate(chans)]
    got = T.tern_concat([(gpu_pack(G, p), p.shape[1]) for p in parts])
    want = oracle.pack(oracle.concat_channels(parts))
    assert got.shape[-1] == (sum(chans) + 31) // 32
    np.testing.assert_array_equal(G.words(got), want)


def test_decoder_step_upsample_crop_concat(G):
    """The decoder step of the U-Net: upsampled tensor first, centre-cropped skip tensor after."""
    import paper_1801_09449_amd as T
    low = tern((2, 48, 1, 6, 5), 31)
    skip = tern((2, 20, 1, 15, 13), 32)
    up = oracle.upsample_nearest(low, (1, 2, 2))
    want = oracle.concat_channels([up, oracle.centre_crop(skip, up.shape[2:])])
    first = tuple((s - u) // 2 for s, u in zip(skip.shape[2:], up.shape[2:]))
    got = T.tern_concat([(gpu_pack(G, low), 48, (1, 2, 2)), (gpu_pack(G, skip), 20, 1, first)],
                        out_spatial=up.shape[2:])
    np.testing.assert_array_equal(G.words(got), oracle.pack(want))


def test_concat_rejects_bad_arguments(G):
    import paper_1801_09449_amd as T
    a = gpu_pack(G, tern((1, 8, 2, 4, 4), 1))
    b = gpu_pack(G, tern((2, 8, 2, 4, 4), 2))
    with pytest.raises(T.TernError) as e:
        T.tern_concat([(a, 8), (b, 8)], out_spatial=(2, 4, 4))          # batch mismatch
    assert e.value.status == -3
    with pytest.raises(T.TernError) as e:
        T.tern_concat([(a, 8, 1, (0, 1, 0))], out_spatial=(2, 4, 4))    # crop runs past the source
    assert e.value.status == -3
    with pytest.raises(T.TernError) as e:
        T.tern_concat([(a, 8)] * 9, out_spatial=(2, 4, 4))              # too many sources
    assert e.value.status == -3


# ---- 2-D convolutions (single output plane) ---------------------------------------------------------
@pytest.mark.parametrize("n,ci,co,hw,k,stride", [(1, 32, 32, (17, 23), (1, 3, 3), 1), (3, 64, 40, (20, 19), (1, 3, 3), 1),
                                                 (2, 15, 32, (30, 26), (1, 3, 3), 1), (1, 128, 64, (33, 9), (1, 1, 1), 1),
                                                 (4, 8, 16, (21, 22), (1, 6, 6), (1, 2, 2)),
                                                 (5, 70, 33, (9, 40), (1, 3, 3), (1, 2, 1))])
def test_conv2d_single_plane(G, n, ci, co, hw, k, stride):
    """D = 1: a lane's voxels are stacked along y, and batch items are folded into planes for the
    packed output.  Both output modes against the oracle."""
    c = synth.conv_case("c2d", n, ci, co, (1,) + hw, k=k, stride=stride, pad=0, seed=n + ci)
    acc, packed = G.run_case(c)
    want = oracle.conv3d(c.act, c.wgt, ConvGeom(c.k, c.stride, c.pad, c.dil))
    np.testing.assert_array_equal(acc, want)
    np.testing.assert_array_equal(packed, oracle.pack(oracle.threshold(want, c.lo, c.hi)))


def test_conv_depth_one_kernel_on_a_volume_with_batch(G):
    """kd = 1 on D > 1 with N > 1 (planes independent: batch folded into depth), padded in-plane."""
    c = synth.conv_case("kd1", 3, 40, 24, (5, 12, 11), k=(1, 3, 3), pad=(0, 1, 1), seed=8)
    acc, packed = G.run_case(c)
    want = oracle.conv3d(c.act, c.wgt, ConvGeom(c.k, c.stride, c.pad, c.dil))
    np.testing.assert_array_equal(acc, want)
    np.testing.assert_array_equal(packed, oracle.pack(oracle.threshold(want, c.lo, c.hi)))


def test_first_layer_of_table1_stack_kernel(G):
    """Row #1 of Table 1: one input channel, kernel spanning the whole stack of 15 slices."""
    c = synth.conv_case("row1", 2, 1, 32, (15, 20, 22), k=(15, 3, 3), pad=0, seed=4)
    acc, packed = G.run_case(c)
    want = oracle.conv3d(c.act, c.wgt, ConvGeom(c.k, c.stride, c.pad, c.dil))
    assert want.shape[2] == 1
    np.testing.assert_array_equal(acc, want)
    np.testing.assert_array_equal(packed, oracle.pack(oracle.threshold(want, c.lo, c.hi)))


# ---- average pooling folded into the next convolution ----------------------------------------------
@pytest.mark.parametrize("vol,k,pool", [((1, 23, 21), (1, 3, 3), (1, 2, 2)), ((6, 10, 9), (3, 3, 3), (2, 2, 2)),
                                        ((1, 13, 11), (1, 1, 1), (1, 2, 2))])
def test_avgpool_folded_into_conv(G, vol, k, pool):
    import paper_1801_09449_amd as T
    x = tern((2, 24) + vol, 17)
    w = tern((40, 24) + k, 18, 0.5, synth.T_WGT)
    lo, hi = synth.threshold_pair(40, 19, lo=-6, hi=6)
    want = oracle.conv3d(oracle.pool_sum(x, pool), w, ConvGeom(k, (1, 1, 1), (0, 0, 0), (1, 1, 1)))
    wf = T.tern_fold_avgpool(w, pool)
    bank = T.tern_pack_filters(G.dev(wf))
    xp = gpu_pack(G, x)
    acc = T.tern_conv3d(xp, 24, bank, 40, wf.shape[2:], pool, 0, 1)
    np.testing.assert_array_equal(acc.cpu().numpy(), want)
    codes = T.tern_conv3d(xp, 24, bank, 40, wf.shape[2:], pool, 0, 1, thr_lo=G.dev(lo), thr_hi=G.dev(hi))
    np.testing.assert_array_equal(G.words(codes), oracle.pack(oracle.threshold(want, lo, hi)))


# ---- prediction layer ------------------------------------------------------------------------------
def real_conv_bound(w, b):
    """|fp32 result - exact| <= terms * 2^-24 * (|bias| + sum|w| of the filter), per output channel."""
    terms = w[0].size + 1
    mass = np.abs(w.astype(np.float64)).reshape(w.shape[0], -1).sum(axis=1) + np.abs(b.astype(np.float64))
    return terms * 2.0 ** -24 * mass


@pytest.mark.parametrize("ci,co,vol,k,stride,pad,dil", [(64, 2, (1, 20, 18), (1, 3, 3), 1, 0, 1),
                                                        (37, 5, (4, 6, 7), (3, 3, 3), (1, 2, 1), (1, 0, 2), (1, 1, 2)),
                                                        (8, 1, (3, 3, 3), (1, 1, 1), 1, 0, 1),
                                                        (300, 2, (3, 4, 5), (3, 3, 3), 1, 1, 1),     # filters too large for LDS
                                                        (130, 7, (2, 9, 70), (1, 3, 3), 1, (0, 1, 1), 1),
                                                        (64, 2, (1, 200, 170), (1, 1, 1), 1, 0, 1),         # tables: two words, two outputs
                                                        (40, 4, (1, 190, 180), (1, 1, 3), 1, (0, 0, 1), 1),  # the same, four, padded
                                                        (8, 3, (1, 190, 180), (1, 3, 3), 1, (0, 1, 1), 1),   # one word, padded
                                                        (130, 2, (1, 12, 13), (1, 3, 5), 1, (0, 1, 2), 1),   # filters in LDS, two outputs
                                                        (130, 7, (1, 9, 20), (1, 3, 5), (1, 2, 1), 0, 1),    # the same, four at a time
                                                        (300, 5, (3, 4, 5), (3, 3, 3), 1, 1, 1)])            # filters too large for LDS
def test_conv3d_real(G, ci, co, vol, k, stride, pad, dil):
    import paper_1801_09449_amd as T
    t3 = lambda v: (v,) * 3 if isinstance(v, int) else tuple(v)
    x = tern((2, ci) + vol, 23)
    w = synth.gaussian((co, ci) + k, 23, synth.T_F32)
    b = synth.gaussian((co,), 24, synth.T_F32)
    want = oracle.conv3d_real(x, w, b, t3(stride), t3(pad), t3(dil))
    got = T.tern_conv3d_real(gpu_pack(G, x), ci, G.dev(w), G.dev(b), stride, pad, dil).cpu().numpy()
    assert got.shape == want.shape and got.dtype == np.float32
    bound = real_conv_bound(w, b)[None, :, None, None, None]
    assert (np.abs(got.astype(np.float64) - want) <= bound).all()
    # without bias
    got0 = T.tern_conv3d_real(gpu_pack(G, x), ci, G.dev(w), None, stride, pad, dil).cpu().numpy()
    want0 = oracle.conv3d_real(x, w, None, t3(stride), t3(pad), t3(dil))
    assert (np.abs(got0.astype(np.float64) - want0) <= bound).all()
    # ternary-valued float weights: every partial sum is a small integer, the result is exact
    wi = tern((co, ci) + k, 25, 0.5, synth.T_WGT)
    exact = oracle.conv3d(x, wi, ConvGeom(k, t3(stride), t3(pad), t3(dil)))
    goti = T.tern_conv3d_real(gpu_pack(G, x), ci, G.dev(wi.astype(np.float32)), None, stride, pad, dil).cpu().numpy()
    np.testing.assert_array_equal(goti, exact.astype(np.float32))


@pytest.mark.parametrize("ci,co,vol,k,stride,pad,dil", [
    (64, 2, (1, 260, 258), (1, 3, 3), 1, 0, 1),             # a workgroup has more than one tile
    (64, 9, (1, 259, 255), (1, 3, 3), 1, (0, 1, 1), 1),     # the same padded; three groups of filters, the last one filter
    (128, 2, (1, 61, 67), (1, 3, 3), 1, (0, 1, 1), 1),      # records of four words, padded, more taps than fetched at a time
    (99, 5, (1, 40, 43), (1, 2, 2), 2, 0, 1),               # four words, the last one part empty; strided
    (96, 3, (1, 190, 180), (1, 3, 3), 1, 0, 1),             # three words, more than one tile
    (150, 2, (1, 21, 35), (1, 3, 3), 1, (0, 2, 1), 2),      # five, dilated
    (192, 4, (3, 9, 11), (1, 3, 3), 1, 0, 1),               # six, two units to a tap
    (200, 1, (1, 13, 17), (1, 3, 3), 1, (0, 1, 0), 1),      # seven
    (224, 6, (2, 9, 9), (1, 1, 1), 1, 0, 1),                # seven, one unit in all
    (256, 2, (1, 20, 19), (2, 2, 2), 1, 1, 1),              # eight, two units to a tap; 64 operand blocks
    (320, 3, (1, 11, 12), (1, 2, 3), 1, 0, 1),              # ten, five units of two words
    (352, 2, (1, 9, 40), (1, 1, 5), 1, 0, 1),               # eleven, word by word
    (32, 4, (3, 9, 10), (3, 3, 3), 1, 1, 1),
    (96, 3, (2, 5, 6), (1, 3, 3), (1, 2, 1), (0, 2, 1), (1, 1, 2)),
    (33, 1, (1, 1, 1), (1, 1, 1), 1, 0, 1),                 # one voxel
    (20, 2, (4, 9, 9), (4, 4, 4), 1, 0, 1),                 # 64 operand blocks, the most that fit
    (20, 2, (5, 13, 7), (5, 13, 1), 1, 0, 1),               # 65: table sums
])
def test_conv3d_real_matrix_blocks(G, ci, co, vol, k, stride, pad, dil):
    """The prediction layer on the matrix cores, and weights over fifty orders of magnitude: each is three bf16
    numbers exactly, so the bound of a 32-bit sum holds whatever the range."""
    import paper_1801_09449_amd as T
    t3 = lambda v: (v,) * 3 if isinstance(v, int) else tuple(v)
    x = tern((2, ci) + vol, 29)
    for spread in (0.0, 25.0):
        w = synth.gaussian((co, ci) + k, 29, synth.T_F32)
        w *= np.float32(10.0) ** (spread * np.tanh(synth.gaussian((co, ci) + k, 30, synth.T_F32))).astype(np.float32)
        b = synth.gaussian((co,), 31, synth.T_F32)
        want = oracle.conv3d_real(x, w, b, t3(stride), t3(pad), t3(dil))
        got = T.tern_conv3d_real(gpu_pack(G, x), ci, G.dev(w), G.dev(b), stride, pad, dil).cpu().numpy()
        bound = real_conv_bound(w, b)[None, :, None, None, None]
        assert (np.abs(got.astype(np.float64) - want) <= bound).all()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3e38, 1e-40, 0.0])
def test_conv3d_real_special_weights(G, value):
    """A zero code takes no part, whatever its weight; the smallest floats are not lost."""
    import paper_1801_09449_amd as T
    x = tern((2, 40, 1, 12, 11), 33)
    w = synth.gaussian((5, 40, 1, 3, 3), 33, synth.T_F32) * (1e-38 if value == 1e-40 else 1)
    w[1, 7, 0, 1, 2] = w[4, 39, 0, 0, 0] = value
    got = T.tern_conv3d_real(gpu_pack(G, x), 40, G.dev(w), None, 1, 0, 1).cpu().numpy().astype(np.float64)
    finite = np.where(np.isfinite(w), w, np.float32(0.0))
    want = oracle.conv3d_real(x, finite, None, (1,) * 3, (0,) * 3, (1,) * 3).astype(np.float64)
    odd = np.zeros_like(want)                                       # what the two odd weights add
    if not np.isfinite(value):
        for o, c, (b, a) in ((1, 7, (1, 2)), (4, 39, (0, 0))):
            code = x[:, c, :, b:b + want.shape[3], a:a + want.shape[4]]
            odd[:, o] = np.where(code == 0, 0.0, np.where(code == 0, 1, code) * np.float64(value))
    bound = real_conv_bound(finite, np.zeros(5, np.float32))[None, :, None, None, None]
    plain = odd == 0
    assert (np.abs(got - want)[plain] <= np.broadcast_to(bound, want.shape)[plain]).all()
    np.testing.assert_array_equal(got[~plain], odd[~plain])


@pytest.mark.parametrize("value", [np.inf, 1e-40])
@pytest.mark.parametrize("ci,co,n,vol,k,pad", [
    (20, 2, 1, (1, 30, 31), (1, 3, 3), (0, 1, 1)),          # one word
    (96, 6, 2, (3, 9, 10), (1, 3, 3), (0, 0, 0)),           # three, a second group of filters
    (160, 2, 1, (1, 12, 13), (1, 3, 3), (0, 1, 0)),         # five, padded
    (256, 1, 1, (1, 12, 13), (1, 2, 2), (0, 1, 1)),         # eight
    (64, 2, 3, (1, 170, 160), (1, 3, 3), (0, 1, 1)),        # two; a workgroup has more than one tile
])
def test_conv3d_real_added_one_by_one(G, ci, co, n, vol, k, pad, value):
    """Weights that are not three bf16 numbers send a workgroup the plain way: every word count's addresses there,
    padding, and several tiles.  An infinite weight shows where its channel's code is not zero, with its sign."""
    import paper_1801_09449_amd as T
    x = tern((n, ci) + vol, 37)
    w = synth.gaussian((co, ci) + k, 37, synth.T_F32)
    at = (co - 1, ci - 1, 0, k[1] - 1, 0)
    w[at] = value
    got = T.tern_conv3d_real(gpu_pack(G, x), ci, G.dev(w), None, 1, pad, 1).cpu().numpy().astype(np.float64)
    finite = np.where(np.isfinite(w), w, np.float32(0.0))
    want = oracle.conv3d_real(x, finite, None, (1,) * 3, pad, (1,) * 3).astype(np.float64)
    bound = np.broadcast_to(real_conv_bound(finite, np.zeros(co, np.float32))[None, :, None, None, None], want.shape)
    odd = np.zeros_like(want)
    if not np.isfinite(value):
        xp = np.pad(x, ((0, 0), (0, 0)) + tuple((a, a) for a in pad))
        code = xp[:, ci - 1, :, at[3]:at[3] + want.shape[3], :want.shape[4]]
        odd[:, co - 1] = np.where(code == 0, 0.0, np.where(code == 0, 1, code) * np.inf)
    plain = odd == 0
    assert (np.abs(got - want)[plain] <= bound[plain]).all()
    np.testing.assert_array_equal(got[~plain], odd[~plain])


# ---- code statistics ---------------------------------------------------------------------------------
@pytest.mark.parametrize("n,c,vol", [(1, 1, (1, 1, 1)), (2, 5, (3, 5, 7)), (1, 33, (4, 9, 11)), (3, 64, (2, 8, 8)),
                                     (1, 100, (5, 13, 6)), (2, 256, (3, 4, 5)), (1, 16, (40, 64, 70))])
def test_count_codes(G, n, c, vol):
    import paper_1801_09449_amd as T
    x = tern((n, c) + vol, 71, p0=0.45)
    nz, ng = T.tern_count_codes(gpu_pack(G, x), c)
    want_nz, want_ng = oracle.count_codes(x)
    np.testing.assert_array_equal(nz.cpu().numpy(), want_nz)
    np.testing.assert_array_equal(ng.cpu().numpy(), want_ng)


def test_count_codes_ignores_sign_under_clear_mask_and_repeats(G):
    import torch
    import paper_1801_09449_amd as T
    x = tern((1, 40, 3, 6, 5), 72)
    p = gpu_pack(G, x).clone()
    p[..., 1, :] = -1                      # every sign bit set, also under clear mask bits
    want_nz, _ = oracle.count_codes(x)
    for _ in range(2):                     # the call overwrites its outputs: same answer twice
        nz, ng = T.tern_count_codes(p, 40)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(nz.cpu().numpy(), want_nz)
        np.testing.assert_array_equal(ng.cpu().numpy(), want_nz)     # every nonzero now reads as -1


# ---- pooled convolutions through two balanced-ternary digits -----------------------------------------
def digits_of(words, c):
    """(low, high) int8 tensors [N][c][D][H][W] from a packed two-digit tensor (numpy words
    [N][D][H][W][2][2*wd])."""
    wd = (c + 31) // 32
    m, s = words[..., 0, :], words[..., 1, :]
    out = []
    for which in (0, 1):
        mm, ss = m[..., which::2], s[..., which::2]                      # [N][D][H][W][wd]
        bits = np.arange(32, dtype=np.uint32)
        mb = ((mm[..., None] >> bits) & 1).reshape(mm.shape[:-1] + (32 * wd,))[..., :c]
        sb = ((ss[..., None] >> bits) & 1).reshape(ss.shape[:-1] + (32 * wd,))[..., :c]
        code = mb.astype(np.int8) * (1 - 2 * sb.astype(np.int8))
        out.append(np.moveaxis(code, -1, 1))
    return out


@pytest.mark.parametrize("c,vol,win", [(5, (3, 6, 8), (1, 2, 2)), (32, (1, 7, 9), (1, 2, 2)), (70, (4, 5, 6), (2, 2, 1)),
                                       (64, (2, 4, 9), (1, 1, 3)), (33, (3, 3, 3), (1, 1, 1)), (96, (2, 8, 8), (2, 1, 2))])
def test_pool_digits(G, c, vol, win):
    import paper_1801_09449_amd as T
    x = synth.ternary((2, c) + vol, 0.3, c + vol[0], synth.T_ACT)
    got, c2 = T.tern_pool_digits(T.tern_pack(G.dev(x)), c, win)
    assert c2 == 64 * ((c + 31) // 32)
    words = G.words(got)
    low, high = digits_of(words, c)
    want_low, want_high = oracle.pool_digits(x, win)
    np.testing.assert_array_equal(low, want_low)
    np.testing.assert_array_equal(high, want_high)
    # canonical packing: no sign bit without its mask bit, padding channels empty
    assert not (words[..., 1, :] & ~words[..., 0, :]).any()
    if c % 32:
        assert not (words[..., 0, -2:] >> np.uint32(c % 32)).any()


@pytest.mark.parametrize("ci,co,vol,k,win", [(64, 40, (1, 30, 26), (1, 3, 3), (1, 2, 2)), (40, 33, (6, 12, 10), (3, 3, 3), (1, 2, 2)),
                                             (128, 64, (2, 21, 18), (1, 3, 3), (1, 2, 2)), (256, 48, (1, 16, 20), (1, 1, 1), (1, 2, 2)),
                                             (32, 16, (4, 9, 9), (2, 3, 1), (2, 1, 2))])
def test_conv_on_pooled_digits_equals_conv_on_window_sums(G, ci, co, vol, k, win):
    """tern_pool_digits + tern_conv3d_digits against the oracle's convolution of the window sums:
    int32 accumulators and fused packed output, both channel-block widths."""
    import paper_1801_09449_amd as T
    x = synth.ternary((2, ci) + vol, 0.35, ci + co, synth.T_ACT)
    w = synth.ternary((co, ci) + k, 0.5, ci + co, synth.T_WGT)
    pvol = win[0] * win[1] * win[2]
    lo, hi = synth.bn_like_thresholds(co, int(np.prod(k)) * pvol, ci, 0.5, 0.65, ci, synth.T_THR)
    pooled = np.ascontiguousarray(oracle.pool_sum(x, win))      # int8 sums in [-4, 4]
    geom = ConvGeom(k, (1, 1, 1), (0, 0, 0), (1, 1, 1))
    want_acc = oracle.conv3d(pooled, w, geom)
    want_packed = oracle.pack(oracle.threshold(want_acc, lo, hi))
    dig, c2 = T.tern_pool_digits(T.tern_pack(G.dev(x)), ci, win)
    bank = T.tern_pack_filters(G.dev(T.tern_digits_weights(w)))
    try:
        for cb in (0, 16, 32):
            T.tern_set_option(3, cb)
            acc = T.tern_conv3d(dig, c2, bank, co, k=k, stride=1, pad=0, dil=1, digits=True)
            packed = T.tern_conv3d(dig, c2, bank, co, k=k, stride=1, pad=0, dil=1, thr_lo=G.dev(lo),
                                   thr_hi=G.dev(hi), digits=True)
            np.testing.assert_array_equal(acc.cpu().numpy(), want_acc)
            np.testing.assert_array_equal(G.words(packed), want_packed)
    finally:
        T.tern_set_option(3, 0)
    # the same through the matrix cores: the two digits of a value become its 4-bit float code,
    # the bank is that of the undoubled weights
    mbank = T.tern_expand_filters(G.dev(w), "f4")
    acc = T.tern_conv3d(dig, c2, mbank, co, k=k, stride=1, pad=0, dil=1, digits=True, mfma="f4")
    packed = T.tern_conv3d(dig, c2, mbank, co, k=k, stride=1, pad=0, dil=1, thr_lo=G.dev(lo), thr_hi=G.dev(hi),
                           digits=True, mfma="f4")
    np.testing.assert_array_equal(acc.cpu().numpy(), want_acc)
    np.testing.assert_array_equal(G.words(packed), want_packed)


def test_two_digit_input_through_the_direct_kernel(G):
    """A dilation whose halo tile no LDS holds: tern_conv3d_digits runs on the direct kernel (odd
    words count three times) and must still equal the convolution of the window sums; the matrix
    route refuses such a halo."""
    import paper_1801_09449_amd as T
    ci, co, win, k = 40, 33, (1, 2, 2), (2, 3, 3)
    x = synth.ternary((1, ci, 110, 18, 18), 0.35, 611, synth.T_ACT)
    w = synth.ternary((co, ci) + k, 0.5, 612, synth.T_WGT)
    lo, hi = synth.bn_like_thresholds(co, 18 * 4, ci, 0.5, 0.65, ci, synth.T_THR)
    pooled = np.ascontiguousarray(oracle.pool_sum(x, win))
    geom = ConvGeom(k, (1, 1, 1), (0, 1, 1), (100, 1, 1))
    want_acc = oracle.conv3d(pooled, w, geom)
    assert want_acc.shape == (1, co, 10, 9, 9)
    want_packed = oracle.pack(oracle.threshold(want_acc, lo, hi))
    dig, c2 = T.tern_pool_digits(T.tern_pack(G.dev(x)), ci, win)
    bank = T.tern_pack_filters(G.dev(T.tern_digits_weights(w)))
    kw = dict(k=k, stride=1, pad=(0, 1, 1), dil=(100, 1, 1), digits=True)
    acc = T.tern_conv3d(dig, c2, bank, co, **kw)
    packed = T.tern_conv3d(dig, c2, bank, co, thr_lo=G.dev(lo), thr_hi=G.dev(hi), **kw)
    np.testing.assert_array_equal(acc.cpu().numpy(), want_acc)
    np.testing.assert_array_equal(G.words(packed), want_packed)
    with pytest.raises(T.TernError) as e:
        T.tern_conv3d(dig, c2, T.tern_expand_filters(G.dev(w), "f4"), co, mfma="f4", **kw)
    assert e.value.status == -2


# ---- the whole network -----------------------------------------------------------------------------
def run_unet(G, u):
    import torch
    from paper_1801_09449_amd import unet
    plan = unet.UNetPlan(u.layers, u.head_w, u.head_b, u.in_lo, u.in_hi)
    pred, kept = unet.unet_forward(plan, G.dev(u.x), keep_layers=True)
    torch.cuda.synchronize()
    return pred.cpu().numpy(), [G.words(t) for t, _ in kept], kept, plan


def check_unet(G, u):
    """Runs the network and compares every module with the oracle; returns the plan."""
    pred, kept, kept_dev, plan = run_unet(G, u)
    codes, want_pred = oracle.unet_forward(u.x, u.in_lo, u.in_hi, u.layers, u.head_w, u.head_b)
    assert len(kept) == len(codes) == 14
    for li, (got, want) in enumerate(zip(kept, codes), start=1):
        np.testing.assert_array_equal(got, oracle.pack(want), err_msg=f"module #{li}")
    # zero fraction per module from the library's statistics = the oracle's
    import paper_1801_09449_amd as T
    for (t, c), want in zip(kept_dev, codes):
        nz, ng = T.tern_count_codes(t, c)
        want_nz, want_ng = oracle.count_codes(want)
        np.testing.assert_array_equal(nz.cpu().numpy(), want_nz)
        np.testing.assert_array_equal(ng.cpu().numpy(), want_ng)
    bound = real_conv_bound(u.head_w, u.head_b)[None, :, None, None, None]
    assert pred.shape == want_pred.shape
    assert (np.abs(pred.astype(np.float64) - want_pred) <= bound).all()
    return plan


def test_unet_reduced(G):
    """Narrow network on small stacks, batch of 3: every module's packed output, bit for bit."""
    check_unet(G, synth.unet_table1(seed=5, n=3, width_div=8, size=(84, 76), slices=5))
    check_unet(G, synth.unet_table1(seed=6, n=1, width_div=3, size=(92, 100), slices=15))


def test_unet_several_stacks_of_narrow_channels(G):
    """Four full-size stacks, narrow channels: a part of a word in every module, and inputs that are joined in
    memory (odd word counts)."""
    check_unet(G, synth.unet_table1(seed=7, n=4, width_div=8))


def test_unet_reduced_with_every_pooled_module_through_two_digits(G, monkeypatch):
    """The same narrow networks with the plan's size threshold at zero, so that modules 4, 6 and 8
    all pool into two digits (tern_module.pool) instead of folding the window into their filters;
    odd extents in front of the pooling drop their last row and column either way."""
    from paper_1801_09449_amd import unet
    monkeypatch.setattr(unet.UNetPlan, "DIGITS_FROM_MACS", 0.0)
    check_unet(G, synth.unet_table1(seed=5, n=3, width_div=8, size=(84, 76), slices=5))
    check_unet(G, synth.unet_table1(seed=6, n=1, width_div=3, size=(92, 100), slices=15))


def test_unet_table1_full_size(G):
    """The network at the paper's size (236 x 172 x 15 stack, full channel counts), one stack."""
    check_unet(G, synth.unet_table1(seed=0, n=1))


def test_net_forward_generic_wiring(G):
    """tern_net_forward beyond the Table 1 pattern: a 3-D network with padded and strided
    modules, upsampling without a skip, a skip without upsampling, a skip of a skip, unaligned
    channel counts, and no prediction layer."""
    import torch
    from paper_1801_09449_amd import unet
    n, vol = 2, (6, 14, 12)
    x = synth.gaussian((n, 3) + vol, 91, synth.T_F32)
    in_lo = np.array([-0.4, -0.5, -0.2], np.float32)
    in_hi = np.array([0.5, 0.3, 0.6], np.float32)
    spec = [
        # c_out, c_in, k, stride, pad, extras
        (20, 3, (3, 3, 3), (1, 1, 1), (1, 1, 1), dict(save="a")),
        (33, 20, (3, 3, 3), (2, 2, 2), (1, 1, 1), dict(save="b")),
        (16, 33, (1, 1, 1), (1, 1, 1), (0, 0, 0), dict()),
        (24, 16 + 33, (3, 3, 3), (1, 1, 1), (1, 1, 1), dict(concat="b")),                 # skip, no upsampling
        (12, 24, (3, 3, 3), (1, 1, 1), (1, 1, 1), dict(up=(2, 2, 2), save="c")),           # upsampling, no skip
        (8, 12 + 20, (3, 3, 3), (1, 1, 1), (0, 0, 0), dict(concat="a")),                   # same extent as "a"
        (5, 8 + 12, (1, 3, 3), (1, 1, 1), (0, 0, 0), dict(concat="c")),                    # "c" is larger: cropped
    ]
    layers = []
    for li, (co, ci, k, st, pd, extra) in enumerate(spec, start=1):
        w = synth.ternary((co, ci) + k, 0.5, 91, synth.T_WGT + 8 * li)
        lo, hi = synth.bn_like_thresholds(co, int(np.prod(k)), ci, 0.5, 0.6, 91, synth.T_THR + 8 * li)
        layers.append(dict(w=w, k=k, stride=st, pad=pd, lo=lo, hi=hi, pool=None, up=extra.get("up"),
                           concat=extra.get("concat"), save=extra.get("save")))
    plan = unet.UNetPlan(layers, None, None, in_lo, in_hi)
    pred, kept = unet.unet_forward(plan, G.dev(x), keep_layers=True)
    torch.cuda.synchronize()
    assert pred is None
    codes, _ = oracle.unet_forward(x, in_lo, in_hi, layers, None, None)
    assert len(kept) == len(codes) == 7
    for li, ((t, c), want) in enumerate(zip(kept, codes), start=1):
        assert c == want.shape[1]
        np.testing.assert_array_equal(G.words(t), oracle.pack(want), err_msg=f"module {li}")
    assert len(np.unique(codes[-1])) == 3


def test_net_forward_one_channel_first_module(G):
    """A plain chain through tern_net_forward whose first module qualifies for the one-launch
    route (one input channel, 3x3x3): same codes as the oracle's chain, module by module."""
    import torch
    from paper_1801_09449_amd import unet
    f = synth.config2(seed=8, vol=(12, 20, 18))
    layers = [dict(w=L["w"], k=L["k"], stride=L["stride"], pad=L["pad"], lo=L["lo"], hi=L["hi"], pool=None,
                   up=None, concat=None, save=None) for L in f.layers]
    plan = unet.UNetPlan(layers, None, None, f.in_lo, f.in_hi)
    _, kept = unet.unet_forward(plan, G.dev(f.x), keep_layers=True)
    torch.cuda.synchronize()
    want = oracle.fcn_forward(f.x, f.in_lo, f.in_hi,
                              [dict(w=L["w"], geom=ConvGeom(L["k"], L["stride"], L["pad"], L["dil"]), lo=L["lo"],
                                    hi=L["hi"]) for L in f.layers])
    for li, ((t, c), code) in enumerate(zip(kept, want), start=1):
        np.testing.assert_array_equal(G.words(t), oracle.pack(code), err_msg=f"module {li}")


@pytest.mark.parametrize("vol,ca,cs,k0,kj,up,stride,pad,read", [
    ((1, 23, 30), 64, 64, (1, 3, 3), (1, 3, 3), (1, 2, 2), (1, 1, 1), (0, 0, 0), True),      # a decoder step; planes of the batch as one stack
    ((1, 40, 27), 128, 50, (1, 3, 3), (1, 3, 3), (1, 1, 4), (1, 1, 1), (0, 1, 1), True),     # a last skip word part empty; padded
    ((5, 12, 9), 64, 128, (3, 3, 3), (3, 3, 3), (2, 2, 2), (1, 1, 1), (1, 1, 1), True),      # a volume, cropped along z
    ((4, 9, 11), 192, 64, (3, 3, 3), (3, 3, 3), (1, 2, 1), (2, 2, 1), (1, 0, 1), True),      # strided
    ((3, 10, 10), 64, 64, (1, 3, 3), (1, 3, 3), (2, 2, 2), (1, 1, 1), (0, 0, 0), True),      # no depth taps but upsampled along z
    ((1, 15, 14), 64, 0, (1, 3, 3), (1, 3, 3), (1, 2, 2), (1, 1, 1), (0, 1, 1), True),       # upsampled, no skip
    ((1, 15, 14), 64, 64, (1, 3, 3), (1, 3, 3), (1, 3, 2), (1, 1, 1), (0, 0, 0), False),      # a factor of three: joined in memory first
    ((1, 15, 14), 32, 32, (1, 3, 3), (1, 3, 3), (1, 2, 2), (1, 1, 1), (0, 0, 0), False),      # odd word counts: likewise
    ((1, 15, 14), 64, 64, (1, 3, 3), (1, 1, 1), (1, 2, 2), (1, 1, 1), (0, 0, 0), False),      # a single tap: likewise
])
def test_net_forward_reads_upsampled_and_skipped_input(G, vol, ca, cs, k0, kj, up, stride, pad, read):
    """A module whose input is an upsampled tensor with the channels of a cropped one behind it, as the
    convolution reads it from both, against the oracle on the joined tensor.  Where it does, the region of the
    workspace for the joined tensor is not written."""
    import torch
    from paper_1801_09449_amd import unet
    n, seed = 3, 40 + ca + cs + vol[1]
    half = np.array([0.5, 0.5], np.float32)
    big = tuple(v * u + a for v, u, a in zip(vol, up, (0 if vol[0] == 1 else 1, 3, 2)))
    # module 1 makes the skip, larger than the upsampled tensor; module 2 goes down to `vol`
    xb = synth.gaussian((n, 2) + big, seed, synth.T_F32)
    same = tuple(kk // 2 for kk in k0)
    kshrink = tuple(b - (v - 1) * u for b, v, u in zip(big, vol, up))
    spec = [(max(cs, 16), 2, k0, (1, 1, 1), same, dict(save="a")),
            (ca, max(cs, 16), kshrink, up, (0, 0, 0), dict()),
            (40, ca + cs, kj, stride, pad, dict(up=up, concat="a" if cs else None))]
    layers = []
    for li, (co, ci, k, st, pd, extra) in enumerate(spec, start=1):
        w = synth.ternary((co, ci) + k, 0.5, seed, synth.T_WGT + 8 * li)
        lo, hi = synth.bn_like_thresholds(co, int(np.prod(k)), ci, 0.5, 0.6, seed, synth.T_THR + 8 * li)
        layers.append(dict(w=w, k=k, stride=st, pad=pd, lo=lo, hi=hi, pool=None, up=extra.get("up"),
                           concat=extra.get("concat"), save=extra.get("save")))
    plan = unet.UNetPlan(layers, None, None, -half, half)
    xd = G.dev(xb)
    ws = plan.workspace(xd).fill_(0xa5)
    _, kept = unet.unet_forward(plan, xd, keep_layers=True)
    torch.cuda.synchronize()
    start, end = (kept[i][0].data_ptr() - ws.data_ptr() for i in (1, 2))
    joined = ws[(start + kept[1][0].numel() * 4 + 255) // 256 * 256:end]
    assert joined.numel() >= n * (ca + cs) // 4 and bool((joined == 0xa5).all()) == read
    codes, _ = oracle.unet_forward(xb, -half, half, layers, None, None)
    for li, ((t, c), want) in enumerate(zip(kept, codes), start=1):
        np.testing.assert_array_equal(G.words(t), oracle.pack(want), err_msg=f"module {li}")
    assert len(np.unique(codes[-1])) == 3


@pytest.mark.parametrize("n,ca,cs,co,hw,blocks", [
    (12, 64, 64, 64, 96, 1),
    (6, 64, 64, 256, 96, 2),
    (12, 128, 50, 128, 94, 2),         # six words, the last one part empty
    (13, 64, 0, 64, 97, 1),            # no skip
])
def test_net_forward_joined_input_in_large_waves(G, n, ca, cs, co, hw, blocks):
    """The same in launches that give waves 128 voxels and 32 or 64 filters, as a U-Net's decoder has on a batch, against
    a float32 convolution of the decoded tensors (sums below 2^24: exact)."""
    import torch
    import paper_1801_09449_amd as T
    g = torch.Generator(device="cuda").manual_seed(ca + cs + co)
    half = hw // 2
    x = torch.randn((n, 1, 1, 2 * half + 3, 2 * half + 6), generator=g, device="cuda")
    cut = torch.full((1,), 0.5, device="cuda")
    mods, weights = [], []
    for c_out, c_in, k, st, pd, extra in (
            (cs or 16, 1, (1, 3, 3), (1, 1, 1), (0, 1, 1), {}),
            (ca, cs or 16, (1, 5, 8), (1, 2, 2), (0, 0, 0), {}),
            (co, ca + cs, (1, 3, 3), (1, 1, 1), (0, 0, 1), dict(up=(1, 2, 2), skip_from=0 if cs else -1))):
        w = torch.randint(-1, 2, (c_out, c_in) + k, generator=g, device="cuda", dtype=torch.int8)
        s = max(1, int(0.3 * (c_in * k[1] * k[2]) ** 0.5))
        lo, hi = (torch.randint(a, a + 3, (c_out,), generator=g, device="cuda", dtype=torch.int32) for a in (-s, s - 2))
        mods.append(T.NetModule(c_out, T.tern_pack_filters(w), lo, hi, k, st, pd, (1, 1, 1), **extra))
        weights.append((w, lo, hi))
    _, views = T.tern_net_forward(x, -cut, cut, mods, return_modules=True)
    plan = T.tern_last_launch()
    assert (plan["voxels_per_lane"], plan["channels_per_pass"]) == (2, 32 * blocks)

    def codes(v):
        t, dm = v
        bits = (t[..., None] >> torch.arange(32, device="cuda", dtype=torch.int32)) & 1      # [n, d, h, w, 2, words, 32]
        bits = bits.flatten(-2)[..., :dm[1]].float()
        return (bits[..., 0, :] * (1 - 2 * bits[..., 1, :])).permute(0, 4, 1, 2, 3)[:, :, 0]
    up = codes(views[1]).repeat_interleave(2, 2).repeat_interleave(2, 3)
    if cs:
        skip = codes(views[0])
        y0, x0 = (skip.shape[2] - up.shape[2]) // 2, (skip.shape[3] - up.shape[3]) // 2
        up = torch.cat([up, skip[:, :, y0:y0 + up.shape[2], x0:x0 + up.shape[3]]], 1)
    w, lo, hi = weights[2]
    up = torch.nn.functional.pad(up, (1, 1))
    oh, ow = up.shape[2] - 2, up.shape[3] - 2
    acc = torch.zeros((n, co, oh * ow), device="cuda")
    for b in range(3):
        for a in range(3):
            tap = w[:, :, 0, b, a].float().contiguous()
            for i in range(n):
                acc[i] += tap @ up[i, :, b:b + oh, a:a + ow].reshape(ca + cs, -1)
    want = T.tern_threshold_pack(acc.view(n, co, 1, oh, ow).int(), lo, hi)
    assert torch.equal(views[2][0], want)
