"""First layers on a scalar volume (one launch from intensities to packed codes), at the edges of the kernel's
tiles and of its dispatch, against the CPU oracle bit for bit."""
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


def run(G, x, in_lo, in_hi, w, lo, hi, stride, pad, dil):
    import paper_1801_09449_amd as T
    L = T.FcnLayer(1, w.shape[0], T.tern_pack_filters(G.dev(w)), G.dev(lo), G.dev(hi), w.shape[2:], stride, pad, dil)
    got = T.tern_fcn_forward(G.dev(x), G.dev(in_lo), G.dev(in_hi), [L])
    want = oracle.fcn_forward(x, in_lo, in_hi, [dict(w=w, geom=ConvGeom(w.shape[2:], stride, pad, dil), lo=lo, hi=hi)])
    np.testing.assert_array_equal(G.words(got), oracle.pack(want[-1]))
    return want[-1]


@pytest.mark.parametrize("k,n,vol,c_out,stride,pad,dil", [
    ((3, 3, 3), 1, (5, 2, 64), 16, (1, 1, 1), (1, 1, 1), (1, 1, 1)),          # one tile exactly, half a block of filters
    ((3, 3, 3), 1, (6, 3, 65), 17, (1, 1, 1), (1, 1, 1), (1, 1, 1)),          # one more of everything
    ((3, 3, 3), 1, (4, 1, 31), 32, (1, 1, 1), (1, 1, 1), (1, 1, 1)),
    ((3, 3, 3), 1, (3, 3, 3), 1, (1, 1, 1), (0, 0, 0), (1, 1, 1)),            # a single voxel
    ((3, 3, 3), 2, (40, 131, 70), 16, (1, 1, 1), (1, 1, 1), (1, 1, 1)),       # four rows to a wave
    ((3, 3, 3), 1, (23, 131, 70), 40, (1, 1, 1), (1, 0, 1), (1, 1, 1)),       # two rows; a second block of filters
    ((3, 3, 3), 1, (9, 40, 150), 24, (1, 2, 2), (1, 1, 1), (1, 1, 1)),
    ((3, 3, 3), 1, (11, 40, 130), 256, (1, 1, 1), (1, 1, 1), (1, 1, 1)),      # more workgroups than are resident: plane by plane
    ((3, 3, 3), 1, (23, 60, 130), 96, (1, 1, 1), (1, 1, 1), (1, 1, 1)),       # two rounds with four or five waves: planes together
    ((3, 3, 3), 2, (83, 131, 70), 16, (1, 1, 1), (1, 1, 1), (1, 1, 1)),       # plane by plane with half a block of filters
    ((3, 3, 3), 2, (7, 30, 80), 16, (1, 1, 3), (2, 5, 4), (1, 3, 2)),         # planes and columns of padding alone
    ((3, 3, 3), 1, (5, 40, 620), 8, (1, 1, 70), (1, 1, 1), (1, 1, 1)),        # columns too far apart for a tile
    ((3, 3, 3), 1, (5, 260, 130), 8, (1, 1, 1), (1, 60, 40), (1, 120, 60)),
    ((3, 3, 3), 1, (6, 196, 25), 16, (1, 1, 70), (1, 0, 0), (1, 2, 1)),       # one output along x, whose taps lie together
    ((3, 3, 3), 1, (5, 60, 141), 17, (1, 3, 4), (1, 5, 60), (1, 5, 60)),      # a narrow output, taps far apart along x
    ((3, 3, 3), 2, (40, 131, 130), 70, (1, 1, 1), (1, 20, 66), (1, 20, 66)),  # far apart along both; all blocks of filters in a workgroup
    ((3, 3, 3), 1, (9, 70, 40), 40, (1, 1, 1), (1, 3, 1), (1, 4, 1)),         # along y alone; a workgroup to a block of filters
    ((1, 3, 3), 1, (7, 40, 200), 33, (1, 1, 1), (0, 9, 70), (1, 9, 70)),
    ((15, 3, 3), 8, (15, 130, 140), 64, (1, 1, 1), (0, 0, 0), (1, 16, 16)),
    ((15, 3, 3), 2, (16, 60, 330), 40, (1, 1, 2), (1, 0, 90), (1, 24, 130)),
    ((1, 3, 3), 1, (7, 8, 64), 16, (1, 1, 1), (0, 1, 1), (1, 1, 1)),
    ((1, 3, 3), 2, (15, 33, 97), 33, (1, 2, 1), (0, 0, 2), (1, 1, 2)),
    ((15, 3, 3), 1, (15, 20, 34), 16, (1, 1, 1), (0, 0, 0), (1, 1, 1)),
    ((15, 3, 3), 2, (17, 11, 70), 33, (1, 1, 1), (1, 1, 1), (1, 1, 1)),       # several output planes, padded along z
    ((15, 3, 3), 5, (15, 236, 172), 32, (1, 1, 1), (0, 0, 0), (1, 1, 1)),
    ((15, 3, 3), 1, (20, 30, 40), 20, (1, 2, 2), (7, 2, 2), (1, 2, 2)),
])
def test_first_layer_tiles(G, k, n, vol, c_out, stride, pad, dil):
    seed = 71 + c_out + vol[0]
    x = synth.gaussian((n, 1) + vol, seed, synth.T_F32)
    w = synth.ternary((c_out, 1) + k, 0.5, seed, synth.T_WGT)
    lo, hi = synth.bn_like_thresholds(c_out, int(np.prod(k)), 1, 0.5, 0.6, seed, synth.T_THR)
    # zeros are no neutral intensity here: padding has to be code 0 whatever the cut points say
    for a, b in ((-0.4, 0.7), (0.1, 0.3)):
        run(G, x, np.array([a], np.float32), np.array([b], np.float32), w, lo, hi, stride, pad, dil)


@pytest.mark.parametrize("k", [(3, 3, 3), (15, 3, 3)])
def test_first_layer_special_intensities(G, k):
    """NaN is code 0, infinities are +-1, and values on a cut point are 0."""
    vol = (16, 9, 66)
    x = synth.gaussian((1, 1) + vol, 5, synth.T_F32)
    flat = x.reshape(-1)
    flat[::7], flat[1::11], flat[2::13], flat[3::5], flat[4::17] = np.nan, np.inf, -np.inf, 0.5, -0.5
    w = synth.ternary((16, 1) + k, 0.5, 6, synth.T_WGT)
    lo, hi = synth.bn_like_thresholds(16, int(np.prod(k)), 1, 0.5, 0.6, 6, synth.T_THR)
    half = np.array([0.5], np.float32)
    run(G, x, -half, half, w, lo, hi, (1, 1, 1), (1, 1, 1), (1, 1, 1))


@pytest.mark.parametrize("vol,c_out", [
    ((1, 2, 131072), 524288),          # a row of output is 2^32 words
])
def test_first_layer_offsets_beyond_32_bits(G, vol, c_out):
    """Against the same layer with some of the filters, and on the two ends of the volume."""
    import torch
    import paper_1801_09449_amd as T
    gen = torch.Generator("cuda").manual_seed(c_out)
    k, pad, half = (1, 3, 3), (0, 1, 1), torch.full((1,), 0.5, device="cuda")
    x = torch.randn((1, 1) + vol, generator=gen, device="cuda")
    w = torch.randint(-1, 2, (c_out, 1) + k, generator=gen, device="cuda", dtype=torch.int8)
    lo, hi = torch.full((c_out,), -2, device="cuda", dtype=torch.int32), torch.arange(c_out, device="cuda", dtype=torch.int32) % 4

    def run_on(x, a, b):
        L = T.FcnLayer(1, b - a, T.tern_pack_filters(w[a:b].contiguous()), lo[a:b].contiguous(), hi[a:b].contiguous(), k, (1, 1, 1), pad, (1, 1, 1))
        return T.tern_fcn_forward(x, -half, half, [L])

    got = run_on(x, 0, c_out)
    part = min(c_out, 4096)
    end = min(vol[2], 131072)
    for a in sorted({0, c_out // 2, c_out - part}):
        words = slice(a // 32, (a + part + 31) // 32)
        if a + part > c_out:
            continue
        left, right = (run_on(x[..., s].contiguous(), a, a + part) for s in (slice(0, end), slice(vol[2] - end, vol[2])))
        cut = end if end == vol[2] else end - 1            # (a slice's inner edge has padding beside it)
        assert torch.equal(got[:, :, :, :cut, :, words], left[:, :, :, :cut])
        assert torch.equal(got[:, :, :, vol[2] - cut:, :, words], right[:, :, :, end - cut:])
    del got, x, left, right
    torch.cuda.empty_cache()
