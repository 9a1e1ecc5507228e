"""The binding's compiled per-call path: it gives what the Python path gives, and leaves every call that is
not plain to it (same errors, nothing launched)."""
import numpy as np
import pytest
import torch

import synth


@pytest.fixture
def B():
    from paper_1801_09449_amd import binding as B
    B.lib()
    assert B._native, "built together with the library"
    yield B
    B.lib()


def test_host_tensors_and_odd_arguments_are_left_to_the_python_checks(B):
    n = B._native
    x = torch.zeros(1, 32, 2, 2, 2, dtype=torch.int8)
    assert n.pack(x, None) is None and n.pack(3, None) is None and n.pack(None, x) is None
    assert n.threshold_pack(x.float(), None, None, None) is None
    assert n.fcn(x, x, x, [], None, None) is None and n.fcn(None, None, None, (), None, None) is None
    assert n.net(x, x, x, [object()], None, None, 1, 0, 1, None, None) is None
    assert n.conv(False, x, 32, x, 32, 3, 1, 1, 1, None, None, None) is None
    with pytest.raises(TypeError):
        n.conv(x)
    with pytest.raises(ValueError, match="GPU"):
        B.tern_pack(x)


def test_an_extension_that_does_not_load_fails_every_call_and_a_missing_one_none(B, tmp_path):
    """Not the first call only, with every later one silently on the slow path."""
    import os
    import shutil
    import subprocess
    import sys
    src = os.path.dirname(B.__file__)
    pkg = tmp_path / "paper_1801_09449_amd"
    pkg.mkdir()
    for f in os.listdir(src):
        if f.endswith(".py") or f == "libtern.so":
            shutil.copy(os.path.join(src, f), pkg / f)
    code = ("import paper_1801_09449_amd as T\n"
            "for _ in range(3):\n"
            "    try: print(T.tern_words(33))\n"
            "    except ImportError as e: print('ImportError', 'build both again' in str(e))\n")
    run = lambda: subprocess.run([sys.executable, "-c", code], cwd=tmp_path, text=True, capture_output=True, check=True).stdout.split("\n")[:3]
    assert run() == ["2"] * 3
    (pkg / "_tern_torch.so").write_bytes(b"of another build")
    assert run() == ["ImportError True"] * 3


@pytest.mark.parametrize("missing", ["g++", "Python.h", "torch's headers", None])
def test_library_builds_without_the_tools_of_the_extension(monkeypatch, tmp_path, missing):
    """build() compiles the library first; what the extension lacks is a warning, no failure, and no
    extension of another build stays beside the new library."""
    from torch.utils import cpp_extension
    from paper_1801_09449_amd import build
    ran = []

    def run(cmd, verbose):
        ran.append(cmd)
        (tmp_path / cmd[cmd.index("-o") + 1].split("/")[-1]).write_text("built")
    monkeypatch.setattr(build, "_run", run)
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libtern.so"))
    monkeypatch.setattr(build, "NATIVE", str(tmp_path / "_tern_torch.so"))
    (tmp_path / "_tern_torch.so").write_text("old")
    if missing == "g++":
        monkeypatch.setattr(build.shutil, "which", lambda name: None)
    elif missing == "Python.h":
        monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    elif missing:
        monkeypatch.setattr(cpp_extension, "include_paths", lambda: [str(tmp_path)])
    if missing:
        with pytest.warns(UserWarning, match=missing.replace("+", "[+]")):
            assert build.build() == str(tmp_path / "libtern.so")
    else:
        build.build()
    assert (tmp_path / "libtern.so").read_text() == "built"
    assert (tmp_path / "_tern_torch.so").exists() == (missing is None)
    assert missing or (tmp_path / "_tern_torch.so").read_text() == "built"


def both(B, call):
    """Results (or the exceptions) of the compiled and of the Python path."""
    got = []
    keep = B._native
    for native in (keep, False):
        B._native = native
        try:
            got.append(call())
        except Exception as e:          # noqa: BLE001 -- compared below
            got.append((type(e), str(e)))
        finally:
            B._native = keep
    return got


@pytest.mark.gpu
@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("binary", [True, False])
def test_convolution_same_results_and_same_errors(B, fused, binary):
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    c = synth.conv_case("native", 2, 40, 33, (5, 6, 7), k=(3, 1, 3), stride=(1, 2, 1), pad=(1, 0, 1), seed=901)
    a, w = B.tern_pack(dev(c.act)), dev(c.wgt)
    bank = B.tern_pack_filters_binary(w) if binary else B.tern_pack_filters(w)
    lo, hi = (dev(c.lo), dev(c.hi)) if fused else (None, None)
    kw = dict(k=c.k, stride=c.stride, pad=c.pad, dil=1, thr_lo=lo, thr_hi=hi, binary=binary)
    x, y = both(B, lambda: B.tern_conv3d(a, 40, bank, 33, **kw))
    assert x.dtype == y.dtype and x.shape == y.shape and torch.equal(x, y)
    out = torch.empty_like(x)
    assert B.tern_conv3d(a, 40, bank, 33, out=out, **kw) is out and torch.equal(out, y)
    lists = dict(kw, k=list(c.k), pad=[1, 0, 1])
    x, z = both(B, lambda: B.tern_conv3d(a, 40, bank, 33, **lists))
    assert torch.equal(x, y) and torch.equal(z, y)
    # lists and numpy integers stay with the compiled path (to leave it costs more than it saves)
    for k, ci in ((list(c.k), 40), (np.array(c.k, np.int64).tolist(), np.int64(40)), (tuple(np.int32(v) for v in c.k), 40), (torch.Size(c.k), 40)):
        got = B._native.conv(binary, a, ci, bank, np.int32(33), k, [1, 2, 1], [1, 0, True], True, lo, hi, None)
        assert got is not None and torch.equal(got, y)
    for k in ((3, 1), (3.0, 1, 3), "313", np.array(c.k), None):
        assert B._native.conv(binary, a, 40, bank, 33, k, 1, 1, 1, lo, hi, None) is None
    bad = [dict(in_packed=a.float()), dict(in_packed=a.cpu()), dict(in_packed=a[:, :, :, ::2]), dict(c_in=70),
           dict(w_bank=bank[:-1]), dict(c_out=65), dict(k=(3, 3, 3)), dict(stride=0), dict(pad=-1), dict(k="3"),
           dict(k=2 ** 40), dict(out=out[:1]), dict(out=out.float()), dict(thr_lo=torch.zeros(2, dtype=torch.int32).cuda(), thr_hi=None)]
    for change in bad:
        args = dict(dict(in_packed=a, c_in=40, w_bank=bank, c_out=33), **kw)
        args.update(change)
        p, q = both(B, lambda: B.tern_conv3d(**args))
        assert isinstance(p, tuple) and p == q, change


@pytest.mark.gpu
def test_packers_and_networks_same_results_and_same_errors(B):
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    src = dev(synth.ternary((2, 33, 3, 4, 5), 0.4, 902, synth.T_ACT))
    for call in (lambda: B.tern_pack(src), lambda: B.tern_pack(src.transpose(2, 3)), lambda: B.tern_pack(src[0]),
                 lambda: B.tern_pack(src, torch.empty(3, dtype=torch.int32).cuda()),
                 lambda: B.tern_threshold_pack(src.float(), torch.full((33,), -0.5).cuda(), torch.full((33,), 0.5).cuda()),
                 lambda: B.tern_threshold_pack(src.int(), torch.full((33,), -0.5).cuda(), torch.full((33,), 0.5).cuda()),
                 lambda: B.tern_threshold_pack(src.double(), src, src)):
        x, y = both(B, call)
        assert (torch.equal(x, y) if isinstance(x, torch.Tensor) else x == y)
    f = synth.config2(seed=3, vol=(16, 16, 8), channels=(16, 32, 40), strides=(1, 2, 1))
    layers = [B.FcnLayer(L["w"].shape[1], L["w"].shape[0], B.tern_pack_filters(dev(L["w"])), dev(L["lo"]), dev(L["hi"]),
                         L["k"], L["stride"], L["pad"], L["dil"]) for L in f.layers]
    mods = [B.NetModule(L["w"].shape[0], B.tern_pack_filters(dev(L["w"])), dev(L["lo"]), dev(L["hi"]), k=L["k"],
                        stride=L["stride"], pad=L["pad"], dil=L["dil"]) for L in f.layers]
    mods.append(B.NetModule(8, B.tern_pack_filters(dev(synth.ternary((8, 56, 3, 3, 3), 0.5, 904, 2))), dev(np.zeros(8, np.int32)),
                            dev(np.ones(8, np.int32)), k=3, pad=1, skip_from=0, up=2))
    x, lo, hi = dev(f.x), dev(f.in_lo), dev(f.in_hi)
    as_lists = [B.FcnLayer(l.c_in, l.c_out, l.w_bank, l.thr_lo, l.thr_hi, list(l.k), list(l.stride), list(l.pad), list(l.dil)) for l in layers]
    for form in (tuple(layers), as_lists, tuple(as_lists)):
        assert torch.equal(B._native.fcn(x, lo, hi, form, None, None), B.tern_fcn_forward(x, lo, hi, layers))
    hw = torch.randn(3, 8, 1, 3, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    for call in (lambda: B.tern_fcn_forward(x, lo, hi, layers), lambda: B.tern_fcn_forward(x, lo, hi, tuple(layers)),
                 lambda: B.tern_fcn_forward(x, lo, hi, layers[1:]), lambda: B.tern_fcn_forward(x, lo, hi, layers, workspace=small),
                 lambda: B.tern_net_forward(x, lo, hi, mods, hw, hw[:, 0, 0, 0, 0].contiguous()),
                 lambda: B.tern_net_forward(x, lo, hi, mods, hw, workspace=small), lambda: B.tern_net_forward(x, lo, hi, mods),
                 lambda: B.tern_net_forward(x, lo, hi, mods[2:], hw)):
        p, q = both(B, call)
        assert (torch.equal(p, q) if isinstance(p, torch.Tensor) else p == q)


def small_net(B, dev):
    """Two modules, the second behind pooling, upsampling and a skip, and a prediction layer."""
    w0, w1 = synth.ternary((40, 2, 3, 3, 3), 0.5, 905, 2), synth.ternary((24, 64 * 3, 1, 3, 3), 0.5, 906, 2)
    bank = lambda w: B.tern_pack_filters(dev(w)) if dev(w).is_cuda else torch.zeros(B.tern_filter_bank_bytes(w.shape[0], w.shape[1], w.shape[2:]) // 4, dtype=torch.int32)
    cut = lambda c, v: dev(np.full(c, v, np.int32))
    class Mod:                          # host stand-in for NetModule, which takes device tensors only
        def __init__(self, c_out, w_bank, thr_lo, thr_hi, k, stride=(1, 1, 1), pad=(0, 0, 0), dil=(1, 1, 1), skip_from=-1, up=(1, 1, 1), pool=(1, 1, 1)):
            self.__dict__.update({n: v for n, v in locals().items() if n != "self"})
    M = B.NetModule if dev(w0).is_cuda else Mod
    mods = [M(40, bank(w0), cut(40, -1), cut(40, 1), k=(3, 3, 3), pad=(1, 1, 1)),
            M(24, bank(w1), cut(24, -2), cut(24, 2), k=(1, 3, 3), skip_from=0, up=(1, 1, 1), pool=(1, 2, 2))]
    g = np.random.default_rng(7)
    return dict(x=dev(g.standard_normal((2, 2, 3, 10, 12)).astype(np.float32)), in_lo=dev(np.full(2, -0.5, np.float32)),
                in_hi=dev(np.full(2, 0.5, np.float32)), mods=mods, head_w=dev(g.standard_normal((3, 24, 1, 2, 2)).astype(np.float32)),
                head_b=dev(np.zeros(3, np.float32)))


def undersized(B, net):
    """Changes to a network's tensors that leave one of them smaller than what the library reads of it."""
    import copy
    yield "in_lo", dict(net, in_lo=net["in_lo"][:1]), "C entries"
    yield "in_hi", dict(net, in_hi=net["in_hi"][:1]), "C entries"
    for i in (0, 1):
        for name, match in (("w_bank", "module %d: w_bank" % i), ("thr_lo", "module %d: cut" % i), ("thr_hi", "module %d: cut" % i)):
            mods = [copy.copy(m) for m in net["mods"]]
            setattr(mods[i], name, getattr(mods[i], name)[:-1])
            yield "%s %d" % (name, i), dict(net, mods=mods), match
    yield "head_b", dict(net, head_b=net["head_b"][:2]), "head_b"
    yield "head_w", dict(net, head_w=net["head_w"][:, :23].contiguous()), "24 input channels"


def test_network_parameters_smaller_than_what_is_read_are_refused_on_the_host(B):
    """The library gets bare pointers, so the binding compares sizes (here on host tensors, through the
    function that stands in front of the call)."""
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a))

    def sizes(n):
        return B._head_sizes(B._net_sizes(n["x"].shape, n["in_lo"], n["in_hi"], n["mods"]), n["head_w"], n["head_b"], 1, 0, 1)
    net = small_net(B, dev)
    assert sizes(net) == (2, 3, 3, 2, 3)
    for name, bad, match in undersized(B, net):
        with pytest.raises(ValueError, match=match):
            sizes(bad)
    large = dict(net, in_lo=torch.zeros(9), head_b=torch.zeros(9))     # as before: more than needed is fine
    assert sizes(large) == sizes(net)


def test_what_a_unet_plan_keeps_by_input_shape_is_bounded(B, monkeypatch):
    from paper_1801_09449_amd import unet
    plan = unet.UNetPlan.__new__(unet.UNetPlan)
    net = small_net(B, lambda a: torch.from_numpy(np.ascontiguousarray(a)))
    plan.mods, plan._digit_mods, plan._macs, plan._ws = net["mods"], {}, {}, None
    plan._shapes, plan._chosen, plan._need = {}, {}, {}
    monkeypatch.setattr(B, "tern_net_workspace_bytes", lambda shape, mods: 16)
    held = lambda: sum(len(d) for d in vars(plan).values() if isinstance(d, dict))
    for i in range(1000):
        x = torch.empty(1, 2, 3, 8 + i, 8, device="meta")
        assert plan.workspace(x).numel() == 16 and plan.modules(x.shape) == net["mods"]
        assert held() <= 256
    assert held() > 0 and plan.modules(x.shape) is plan.modules((1, 2, 3, 8 + i, 8))


@pytest.mark.gpu
def test_network_parameters_smaller_than_what_is_read_raise_before_a_launch(B):
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    net = small_net(B, dev)
    want, other = both(B, lambda: B.tern_net_forward(**net))
    assert torch.equal(want, other) and want.shape == (2, 3, 3, 2, 3)
    out = torch.empty(want.numel() + 5, device="cuda")
    for case in [net, dict(net, head_w=None, head_b=None)]:
        p, q = both(B, lambda: B.tern_net_forward(**case))
        assert p is q is None or torch.equal(p, q)
    assert B.tern_net_forward(**net, head_out=out) is out and torch.equal(out[:want.numel()].view_as(want), want)
    for name, bad, match in list(undersized(B, net)) + [("head_out", dict(net, head_out=out[:want.numel() - 1]), "head_out")]:
        p, q = both(B, lambda: B.tern_net_forward(**bad))
        assert isinstance(p, tuple) and p[0] is ValueError and match in p[1] and p == q, (name, p, q)


@pytest.mark.gpu
def test_calls_go_to_the_current_stream(B):
    src = torch.from_numpy(synth.ternary((1, 64, 8, 8, 8), 0.4, 903, synth.T_ACT)).cuda()
    want = B.tern_pack(src)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        g = torch.cuda.CUDAGraph()
        out = torch.zeros_like(want)
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=s):      # captured only if it went to this stream
            B.tern_pack(src, out)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
