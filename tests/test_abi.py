"""The C-ABI library loads and exports every entry point include/adapt_fxp.h declares (CPU only:
no compute call is made)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "adapt_fxp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(adapt_[a-z0-9_]+)\s*\(", text)))


def test_header_declares_the_documented_entry_points():
    names = _declared()
    for must in ("adapt_create", "adapt_destroy", "adapt_quantize", "adapt_quantize_batched", "adapt_fxp_gemm",
                 "adapt_conv_fwd", "adapt_conv_dgrad", "adapt_conv_wgrad", "adapt_kld_precision_search",
                 "adapt_kld_precision_search_batched", "adapt_acc_bits", "adapt_error_string"):
        assert must in names


def test_library_exports_every_declared_symbol():
    import paper_2107_13490_amd as pkg
    path = pkg.library_path()
    if not os.path.exists(path):
        import __graft_entry__
        __graft_entry__.build()
    lib = ctypes.CDLL(path)
    for name in _declared():
        assert hasattr(lib, name), name
    lib.adapt_error_string.restype = ctypes.c_char_p
    assert lib.adapt_error_string(0) == b"ok"
    assert lib.adapt_version() >= 1


def test_acc_bits_rule():
    import paper_2107_13490_amd as pkg
    from paper_2107_13490_amd import Fmt
    assert pkg.acc_bits(256, Fmt(8, 6), Fmt(8, 6)) == 32
    assert pkg.acc_bits((1 << 17) - 1, Fmt(8, 0), Fmt(8, 0)) == 32        # (2^17-1) * 2^14 < 2^31
    assert pkg.acc_bits(1 << 17, Fmt(8, 0), Fmt(8, 0)) == 64
    assert pkg.acc_bits(1, Fmt(16, 0), Fmt(16, 0)) == 32                  # 2^30
    assert pkg.acc_bits(2, Fmt(16, 0), Fmt(16, 0)) == 64
    assert pkg.acc_bits(1152, Fmt(12, 9), Fmt(12, 9)) == 64


def test_no_cpu_fallback():
    import torch
    import paper_2107_13490_amd as pkg
    if torch.cuda.is_available():
        pytest.skip("GPU present")
    with pytest.raises(RuntimeError):
        pkg.Context()


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 2 and "one GPU" in r.stderr


def test_header_is_plain_c(tmp_path):
    """The boundary is a C ABI: the header must compile as C99 on its own, and every declared function must be usable
    from C (its address is taken below)."""
    import subprocess
    names = _declared()
    src = tmp_path / "use_header.c"
    body = ",\n".join(f"    (fn){n}" for n in names)
    src.write_text('#include "adapt_fxp.h"\n\ntypedef void (*fn)(void);\nfn table[] = {\n' + body + "\n};\n")
    inc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include")
    r = subprocess.run(["gcc", "-std=c99", "-Wall", "-Werror", "-pedantic", "-fsyntax-only", "-I", inc, str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_host_side_sizing_needs_no_gpu():
    """Workspace queries and the chain's layout are host arithmetic: they answer without a device."""
    import ctypes as C
    import paper_2107_13490_amd as pkg
    from paper_2107_13490_amd import ConvDesc, Fmt, LayerDesc, NodeDesc
    from paper_2107_13490_amd.binding import WorkspaceQuery
    lib = pkg.load_library()
    assert pkg.acc_bits(64, Fmt(24, 0), Fmt(8, 0)) == 128 and pkg.acc_bits(64, Fmt(8, 0), Fmt(32, 0)) == 128
    assert pkg.acc_bits(64, Fmt(33, 0), Fmt(8, 0)) < 0

    def need(call, **kw):
        q = WorkspaceQuery()
        q.call = call
        for k, v in kw.items():
            setattr(q, k, v)
        return lib.adapt_workspace_bytes(None, C.byref(q))

    d = ConvDesc(128, 16, 16, 64, 192, 3, 3, 1, 1)
    narrow = need(pkg.CALL_CONV_FWD, conv=d, fa=Fmt(8, 5), fb=Fmt(8, 5))
    two = need(pkg.CALL_CONV_FWD, conv=d, fa=Fmt(12, 9), fb=Fmt(12, 9))
    wide = need(pkg.CALL_CONV_FWD, conv=d, fa=Fmt(24, 20), fb=Fmt(24, 20))
    assert 0 < narrow <= two < wide
    # the parts of the operands and the exact sums of the outputs are part of a wide call's need
    outputs = 128 * 16 * 16 * 192
    assert wide >= 8 * outputs + 16 * outputs
    back = need(pkg.CALL_CONV_BACKWARD, conv=d, fa=Fmt(32, 0), fb=Fmt(32, 28), fc=Fmt(32, 28))
    assert back == max(need(pkg.CALL_CONV_DGRAD, conv=d, fa=Fmt(32, 0), fb=Fmt(32, 28)), need(pkg.CALL_CONV_WGRAD, conv=d, fa=Fmt(32, 0), fb=Fmt(32, 28)))
    assert need(pkg.CALL_CONV_FWD, conv=d, fa=Fmt(33, 5), fb=Fmt(8, 5)) == 0              # no such format
    assert need(pkg.CALL_KLD_SEARCH, n=1 << 20, wl_lo=2, wl_hi=32, bins=2048) > need(pkg.CALL_KLD_SEARCH, n=1 << 20, wl_lo=4, wl_hi=16, bins=2048) > 0

    layers = (LayerDesc * 2)(LayerDesc(ConvDesc(4, 8, 8, 4, 8, 3, 3, 1, 1), 1, 1), LayerDesc(ConvDesc(4, 1, 1, 128, 10, 1, 1, 1, 0), 0, 0))
    w16 = lib.adapt_net_workspace_bytes(layers, 2, 0)
    w32 = lib.adapt_net_workspace_bytes_wide(layers, 2, 0, 32)
    assert 0 < w16 < w32 <= 2 * w16 + 4096 and lib.adapt_net_workspace_bytes_wide(layers, 2, 0, 16) == w16
    assert lib.adapt_net_workspace_bytes_wide(layers, 2, 0, 24) == 0                          # 16 or 32
    assert lib.adapt_net_workspace_bytes(layers, 2, 4) > w16                                  # the lookback rings
    bad = (LayerDesc * 2)(layers[0], LayerDesc(ConvDesc(4, 1, 1, 100, 10, 1, 1, 1, 0), 0, 0))  # 128 values do not feed 100 inputs
    assert lib.adapt_net_workspace_bytes(bad, 2, 0) == 0
    c = ConvDesc(2, 4, 4, 8, 8, 3, 3, 1, 1)
    nodes = (NodeDesc * 3)(NodeDesc(c, 1, 0, 1, -1, -1, 0), NodeDesc(c, 1, 0, 1, -1, -1, 0), NodeDesc(c, 1, 0, 1, -1, 0, 1))
    g16 = lib.adapt_graph_workspace_bytes(nodes, 3, 0)
    assert 0 < g16 < lib.adapt_graph_workspace_bytes_wide(nodes, 3, 0, 32)
    assert lib.adapt_bn_state_bytes(64) >= 64 + 64 * 52 and lib.adapt_bn_state_bytes(0) == 0 and lib.adapt_bn_state_bytes(5000) == 0


@pytest.mark.parametrize("bad", [(8.0, 6), (8, None), ("8", 6), (8, 6, 1)])
def test_kept_formats_refuse_what_the_structure_refuses(bad):
    from paper_2107_13490_amd import binding
    with pytest.raises((TypeError, ValueError)):
        binding._fmt(bad)
    f = binding._fmt((8, 6))
    assert (f.wl, f.fl) == (8, 6)


def test_batched_descriptors_are_those_of_the_structures():
    import numpy as np
    import torch
    from paper_2107_13490_amd import binding as b

    class Recorder:
        def __getattr__(self, name):
            return lambda h, items, *rest: (setattr(self, "items", bytes(items)), 0)[1]

    cx = b.Context.__new__(b.Context)
    cx._lib, cx._torch, cx._h = Recorder(), torch, None
    ts = [torch.zeros(4 + t) for t in range(3)]
    kw = dict(outs=ts, counters=torch.zeros(6, dtype=torch.int64))

    def check(cls, rows):
        got = (cls * len(rows)).from_buffer_copy(cx._lib.items)
        for g, row in zip(got, rows):
            want = cls(*row)
            assert [getattr(g, f) for f, _ in cls._fields_] == [getattr(want, f) for f, _ in cls._fields_]
    # what the fields take: plain and numpy integers, negative and oversized ones (they wrap)
    for streams in ([1, 2, 3], np.arange(3), list(np.arange(3, dtype=np.uint64)), [-1, 1 << 64, 5], torch.arange(3)):
        for wl in (8, np.int32(8), (1 << 32) + 8):
            cx.quantize_batched(ts, [(wl, 5)] * 3, streams, **kw)
            check(b.QuantizeItem, [(t.data_ptr(), t.data_ptr(), t.numel(), wl, 5, s) for t, s in zip(ts, streams)])
        kld, sel = torch.zeros(3, 15, dtype=torch.float64), torch.zeros(3, 2, dtype=torch.int32)
        cx.kld_precision_search_batched(ts, [2, 2, 2], [64, np.int64(65), 66], streams, 2, 16, 0.1, kld=kld, sel=sel)
        check(b.KldItem, [(t.data_ptr(), t.numel(), 2, 64 + i, s) for i, (t, s) in enumerate(zip(ts, streams))])
    same = [ts[0]] * 2
    cx.gradient_diversity(same, [(8, 5), (np.int64(9), -1)], sums=ts[0], out=ts[0])
    check(b.GradItem, [(ts[0].data_ptr(), 8, 5), (ts[0].data_ptr(), 9, -1)])
    cx.quantize_batched([], [], [], counters=ts[0])
    assert cx._lib.items == bytes(40)
    # and what they refuse
    for bad in ((8.5, 5), (8, "5"), (None, 5)):
        with pytest.raises(TypeError):
            cx.quantize_batched(ts, [bad] * 3, [1, 2, 3], **kw)
        with pytest.raises(TypeError):
            cx.gradient_diversity(same, [bad] * 2, sums=ts[0], out=ts[0])
    for call in (lambda: cx.quantize_batched(ts, [(8, 5)] * 3, [1, 2], **kw), lambda: cx.quantize_batched(ts, [(8, 5)] * 2, [1, 2, 3], **kw),
                 lambda: cx.gradient_diversity(same, [(8, 5)], sums=ts[0], out=ts[0])):
        with pytest.raises(IndexError):
            call()
    assert (b._fmt((8,)).wl, b._fmt((8,)).fl) == (8, 0) and b._fmt(np.array([9, 4])).fl == 4
