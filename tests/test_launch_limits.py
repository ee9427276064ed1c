"""What the library launches, on a stand-in for the HIP runtime (tests/fake_hip.cpp: no GPU): no launch takes more LDS than has been
requested for its kernel, whatever was launched before it in this or another context; which kernels calls of stated sizes take."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)      # ahead of the HIP runtime that the library loads
from paper_2107_13490_amd import binding as b
fake.fake_launched.restype = C.c_char_p
lib = b.load_library()
at = 1 << 40      # operands are never read
def context():
    h = C.c_void_p()
    assert lib.adapt_create(C.byref(h), None, 64 << 20) == 0
    return h
"""
LAYERS = """
def layer(h, shape, wx, ww):
    d, fx, fw, ep = b.ConvDesc(*shape), b.Fmt(wx, 4), b.Fmt(ww, 4), b.Epilogue.exact()
    assert lib.adapt_conv_fwd(h, d, at, fx, 2 * at, fw, 3 * at, ep) == 0
    assert lib.adapt_conv_backward(h, d, at, fx, 2 * at, fw, 3 * at, fx, 4 * at, ep, 5 * at, ep) == 0
# layers whose patches differ: the smaller ones first, and again in a second context after the larger ones
shapes = [(256, 16, 16, 64, 128, 3, 3, 1, 1), (256, 16, 16, 128, 128, 3, 3, 1, 1), (171, 19, 20, 64, 128, 3, 3, 1, 1), (64, 32, 32, 64, 128, 5, 5, 1, 2),
          (64, 32, 32, 128, 128, 5, 5, 1, 2), (256, 8, 8, 192, 256, 3, 3, 1, 1), (64, 32, 32, 64, 64, 3, 3, 1, 1), (96, 32, 32, 64, 64, 5, 5, 1, 2)]
first, second = context(), context()
for wx, ww in ((12, 12), (8, 13), (16, 8), (16, 16)):
    for h, order in ((first, shapes), (second, shapes[:2]), (first, shapes[::-1])):
        for s in order:
            layer(h, s, wx, ww)
print(fake.fake_launches(), fake.fake_big_launches(), fake.fake_over_limit())
"""


def _run(calls, tmp_path):
    from paper_2107_13490_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    lib = str(tmp_path / "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", lib], check=True)
    return subprocess.run([sys.executable, "-c", PRELUDE + calls, lib], stdout=subprocess.PIPE, text=True, cwd=ROOT, check=True).stdout


def test_launches_stay_within_the_lds_requested_for_their_kernels(tmp_path):
    launches, big, over = (int(v) for v in _run(LAYERS, tmp_path).split()[-3:])
    assert launches > 100 and big > 20
    assert over == 0


QUANTIZE = """
h = context()
for n, wl in ((45 << 20, 12), (1 << 26, 12), (1 << 27, 12), ((1 << 27) + 1, 12), (1 << 28, 8), ((1 << 28) + 1, 8)):
    assert lib.adapt_quantize(h, at, n, b.Fmt(wl, 4), b.Rng(1, 1, 1), 2 * at, 3 * at, 4 * at) == 0
    one = fake.fake_launched().decode()
    items = (b.QuantizeItem * 4)(*(b.QuantizeItem(at, 2 * at, n // 4 + (n % 4 if i == 0 else 0), wl, 4, i) for i in range(4)))
    assert lib.adapt_quantize_batched(h, items, 4, 1, 1, 3 * at) == 0
    print(n, wl, int("quantize_kernelI%sLb0ELb1E" % ("a" if wl <= 8 else "s") in one), int("quantize_batched_kernelILb0ELb1E" in fake.fake_launched().decode()))
"""


def test_codes_are_stored_past_the_caches_only_where_they_exceed_the_last_one(tmp_path):
    rows = [[int(v) for v in line.split()] for line in _run(QUANTIZE, tmp_path).splitlines()]
    assert len(rows) == 6
    for n, wl, one, batch in rows:
        past = n * (1 if wl <= 8 else 2) > 256 << 20
        assert (one, batch) == (past, past), (n, wl)


PATCHES = """
h = context()
for n, hh, c, k in ((192, 16, 64, 128), (355, 8, 64, 240), (13, 32, 64, 400), (256, 32, 64, 64)):
    for wx, ww in ((12, 12), (16, 16), (8, 13), (12, 9)):
        f = b.Fmt(wx, 4), b.Fmt(ww, 4)
        fake.fake_launched()
        assert lib.adapt_conv_fwd(h, b.ConvDesc(n, hh, hh, c, k, 3, 3, 1, 1), at, f[0], 2 * at, f[1], 3 * at, b.Epilogue.exact()) == 0
        assert lib.adapt_conv_dgrad(h, b.ConvDesc(n, hh, hh, k, c, 3, 3, 1, 1), at, f[0], 2 * at, f[1], 3 * at, b.Epilogue.exact()) == 0
        for launch in fake.fake_launched().decode().split():
            name, lds = launch.rsplit("/", 1)
            if "halo_kernel" in name and "Li128ELi64E" in name:
                print(c, lds)
"""


def test_patches_of_one_chunk_of_channels_leave_room_for_three_blocks(tmp_path):
    rows = [[int(v) for v in line.split()] for line in _run(PATCHES, tmp_path).splitlines()]
    assert len(rows) >= 16 and all(3 * lds <= 160 * 1024 for _, lds in rows), rows
