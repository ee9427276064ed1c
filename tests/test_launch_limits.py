"""No launch takes more LDS than the library has requested for its kernel, whatever was launched before it in this or another
context (on a stand-in for the HIP runtime, tests/fake_hip.cpp: no GPU)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CALLS = """
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)      # ahead of the HIP runtime that the library loads
from paper_2107_13490_amd import binding as b
lib = b.load_library()
at = 1 << 40      # operands are never read
def context():
    h = C.c_void_p()
    assert lib.adapt_create(C.byref(h), None, 64 << 20) == 0
    return h
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


def test_launches_stay_within_the_lds_requested_for_their_kernels(tmp_path):
    from paper_2107_13490_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    lib = str(tmp_path / "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", lib], check=True)
    r = subprocess.run([sys.executable, "-c", CALLS, lib], stdout=subprocess.PIPE, text=True, cwd=ROOT, check=True)
    launches, big, over = (int(v) for v in r.stdout.split()[-3:])
    assert launches > 100 and big > 20
    assert over == 0
