"""What planned contractions read lies inside their operands (a host program, tests/plan_extents.hip; no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_planned_reads_stay_inside_the_operands(tmp_path):
    from paper_2107_13490_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    lib = os.path.dirname(build.LIB)
    exe = str(tmp_path / "plan_extents")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17",
                    "-Wno-unused-function", "-I", os.path.join(ROOT, "include"), "-I", build.CSRC,
                    os.path.join(ROOT, "tests", "plan_extents.hip"), "-o", exe, "-L", lib, "-ladapt_fxp", "-Wl,-rpath," + lib], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
