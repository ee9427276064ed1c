"""What planned contractions read lies inside their operands, and which kernels calls take (host programs, tests/plan_extents.hip
and tests/plan_routes.hip; no GPU)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _host_program(name, out):
    from paper_2107_13490_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    lib = os.path.dirname(build.LIB)
    exe = str(out / name)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17",
                    "-Wno-unused-function", "-I", os.path.join(ROOT, "include"), "-I", build.CSRC,
                    os.path.join(ROOT, "tests", name + ".hip"), "-o", exe, "-L", lib, "-ladapt_fxp", "-Wl,-rpath," + lib], check=True)
    return exe


def test_planned_reads_stay_inside_the_operands(tmp_path):
    r = subprocess.run([_host_program("plan_extents", tmp_path)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout[-2000:]


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    """call -> (rows, splits, positions and threads of the slab sum) of its weight gradient alone, and beside the data gradient"""
    exe = _host_program("plan_routes", tmp_path_factory.mktemp("routes"))

    def plan(calls):
        out = subprocess.run([exe], input="\n".join(" ".join(map(str, c)) for c in calls), stdout=subprocess.PIPE, text=True, check=True).stdout
        lines = [[int(v) for v in line.split()] for line in out.splitlines()]
        assert len(lines) == len(calls)
        return [(tuple(v[:4]), tuple(v[4:])) for v in lines]
    return plan


def test_weight_gradients_take_image_rows_only_where_they_are_faster(routes):
    # n, h, w, c, k, r, s, stride, pad, bits of dy, w, x; measured in us on the implicit GEMM and on image rows
    slower = [
        (414, 12, 9, 72, 344, 3, 3, 1, 1, 16, 16, 16),       # 96.4, 121.2: row sums, against the double-buffered tiles
        (100, 20, 19, 144, 224, 3, 3, 1, 1, 16, 16, 16),     # 83.6, 98.8
        (24, 28, 27, 176, 352, 3, 3, 1, 1, 16, 16, 16),      # 79.9, 88.8
        (17, 16, 13, 400, 512, 3, 3, 1, 1, 16, 16, 16),      # 60.0, 66.1: no slabs on either side
        (3, 32, 29, 464, 304, 3, 3, 1, 1, 12, 12, 12),       # 35.1, 36.6: twelve stages against no slabs
        (14, 12, 9, 448, 432, 3, 3, 1, 1, 16, 12, 8),        # 18.2, 23.9
    ]
    faster = [
        (256, 16, 16, 128, 128, 3, 3, 1, 1, 12, 12, 12),     # 65.2, 54.7
        (256, 32, 32, 64, 64, 3, 3, 1, 1, 12, 12, 12),       # 68.0, 49.5
        (256, 32, 32, 64, 64, 3, 3, 1, 1, 16, 16, 16),       # 84.5, 62.2
        (128, 8, 8, 384, 256, 3, 3, 1, 1, 12, 12, 8),        # 47.6, 34.9
        (256, 16, 16, 128, 128, 3, 3, 1, 1, 8, 12, 12),      # 51.3, 37.2
    ]
    plans = routes(slower + faster)
    assert [p[0][0] for p in plans] == [0] * len(slower) + [1] * len(faster)


def test_backward_calls_give_up_a_shared_launch_only_for_less_time(routes):
    # the weight gradient alone is faster on image rows in all of them; us of the whole call, one launch and two
    shared = [
        (128, 4, 4, 512, 512, 3, 3, 1, 1, 12, 12, 12),       # 61.3, 87.7
        (192, 4, 4, 512, 512, 3, 3, 1, 1, 16, 16, 16),       # 106.6, 130.6
        (128, 8, 8, 192, 384, 3, 3, 1, 1, 12, 12, 12),       # 74.9, 82.3
        (24, 20, 19, 96, 448, 3, 3, 1, 1, 12, 12, 12),       # 62.3, 84.3
        (198, 6, 6, 192, 272, 3, 3, 1, 1, 12, 12, 12),       # 54.3, 65.6
    ]
    apart = [
        (154, 20, 20, 304, 48, 3, 3, 1, 1, 10, 16, 9),       # 190.1, 131.9
        (386, 31, 30, 64, 144, 1, 3, 1, 1, 12, 14, 13),      # 178.3, 134.2
        (303, 7, 7, 304, 144, 3, 3, 1, 1, 15, 16, 9),        # 146.1, 102.1
        (128, 8, 8, 384, 256, 3, 3, 1, 1, 12, 12, 12),       # 91.4, 87.8
        (256, 16, 16, 128, 128, 3, 3, 1, 1, 12, 12, 12),     # no shared launch: the data gradient runs on patches
    ]
    plans = routes(shared + apart)
    assert all(alone[0] == 1 for alone, _ in plans)
    assert [both[0] for _, both in plans] == [0] * len(shared) + [1] * len(apart)


def test_the_gpu_tests_of_image_rows_and_of_the_slab_sum_reach_them(routes):
    from test_gpu_contract import ROWS_CASES, SLAB_SUM_CASES
    from test_gpu_net import ROWS_NETS
    calls = [(n, h, w, c, k, r, s, 1, pad, dy, dy, x) for n, h, w, c, k, r, s, pad, dy, x, _ in ROWS_CASES]
    for call, case, (alone, _) in zip(calls, ROWS_CASES, routes(calls)):
        assert (alone[0], alone[3]) == (1, case[-1]), (case, alone)
        assert (alone[1] == 1 and alone[2] == 0) == (case[-1] == 0), (case, alone)
    calls = [(n, h, w, c, k, r, 3, 1, 1, dy, dy, x) for n, h, w, c, k, r, x, dy, _ in ROWS_NETS]
    for case, (alone, both) in zip(ROWS_NETS, routes(calls)):
        route = alone if case[6] == case[7] else both        # a layer in front: both gradients in one call
        assert (route[0], route[3]) == (1, case[-1]), (case, route)
    calls = [(40, 32, 32, c, k, 3, 3, 1, 1, wl, wl, wl) for c, k, _ in SLAB_SUM_CASES for wl in (8, 12)]
    threads = [t for *_, t in SLAB_SUM_CASES for _ in range(2)]
    assert [(alone[0], alone[3]) for alone, _ in routes(calls)] == [(0, t) for t in threads]


def test_slab_positions_on_image_rows_fit_32_bits(routes):
    # the widest slabs: half of the output channels' tiles empty, weights just below the 2^31 that calls may have
    plans = routes([(1, p + r - 1, 130, c, 33, r, 3, 1, 0, 12, 12, 8) for p, r, c in ((16, 33, 343999), (16, 51, 249999), (16, 71, 191991))])
    assert all(alone[0] == 1 and 1 << 31 < alone[2] < (1 << 32) - (1 << 20) for alone, _ in plans), plans
