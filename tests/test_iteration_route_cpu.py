"""What cronus_iteration enqueues, on the host: api.cpp and plan.cpp as they are, with stubs for the launches and the HIP calls
(tests/native/iteration_check_main.cpp).  A decode iteration's rows are placed by the attention launch itself or by a scatter in
front of it; the results are the same bits, so only the route can tell which of the two ran."""
import os
import shutil
import subprocess

import pytest

from test_gpu_rows_in_launch import CASES, SCATTERED

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_17357_amd", "csrc")
SCATTER, PLACED = "0 rows attention", "0 attention+rows"
K, V, CU, START, OUT, WS = (0x100000000 * (i + 1) for i in range(6))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    cxx, rocm = shutil.which("g++"), os.environ.get("ROCM_PATH", "/opt/rocm")
    if cxx is None or not os.path.exists(os.path.join(rocm, "include", "hip", "hip_runtime.h")):
        pytest.skip("no host C++ compiler or no HIP headers")
    out = str(tmp_path_factory.mktemp("iteration") / "iteration_check")
    flags = ["-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-w", "-D__HIP_PLATFORM_AMD__",
             "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-isystem", os.path.join(rocm, "include")]
    subprocess.run([cxx, *flags, "-Drows_in_launch=rule_of_plan_cpp", "-c", os.path.join(CSRC, "plan.cpp"), "-o", out + ".plan.o"], check=True)
    subprocess.run([cxx, *flags, os.path.join(ROOT, "tests", "native", "iteration_check_main.cpp"), os.path.join(CSRC, "api.cpp"),
                    os.path.join(CSRC, "balancer.cpp"), out + ".plan.o", "-o", out], check=True)
    return out


def route(exe, P, C, heads=(32, 8, 128), fp8=False, failure="none", rows=None, second=0, k=K, v=V, cu=CU, start=START, out=OUT, ws=WS, ws_bytes=1 << 28):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
    env.pop("LD_PRELOAD", None)  # the sanitizer runtime must come first in the library list
    args = [*heads, int(fp8), failure, sum(C) if rows is None else rows, second, k, v, cu, start, out, ws, ws_bytes, len(P)]
    r = subprocess.run([exe, *map(str, args), *(str(x) for pc in zip(P, C) for x in pc)], capture_output=True, text=True, env=env, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr[-3000:]
    return r.stdout.strip()


def test_rows_that_lie_in_what_the_attention_writes(exe):
    """They are read before it starts, by the scatter, whichever of their arrays it is; next to it they may lie."""
    P, C = [100, 600, 40], [1, 1, 1]
    row, head_row = 3 * 8 * 128 * 2, 3 * 32 * 128 * 2
    assert route(exe, P, C) == PLACED
    for area, bytes_ in ((OUT, head_row), (WS, 1 << 28)):
        for name, size in (("k", row), ("v", row), ("cu", 16), ("start", 12)):
            for at, want in ((area - size, PLACED), (area - size + 1, SCATTER), (area, SCATTER), (area + bytes_ - 1, SCATTER), (area + bytes_, PLACED)):
                assert route(exe, P, C, **{name: at}) == want, (name, hex(at))


@pytest.mark.parametrize("rows", ["placed in the launch", "scattered"])
def test_rows_are_placed_where_the_attention_is_not_enqueued(exe, rows):
    """Errors that are found after the checks leave the rows placed, whichever route they were to take."""
    P, C = ([100, 9000, 40], [1, 1, 1]) if rows == "placed in the launch" else ([100, 9000], [50, 1])
    assert route(exe, P, C) == (PLACED if rows == "placed in the launch" else SCATTER)
    assert route(exe, P, C, ws_bytes=256) == "3 rows"
    for failure in ("setup", "buffer", "launch"):
        assert route(exe, P, C, failure=failure) == "4 rows"


def test_more_heads_than_the_scatter_takes_are_refused(exe):
    assert route(exe, [20], [1], heads=(65535, 65535, 64)).startswith("0 ")
    for P, C in (([20], [1]), ([20], [50])):
        assert route(exe, P, C, heads=(65536, 65536, 64)) == "1"


@pytest.mark.parametrize("name", CASES)
def test_route_of_the_cases_on_the_gpu(exe, name):
    shape, P, C, given = CASES[name]
    rows = sum(given[0]) if isinstance(given, tuple) else None
    heads = shape.n_q_heads, shape.n_kv_heads, shape.head_dim
    assert route(exe, P, C, heads, shape.kv_dtype == "fp8", rows=rows) == (SCATTER if name in SCATTERED else PLACED)


def test_rule_for_rows_in_the_launch(exe):
    """One set, one row for each of at most 64 decodes (8 sequences where any is skipped), at most 4400 keys a CU (a row counts as 900, heads beyond 32 a KV head twice)."""
    for n, want in ((1, PLACED), (63, PLACED), (64, PLACED), (65, SCATTER)):
        assert route(exe, [100] * n, [1] * n) == want
    P = [100, 600, 40]
    assert route(exe, P, [1, 1, 1], rows=2) == route(exe, P, [1, 1, 1], rows=4) == SCATTER
    assert route(exe, P, [1, 1, 1], rows=0, second=3) == PLACED
    assert route(exe, P, [1, 1, 1], rows=3, second=3) == SCATTER
    assert route(exe, P, [1, 2, 1]) == route(exe, P, [1, 2, 1], rows=3) == SCATTER
    assert route(exe, P, [1, 0, 1]) == PLACED and route(exe, P, [1, 0, 1], rows=3) == SCATTER
    for n, want in ((8, PLACED), (9, SCATTER)):
        assert route(exe, [100] * n, [1] * (n - 1) + [0]) == route(exe, [100] * n, [0] * (n - 1) + [1]) == want
    cus, row = 4400 * 256, 900
    for heads, copies in (((32, 8, 128), 8), ((28, 4, 128), 4), ((48, 2, 64), 2), ((80, 2, 128), 4), ((64, 2, 64), 2), ((66, 2, 64), 4)):
        for fp8 in (False, True):
            keys = cus // copies - 16 * row  # of 16 decodes, at most
            P = [keys // 16 - 1] * 15
            last = keys - 15 * (keys // 16) - 1
            assert route(exe, P + [last], [1] * 16, heads, fp8) == PLACED
            assert route(exe, P + [last + 1], [1] * 16, heads, fp8) == SCATTER
    assert route(exe, [1048575] * 64, [1] * 64, (64, 64, 64), ws_bytes=1 << 40) == SCATTER  # 2^32 keys


def test_launches_with_chunk_tiles_never_place_rows(exe):
    """Whatever the rule says: the kernels that place rows would run a tile as a narrow item."""
    for P, C in (([100], [50]), ([100, 9000], [50, 1]), ([3000, 100], [200, 9])):
        assert route(exe, P, C, failure="rule") == SCATTER
    assert route(exe, [100, 9000], [2, 8], failure="rule") == PLACED
