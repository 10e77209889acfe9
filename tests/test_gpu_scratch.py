"""Calls on a device without room for their large buffers, on the GPU: the results are those of one with room.  Each
case runs in a process of its own, where hipMalloc refuses requests above a limit (native/alloc_limit.cpp)."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes as C, sys
limiter = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)
limiter.alloc_limit.argtypes, limiter.alloc_refuse.argtypes = [C.c_uint64], [C.c_uint64, C.c_int64]
limiter.alloc_failed.restype = C.c_int64
import numpy as np, torch
import paper_2408_08933_amd as rg
g = torch.Generator().manual_seed(4)
def with_room_and_without(call, limit=0, refuse=0, times=-1):
    a = call()
    torch.cuda.synchronize()
    print("with room", flush=True)
    limiter.alloc_limit(limit)
    limiter.alloc_refuse(refuse, times)
    b = call()
    torch.cuda.synchronize()
    limiter.alloc_limit(0)
    limiter.alloc_refuse(0, 0)
    assert limiter.alloc_failed() > 0
    print("without", flush=True)
    return a, b
"""


@pytest.fixture(scope="module")
def limiter(tmp_path_factory):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    so = str(tmp_path_factory.mktemp("limit") / "alloc_limit.so")
    subprocess.run([shutil.which("g++") or "c++", "-std=c++17", "-O1", "-shared", "-fPIC",
                    os.path.join(ROOT, "tests", "native", "alloc_limit.cpp"), "-o", so, "-ldl"], check=True)
    return so


def run(limiter, body):
    r = subprocess.run([sys.executable, "-u", "-c", PRELUDE + textwrap.dedent(body), limiter], cwd=ROOT,
                       capture_output=True, text=True, timeout=100)
    print(r.stdout, r.stderr, flush=True)
    assert r.returncode == 0


def test_knn_without_room_for_the_sweep(limiter):
    # 40,000 queries: 655 MB of buffers for the sweep, none of the running top-K's above 300 MB
    run(limiter, """
        X, Q = torch.randn(9000, 24, generator=g).cuda(), torch.randn(40_000, 24, generator=g).cuda()
        a, b = with_room_and_without(lambda: rg.rg_knn(Q, X, 20), 400 << 20)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    """)


def test_knn_in_parts(limiter):
    # 200,000 queries: 320 MB of candidates, none of the running top-K's buffers above 269 MB
    run(limiter, """
        X, Q = torch.randn(5000, 8, generator=g).cuda(), torch.randn(200_000, 8, generator=g).cuda()
        a, b = with_room_and_without(lambda: rg.rg_knn(Q, X, 100), 300 << 20)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
        assert sum(rg.rg_knn_last_stats().values()) == 200_000
    """)


def test_knn_out_of_fp16_range_without_room_for_fp16_rows(limiter):
    # 1.25M x 128: FP16 rows of 320 MB
    run(limiter, """
        X, Q = 1e5 * torch.randn(1_250_000, 128, generator=g).cuda(), torch.randn(200, 128, generator=g).cuda()
        a, b = with_room_and_without(lambda: rg.rg_knn(Q, X, 20), 300 << 20)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    """)


# 150,000 rows, lists of 31: no room for the selected distances of all nodes, or for the offsets of the reverse updates
# (8 bytes a row), where the projection goes to the host too
@pytest.mark.parametrize("refuse", [8 * 31 * 150_000, 8 * 150_001])
def test_build_without_room_for_all_selections(limiter, refuse):
    run(limiter, f"""
        X, T = torch.randn(150_000, 16, generator=g).cuda(), torch.randn(20_000, 16, generator=g).cuda()
        a, b = with_room_and_without(lambda: rg.rg_build(X, T, 16, 64, L_build=48).graph(), refuse={refuse})
        assert a[2] == b[2] and np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    """)


def test_build_without_room_for_rows_beside_the_lists(limiter):
    # the padded rows are refused while the lists are on the device: 48 coordinates are not padded, so that no other
    # buffer has their size
    run(limiter, """
        X, T = torch.randn(20_000, 48, generator=g).cuda(), torch.randn(20_000, 48, generator=g).cuda()
        a, b = with_room_and_without(lambda: rg.rg_build(X, T, 16, 24, L_build=64).graph(), refuse=4 * 48 * 20_000, times=1)
        assert a[2] == b[2] and np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    """)
