"""What the library asks of the device, on the CPU: a runtime without a device (native/fake_hip.cpp) takes the place
of HIP's, records launches instead of running them and keeps two of its rules, grids of fewer than 2^32 threads and an
amount of memory.  Each case runs in a process of its own, which never loads the real runtime's calls."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

import paper_2408_08933_amd as rg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++")
pytestmark = pytest.mark.skipif(not CXX, reason="needs g++")

PRELUDE = """
import ctypes as C, sys
import numpy as np
fake, lib = C.CDLL(sys.argv[1], C.RTLD_GLOBAL), C.CDLL(sys.argv[2])
lib.rg_last_error.restype = C.c_char_p
fake.fake_launch.restype = C.c_char_p
fake.fake_launches.restype = C.c_int64
fake.fake_most.restype = fake.fake_in_use.restype = fake.fake_shared.restype = C.c_uint64
fake.fake_limit.argtypes, fake.fake_amax.argtypes = [C.c_uint64], [C.c_float]
I64, P = C.c_int64, lambda a: C.c_void_p(a.ctypes.data)
class Opts(C.Structure):
    _fields_ = [(k, C.c_int32) for k in ("L_build", "m_pj", "m_ce", "threads", "knn_slack", "keep_stages")]
def ok(rc):
    assert rc == 0, (rc, lib.rg_last_error())
def launches(*names):
    g, b, out = C.c_uint64(), C.c_uint64(), []
    for i in range(fake.fake_launches()):
        name = fake.fake_launch(I64(i), C.byref(g), C.byref(b)).decode()
        if any(n in name for n in names):
            out.append((name, g.value, b.value))
    return out
def build(X, T, Nq, M, L, m_pj=0, m_ce=0, keep=0):
    ix, o = C.c_void_p(), Opts(L, m_pj, m_ce, 8, 0, keep)
    rc = lib.rg_build(P(X), I64(X.shape[0]), X.shape[1], P(T), I64(T.shape[0]), Nq, M, 0, C.byref(o), None, C.byref(ix))
    if rc == 0:
        lib.rg_free(ix)
    return rc
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run([CXX, "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "native", "fake_hip.cpp"),
                    "-o", so], check=True, capture_output=True, text=True)
    return so


def run(fake, body, timeout=300):
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), fake, rg.LIB_PATH], capture_output=True,
                       text=True, timeout=timeout)
    assert r.returncode == 0, r.stdout + r.stderr


def test_build_past_2_to_24_rows(fake):
    # the smallest n whose one workgroup of 256 per node is a grid of 2^32 threads, and one more
    run(fake, """
        n = (1 << 24) + 1
        ok(build(np.zeros((n, 1), np.float32), np.zeros((8, 1), np.float32), 2, 3, 4, 1, 1))
        for kernel, times in (("k_sort_events", 2), ("k_replay_fill", 1), ("k_replayE", 1)):
            at = launches(kernel)
            assert sum(g for _, g, _ in at) == times * n, (kernel, at)
            assert max(g for _, g, _ in at) <= 1 << 22, (kernel, at)
    """)


@pytest.mark.parametrize("n", [300, 40_000])
def test_search_of_2_to_26_queries(fake, n):
    # n: a base whose visited bitmap lies in LDS, and one with a visited table.  No kernel runs, so neither queries nor
    # results are touched
    run(fake, f"""
        n, nq = {n}, (1 << 26) + 1
        X, off, idx = np.zeros((n, 64), np.float32), np.arange(n + 1), np.zeros(n, np.uint32)
        ix = C.c_void_p()
        ok(lib.rg_index_from_csr(P(X), I64(n), 64, P(off), P(idx), 0, 0, None, C.byref(ix)))
        ok(lib.rg_search(ix, P(X), I64(nq), 1, 50, P(idx), P(X), None, None, None))
        at = launches("k_search")
        assert sum(g for _, g, _ in at) == nq and max(g for _, g, _ in at) <= 1 << 25, at
        lib.rg_free(ix)
    """)


def test_knn_without_room_for_the_sweep(fake):
    # 131,072 queries: the sweep's buffers take 2.4 GB beside what the running top-K needs too, which fits
    run(fake, """
        n, nq, d, k = 8192, 1 << 17, 8, 16
        X, Q = np.zeros((n, d), np.float32), np.zeros((nq, d), np.float32)
        ids, ds = np.zeros((nq, k), np.uint32), np.zeros((nq, k), np.float32)
        fake.fake_limit(1 << 30)
        ok(lib.rg_knn(P(Q), I64(nq), P(X), I64(n), d, k, P(ids), P(ds), None))
        assert launches("k_knn16") and not launches("k_scan16")
        assert fake.fake_in_use() == 0
    """)


def test_knn_out_of_fp16_range_needs_no_fp16_rows(fake):
    # 4M x 64: FP16 rows of 537 MB, while the FP32 passes that such values take need 300 MB
    run(fake, """
        n, nq, d, k = 4 << 20, 1000, 64, 10
        X, Q = np.zeros((n, d), np.float32), np.zeros((nq, d), np.float32)
        ids, ds = np.zeros((nq, k), np.uint32), np.zeros((nq, k), np.float32)
        fake.fake_amax(1e6)
        fake.fake_limit(400 << 20)
        ok(lib.rg_knn(P(Q), I64(nq), P(X), I64(n), d, k, P(ids), P(ds), None))
        assert launches("k_knnE") and not launches("k_knn16", "k_scan16")
        fake.fake_amax(1.0)
        assert lib.rg_knn(P(Q), I64(nq), P(X), I64(n), d, k, P(ids), P(ds), None) == -2
        assert fake.fake_in_use() == 0
    """)


def test_knn_without_room_for_the_sample(fake):
    # 16M x 64: FP16 rows of 2.15 GB, a sample of 0.54 GB, 0.3 GB for the running top-K
    run(fake, """
        n, nq, d, k = 16 << 20, 1000, 64, 10
        X, Q = np.zeros((n, d), np.float32), np.zeros((nq, d), np.float32)
        ids, ds = np.zeros((nq, k), np.uint32), np.zeros((nq, k), np.float32)
        fake.fake_limit(2500 << 20)
        ok(lib.rg_knn(P(Q), I64(nq), P(X), I64(n), d, k, P(ids), P(ds), None))
        ok(lib.rg_knn_candidates_f16(P(Q), I64(nq), P(X), I64(n), d, 58, P(ids), P(ds), None))
        assert len(launches("k_knn16")) == 2 and not launches("k_scan16")
    """)


def test_build_knn_in_parts(fake):
    # 1M lists of 100: 1.6 GB of candidates and 0.5 GB of buffers beside the lists themselves (0.4 GB), which stay
    run(fake, """
        n, nt, d = 8192, 1 << 20, 8
        fake.fake_limit(2250 << 20)
        ok(build(np.zeros((n, d), np.float32), np.zeros((nt, d), np.float32), 100, 16, 32))
        assert sum(g for _, g, _ in launches("k_knn_certify")) == nt
        assert fake.fake_in_use() == 0
    """)


# MB: the selections of all nodes do not fit, or the lists after the reverse updates do not
@pytest.mark.parametrize("limit", [180, 345])
def test_build_without_room_for_all_selections(fake, limit):
    # 400,000 rows of 16: the base takes 26 MB, the projected graph 51 MB and a batch of searches and selections 56 MB;
    # the selections of all nodes take 150 MB and their first candidates 51 MB, their reverse updates 54 MB
    run(fake, f"""
        n, d = 400_000, 16
        fake.fake_limit({limit} * 1000 * 1000)
        ok(build(np.zeros((n, d), np.float32), np.zeros((1000, d), np.float32), 16, 64, 100))
        assert not launches("k_replayE") and sum(g for _, g, _ in launches("k_sort_events")) == ({limit} > 300) * 2 * n
        assert fake.fake_in_use() == 0
    """)


def test_build_without_room_for_rows_beside_the_lists(fake):
    # 3M rows of 128 (1.57 GB, 0.8 GB as FP16) and 4M lists of 32 (0.54 GB): rows and graph fit, rows and lists do not
    run(fake, """
        n, nt, d = 3 << 20, 4 << 20, 128
        X, T = np.zeros((n, d), np.float32), np.zeros((nt, d), np.float32)
        fake.fake_limit(2050 * 1000 * 1000)
        ok(build(X, T, 32, 8, 16))
        assert fake.fake_in_use() == 0
    """)


# rows of ids, d, L, KB of the table: short queues on wide rows keep 4 KB where one of 2 KB lets more workgroups share a
# CU; longer queues, other rows and narrow coordinates do not
@pytest.mark.parametrize("deg,d,L,kb", [(100, 200, 50, 4), (100, 96, 128, 4), (200, 200, 60, 4), (112, 256, 128, 4),
                                        (100, 200, 129, 2), (128, 200, 50, 2), (100, 64, 100, 2), (56, 200, 200, 2)])
def test_visited_table_of_wide_rows(fake, deg, d, L, kb):
    run(fake, f"""
        n, deg, d, L = 5000, {deg}, {d}, {L}
        X, idx = np.zeros((n, d), np.float32), np.zeros(n * deg, np.uint32)
        off, ix = np.arange(n + 1, dtype=np.int64) * deg, C.c_void_p()
        ok(lib.rg_index_from_csr(P(X), I64(n), d, P(off), P(idx), 0, 0, None, C.byref(ix)))
        ok(lib.rg_index_set_storage(ix, 1, None))
        fake.fake_reset()
        ok(lib.rg_search(ix, P(X), I64(10_000), 10, L, P(idx), P(X), None, None, None))
        assert len(launches("k_search")) == fake.fake_launches() == 1
        cand, pad = 64 if deg <= 64 else 128, (d + 15) // 16 * 16
        assert fake.fake_shared(I64(0)) - (4 * pad + 8 * L + 20 * cand) == {kb} << 10
        lib.rg_free(ix)
    """)


def test_calls_after_one_without_room(fake):
    # each call that finds no room says so, and leaves nothing behind for the next one
    run(fake, """
        n, d = 50_000, 64
        X, off, idx = np.zeros((n, d), np.float32), np.arange(n + 1), np.zeros(n, np.uint32)
        def index():
            ix = C.c_void_p()
            rc = lib.rg_index_from_csr(P(X), I64(n), d, P(off), P(idx), 0, 0, None, C.byref(ix))
            return rc, ix
        def search(nq, evals):
            return lib.rg_search(ix, P(X), I64(nq), 10, 100, P(idx), P(X), None, P(idx) if evals else None, None)
        rc, ix = index()
        ok(rc)
        calls = [lambda: search(1, False), lambda: search(2000, True), lambda: lib.rg_index_set_storage(ix, 1, None),
                 lambda: lib.rg_index_set_storage(ix, 2, None), lambda: index()[0],
                 lambda: lib.rg_knn(P(X), I64(10), P(X), I64(n), d, 5, P(idx), P(X), None)]
        for call in calls:
            fake.fake_limit(fake.fake_in_use() + 5000)
            assert call() == -2, lib.rg_last_error()
            fake.fake_limit(0)
            ok(search(2000, False))
        lib.rg_free(ix)
    """)
