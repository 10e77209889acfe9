"""Builds on the GPU at the edges of the enhancement's kernels, bit for bit against the oracle."""
import numpy as np
import pytest

import datagen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
rg = pytest.importorskip("paper_2408_08933_amd")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rg.lib()
    return torch.device("cuda:0")


def check(dev, oracle_lib, X, T, Nq, M, L, m_pj=0, m_ce=0):
    print(f"build {X.shape[0]} x {X.shape[1]} Nq={Nq} M={M} L={L} m_pj={m_pj} m_ce={m_ce}", flush=True)
    ix = rg.rg_build(torch.from_numpy(X).to(dev), torch.from_numpy(T).to(dev), Nq, M, L_build=L, m_pj=m_pj, m_ce=m_ce)
    G = oracle_lib.Graph(X, T, Nq, M, L, m_pj, m_ce)
    off, idx, entry = ix.graph()
    assert entry == G.entry and ix.build_stats()["repairs"] == G.repairs
    assert np.array_equal(off, G.offsets) and np.array_equal(idx, G.indices)


# copies: equal distances everywhere, which the shared sums cannot order; hub:
# one row that every node selects (a list of 2,499 reverse updates, and lists
# just above 64); lists: up to 107 enhancement and 20 projected neighbours;
# the odd sizes: rows shorter than a 16-lane piece, fewer nodes than a
# wavefront, a queue longer than the base
@pytest.mark.parametrize("case,n,nt,d,Nq,M,L,m_pj,m_ce", [
    ("copies", 2000, 1500, 40, 24, 32, 150, 0, 0), ("hub", 2500, 1500, 40, 24, 32, 150, 0, 0),
    ("lists", 1500, 1500, 24, 40, 128, 300, 20, 107), ("plain", 61, 40, 3, 9, 8, 200, 0, 0),
    ("plain", 900, 2000, 230, 100, 64, 500, 0, 0), ("plain", 3000, 200, 65, 32, 7, 64, 2, 4),
    ("projected", 1500, 3000, 24, 60, 128, 200, 100, 27)])
def test_build_edges(dev, oracle_lib, case, n, nt, d, Nq, M, L, m_pj, m_ce):
    g = datagen.Generator(2, n=n, n_train=nt, n_test=1, d=max(d, 32))
    X, T = np.ascontiguousarray(g.base()[:, :d]), np.ascontiguousarray(g.train()[:, :d])
    if case == "copies":
        X[1::3] = X[0::3][:len(X[1::3])]
        X[700:760] = X[3]
    if case == "hub":
        X[5] *= 6
        X[17] *= 1.5
    check(dev, oracle_lib, X, T, Nq, M, L, m_pj, m_ce)


# the projection: lists of 63 and 64 entries (one and two slots per lane) that
# overflow, few pivots with many bridges (over 512 candidates), lists of two
# entries, pivots with fewer candidates than places
@pytest.mark.parametrize("case,n,nt,d,Nq,M,L,m_pj,m_ce", [
    ("plain", 1200, 4000, 24, 120, 128, 200, 63, 40), ("copies", 1200, 4000, 24, 120, 128, 200, 64, 40),
    ("few", 1000, 3000, 40, 224, 64, 500, 0, 0), ("hub", 1500, 3000, 20, 50, 8, 100, 2, 3),
    ("plain", 400, 60, 130, 2, 40, 64, 20, 8)])
def test_projection_edges(dev, oracle_lib, case, n, nt, d, Nq, M, L, m_pj, m_ce):
    g = datagen.Generator(3, n=n, n_train=nt, n_test=1, d=max(d, 32))
    X, T = np.ascontiguousarray(g.base()[:, :d]), np.ascontiguousarray(g.train()[:, :d])
    if case == "copies":
        X[1::3] = X[0::3][:len(X[1::3])]
        X[700:760] = X[3]
    if case == "hub":
        X[5:9] *= 5
    if case == "few":
        X[::40] *= 3
    check(dev, oracle_lib, X, T, Nq, M, L, m_pj, m_ce)
