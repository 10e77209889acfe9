"""Builds and insertions of rows near the ends of FP32's range, on the GPU, bit for bit against the oracle: the FP32
sums that turn candidates away must not overflow or underflow into a decision."""
import numpy as np
import pytest

from oracle.updates import Updatable

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
rg = pytest.importorskip("paper_2408_08933_amd")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rg.lib()
    return torch.device("cuda:0")


def check(dev, oracle_lib, X, T, Nq, M, L):
    ix = rg.rg_build(torch.from_numpy(X).to(dev), torch.from_numpy(T).to(dev), Nq, M, L_build=L)
    G = oracle_lib.Graph(X, T, Nq, M, L)
    off, idx, entry = ix.graph()
    assert entry == G.entry and ix.build_stats()["repairs"] == G.repairs
    assert np.array_equal(off, G.offsets) and np.array_equal(idx, G.indices)


def clusters(rng, n, d, norm):
    """Two opposite clusters of n / 2 rows: a longer queue compares rows whose distances are as large as norm^2."""
    X = rng.standard_normal((n, d)) * 0.6
    c = rng.standard_normal(d)
    X += np.where(np.arange(n) % 2, 1.0, -1.0)[:, None] * c
    return (X / np.linalg.norm(X, axis=1, keepdims=True) * norm).astype(np.float32)


# norms: |q||x| below FP32's largest value, around it and far above
@pytest.mark.parametrize("norm", [1.5e19, 2e19, 3e19, 1e22, 1e30])
def test_build_of_very_long_rows(dev, oracle_lib, norm):
    print(f"build of norm {norm}", flush=True)
    rng = np.random.default_rng(3)
    X, T = clusters(rng, 600, 200, norm), rng.standard_normal((400, 200)).astype(np.float32)
    check(dev, oracle_lib, X, T, 16, 24, 400)


def test_insertion_of_very_long_rows(dev, oracle_lib):
    print("insertion", flush=True)
    rng = np.random.default_rng(4)
    X, T = clusters(rng, 600, 200, 3e19), rng.standard_normal((400, 200)).astype(np.float32)
    ix = rg.rg_build(torch.from_numpy(X).to(dev), torch.from_numpy(T).to(dev), 16, 24, L_build=400, keep_stages=True)
    st = Updatable.from_graph(oracle_lib.Graph(X, T, 16, 24, 400), X, T)
    V = clusters(rng, 40, 200, 4e19)
    ix.insert(V)
    st.insert(V)
    off, idx, entry = ix.graph()
    o2, i2 = st.csr()
    assert np.array_equal(off, o2) and np.array_equal(idx, i2) and entry == st.entry


# scale of the short rows: their squares are FP32 normal numbers, subnormal ones and zero
@pytest.mark.parametrize("short", [1e-10, 1e-19, 1e-23, 1e-30])
def test_build_of_short_rows_among_long_ones(dev, oracle_lib, short):
    # Long rows in groups that differ by an FP32 rounding or two per coordinate: a short row is about as near to one of
    # them as to another, so only the last bits of the sums decide which of them keep it out
    print(f"build of rows of {short} among rows of 1e10", flush=True)
    rng = np.random.default_rng(5)
    d, groups, copies = 200, 24, 12
    X = np.repeat(rng.standard_normal((groups, d)), copies, axis=0) * 1e10
    X *= 1 + rng.integers(-3, 4, X.shape) * 2.0 ** -23
    X = np.concatenate([X, rng.standard_normal((300, d)) * short]).astype(np.float32)
    X = X[rng.permutation(len(X))]
    T = rng.standard_normal((400, d)).astype(np.float32)
    check(dev, oracle_lib, X, T, 100, 32, 500)
