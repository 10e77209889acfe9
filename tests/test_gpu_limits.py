"""Calls past the launches and buffers of ordinary sizes, on the GPU."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
rg = pytest.importorskip("paper_2408_08933_amd")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rg.lib()
    return torch.device("cuda:0")


def test_build_of_several_launches_per_step(dev):
    # one launch holds 2^18 nodes; the host's construction has no such steps
    n, nt, d, Nq, M, L = (1 << 18) + 777, 30_000, 16, 16, 12, 24
    g = torch.Generator().manual_seed(11)
    X, T = torch.randn(n, d, generator=g), torch.randn(nt, d, generator=g)
    print(f"build {n} x {d}", flush=True)
    ix = rg.rg_build(X.to(dev), T.to(dev), Nq, M, L_build=L)
    knn, _ = rg.rg_knn(T.to(dev), X.to(dev), Nq)
    print("the same on the host", flush=True)
    host = rg.rg_build_from_knn(X.numpy(), rg.as_u32(knn), Nq, M, L_build=L)
    a, b = ix.graph(), host.graph()
    assert a[2] == b[2] and np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


# n: a base whose visited bitmap lies in LDS, and one with a visited table
@pytest.mark.parametrize("n", [300, 40_000])
def test_search_of_several_launches(dev, n):
    # one launch holds 2^25 queries; the same 1,000 queries over and over
    g = torch.Generator().manual_seed(n)
    X, Q = torch.randn(n, 4, generator=g).to(dev), torch.randn(1000, 4, generator=g).to(dev)
    off, idx = np.arange(n + 1, dtype=np.int64) * 2, ((np.arange(n)[:, None] + [[1, 7]]) % n).astype(np.uint32).reshape(-1)
    ix = rg.rg_index_from_csr(X, off, idx, 3)
    one = rg.rg_search(ix, Q, 2, 4)
    times = (1 << 25) // 1000 + 2
    print(f"search n={n} nq={1000 * times}", flush=True)
    ids, ds = rg.rg_search(ix, Q.repeat(times, 1), 2, 4)
    torch.cuda.synchronize()
    assert torch.equal(ids, one[0].repeat(times, 1)) and torch.equal(ds, one[1].repeat(times, 1))
