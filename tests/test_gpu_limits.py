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
