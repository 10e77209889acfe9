"""The FP16 candidate pass against a threshold (k_scan16) on the GPU: tile and
register-class edges, and the queries that fall back to the running top-K."""
import sys

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


def check_topk(Q, X, K, ids, sc):
    """ids / sc are the K best rows of X by the FP32 sum of the FP16-rounded products, (score desc, id asc): every
    score is its pair's sum up to FP32 accumulation of dp terms (two units per add, so any adder and order), and no
    row left out can score more than the K-th."""
    q, x = Q.half().double(), X.half().double()
    S, A = q @ x.T, q.abs() @ x.abs().T
    dp = (Q.shape[1] + 31) // 32 * 32
    gacc = 2 * dp * 2.0 ** -24 / (1 - 2 * dp * 2.0 ** -24)
    ids, sc = ids.long(), sc.double()
    assert ((ids >= 0) & (ids < X.shape[0])).all()
    assert (ids.sort(dim=1).values.diff(dim=1) > 0).all()
    assert ((S.gather(1, ids) - sc).abs() <= gacc * A.gather(1, ids)).all()
    step = sc.diff(dim=1)
    assert ((step < 0) | ((step == 0) & (ids.diff(dim=1) > 0))).all()
    left = (S - gacc * A).scatter(1, ids, -np.inf)
    assert (left.amax(dim=1) <= sc[:, -1]).all()


# widths: one and seven 32-coordinate blocks in registers, the last of them
# partly filled, and the any-width kernel; n: the smallest that is sampled, a
# ragged last tile, and several splits of the base
@pytest.mark.parametrize("nq,n,d,K", [(1, 4096, 32, 49), (129, 4097, 1, 60), (300, 5003, 33, 1), (64, 20011, 200, 200),
                                      (130, 9000, 224, 256), (65, 6000, 225, 58), (128, 5000, 256, 100),
                                      (40, 12345, 300, 58), (1500, 50001, 96, 128)])
def test_scan_is_fp16_topk(dev, nq, n, d, K):
    print(f"knn scan nq={nq} n={n} d={d} K={K}", flush=True)
    g = torch.Generator().manual_seed(nq + n + d + K)
    X, Q = torch.randn(n, d, generator=g).to(dev), torch.randn(nq, d, generator=g).to(dev)
    ids, sc = rg.rg_knn_candidates_f16(Q, X, K)
    torch.cuda.synchronize()
    check_topk(Q, X, K, ids, sc)


@pytest.mark.parametrize("case", ["overflow", "underflow", "one tile"])
def test_wrong_threshold_falls_back(dev, case):
    # overflow: more rows tie for the best than a buffer holds; underflow: the
    # sampled rows are the best ones, so their threshold passes too few; one
    # tile: all the best rows in one tile of the base, more than the LDS queue
    # holds
    print(f"knn scan {case}", flush=True)
    g = torch.Generator().manual_seed(5)
    n, d, K = 8192, 40, 58
    X, Q = 0.1 * torch.randn(n, d, generator=g), torch.randn(1, d, generator=g) + 0.1 * torch.randn(200, d, generator=g)
    if case == "overflow":
        X[1000:6000] = Q[0]
    elif case == "underflow":
        X[::4] += Q[0]   # K = 58: every fourth row is sampled
    else:
        X[1024:1152] += Q[0]
    X, Q = X.to(dev), Q.to(dev)
    ids, sc = rg.rg_knn_candidates_f16(Q, X, K)
    torch.cuda.synchronize()
    check_topk(Q, X, K, ids, sc)
    if case == "overflow":
        assert (ids == torch.arange(1000, 1000 + K, device=dev)).all()
    sys.stdout.flush()
