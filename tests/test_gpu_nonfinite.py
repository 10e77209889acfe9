"""Searches that meet distances that are no numbers, or infinite, on the GPU: such a row ranks behind all nearer ones
and enters the queue once, whichever kernel runs the search.  Finite coordinates are small whole numbers, so every
finite distance is exact in every storage form."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
rg = pytest.importorskip("paper_2408_08933_amd")
N, D = 3000, 24


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rg.lib()
    return torch.device("cuda:0")


def data(kind, deg=24):
    rng = np.random.default_rng(9)
    X, Q = rng.integers(-7, 8, (N, D)).astype(np.float32), rng.integers(-7, 8, (1300, D)).astype(np.float32)
    odd = rng.permutation(N)[:400]
    if kind != "none":
        X[odd[:200], rng.integers(0, D, 200)] = np.nan
    if kind == "nan and inf":
        X[odd[200:300], 3] = np.inf
        X[odd[300:], 5] = -np.inf
    if kind == "queries":
        Q[::7, 2] = np.nan
    nb = rng.integers(0, N, (N, deg), dtype=np.int64)
    nb[:, 0] = (np.arange(N) + 1) % N
    return X, Q, np.arange(N + 1, dtype=np.int64) * deg, nb.astype(np.uint32)


def reference(X, q, nb, entry, L):
    """The final queue, (delta, id) ascending, a NaN counted as +inf; distances as they are, and the expansions."""
    with np.errstate(invalid="ignore"):
        raw = -(X.astype(np.float64) @ q.astype(np.float64))
    key = np.where(np.isnan(raw), np.inf, raw)
    queue, done, seen, hops = [(key[entry], entry)], set(), {entry}, 0
    while True:
        todo = next((i for _, i in queue if i not in done), None)
        if todo is None:
            return [i for _, i in queue], [raw[i] for _, i in queue], hops
        done.add(todo)
        hops += 1
        new = set(nb[todo].tolist()) - seen
        seen |= new
        queue = sorted(queue + [(key[i], i) for i in new])[:L]


# deg: rows of one turn, of two (a batch may hold more than 64 candidates) and CSR
@pytest.mark.parametrize("deg", [24, 100, 140])
@pytest.mark.parametrize("kind", ["none", "nan", "nan and inf", "queries"])
@pytest.mark.parametrize("storage", ["fp32", "bf16", "fp8"])
def test_every_kernel_returns_the_same(dev, kind, storage, deg):
    print(f"{kind} {storage} {deg}", flush=True)
    X, Q, off, nb = data(kind, deg)
    ix = rg.rg_index_from_csr(torch.from_numpy(X).to(dev), off, nb.reshape(-1), 3)
    if storage != "fp32":
        rg.rg_index_set_storage(ix, rg.RG_STORE_BF16 if storage == "bf16" else rg.RG_STORE_FP8E4M3)
    q = torch.from_numpy(Q).to(dev)
    for k, L in ((10, 40), (100, 200), (300, 600)):
        ids = torch.empty((len(Q), k), dtype=torch.int32, device=dev)
        ds, hops, ev = torch.empty((len(Q), k), device=dev), ids[:, 0].clone(), ids[:, 0].clone()
        rg.rg_search_noalloc_into(ix, q, k, L, ids, ds, hops, ev)
        for nq in (1, 16, 300, 600, 1300):
            for stats in (False, True):
                a = rg.rg_search(ix, q[:nq].contiguous(), k, L, stats=stats)
                torch.cuda.synchronize()
                assert torch.equal(a[0], ids[:nq]), (k, L, nq, stats)
                assert np.array_equal(a[1].cpu().numpy(), ds[:nq].cpu().numpy(), equal_nan=True), (k, L, nq, stats)
                assert not stats or torch.equal(a[2], hops[:nq]), (k, L, nq)
        assert all(len(set(r)) == k for r in ids.cpu().tolist())   # no node twice
        if storage == "fp32":
            for j in range(0, 42 if deg == 24 else 9):
                i, d, h = reference(X, Q[j], nb, 3, L)
                assert ids[j].cpu().tolist() == i[:k] and int(hops[j]) == h, (k, L, j)
                assert np.array_equal(ds[j].cpu().numpy().astype(np.float64), d[:k], equal_nan=True), (k, L, j)


def test_server_returns_the_same(dev):
    X, Q, off, nb = data("nan and inf")
    ix = rg.rg_index_from_csr(torch.from_numpy(X).to(dev), off, nb.reshape(-1), 3)
    ids, ds = rg.rg_search(ix, torch.from_numpy(Q).to(dev), 100, 200)
    ids, ds = rg.as_u32(ids), ds.cpu().numpy()
    s = rg.Server(ix, max_slots=256, hops_per_step=16)
    tags, sent, got = np.arange(len(Q), dtype=np.uint64), 0, 0
    k, L = np.full(len(Q), 100, np.int32), np.full(len(Q), 200, np.int32)
    while got < len(Q):
        if sent < len(Q):
            sent += s.submit_batch(Q[sent:], k[sent:], L[sent:], tags[sent:])
        for r in s.poll():
            assert np.array_equal(r["ids"], ids[r["tag"]]) and np.array_equal(r["dists"], ds[r["tag"]], equal_nan=True)
            got += 1
    s.close()


# deg of the projected graph: one turn and two; a base smaller than a list of candidates
@pytest.mark.parametrize("n,M,m_pj,m_ce", [(900, 24, 0, 0), (900, 128, 100, 27), (3000, 64, 0, 0)])
@pytest.mark.parametrize("kind", ["nan", "nan and inf", "queries"])
def test_build_equals_the_host(dev, kind, n, M, m_pj, m_ce):
    # rows: few NaNs, so that each training query has its neighbours at distances that are numbers
    rng = np.random.default_rng(n)
    X, T = rng.standard_normal((n, 40)).astype(np.float32), rng.standard_normal((n, 40)).astype(np.float32)
    at = rng.permutation(n)[:n // 20]
    if kind == "queries":
        T[at, 3] = np.nan
    else:
        X[at, 3] = np.nan
        if kind == "nan and inf":
            X[at[::2], 3] = np.inf
    Nq, L = 20, 100
    print(f"build {kind} n={n} M={M} m_pj={m_pj}", flush=True)
    ix = rg.rg_build(torch.from_numpy(X).to(dev), torch.from_numpy(T).to(dev), Nq, M, L_build=L, m_pj=m_pj, m_ce=m_ce)
    print("built", flush=True)
    knn, _ = rg.rg_knn(torch.from_numpy(T).to(dev), torch.from_numpy(X).to(dev), Nq)
    host = rg.rg_build_from_knn(X, rg.as_u32(knn), Nq, M, L_build=L, m_pj=m_pj, m_ce=m_ce)
    a, b = ix.graph(), host.graph()
    assert a[2] == b[2] and np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    assert np.diff(a[0]).max() <= M and a[1].max() < n


def test_build_refuses_lists_that_are_too_short(dev):
    rng = np.random.default_rng(1)
    X, T = rng.standard_normal((200, 16)).astype(np.float32), rng.standard_normal((50, 16)).astype(np.float32)
    T[7, 3] = np.nan
    with pytest.raises(rg.RGError) as e:
        rg.rg_build(torch.from_numpy(X).to(dev), torch.from_numpy(T).to(dev), 10, 16, L_build=32)
    assert e.value.code == -1
