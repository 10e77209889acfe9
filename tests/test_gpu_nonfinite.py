"""Searches that meet distances that are no numbers, or infinite, on the GPU: such a row ranks behind all nearer ones
and enters the queue once, whichever kernel runs the search.  Finite coordinates are small whole numbers, so every
finite distance is exact in every storage form."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
rg = pytest.importorskip("paper_2408_08933_amd")
N, D, DEG = 3000, 24, 24


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rg.lib()
    return torch.device("cuda:0")


def data(kind):
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
    nb = rng.integers(0, N, (N, DEG), dtype=np.int64)
    nb[:, 0] = (np.arange(N) + 1) % N
    return X, Q, np.arange(N + 1, dtype=np.int64) * DEG, nb.astype(np.uint32)


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


@pytest.mark.parametrize("kind", ["none", "nan", "nan and inf", "queries"])
@pytest.mark.parametrize("storage", ["fp32", "bf16", "fp8"])
def test_every_kernel_returns_the_same(dev, kind, storage):
    print(f"{kind} {storage}", flush=True)
    X, Q, off, nb = data(kind)
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
            for j in range(0, 42):
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
