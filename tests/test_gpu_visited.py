"""The forgetting visited tables of the search against the exact bitmap, on the GPU: the results never depend on
what a table remembers."""
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


def exact(ix, Q, k, L):
    nq = Q.shape[0]
    ids = torch.empty((nq, k), dtype=torch.int32, device=Q.device)
    ds = torch.empty((nq, k), device=Q.device)
    ev = torch.empty(nq, dtype=torch.int32, device=Q.device)
    hops = torch.empty(nq, dtype=torch.int32, device=Q.device)
    rg.rg_search_noalloc_into(ix, Q, k, L, ids, ds, hops, ev)
    return ids, ds, hops, ev


def graph(n, deg, seed, special=None):
    """Rows of deg random ids, some of them twice in a row, the first rows holding the special ids twice each."""
    rng = np.random.default_rng(seed)
    nb = rng.integers(0, n, size=(n, deg), dtype=np.int64)
    nb[:, 0] = (np.arange(n) + 1) % n
    nb[::3, deg // 2] = nb[::3, 1]          # a copy far from its first place
    nb[::5, 2] = nb[::5, 1]                 # and next to it
    if special is not None:
        s = np.resize(special, (64, deg // 2))
        nb[:64, :deg // 2] = s
        nb[:64, deg // 2:deg // 2 * 2] = s
    return np.arange(n + 1, dtype=np.int64) * deg, nb.astype(np.uint32).reshape(-1)


# n: 16-bit entries with room to spare, entries of exactly 16 bits at 2^8
# (where one entry per set is the mark of a free place), and more than 16 bits
# at 2^8 (a table of ids); deg: a full 64-id turn, and rows of several turns
@pytest.mark.parametrize("n,deg", [(3000, 16), (3000, 64), (3000, 90), ((1 << 22) + 77, 16), ((1 << 23) + 5, 8)])
@pytest.mark.parametrize("storage", ["fp32", "fp8"])
def test_tables_return_the_exact_results(dev, n, deg, storage):
    print(f"visited tables n={n} deg={deg} {storage}", flush=True)
    g = torch.Generator().manual_seed(n + deg)
    X = torch.randn(n, 8, generator=g)
    bits = max(1, (n - 1).bit_length())
    u = np.arange(n, dtype=np.uint64)
    h = (u * np.uint64(2654435761)) & np.uint64((1 << bits) - 1)
    marked = u[(h & np.uint64(0xFFFF)) == np.uint64(0xFFFF)]
    off, idx = graph(n, deg, n + deg, marked if len(marked) else None)
    Q = torch.randn(40, 8, generator=g).to(dev)
    ix = rg.rg_index_from_csr(X.to(dev), off, idx, 3)
    if storage == "fp8":
        rg.rg_index_set_storage(ix, rg.RG_STORE_FP8E4M3)
    for k, L in ((10, 20), (50, 200)):
        ids, ds, hops, ev = exact(ix, Q, k, L)
        for hb in (8, 9, 11, None):
            if hb == 8 and deg > 64:
                continue
            a = rg.rg_search(ix, Q, k, L, stats=True, hash_bits=hb)
            torch.cuda.synchronize()
            assert torch.equal(a[0], ids) and torch.equal(a[1], ds) and torch.equal(a[2], hops), (k, L, hb)
            assert (a[3] >= ev).all()
        assert all(len(set(r.tolist())) == k for r in ids)   # no node twice


# nq: the limits of 8, 4 and 2 wavefronts per query, and one past them; L: the
# limits of 2, 8 and 16 queue entries per lane; n = 60000 visits more nodes at
# L = 1024 than the exact table in LDS holds, so it overflows into the bitmap
# (several times at 4 wavefronts), n = 3000 keeps its bitmap in LDS past 512
# queries.  Rows hold copies.
@pytest.mark.parametrize("storage", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("n,d,deg", [(3000, 40, 24), (60000, 8, 48), (300, 230, 64)])
def test_few_queries_equal_the_sequential_search(dev, n, d, deg, storage):
    g = torch.Generator().manual_seed(n + d)
    X, Q = torch.randn(n, d, generator=g), torch.randn(1030, d, generator=g).to(dev)
    off, idx = graph(n, deg, n + d)
    ix = rg.rg_index_from_csr(X.to(dev), off, idx, 7)
    if storage != "fp32":
        rg.rg_index_set_storage(ix, rg.RG_STORE_BF16 if storage == "bf16" else rg.RG_STORE_FP8E4M3)
    for nq, k, L in ((1, 1, 1), (1, 10, 128), (5, 10, 129), (256, 100, 512), (257, 5, 513), (300, 10, 1024),
                     (2, 10, 1024), (512, 10, 64), (513, 10, 100), (1024, 10, 20), (1025, 10, 20)):
        print(f"few queries n={n} {storage} nq={nq} k={k} L={L}", flush=True)
        ids, ds, hops, ev = exact(ix, Q[:nq].contiguous(), k, L)
        a = rg.rg_search(ix, Q[:nq].contiguous(), k, L, stats=True)
        torch.cuda.synchronize()
        assert torch.equal(a[0], ids) and torch.equal(a[1], ds) and torch.equal(a[2], hops), (nq, k, L)
        assert torch.equal(a[3], ev) if storage == "fp32" and n / 8 <= 8.0 * L * d else (a[3] >= ev).all(), (nq, k, L)


# Batches past the few-query kernel: sets in LDS (8 KB for FP32 rows of d > 128)
# unless the rows scored of FP32 are asked for; rows of more than 64 ids stay
# with the bitmap; two wavefronts per query up to four queries per CU for rows
# of 512 bytes and more.  Longest queues leave the least LDS.
@pytest.mark.parametrize("n,d,deg,storage", [(40000, 8, 48, "fp32"), (40000, 60, 24, "fp32"), (33000, 129, 64, "fp32"),
                                             (40000, 100, 90, "fp32"), (33000, 256, 32, "bf16"), (33000, 513, 32, "fp8")])
def test_batches_equal_the_sequential_search(dev, n, d, deg, storage):
    g = torch.Generator().manual_seed(n + d)
    X, Q = torch.randn(n, d, generator=g), torch.randn(1300, d, generator=g).to(dev)
    off, idx = graph(n, deg, n + d)
    ix = rg.rg_index_from_csr(X.to(dev), off, idx, 7)
    if storage != "fp32":
        rg.rg_index_set_storage(ix, rg.RG_STORE_BF16 if storage == "bf16" else rg.RG_STORE_FP8E4M3)
    for nq, k, L in ((513, 10, 100), (1024, 10, 130), (1025, 10, 200), (1300, 10, 20), (1100, 1, 512), (600, 700, 1024)):
        print(f"batch n={n} d={d} {storage} nq={nq} k={k} L={L}", flush=True)
        ids, ds, hops, ev = exact(ix, Q[:nq].contiguous(), k, L)
        a = rg.rg_search(ix, Q[:nq].contiguous(), k, L)
        b = rg.rg_search(ix, Q[:nq].contiguous(), k, L, stats=True)
        torch.cuda.synchronize()
        assert torch.equal(a[0], ids) and torch.equal(a[1], ds), (nq, k, L)
        assert torch.equal(b[0], ids) and torch.equal(b[1], ds) and torch.equal(b[2], hops), (nq, k, L)
        if storage == "fp32" and n / 8 <= 8.0 * max(k, L) * d:
            assert torch.equal(b[3], ev), (nq, k, L)
