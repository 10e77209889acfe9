"""Workloads of the public entry points, for timing and for comparing results.

Each case is one thing a program that uses the library does over and over: search an index with a few or many
queries (rg_search), compute exact nearest neighbours (rg_knn), build an index (rg_build) or serve a stream of
requests (Server).  prepare() makes what such a program holds before the call, run() is one call, work() the bytes
and operations the call cannot do without, exact() the same results from plain torch in 64 bits.

Vectors follow the synthetic out-of-distribution law of datagen (a Gaussian mixture in a shared low-rank subspace,
the queries scaled and shifted by a fixed gap), drawn on the GPU.  The indexes that are searched are made from a graph
of the shape a built index has where its searches run: about 30 near rows and 20 far ones per node.  Building one with
rg_build takes from seconds to minutes at these sizes and is a case of its own.
"""
import math
import time

import numpy as np
import torch

import paper_2408_08933_amd as rg

STORAGE = {"fp32": rg.RG_STORE_FP32, "bf16": rg.RG_STORE_BF16, "fp8": rg.RG_STORE_FP8E4M3}
ROW_BYTES = {"fp32": 4, "bf16": 2, "fp8": 1}
NEAR, FAR = 32, 24   # edges of a node to near rows and to any rows
WINDOW = 2048        # rows among which the near ones are looked for


def listed():
    return [
        # one interactive lookup: latency is all that counts
        {"name": "search one query", "do": "search", "n": 300_000, "d": 200, "store": "fp32", "nq": 1, "k": 10, "L": 100},
        # a page of lookups of one user request against image-text embeddings
        {"name": "search 16 queries bf16", "do": "search", "n": 200_003, "d": 512, "store": "bf16", "nq": 16, "k": 100,
         "L": 200},
        # the tiny workload's index, a thousand queries at once
        {"name": "search tiny index", "do": "search", "n": 10_000, "d": 64, "store": "fp32", "nq": 1000, "k": 10, "L": 50},
        # many rows, a short queue: the quick first stage of a retrieval pipeline
        {"name": "search short queue", "do": "search", "n": 700_001, "d": 100, "store": "fp32", "nq": 4096, "k": 1,
         "L": 32},
        # the benchmark's batch of 10k queries at its 1M x 200 operating point
        {"name": "search batch fp32", "do": "search", "n": 1_000_000, "d": 200, "store": "fp32", "nq": 10_000, "k": 10,
         "L": 175},
        # the 2M x 512 workload held in FP8 at its operating point
        {"name": "search batch fp8", "do": "search", "n": 2_000_000, "d": 512, "store": "fp8", "nq": 10_000, "k": 10,
         "L": 409},
        # recall above 0.9 on the hardest workload: a queue over 512 entries
        {"name": "search long queue", "do": "search", "n": 500_009, "d": 200, "store": "bf16", "nq": 3001, "k": 100,
         "L": 805},
        # ground truth of the benchmark's test queries
        {"name": "knn ground truth", "do": "knn", "n": 1_000_000, "d": 200, "nq": 10_000, "k": 100},
        # exact neighbours of a few vectors in a small table of odd sizes
        {"name": "knn small odd", "do": "knn", "n": 30_011, "d": 77, "nq": 257, "k": 10},
        # the tiny workload's build: a test or a notebook
        {"name": "build tiny", "do": "build", "n": 10_000, "d": 64, "nt": 10_000, "Nq": 32, "M": 32, "L": 200},
        # an ordinary build with the paper's parameters
        {"name": "build ordinary", "do": "build", "n": 60_000, "d": 200, "nt": 60_000, "Nq": 100, "M": 64, "L": 500},
        # a burst of requests with mixed k and L on the serving loop
        {"name": "serve burst", "do": "serve", "n": 300_000, "d": 200, "store": "fp32", "nq": 4000, "slots": 6144,
         "hops": 24},
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    do = rng.choice(["search"] * 5 + ["knn", "build", "serve"])
    if do == "search":
        d = rng.choice([64, 77, 96, 128, 200, 256, 384, 512, rng.randrange(33, 512)])
        L = _log(rng, 10, 1000)
        k = min(L, rng.choice([1, 10, 100, rng.randrange(1, 101)]))
        n = _log(rng, 10_000, max(10_000, min(1_000_000, 200_000_000 // d)))
        nq = _log(rng, 1, max(1, min(10_000, 4_000_000_000 // (ROW_BYTES["fp32"] * 5 * L * d))))
        return {"do": do, "n": n, "d": d, "store": rng.choice(["fp32", "bf16", "fp8"]), "nq": nq, "k": k, "L": L}
    if do == "knn":
        d = rng.choice([64, 200, 512, rng.randrange(17, 400)])
        n = _log(rng, 3000, 200_000_000 // max(d, 200))
        return {"do": do, "n": n, "d": d, "nq": _log(rng, 1, 10_000), "k": rng.choice([1, 10, 100, rng.randrange(1, 129)])}
    if do == "build":
        d = rng.choice([64, 200, rng.randrange(33, 200)])
        n = _log(rng, 2000, 50_000)
        return {"do": do, "n": n, "d": d, "nt": max(1000, int(n * rng.choice([0.3, 0.5, 1.0]))), "Nq": rng.choice([32, 50, 100]),
                "M": rng.choice([16, 32, 64]), "L": rng.choice([100, 200, 500])}
    return {"do": do, "n": _log(rng, 20_000, 300_000), "d": rng.choice([64, 200, 256]), "store": rng.choice(["fp32", "bf16", "fp8"]),
            "nq": _log(rng, 100, 4000), "slots": rng.choice([1024, 4096, 6144]), "hops": rng.choice([16, 24, 32])}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class Law:
    """Base rows and queries of one seed, drawn on the GPU (the laws of datagen)."""

    def __init__(self, d, seed):
        self.d = d
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.wide = d > 64                 # a low-rank mixture; narrow rows an isotropic one
        self.unit = d <= 64 or d >= 384    # cosine workloads: rows of unit length
        r = 32 if self.wide else d
        if self.wide:
            self.basis = torch.linalg.qr(self._randn(d, r))[0].contiguous()
        centres = 256 if self.wide else 16
        self.cx, self.cq = self._randn(centres, r), self._randn(centres, r)
        if not self.wide:
            self.cx, self.cq = (c / c.norm(dim=1, keepdim=True) for c in (self.cx, self.cq))
        gap = self._randn(d)
        self.gap = (1.5 if not self.unit else 0.8) * gap / gap.norm()
        self.scale = torch.ones(d, device="cuda") if self.unit else 0.5 + torch.rand(d, generator=self.g, device="cuda")

    def _randn(self, *shape):
        return torch.randn(*shape, generator=self.g, device="cuda")

    def _points(self, n, centres):
        z = torch.randint(centres.shape[0], (n,), generator=self.g, device="cuda")
        if not self.wide:
            return centres[z] + 0.3 * self._randn(n, self.d), z
        x = (centres[z] + 0.5 * self._randn(n, 32)) @ self.basis.T
        x += (0.6 * math.sqrt(200 / max(200, self.d))) * self._randn(n, self.d)
        return x / math.sqrt(32), z

    def base(self, n):
        x, z = self._points(n, self.cx)
        return (x / x.norm(dim=1, keepdim=True) if self.unit else x).contiguous(), z

    def queries(self, n):
        q = self._points(n, self.cq)[0] * self.scale + self.gap
        return (q / q.norm(dim=1, keepdim=True) if self.unit else q).contiguous()


def _graph(x, z, g):
    """Sorted adjacency (n x NEAR + FAR, repeats and the node itself as -1) and the entry."""
    n = x.shape[0]
    near, w = min(NEAR, n - 1), min(WINDOW, n)
    order = torch.argsort(z, stable=True)
    ids = torch.empty((n, near + FAR), dtype=torch.int64, device="cuda")
    for s in range(0, n, w):
        rows = order[s:s + w] if s + w <= n else order[n - w:]
        sim = x[rows] @ x[rows].T
        sim.fill_diagonal_(-math.inf)
        ids[rows, :near] = rows[sim.topk(near, dim=1).indices]
    ids[:, near:] = torch.randint(n, (n, FAR), generator=g, device="cuda")
    ids = ids.sort(dim=1).values
    drop = ids == torch.arange(n, device="cuda")[:, None]
    drop[:, 1:] |= ids[:, 1:] == ids[:, :-1]
    entry = int((x - x.mean(dim=0)).norm(dim=1).argmin())
    return ids.masked_fill_(drop, -1), entry


def _data(case, seed):
    law = Law(case["d"], seed)
    x, z = law.base(case["n"])
    adj, entry = _graph(x, z, law.g)
    return x, adj, entry, law.queries(case["nq"])


def _index(case, x, adj, entry):
    keep = adj >= 0
    off = np.zeros(x.shape[0] + 1, dtype=np.int64)
    off[1:] = keep.sum(dim=1).cumsum(0).cpu().numpy()
    ix = rg.rg_index_from_csr(x, off, adj[keep].to(torch.int32).cpu().numpy().view(np.uint32), entry)
    if case["store"] != "fp32":
        rg.rg_index_set_storage(ix, STORAGE[case["store"]])
    return ix


def _requests(case, seed):
    """k and L of each request of a burst: the serving mix of the benchmark."""
    r = np.random.Generator(np.random.PCG64(seed))
    return r.choice(np.asarray([1, 10, 100], np.int32), case["nq"]), r.choice(np.asarray([32, 128, 512], np.int32), case["nq"])


def prepare(case, seed):
    if case["do"] == "knn":
        law = Law(case["d"], seed)
        return {"do": "knn", "x": law.base(case["n"])[0], "q": law.queries(case["nq"]), "k": case["k"]}
    if case["do"] == "build":
        law = Law(case["d"], seed)
        return {"do": "build", "x": law.base(case["n"])[0], "t": law.queries(case["nt"]), "case": case}
    x, adj, entry, q = _data(case, seed)
    ix = _index(case, x, adj, entry)
    if case["do"] == "search":
        return {"do": "search", "ix": ix, "q": q, "k": case["k"], "L": case["L"]}
    k, L = _requests(case, seed)
    server = rg.Server(ix, max_slots=case["slots"], hops_per_step=case["hops"])
    return {"do": "serve", "server": server, "q": q.cpu().numpy(), "k": k, "L": L, "tags": np.arange(case["nq"], dtype=np.uint64)}


def run(state):
    if state["do"] == "search":
        ids, dists = rg.rg_search(state["ix"], state["q"], state["k"], state["L"])
        return {"ids": ids, "dists": dists}
    if state["do"] == "knn":
        ids, dists = rg.rg_knn(state["q"], state["x"], state["k"])
        return {"ids": ids, "dists": dists}
    if state["do"] == "build":
        c = state["case"]
        off, idx, entry = rg.rg_build(state["x"], state["t"], c["Nq"], c["M"], L_build=c["L"]).graph()
        edges = np.full(c["n"] * c["M"], -1, dtype=np.int32)
        edges[:len(idx)] = idx.view(np.int32)
        return {"offsets": off, "indices": edges, "entry": entry}
    server, n = state["server"], len(state["tags"])
    ids = np.full((n, 100), -1, dtype=np.int32)
    dists = np.full((n, 100), np.inf, dtype=np.float32)
    sent = got = 0
    while got < n:
        if sent < n:
            sent += server.submit_batch(state["q"][sent:], state["k"][sent:], state["L"][sent:], state["tags"][sent:])
        done = server.poll()
        for r in done:
            ids[r["tag"], :r["k"]] = r["ids"].view(np.int32)
            dists[r["tag"], :r["k"]] = r["dists"]
        got += len(done)
        if not done:
            time.sleep(2e-5)
    return {"ids": ids, "dists": dists}


# ---------------------------------------------------------------------------
# what a call cannot do without
# ---------------------------------------------------------------------------
def work(case):
    n, d = case["n"], case["d"]
    if case["do"] == "knn":
        return {"bytes": 4 * (n + case["nq"]) * d + 8 * case["nq"] * case["k"], "flops": 2 * case["nq"] * n * d}
    if case["do"] == "build":
        # the exact nearest rows of every training query, and one search per row that scores at least its queue of L
        return {"bytes": 4 * (n + case["nt"]) * d + 4 * n * case["M"], "flops": 2 * case["nt"] * n * d + 2 * n * case["L"] * d}
    # per queue entry about 1.15 expansions, each reading the row of its neighbours' ids, and 40 rows not seen before
    # (counted on these indexes: 33 to 53)
    if case["do"] == "serve":
        entries, k = case["nq"] * (32 + 128 + 512 + 100) / 3, 37
    else:
        entries, k = case["nq"] * max(case["L"], case["k"]), case["k"]
    rows = min(40 * entries, case["nq"] * n)
    rerank = 4 * d * entries if case["store"] != "fp32" else 0
    return {"bytes": rows * d * ROW_BYTES[case["store"]] + 1.15 * entries * 4 * (NEAR + FAR) + rerank + case["nq"] * (4 * d + 8 * k),
            "flops": 2 * d * rows}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------
def _stored(x, store):
    """The rows a search scores against, in 64 bits."""
    if store == "fp32":
        return x.double()
    if store == "bf16":
        return x.bfloat16().double()
    amax = x.abs().amax(dim=1, keepdim=True).double()
    s = torch.exp2(torch.ceil(torch.log2(amax / 448)))
    s = torch.where(448 * s / 2 >= amax, s / 2, s)
    return (x.double() / s).float().to(torch.float8_e4m3fn).double() * s


def _beam(rows, adj, entry, q, L):
    """Best-first searches of all queries at once: (delta, id) of the final queues, ascending."""
    nq, none = q.shape[0], rows.shape[0]
    dist = torch.full((nq, L), math.inf, dtype=torch.float64, device="cuda")
    ids = torch.full((nq, L), none, dtype=torch.int64, device="cuda")
    todo = torch.zeros((nq, L), dtype=torch.bool, device="cuda")
    dist[:, 0], ids[:, 0], todo[:, 0] = -(q @ rows[entry]), entry, True
    live = torch.arange(nq, device="cuda")
    while live.numel():
        at = todo[live].to(torch.uint8).argmax(dim=1)
        node = ids[live, at]
        todo[live, at] = False
        nb = adj[node]
        delta = -torch.bmm(rows[nb.clamp_min(0)], q[live][:, :, None].contiguous())[:, :, 0]
        place = torch.searchsorted(dist[live], delta)        # a row that is queued already stands at its distance
        old = nb < 0
        for o in (-1, 0, 1):
            old |= ids[live].gather(1, (place + o).clamp(0, L - 1)) == nb
        delta = torch.where(old, math.inf, delta)
        order = torch.cat([dist[live], delta], dim=1).sort(dim=1, stable=True)
        dist[live] = order.values[:, :L]
        ids[live] = torch.cat([ids[live], torch.where(old, none, nb)], dim=1).gather(1, order.indices[:, :L])
        todo[live] = torch.cat([todo[live], ~old], dim=1).gather(1, order.indices[:, :L])
        live = live[todo[live].any(dim=1)]
    return dist, ids


def _found(case, x, adj, entry, q, L):
    """The final queue of each search by its exact distance, padded with infinity."""
    rows = _stored(x, case["store"])
    dist, ids = _beam(rows, adj, entry, q.double(), L)
    if case["store"] != "fp32":
        exact = -torch.bmm(x.double()[ids.clamp_max(x.shape[0] - 1)], q.double()[:, :, None].contiguous())[:, :, 0]
        dist = torch.where(ids < x.shape[0], exact, math.inf).sort(dim=1).values
    return dist


def exact(case, seed):
    if case["do"] == "build":
        return None  # a graph: whole numbers
    if case["do"] == "knn":
        law = Law(case["d"], seed)
        x = law.base(case["n"])[0].double()
        q = law.queries(case["nq"]).double()
        step = max(1, 400_000_000 // case["n"])
        d = [-(q[s:s + step] @ x.T).topk(case["k"], dim=1).values for s in range(0, case["nq"], step)]
        return {"ids": None, "dists": torch.cat(d)}
    if case["do"] == "search":
        L, step = max(case["L"], case["k"]), max(1, 40_000_000 // max(case["d"] * 8, 16 * case["L"]))
        x, adj, entry, q = _data(case, seed)
        d = [_found(case, x, adj, entry, q[s:s + step], L)[:, :case["k"]] for s in range(0, case["nq"], step)]
        return {"ids": None, "dists": torch.cat(d)}
    x, adj, entry, q = _data(case, seed)
    k, L = _requests(case, seed)
    out = np.full((case["nq"], 100), np.inf)
    for kk in (1, 10, 100):
        for ll in (32, 128, 512):
            at = np.nonzero((k == kk) & (L == ll))[0]
            if len(at):
                out[at, :kk] = _found(case, x, adj, entry, q[torch.from_numpy(at).cuda()], max(kk, ll))[:, :kk].cpu().numpy()
    return {"ids": None, "dists": out}
