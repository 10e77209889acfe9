// C ABI: argument checking, device memory of the index, the exact kNN
// (GPU candidates + certified FP64 rerank), search dispatch, index files.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <thread>

#include "rg_internal.h"

namespace rg {

static thread_local std::string g_err;
// rows certified from FP16 candidates, from FP32 candidates, by the host scan
static thread_local int64_t g_knn_rows[3];

void set_error(const std::string &msg) { g_err = msg; }

int no_memory(const std::string &msg) {
    (void)hipGetLastError();
    set_error(msg);
    return RG_ENOMEM;
}

namespace {

int32_t round_up(int32_t v, int32_t m) { return (v + m - 1) / m * m; }

template <class F>
void par_rows(int64_t n, int threads, F &&f) {
    threads = (int)std::max<int64_t>(1, std::min<int64_t>(threads, n));
    std::atomic<int64_t> next(0);
    auto work = [&]() {
        for (;;) {
            const int64_t s = next.fetch_add(64);
            if (s >= n) break;
            for (int64_t i = s; i < std::min(n, s + 64); ++i) f(i);
        }
    };
    std::vector<std::thread> pool;
    for (int t = 1; t < threads; ++t) pool.emplace_back(work);
    work();
    for (auto &th : pool) th.join();
}

struct DevBuf {
    void *p = nullptr;
    ~DevBuf() { release(); }
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr;
    }
    int alloc(size_t bytes) {
        if (hipMalloc(&p, bytes ? bytes : 1) != hipSuccess) {
            p = nullptr;
            return no_memory("out of device memory (" + std::to_string(bytes) + " bytes)");
        }
        return RG_OK;
    }
    template <class T>
    T *as() const {
        return static_cast<T *>(p);
    }
};

void free_index_device(rg_index *ix) {
    if (ix->d_base) (void)hipFree(ix->d_base);
    if (ix->d_adj) (void)hipFree(ix->d_adj);
    if (ix->d_adj_off) (void)hipFree(ix->d_adj_off);
    if (ix->d_tomb) (void)hipFree(ix->d_tomb);
    if (ix->d_bf16) (void)hipFree(ix->d_bf16);
    if (ix->d_fp8) (void)hipFree(ix->d_fp8);
    if (ix->d_scale) (void)hipFree(ix->d_scale);
    ix->d_base = nullptr;
    ix->d_adj = nullptr;
    ix->d_adj_off = nullptr;
    ix->d_tomb = nullptr;
    ix->d_bf16 = nullptr;
    ix->d_fp8 = nullptr;
    ix->d_scale = nullptr;
}

// Device copy of the base, rows padded to a 64-byte multiple.
int upload_base(rg_index *ix, const float *base_dev, hipStream_t st) {
    ix->pitch = round_up(ix->d, 16);
    if (hipMalloc(&ix->d_base, sizeof(float) * (size_t)ix->n * ix->pitch) != hipSuccess) {
        ix->d_base = nullptr;
        return no_memory("index: out of device memory for the base rows");
    }
    return launch_pad_rows(base_dev, ix->n, ix->d, ix->d_base, ix->pitch, st);
}

// Device adjacency: ELL rows of width ell = max degree rounded up to 8
// (kNone padded) when the degree allows, else CSR (offsets + indices, ell = 0).
int upload_adj(rg_index *ix, hipStream_t st) {
    const int64_t n = ix->n;
    int64_t maxdeg = 1;
    for (int64_t x = 0; x < n; ++x) maxdeg = std::max<int64_t>(maxdeg, ix->offsets[x + 1] - ix->offsets[x]);
    if (maxdeg > kMaxEll) {
        if (maxdeg >= (1ll << 31)) {
            set_error("index: out-degree does not fit 32 bits");
            return RG_EINVAL;
        }
        const int64_t nnz = ix->offsets[n];
        ix->ell = 0;
        if (hipMalloc(&ix->d_adj, sizeof(uint32_t) * (size_t)std::max<int64_t>(nnz, 1)) != hipSuccess) {
            ix->d_adj = nullptr;
            return no_memory("index: out of device memory for the adjacency");
        }
        if (hipMalloc(&ix->d_adj_off, sizeof(int64_t) * (size_t)(n + 1)) != hipSuccess) {
            ix->d_adj_off = nullptr;
            return no_memory("index: out of device memory for the adjacency");
        }
        RG_HIP(hipMemcpyAsync(ix->d_adj, ix->indices.data(), sizeof(uint32_t) * (size_t)nnz, hipMemcpyHostToDevice,
                              st));
        RG_HIP(hipMemcpyAsync(ix->d_adj_off, ix->offsets.data(), sizeof(int64_t) * (size_t)(n + 1),
                              hipMemcpyHostToDevice, st));
        RG_HIP(hipStreamSynchronize(st));
        return RG_OK;
    }
    ix->ell = round_up((int32_t)maxdeg, 8);
    if (hipMalloc(&ix->d_adj, sizeof(uint32_t) * (size_t)n * ix->ell) != hipSuccess) {
        ix->d_adj = nullptr;
        return no_memory("index: out of device memory for the adjacency");
    }
    std::vector<uint32_t> ell((size_t)n * ix->ell, kNone);
    for (int64_t x = 0; x < n; ++x)
        std::copy(ix->indices.begin() + ix->offsets[x], ix->indices.begin() + ix->offsets[x + 1],
                  ell.begin() + x * ix->ell);
    RG_HIP(hipMemcpyAsync(ix->d_adj, ell.data(), sizeof(uint32_t) * ell.size(), hipMemcpyHostToDevice, st));
    RG_HIP(hipStreamSynchronize(st));
    return RG_OK;
}

}  // namespace

// The visited table of the LDS-table search at 4 << hash_bits bytes: sets of
// 16-bit entries, or ids where an entry would need more bits (n > 2^(15 +
// hash_bits)) or an expansion more than one turn (rows over 64 ids, CSR).
void set_table(SearchArgs &a, int hash_bits) {
    int bits = 1;
    while (bits < 31 && (a.n_rows - 1) >> bits) ++bits;
    a.hash_bits = hash_bits;
    a.id_bits = std::max(bits, hash_bits - 1);
    a.sets = !a.adj_off && a.ell <= 64 && a.id_bits - (hash_bits - 1) <= 16;
}

namespace {

// The size: the largest of 4, 2 and 1 KB that keeps the most wavefronts per
// SIMD at work, up to five, as far as there are queries for them.  A smaller
// table scores more rows (about 7% from one size to the next), fewer
// wavefronts wait longer for each: per row, E4M3 d = 200 L = 409 takes 0.69 /
// 0.80 / 1.00 (us x 1e-3) at 20 / 16 / 11 workgroups per CU, and counts between
// two multiples of 4 run like the lower one (a SIMD more or less).  A sixth per
// SIMD is not worth a smaller table (BF16 1M x 100 L = 200 at 20 / 24: 4.5 /
// 5.2 ms; 1M x 256 L = 300 11.1 / 12.0).  The LDS is handed out in 1,280-byte
// pieces, which the occupancy query leaves out.  Long rows keep more loads in
// flight on fewer wavefronts, so rescoring costs them more than the wavefronts
// do: d > 256 takes 4 KB (4 / 2 / 1 KB, ms for 10,000 queries: E4M3 2M x 512 L
// = 409 29.4 / 30.4 / 31.6, 1M x 384 L = 300 17.3 / 18.0 / 18.6; BF16 1M x 512
// L = 409 28.1 / 30.2 / 32.4), and FP32 rows of d > 128 8 KB while that leaves
// two wavefronts per SIMD (16 / 8 / 4 KB: 1M x 200 L = 100 10.3 / 10.3 / 10.8,
// L = 400 24.0 / 21.1 / 22.6, 1M x 150 L = 200 9.97 / 8.42 / 8.69, 1M x 384
// 20.6 / 20.9 / 21.7; 1M x 128 L = 400 19.2 / 13.9 / 12.8).
int choose_table(SearchArgs &a, int cus) {
    const int width = a.adj_off ? kMaxEll : a.ell;  // ids inserted per batch
    const int64_t want = (a.nq + cus - 1) / std::max(1, cus);
    int best = 10, occ = -1;
    // A table of ids is cleared at half load, so short queues lose more to a
    // smaller one than a fifth wavefront gives back: 4 KB for up to 128 entries
    // on graphs of 65 to 112 ids a row and CSR, 64 < d <= 256.  4 / 2 KB, ms for
    // 10,000 queries: E4M3 100k x 200, 100 ids, L = 50 4.2 / 4.5, 200 ids (CSR)
    // 7.2 / 7.8, BF16 100k x 96, 100 ids, L = 100 1.19 times as fast; but 128 ids
    // 0.96 times, and d = 64, 100 ids, L = 100 6.4 / 5.9.
    set_table(a, best);
    if (!a.sets && (a.adj_off || (a.ell > 64 && a.ell <= 112)) && a.d > 64 && a.d <= 256 && a.Leff <= 128 &&
        !(a.storage == RG_STORE_FP32 && a.d > 128))
        return RG_OK;
    for (int hb = a.storage == RG_STORE_FP32 && a.d > 128 ? 11 : 10; hb >= 8; --hb) {
        if ((1 << hb) < 2 * width + 2) break;
        int o = 0;
        set_table(a, hb);
        const int rc = table_search_occupancy(a, &o);
        if (rc) return rc;
        const int piece = 1280, lds = (int)search_lds_bytes(a.Leff, a.qpad, hb, a.cand);
        o = std::min(o, (160 << 10) / ((lds + piece - 1) / piece * piece));
        if (o >= 4) o &= ~3;
        o = (int)std::min<int64_t>(std::min(o, 20), want);
        if (o > occ) {
            occ = o;
            best = hb;
        }
        if ((hb == 11 || (hb == 10 && a.d > 256)) && o >= 8) {
            best = hb;
            break;
        }
    }
    set_table(a, best);
    return RG_OK;
}

// Search parameters common to every search entry point.
SearchArgs search_args(const rg_index *ix, const float *queries, int64_t nq, int32_t k, int32_t L, uint32_t *ids,
                       float *dists, uint32_t *hops, uint32_t *evals) {
    SearchArgs a{};
    a.base = ix->d_base;
    a.base_bf16 = ix->d_bf16;
    a.base_fp8 = ix->d_fp8;
    a.adj = ix->d_adj;
    a.adj_off = ix->d_adj_off;
    a.tomb = ix->d_tomb;
    a.queries = queries;
    a.out_ids = ids;
    a.out_d = dists;
    a.out_hops = hops;
    a.out_evals = evals;
    a.nq = nq;
    a.d = ix->d;
    a.pitch = ix->pitch;
    a.pitch8 = ix->pitch8;
    a.qpad = query_pad(ix->d, ix->pitch, ix->storage);
    a.ell = ix->ell;
    a.k = k;
    a.Leff = std::max(k, L);
    a.cand = cand_capacity(ix->ell, ix->d_adj_off != nullptr);
    a.hash_bits = 0;
    a.n_rows = ix->n;
    a.entry = ix->entry;
    a.storage = ix->storage;
    return a;
}

int upload_index(rg_index *ix, const float *base_dev, hipStream_t st) {
    int rc = upload_base(ix, base_dev, st);
    if (!rc) rc = upload_adj(ix, st);
    return rc;
}

int check_csr(int64_t n, const int64_t *off, const uint32_t *idx, uint32_t entry) {
    if (off[0] != 0) return RG_EINVAL;
    for (int64_t x = 0; x < n; ++x)
        if (off[x + 1] < off[x]) return RG_EINVAL;
    for (int64_t e = 0; e < off[n]; ++e)
        if (idx[e] >= (uint64_t)n) return RG_EINVAL;
    if (entry >= (uint64_t)n) return RG_EINVAL;
    return RG_OK;
}

int copy_to_host(const float *dev, int64_t count, std::vector<float> &h, hipStream_t st) {
    h.resize((size_t)count);
    RG_HIP(hipMemcpyAsync(h.data(), dev, sizeof(float) * (size_t)count, hipMemcpyDeviceToHost, st));
    RG_HIP(hipStreamSynchronize(st));
    return RG_OK;
}

uint64_t fnv1a(uint64_t h, const void *p, size_t n) {
    const unsigned char *b = static_cast<const unsigned char *>(p);
    for (size_t i = 0; i < n; ++i) {
        h ^= b[i];
        h *= 1099511628211ull;
    }
    return h;
}

}  // namespace

// ---------------------------------------------------------------------------
// exact kNN
// ---------------------------------------------------------------------------
namespace {

// Canonical FP64 kNN of one query row by a full scan of the base on the
// host: the last resort for a row whose candidates cannot be certified
// (ties wider than the largest candidate list).
void knn_scan_row(const float *q, const float *X, int64_t n, int32_t d, int32_t k, int threads, uint32_t *ids,
                  double *ds) {
    std::vector<std::pair<double, uint32_t>> all((size_t)n);
    par_rows(n, threads, [&](int64_t i) {
        double s = 0.0;
        for (int j = 0; j < d; ++j) s += (double)q[j] * (double)X[i * d + j];
        all[i] = {-s, (uint32_t)i};
    });
    std::partial_sort(all.begin(), all.begin() + k, all.end());
    for (int j = 0; j < k; ++j) {
        ids[j] = all[j].second;
        if (ds) ds[j] = all[j].first;
    }
}

}  // namespace

// Exact k nearest base rows of every query row, in canonical (delta, id)
// order, to device memory.  The GPU proposes K candidates per row (first from
// FP16 rows, at the FP16 matrix rate, when every value fits FP16's range; rows
// it cannot certify then from FP32 rows with K doubling up to 256); the
// candidates are rescored with the canonical FP64 distance and a row is kept
// when its certificate shows no other base row can be among its k nearest.
// Rows no list of 256 certifies are scanned in full on the host.
//
// The values the certificate needs (the largest row norm and element) come
// from the pass that makes the FP16 rows, results stay on the device, and the
// host sees the count of rows not certified; the base comes back to the host
// only for the scan.  Before, both matrices were copied to the host for the
// norms and the lists went through it: on 10k x 1M x 200 that was 215 of 270
// ms.
int knn_rows(const float *Qdev, int64_t nq, const float *Xdev, int64_t n, int32_t d, int32_t k, int32_t slack,
             const float *Xhost, int threads, uint32_t *ids, float *dists, int64_t (&done)[3], hipStream_t st) {
    const bool log = std::getenv("RG_LOG") != nullptr;
    const double u32 = std::ldexp(1.0, -24), u64 = std::ldexp(1.0, -53), u16 = std::ldexp(1.0, -11);
    const double g64 = (d + 1) * u64 / (1.0 - (d + 1) * u64);
    const int32_t dp = knn16_width(d);
    const int32_t K16 = (int32_t)std::min<int64_t>(std::min<int64_t>(256, n), std::max(2 * k, k + 48));
    const int32_t s16 = knn16_sample(n, K16);

    // lists of rows still open (this pass's and the next one's) and their count
    DevBuf lists, small;
    int rc = lists.alloc(2 * sizeof(uint32_t) * (size_t)nq);
    if (!rc) rc = small.alloc(2 * sizeof(PackStats) + 16);
    if (rc) return rc;
    uint32_t *open_rows = lists.as<uint32_t>(), *next_rows = open_rows + nq;
    PackStats *st_q = small.as<PackStats>(), *st_x = st_q + 1;
    uint32_t *n_fail = reinterpret_cast<uint32_t *>(st_x + 1);
    int64_t m = nq;  // rows open; all of them in order while m == nq
    bool all = true;

    // One pass: candidates of the open rows, certification, results of the
    // certified rows; the others stay open.
    double xmax = 0.0;
    auto certify = [&](const float *qd, const uint32_t *cid, const float *csc, bool f16, int32_t K, double gsum,
                       double eta, double abs0) -> int {
        int r = launch_knn_certify(qd, m, d, Xdev, n, d, d, cid, csc, K, k, gsum, xmax, eta, abs0,
                                   all ? nullptr : open_rows, ids, dists, next_rows, n_fail, st);
        if (r) return r;
        uint32_t nf = 0;
        RG_HIP(hipMemcpyAsync(&nf, n_fail, 4, hipMemcpyDeviceToHost, st));
        RG_HIP(hipStreamSynchronize(st));
        done[f16 ? 0 : 1] += m - (int64_t)nf;
        if (log)
            std::fprintf(stderr, "[rg] knn %s candidates: %lld rows, K=%d, %lld not certified\n", f16 ? "FP16" : "FP32",
                         (long long)m, K, (long long)nf);
        std::swap(open_rows, next_rows);
        m = nf;
        all = false;
        return RG_OK;
    };

    // FP16 pass.  Rounding each input to FP16 errs by at most u16 |v| + eta0
    // (eta0 = 2^-25, half the subnormal spacing), the products of the
    // rounded values are exact in FP32, and the FP32 accumulation of dp of
    // them errs by at most gacc (2 units per add allows truncating adders).
    // So a candidate score errs by at most
    //   (2 u16 + u16^2 + gacc (1 + u16)^2) sum|t_i x_i|
    //   + (1 + gacc) (1 + u16) eta0 (|t|_1 + |x|_1) + (1 + gacc) d eta0^2,
    // with sum|t_i x_i| <= |t| xmax and |v|_1 <= sqrt(d) |v|.
    {
        const size_t hq = 2 * (size_t)knn16_rows(nq) * dp, hx = 2 * (size_t)knn16_rows(n) * dp;
        const size_t hs = s16 > 0 ? 2 * (size_t)knn16_rows((n + s16 - 1) / s16) * dp : 0;
        DevBuf half, cand;
        // with no room for the sample the running top-K does without; with
        // none for the copies only values out of FP16's range, which need
        // none, can go on
        int32_t s = s16;
        if (half.alloc(hq + hx + hs) && (s == 0 || (s = 0, half.alloc(hq + hx)))) s = -1;
        char *q16 = s < 0 ? nullptr : half.as<char>(), *x16 = s < 0 ? nullptr : q16 + hq, *smp = s > 0 ? x16 + hx : nullptr;
        rc = launch_pack16(Qdev, nq, d, d, q16, knn16_rows(nq), dp, nullptr, 0, st_q, st);
        if (!rc) rc = launch_pack16(Xdev, n, d, d, x16, knn16_rows(n), dp, smp, std::max(s, 0), st_x, st);
        if (rc) return rc;
        PackStats h[2];
        RG_HIP(hipMemcpyAsync(h, st_q, sizeof(h), hipMemcpyDeviceToHost, st));
        RG_HIP(hipStreamSynchronize(st));
        double norm2;
        float aq, ax;
        std::memcpy(&norm2, &h[1].norm2, 8);
        std::memcpy(&aq, &h[0].amax, 4);
        std::memcpy(&ax, &h[1].amax, 4);
        // the sums of squares, in another order, may be off by d ulps
        xmax = h[1].nan0 ? NAN : std::sqrt(norm2) * (1.0 + 1e-12 + d * u64);
        if (std::max(aq, ax) < 32768.f) {
            if (s < 0) {
                set_error("knn: out of device memory for the FP16 rows");
                return RG_ENOMEM;
            }
            const double eta0 = std::ldexp(1.0, -25);
            const double gacc = 2.0 * dp * u32 / (1.0 - 2.0 * dp * u32);
            const double gsum = 2 * u16 + u16 * u16 + gacc * (1 + u16) * (1 + u16) + g64;
            const double eta = (1 + gacc) * (1 + u16) * eta0 * std::sqrt((double)d);
            const double abs0 = (1 + gacc) * d * eta0 * eta0;
            rc = cand.alloc(8 * (size_t)nq * K16);
            if (rc) return rc;
            uint32_t *cid = cand.as<uint32_t>();
            float *csc = reinterpret_cast<float *>(cid + (size_t)nq * K16);
            rc = launch_knn16_candidates(q16, nq, x16, n, d, dp, smp, s, K16, cid, csc, st);
            if (!rc) rc = certify(Qdev, cid, csc, true, K16, gsum, eta, abs0);
            if (rc) return rc;
        }
    }
    // FP32 passes for what is left, K doubling
    const double g32 = (d + 1) * u32 / (1.0 - (d + 1) * u32);
    int32_t K = (int32_t)std::min<int64_t>(n, (int64_t)k + slack);
    if (K > 256) K = std::max(k, 256);
    while (m > 0) {
        DevBuf qbuf, cand;
        const float *qd = Qdev;
        if (!all) {
            rc = qbuf.alloc(sizeof(float) * (size_t)m * d);
            if (!rc) rc = launch_gather_rows(Qdev, open_rows, m, d, qbuf.as<float>(), st);
            if (rc) return rc;
            qd = qbuf.as<float>();
        }
        rc = cand.alloc(8 * (size_t)m * K);
        if (rc) return rc;
        uint32_t *cid = cand.as<uint32_t>();
        float *csc = reinterpret_cast<float *>(cid + (size_t)m * K);
        rc = launch_knn_candidates(qd, m, d, Xdev, n, d, d, K, cid, csc, st);
        if (!rc) rc = certify(qd, cid, csc, false, K, g32 + g64, 0.0, 0.0);
        if (rc) return rc;
        if (m == 0 || K >= 256 || K >= n) break;
        K = (int32_t)std::min<int64_t>(std::min<int64_t>(256, n), 2 * (int64_t)K);
    }
    if (m == 0) return RG_OK;
    // the rest by a full canonical scan on the host
    if (log) std::fprintf(stderr, "[rg] knn: %lld rows scanned on the host\n", (long long)m);
    std::vector<float> xh, q((size_t)d), hd((size_t)k);
    if (!Xhost) {
        rc = copy_to_host(Xdev, n * d, xh, st);
        if (rc) return rc;
        Xhost = xh.data();
    }
    std::vector<uint32_t> rows((size_t)m), hid((size_t)k);
    std::vector<double> dd((size_t)k);
    if (!all) {
        RG_HIP(hipMemcpyAsync(rows.data(), open_rows, sizeof(uint32_t) * (size_t)m, hipMemcpyDeviceToHost, st));
        RG_HIP(hipStreamSynchronize(st));
    } else {
        for (int64_t i = 0; i < m; ++i) rows[i] = (uint32_t)i;
    }
    for (uint32_t r : rows) {
        rc = copy_to_host(Qdev + (int64_t)r * d, d, q, st);
        if (rc) return rc;
        knn_scan_row(q.data(), Xhost, n, d, k, threads, hid.data(), dd.data());
        for (int j = 0; j < k; ++j) hd[j] = (float)dd[j];
        RG_HIP(hipMemcpyAsync(ids + (int64_t)r * k, hid.data(), sizeof(uint32_t) * k, hipMemcpyHostToDevice, st));
        if (dists)
            RG_HIP(hipMemcpyAsync(dists + (int64_t)r * k, hd.data(), sizeof(float) * k, hipMemcpyHostToDevice, st));
        RG_HIP(hipStreamSynchronize(st));
    }
    done[2] += m;
    return RG_OK;
}

// The same for all rows, with half of them at a time where their lists do not
// fit.
int knn_exact(const float *Qdev, int64_t nq, const float *Xdev, int64_t n, int32_t d, int32_t k, int32_t slack,
              const float *Xhost, int threads, uint32_t *ids, float *dists, hipStream_t st) {
    threads = hw_threads(threads);
    if (slack <= 0) slack = std::max(16, k / 4);
    g_knn_rows[0] = g_knn_rows[1] = g_knn_rows[2] = 0;
    int64_t part = nq;
    for (int64_t q0 = 0; q0 < nq;) {
        const int64_t cnt = std::min(part, nq - q0);
        int64_t done[3] = {0, 0, 0};
        const int rc = knn_rows(Qdev + q0 * d, cnt, Xdev, n, d, k, slack, Xhost, threads, ids + q0 * k,
                                dists ? dists + q0 * k : nullptr, done, st);
        if (rc == RG_ENOMEM && cnt >= 4096) {
            part = (cnt + 1) / 2;
            continue;
        }
        if (rc) return rc;
        for (int i = 0; i < 3; ++i) g_knn_rows[i] += done[i];
        q0 += cnt;
    }
    return RG_OK;
}

}  // namespace rg

using namespace rg;

extern "C" {

const char *rg_last_error(void) { return g_err.c_str(); }

int rg_knn_candidates(const float *queries, int64_t nq, const float *base, int64_t n, int32_t d, int32_t K,
                      uint32_t *ids, float *scores, void *stream) {
    if (!queries || !base || !ids || !scores || nq < 0 || n < 1 || d < 1 || K < 1 || K > n) {
        set_error("rg_knn_candidates: invalid argument");
        return RG_EINVAL;
    }
    return launch_knn_candidates(queries, nq, d, base, n, d, d, K, ids, scores, (hipStream_t)stream);
}

int rg_knn_candidates_f16(const float *queries, int64_t nq, const float *base, int64_t n, int32_t d, int32_t K,
                          uint32_t *ids, float *scores, void *stream) {
    if (!queries || !base || !ids || !scores || nq < 0 || n < 1 || n >= (1ll << 31) || d < 1 || K < 1 || K > n ||
        K > 256) {
        set_error("rg_knn_candidates_f16: invalid argument");
        return RG_EINVAL;
    }
    if (nq == 0) return RG_OK;
    hipStream_t st = (hipStream_t)stream;
    const int32_t dp = knn16_width(d);
    int32_t s = knn16_sample(n, K);
    DevBuf q16, x16, smp, stats;
    int rc = q16.alloc(2 * (size_t)knn16_rows(nq) * dp);
    if (!rc) rc = x16.alloc(2 * (size_t)knn16_rows(n) * dp);
    if (!rc && s > 0 && smp.alloc(2 * (size_t)knn16_rows((n + s - 1) / s) * dp)) s = 0;  // the running top-K
    if (!rc) rc = stats.alloc(2 * sizeof(PackStats));
    if (!rc)
        rc = launch_pack16(queries, nq, d, d, q16.p, knn16_rows(nq), dp, nullptr, 0, stats.as<PackStats>(), st);
    if (!rc) rc = launch_pack16(base, n, d, d, x16.p, knn16_rows(n), dp, smp.p, s, stats.as<PackStats>() + 1, st);
    if (rc) return rc;
    PackStats h[2];
    RG_HIP(hipMemcpyAsync(h, stats.p, sizeof(h), hipMemcpyDeviceToHost, st));
    RG_HIP(hipStreamSynchronize(st));
    for (int i = 0; i < 2; ++i)
        if (h[i].bad) {
            set_error(std::string("rg_knn_candidates_f16: a ") + (i == 0 ? "query" : "base") +
                      " value is out of the FP16 range used (|v| < 2^15)");
            return RG_EINVAL;
        }
    return launch_knn16_candidates(q16.p, nq, x16.p, n, d, dp, smp.p, s, K, ids, scores, st);
}

int rg_knn_last_stats(int64_t *rows_f16, int64_t *rows_f32, int64_t *rows_host) {
    if (rows_f16) *rows_f16 = g_knn_rows[0];
    if (rows_f32) *rows_f32 = g_knn_rows[1];
    if (rows_host) *rows_host = g_knn_rows[2];
    return RG_OK;
}

int rg_knn(const float *queries, int64_t nq, const float *base, int64_t n, int32_t d, int32_t k, uint32_t *ids,
           float *dists, void *stream) {
    if (!queries || !base || !ids || !dists || nq < 0 || n < 1 || d < 1 || k < 1 || k > n || k > 224 ||
        n >= (1ll << 31)) {
        set_error("rg_knn: invalid argument (need 1 <= k <= min(n, 224), n < 2^31)");
        return RG_EINVAL;
    }
    if (nq == 0) return RG_OK;
    hipStream_t st = (hipStream_t)stream;
    return knn_exact(queries, nq, base, n, d, k, 0, nullptr, 0, ids, dists, st);
}

int rg_build(const float *base, int64_t n, int32_t d, const float *train, int64_t nt, int32_t Nq, int32_t M,
             int32_t metric, const rg_build_opts *opts, void *stream, rg_index **out) {
    if (!base || !train || !out || n < 1 || n >= (1ll << 31) || d < 1 || nt < 1 || Nq < 2 || Nq > n || M < 3 ||
        M > kMaxEll || metric != RG_METRIC_IP || Nq > 224) {
        set_error("rg_build: invalid argument");
        return RG_EINVAL;
    }
    *out = nullptr;
    rg_build_opts o{};
    if (opts) o = *opts;
    const int32_t L = o.L_build > 0 ? o.L_build : 500;
    const int32_t m_pj = o.m_pj > 0 ? o.m_pj : M / 2;
    const int32_t m_ce = o.m_ce > 0 ? o.m_ce : (M - 1) / 2;
    if (m_pj + m_ce > M - 1) {
        set_error("rg_build: m_pj + m_ce must be <= M - 1");
        return RG_EINVAL;
    }
    hipStream_t st = (hipStream_t)stream;
    const int threads = hw_threads(o.threads);
    const auto t0 = std::chrono::steady_clock::now();
    std::vector<float> xh, th;
    int rc = copy_to_host(base, n * d, xh, st);
    if (!rc && o.keep_stages) rc = copy_to_host(train, nt * d, th, st);
    if (rc) return rc;
    if (std::getenv("RG_LOG")) std::fprintf(stderr, "[rg] build: n=%lld d=%d nt=%lld Nq=%d M=%d L=%d\n", (long long)n, d, (long long)nt, Nq, M, L);
    // the lists stay on the device for the projection
    DevBuf lists;
    rc = lists.alloc(sizeof(uint32_t) * (size_t)nt * Nq);
    if (!rc)
        rc = knn_exact(train, nt, base, n, d, Nq, o.knn_slack, xh.data(), threads, lists.as<uint32_t>(), nullptr, st);
    if (rc) return rc;
    std::vector<uint32_t> knn;
    if (o.keep_stages || n <= 256) {
        knn.resize((size_t)nt * Nq);
        RG_HIP(hipMemcpyAsync(knn.data(), lists.p, sizeof(uint32_t) * knn.size(), hipMemcpyDeviceToHost, st));
    }
    RG_HIP(hipStreamSynchronize(st));
    // a list of the whole base is certified as it is, and lacks the rows whose
    // scores are NaN
    if (n <= 256 && std::find(knn.begin(), knn.end(), kNone) != knn.end()) {
        set_error("rg_build: a training query has fewer than Nq base rows at a distance that is a number");
        return RG_EINVAL;
    }
    if (!o.keep_stages) std::vector<uint32_t>().swap(knn);
    if (std::getenv("RG_LOG"))
        std::fprintf(stderr, "[rg] kNN preprocessing done in %.2f s\n",
                     std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count());
    const auto t1 = std::chrono::steady_clock::now();
    rg_index *ix = new rg_index();
    ix->n = n;
    ix->d = d;
    ix->metric = metric;
    ix->Nq = Nq;
    ix->M = M;
    ix->L_build = L;
    ix->m_pj = m_pj;
    ix->m_ce = m_ce;
    (void)hipGetDevice(&ix->device);
    rc = upload_base(ix, base, st);
    if (rc == RG_ENOMEM && lists.p) {
        // no room for the rows beside the lists: these go to the host, and the
        // projection with them
        knn.resize((size_t)nt * Nq);
        rc = hipMemcpyAsync(knn.data(), lists.p, sizeof(uint32_t) * knn.size(), hipMemcpyDeviceToHost, st) == hipSuccess &&
                     hipStreamSynchronize(st) == hipSuccess
                 ? RG_OK
                 : RG_EDEVICE;
        lists.release();
        if (!rc) rc = upload_base(ix, base, st);
    }
    HostGraph g;
    if (!rc) {
        GpuCtx gpu{ix->d_base,  ix->pitch,     st,            lists.as<uint32_t>(),     canon_pivots,
                   canon_lists, canon_project, canon_enhance, [&] { lists.release(); }};
        rc = host_construct(xh.data(), n, d, knn.empty() ? nullptr : knn.data(), nt, Nq, M, L, m_pj, m_ce, threads, &gpu, o.keep_stages != 0,
                            &g);
    }
    if (!rc) {
        ix->entry = g.entry;
        ix->repairs = g.repairs;
        ix->offsets.swap(g.offsets);
        ix->indices.swap(g.indices);
        ix->stages = std::move(g.stages);
        if (ix->stages.kept) {
            ix->stages.base.swap(xh);
            ix->stages.train.swap(th);
        }
        rc = upload_adj(ix, st);
    }
    if (rc) {
        free_index_device(ix);
        delete ix;
        return rc;
    }
    const auto t2 = std::chrono::steady_clock::now();
    ix->t_knn = std::chrono::duration<double>(t1 - t0).count();
    ix->t_project = g.t_project;
    ix->t_enhance = g.t_enhance;
    ix->t_total = std::chrono::duration<double>(t2 - t0).count();
    *out = ix;
    return RG_OK;
}

int rg_build_from_knn(const float *base_host, int64_t n, int32_t d, const uint32_t *knn_host,
                      const float *train_host, int64_t nt, int32_t Nq, int32_t M, const rg_build_opts *opts,
                      rg_index **out) {
    if (!base_host || !knn_host || !out || n < 1 || n >= (1ll << 31) || d < 1 || nt < 1 || Nq < 2 || Nq > n ||
        M < 3 || M > kMaxEll) {
        set_error("rg_build_from_knn: invalid argument");
        return RG_EINVAL;
    }
    *out = nullptr;
    for (int64_t i = 0; i < nt * (int64_t)Nq; ++i)
        if (knn_host[i] >= (uint64_t)n) {
            set_error("rg_build_from_knn: kNN id out of range");
            return RG_EINVAL;
        }
    rg_build_opts o{};
    if (opts) o = *opts;
    const int32_t L = o.L_build > 0 ? o.L_build : 500;
    const int32_t m_pj = o.m_pj > 0 ? o.m_pj : M / 2;
    const int32_t m_ce = o.m_ce > 0 ? o.m_ce : (M - 1) / 2;
    if (m_pj + m_ce > M - 1) {
        set_error("rg_build_from_knn: m_pj + m_ce must be <= M - 1");
        return RG_EINVAL;
    }
    HostGraph g;
    const int rc = host_construct(base_host, n, d, knn_host, nt, Nq, M, L, m_pj, m_ce, hw_threads(o.threads),
                                  nullptr, o.keep_stages != 0, &g);
    if (rc) return rc;
    rg_index *ix = new rg_index();
    ix->n = n;
    ix->d = d;
    ix->entry = g.entry;
    ix->Nq = Nq;
    ix->M = M;
    ix->L_build = L;
    ix->m_pj = m_pj;
    ix->m_ce = m_ce;
    ix->repairs = g.repairs;
    ix->offsets.swap(g.offsets);
    ix->indices.swap(g.indices);
    ix->stages = std::move(g.stages);
    if (ix->stages.kept) {
        ix->stages.base.assign(base_host, base_host + n * d);
        if (train_host) ix->stages.train.assign(train_host, train_host + nt * d);
    }
    ix->t_project = g.t_project;
    ix->t_enhance = g.t_enhance;
    ix->t_total = g.t_total;
    *out = ix;
    return RG_OK;
}

int rg_index_from_csr(const float *base, int64_t n, int32_t d, const int64_t *offsets, const uint32_t *indices,
                      uint32_t entry, int32_t metric, void *stream, rg_index **out) {
    if (!base || !offsets || !out || n < 1 || n >= (1ll << 31) || d < 1 || metric != RG_METRIC_IP ||
        (offsets[n] > 0 && !indices)) {
        set_error("rg_index_from_csr: invalid argument");
        return RG_EINVAL;
    }
    *out = nullptr;
    if (check_csr(n, offsets, indices, entry)) {
        set_error("rg_index_from_csr: malformed CSR or entry");
        return RG_EINVAL;
    }
    rg_index *ix = new rg_index();
    ix->n = n;
    ix->d = d;
    ix->metric = metric;
    ix->entry = entry;
    ix->offsets.assign(offsets, offsets + n + 1);
    ix->indices.assign(indices, indices + offsets[n]);
    (void)hipGetDevice(&ix->device);
    const int rc = upload_index(ix, base, (hipStream_t)stream);
    if (rc) {
        free_index_device(ix);
        delete ix;
        return rc;
    }
    *out = ix;
    return RG_OK;
}

int rg_index_graph(const rg_index *ix, const int64_t **offsets, const uint32_t **indices, int64_t *nnz,
                   uint32_t *entry) {
    if (!ix) {
        set_error("rg_index_graph: null index");
        return RG_EINVAL;
    }
    if (offsets) *offsets = ix->offsets.data();
    if (indices) *indices = ix->indices.data();
    if (nnz) *nnz = ix->offsets[ix->n];
    if (entry) *entry = ix->entry;
    return RG_OK;
}

int rg_index_stage_graph(const rg_index *ix, int32_t stage, const int64_t **offsets, const uint32_t **indices,
                         int64_t *nnz, uint32_t *entry) {
    if (!ix || (stage != RG_STAGE_PROJECTED && stage != RG_STAGE_BIPARTITE)) {
        set_error("rg_index_stage_graph: invalid argument");
        return RG_EINVAL;
    }
    const StageGraphs &sg = ix->stages;
    if (!sg.kept) {
        set_error("rg_index_stage_graph: the build did not keep its stage graphs (keep_stages)");
        return RG_EINVAL;
    }
    const bool pj = stage == RG_STAGE_PROJECTED;
    const std::vector<int64_t> &off = pj ? sg.pj_off : sg.bi_off;
    const std::vector<uint32_t> &idx = pj ? sg.pj_idx : sg.bi_idx;
    if (offsets) *offsets = off.data();
    if (indices) *indices = idx.data();
    if (nnz) *nnz = off[ix->n];
    if (entry) *entry = pj ? ix->entry : sg.entry_bi;
    return RG_OK;
}

int rg_index_bipartite(const rg_index *ix, const int64_t **bridge_offsets, const uint32_t **bridges,
                       int64_t *n_built, const int64_t **nout_offsets, const uint32_t **nout, int64_t *nt) {
    if (!ix || !ix->stages.kept) {
        set_error("rg_index_bipartite: the build did not keep its stage graphs (keep_stages)");
        return RG_EINVAL;
    }
    const StageGraphs &sg = ix->stages;
    if (sg.nout_view_off.empty()) {  // N_out(t) as built, then the ids inserted into it
        sg.nout_view_off.assign((size_t)sg.nt + 1, 0);
        for (int64_t t = 0; t < sg.nt; ++t)
            sg.nout_view_off[t + 1] =
                sg.nout_view_off[t] + sg.q1 + (sg.nout_add.empty() ? 0 : (int64_t)sg.nout_add[t].size());
        sg.nout_view_idx.resize((size_t)sg.nout_view_off[sg.nt]);
        for (int64_t t = 0; t < sg.nt; ++t) {
            auto o = std::copy(sg.nout.begin() + t * sg.q1, sg.nout.begin() + (t + 1) * sg.q1,
                               sg.nout_view_idx.begin() + sg.nout_view_off[t]);
            if (!sg.nout_add.empty()) std::copy(sg.nout_add[t].begin(), sg.nout_add[t].end(), o);
        }
    }
    if (bridge_offsets) *bridge_offsets = sg.b_off.data();
    if (bridges) *bridges = sg.b_idx.data();
    if (n_built) *n_built = sg.n_built;
    if (nout_offsets) *nout_offsets = sg.nout_view_off.data();
    if (nout) *nout = sg.nout_view_idx.data();
    if (nt) *nt = sg.nt;
    return RG_OK;
}

// Grow the device base by nv rows taken from host memory; the reduced-
// precision copies are dropped (they are made again for the new size).
int grow_device_base(rg_index *ix, const float *rows_host, int64_t nv, hipStream_t st) {
    DevBuf tmp;
    int rc = tmp.alloc(sizeof(float) * (size_t)nv * ix->d);
    if (rc) return rc;
    RG_HIP(hipMemcpyAsync(tmp.p, rows_host, sizeof(float) * (size_t)nv * ix->d, hipMemcpyHostToDevice, st));
    float *nb = nullptr;
    if (hipMalloc(&nb, sizeof(float) * (size_t)(ix->n + nv) * ix->pitch) != hipSuccess) {
        return no_memory("insert: out of device memory for the base rows");
    }
    if (hipMemcpyAsync(nb, ix->d_base, sizeof(float) * (size_t)ix->n * ix->pitch, hipMemcpyDeviceToDevice, st) !=
            hipSuccess ||
        launch_pad_rows(tmp.as<float>(), nv, ix->d, nb + (size_t)ix->n * ix->pitch, ix->pitch, st) != RG_OK ||
        hipStreamSynchronize(st) != hipSuccess) {
        (void)hipFree(nb);
        set_error("insert: device copy of the base rows failed");
        return RG_EDEVICE;
    }
    (void)hipFree(ix->d_base);
    ix->d_base = nb;
    for (void **p : {(void **)&ix->d_bf16, (void **)&ix->d_fp8, (void **)&ix->d_scale})
        if (*p) {
            (void)hipFree(*p);
            *p = nullptr;
        }
    return RG_OK;
}

int upload_tomb(rg_index *ix, hipStream_t st) {
    if (ix->d_tomb) (void)hipFree(ix->d_tomb);
    ix->d_tomb = nullptr;
    if (ix->n_deleted == 0 || !ix->d_base) return RG_OK;
    if (hipMalloc(&ix->d_tomb, sizeof(uint32_t) * ix->tomb.size()) != hipSuccess) {
        ix->d_tomb = nullptr;
        return no_memory("delete: out of device memory for the tombstones");
    }
    RG_HIP(hipMemcpyAsync(ix->d_tomb, ix->tomb.data(), sizeof(uint32_t) * ix->tomb.size(), hipMemcpyHostToDevice, st));
    RG_HIP(hipStreamSynchronize(st));
    return RG_OK;
}

int rg_insert(rg_index *ix, const float *vectors, int64_t nv, int32_t L, void *stream) {
    if (!ix || nv < 0 || (nv > 0 && !vectors) || L < 0 || L > kMaxL) {
        set_error("rg_insert: invalid argument");
        return RG_EINVAL;
    }
    StageGraphs &sg = ix->stages;
    if (!sg.kept || sg.train.empty()) {
        set_error("rg_insert: needs an index built with keep_stages (and, from kNN lists, the training queries)");
        return RG_EINVAL;
    }
    if (ix->n + nv >= (1ll << 31)) {
        set_error("rg_insert: too many rows");
        return RG_EINVAL;
    }
    if (nv == 0) return RG_OK;
    if (ix->d_base && ix->d_adj_off) {
        set_error("rg_insert: the index graph is held as CSR (out-degree > 128)");
        return RG_EINVAL;
    }
    for (int64_t i = 0; i < nv * (int64_t)ix->d; ++i)
        if (!std::isfinite(vectors[i])) {
            set_error("rg_insert: a vector holds a value that is not finite");
            return RG_EINVAL;
        }
    if (L == 0) L = ix->L_build;
    const auto t0 = std::chrono::steady_clock::now();
    hipStream_t st = (hipStream_t)stream;
    // the reduced-precision copies are remade for the new size at the end;
    // until then the index searches its FP32 rows
    const int32_t storage = ix->storage;
    ix->storage = RG_STORE_FP32;
    const int64_t n0 = ix->n;
    const int32_t d = ix->d;
    sg.base.insert(sg.base.end(), vectors, vectors + nv * d);
    // on a failure past this point: the index keeps its n0 rows and graph
    // (a grown device base holds them first), and its storage form, whose
    // reduced copies are remade if they were released
    auto undo = [&](int code) {
        sg.base.resize((size_t)n0 * d);
        if (storage != RG_STORE_FP32 && ix->d_base) {
            const std::string err = g_err;
            (void)rg_index_set_storage(ix, storage, stream);
            g_err = err;
        }
        return code;
    };
    std::vector<uint32_t> qid((size_t)nv * L);
    std::vector<int32_t> qn((size_t)nv);
    int rc = RG_OK;
    if (ix->d_base) {
        // canonical searches of the new rows on the device, graph as it stands
        rc = grow_device_base(ix, vectors, nv, st);
        if (rc) return undo(rc);
        const int64_t B = std::min<int64_t>(nv, 1 << 15);
        DevBuf di, dd, dn, dm;
        rc = dm.alloc(8);
        if (!rc) rc = launch_max_norm(ix->d_base, n0, ix->pitch, dm.as<double>(), st);
        if (!rc) rc = di.alloc(sizeof(uint32_t) * B * L);
        if (!rc) rc = dd.alloc(sizeof(double) * B * L);
        if (!rc) rc = dn.alloc(sizeof(int32_t) * B);
        for (int64_t x0 = 0; x0 < nv && !rc; x0 += B) {
            const int64_t cnt = std::min(B, nv - x0);
            rc = launch_canon_search(ix->d_base, n0, d, ix->pitch, ix->d_adj, ix->ell, ix->entry, L, n0 + x0, cnt,
                                     dm.as<double>(), di.as<uint32_t>(), dd.as<double>(), dn.as<int32_t>(), st);
            if (!rc && (hipMemcpyAsync(qid.data() + x0 * L, di.p, sizeof(uint32_t) * cnt * L, hipMemcpyDeviceToHost,
                                       st) != hipSuccess ||
                        hipMemcpyAsync(qn.data() + x0, dn.p, sizeof(int32_t) * cnt, hipMemcpyDeviceToHost, st) !=
                            hipSuccess ||
                        hipStreamSynchronize(st) != hipSuccess)) {
                set_error("rg_insert: device search failed");
                rc = RG_EDEVICE;
            }
        }
    } else {
        host_canon_searches(sg.base.data(), d, ix->offsets.data(), ix->indices.data(), ix->entry, L, n0, nv, 0,
                            qid.data(), qn.data());
    }
    const auto t_search = std::chrono::steady_clock::now();
    if (!rc)
        rc = host_insert(sg, d, ix->M, ix->m_pj, L, ix->entry, n0, nv, qid.data(), qn.data(), ix->offsets,
                         ix->indices, 0);
    const auto t_merge = std::chrono::steady_clock::now();
    if (rc) return undo(rc);
    ix->n = n0 + nv;
    if (!ix->tomb.empty()) ix->tomb.resize((size_t)((ix->n + 31) / 32), 0u);
    if (ix->d_base) {
        if (ix->d_adj) (void)hipFree(ix->d_adj);
        ix->d_adj = nullptr;
        rc = upload_adj(ix, st);
        if (!rc) rc = upload_tomb(ix, st);
        if (!rc && storage != RG_STORE_FP32) rc = rg_index_set_storage(ix, storage, stream);
    } else {
        ix->storage = storage;
    }
    if (std::getenv("RG_LOG")) {
        auto sec = [](auto a, auto b) { return std::chrono::duration<double>(b - a).count(); };
        std::fprintf(stderr, "[rg] insert %lld rows: searches %.2f s, merge %.2f s, device update %.2f s\n",
                     (long long)nv, sec(t0, t_search), sec(t_search, t_merge),
                     sec(t_merge, std::chrono::steady_clock::now()));
    }
    return rc;
}

int rg_delete(rg_index *ix, const uint32_t *ids, int64_t count, void *stream) {
    if (!ix || count < 0 || (count > 0 && !ids)) {
        set_error("rg_delete: invalid argument");
        return RG_EINVAL;
    }
    for (int64_t i = 0; i < count; ++i)
        if (ids[i] >= (uint64_t)ix->n) {
            set_error("rg_delete: id out of range");
            return RG_EINVAL;
        }
    if (ix->tomb.empty()) ix->tomb.assign((size_t)((ix->n + 31) / 32), 0u);
    for (int64_t i = 0; i < count; ++i) {
        uint32_t &w = ix->tomb[ids[i] >> 5];
        const uint32_t bit = 1u << (ids[i] & 31u);
        if (!(w & bit)) {
            w |= bit;
            ++ix->n_deleted;
        }
    }
    return upload_tomb(ix, (hipStream_t)stream);
}

int rg_index_tombstones(const rg_index *ix, const uint32_t **bits, int64_t *count) {
    if (!ix) {
        set_error("rg_index_tombstones: null index");
        return RG_EINVAL;
    }
    if (bits) *bits = ix->tomb.empty() ? nullptr : ix->tomb.data();
    if (count) *count = ix->n_deleted;
    return RG_OK;
}

int rg_index_info(const rg_index *ix, int64_t *n, int32_t *d, int32_t *pitch, int32_t *ell, int64_t *bytes) {
    if (!ix) {
        set_error("rg_index_info: null index");
        return RG_EINVAL;
    }
    if (n) *n = ix->n;
    if (d) *d = ix->d;
    if (pitch) *pitch = ix->pitch;
    if (ell) *ell = ix->ell;
    if (bytes) {
        int64_t b = (int64_t)ix->n * ix->pitch * 4;
        b += ix->d_adj_off ? ix->offsets[ix->n] * 4 + (ix->n + 1) * 8 : (int64_t)ix->n * ix->ell * 4;
        if (ix->d_bf16) b += (int64_t)ix->n * ix->pitch * 2;
        if (ix->d_fp8) b += (int64_t)ix->n * ix->pitch8 + ix->n * 4;
        *bytes = b;
    }
    return RG_OK;
}

// build statistics: seconds for kNN, projection, enhancement, total; repairs
int rg_index_build_stats(const rg_index *ix, double *t_knn, double *t_project, double *t_enhance, double *t_total,
                         int64_t *repairs) {
    if (!ix) return RG_EINVAL;
    if (t_knn) *t_knn = ix->t_knn;
    if (t_project) *t_project = ix->t_project;
    if (t_enhance) *t_enhance = ix->t_enhance;
    if (t_total) *t_total = ix->t_total;
    if (repairs) *repairs = ix->repairs;
    return RG_OK;
}

int rg_index_set_storage(rg_index *ix, int32_t storage, void *stream) {
    if (!ix || !ix->d_base || storage < RG_STORE_FP32 || storage > RG_STORE_FP8E4M3) {
        set_error("rg_index_set_storage: invalid argument");
        return RG_EINVAL;
    }
    hipStream_t st = (hipStream_t)stream;
    if (storage == RG_STORE_BF16 && !ix->d_bf16) {
        if (hipMalloc(&ix->d_bf16, sizeof(uint16_t) * (size_t)ix->n * ix->pitch) != hipSuccess) {
            ix->d_bf16 = nullptr;
            return no_memory("set_storage: out of device memory");
        }
        const int rc = launch_quant_bf16(ix->d_base, ix->n, ix->pitch, ix->d_bf16, st);
        if (rc) return rc;
    }
    if (storage == RG_STORE_FP8E4M3 && !ix->d_fp8) {
        ix->pitch8 = fp8_pitch(ix->d);
        if (hipMalloc(&ix->d_fp8, (size_t)ix->n * ix->pitch8) != hipSuccess ||
            hipMalloc(&ix->d_scale, sizeof(float) * (size_t)ix->n) != hipSuccess) {
            if (ix->d_fp8) (void)hipFree(ix->d_fp8);
            ix->d_fp8 = nullptr;
            ix->d_scale = nullptr;
            return no_memory("set_storage: out of device memory");
        }
        const int rc = launch_quant_fp8(ix->d_base, ix->n, ix->d, ix->pitch, ix->d_fp8, ix->pitch8, ix->d_scale, st);
        if (rc) return rc;
    }
    RG_HIP(hipStreamSynchronize(st));
    ix->storage = storage;
    return RG_OK;
}

// Device copies of the reduced-precision rows (for tests): codes/scales or bf16 bits.
int rg_index_storage_ptrs(const rg_index *ix, const void **bf16, const void **fp8, const float **scales,
                          int32_t *pitch8) {
    if (!ix) return RG_EINVAL;
    if (bf16) *bf16 = ix->d_bf16;
    if (fp8) *fp8 = ix->d_fp8;
    if (scales) *scales = ix->d_scale;
    if (pitch8) *pitch8 = ix->pitch8;
    return RG_OK;
}

int rg_search(const rg_index *ix, const float *queries, int64_t nq, int32_t k, int32_t L, uint32_t *ids,
              float *dists, uint32_t *hops, uint32_t *evals, void *stream) {
    if (!ix || nq < 0 || (nq > 0 && (!queries || !ids || !dists)) || k < 1 || L < 1 || k > kMaxSearchL ||
        L > kMaxSearchL || nq >= (1ll << 31)) {
        set_error("rg_search: invalid argument (need 1 <= k, L <= 1024)");
        return RG_EINVAL;
    }
    if (!ix->d_base) {
        set_error("rg_search: index has no device data (built by rg_build_from_knn)");
        return RG_EINVAL;
    }
    if (nq == 0) return RG_OK;
    hipStream_t st = (hipStream_t)stream;
    SearchArgs a = search_args(ix, queries, nq, k, L, ids, dists, hops, evals);
    int cus = 0;
    RG_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ix->device));
    // FP32 rows have an exact visited set where a bitmap (about n/8 bytes per
    // query) stays below 5% of a query's expected row bytes (about 40 L_eff
    // rows of 4d bytes, as measured on built indexes: the graph's mean degree
    // says little, the expanded nodes being its dense part) and either LDS
    // holds it, the caller asks for the number of rows scored, or a table could
    // not have sets, and always for CSR graphs, whose wide rows would overflow
    // a table at every expansion.  A bitmap in device memory costs more than the rows that a
    // table scores again: its lines miss the caches, and each of its atomics
    // reads and writes one.  Bitmap / table, 10,000 queries: 1M x 200 L = 100
    // 14.0 / 10.3 ms (7,503 / 7,671 rows per query), L = 400 28.1 / 21.1, L =
    // 800 51.2 / 44.0, 1M x 96 L = 200 9.0 / 5.0, 1M x 384 L = 200 29.1 / 20.9.
    const bool exact = ix->storage == RG_STORE_FP32 &&
                       (ix->d_adj_off || (double)ix->n / 8.0 <= 0.05 * 40.0 * std::max(L, k) * 4.0 * ix->d);
    a.bm_words = ((ix->n + 31) / 32 + 63) / 64 * 64;
    int rc = RG_OK;
    // Few queries: 8 wavefronts per query while that is one workgroup per CU
    // (two wavefronts per SIMD with this kernel's registers), 4 up to two
    // workgroups, both with an exact set where one is due, and 2 up to four
    // with a table.  Beyond, and at two wavefronts with queues over 512 entries
    // or on a base whose bitmap LDS holds or with rows of under 512 bytes, one
    // wavefront per query is faster.  Measured, us, one wavefront / several:
    // FP32 300k x 200 L = 100 1 query 720 / 510, 512 1,390 / 1,140, 1M x 200 L =
    // 200 700 queries 2,740 / 2,440, 1M x 512 L = 100 1,000 2,990 / 2,370, 1M x
    // 96 L = 200 800 2,210 / 2,310, 10k x 64 L = 200 1,000 900 / 1,270; BF16
    // 200k x 512 L = 200 16 queries 2,090 / 1,190, 500k x 512 L = 400 1,024
    // 5,870 / 4,690, 500 with L = 800 9,620 / 6,410, 300k x 200 L = 400 700
    // 3,570 / 4,190; E4M3 500k x 512 L = 400 1,024 7,300 / 5,800, 300k x 100 L =
    // 200 1,000 1,750 / 2,250; BF16 500k x 200 L = 805 768 7,540 / 9,330.
    set_table(a, 10);
    // evals asks for the exact counts
    const bool counts = exact && (evals || !a.sets);
    const int row_bytes = ix->d * (ix->storage == RG_STORE_FP32 ? 4 : ix->storage == RG_STORE_BF16 ? 2 : 1);
    const int64_t most = (counts || a.Leff > kMaxL || row_bytes < 512 ? 2 : 4) * (int64_t)cus;
    const bool bits = exact && !a.adj_off && ix->n <= 32 << 10;
    if (!a.adj_off && a.ell <= 64 && nq <= most && ((exact && nq <= 2 * (int64_t)cus) || (a.sets && !bits))) {
        a.grid = nq <= cus ? 8 : nq <= 2 * (int64_t)cus ? 4 : 2;
        void *ws = nullptr;
        if (exact && nq <= 2 * (int64_t)cus) {
            // room for twice the expected nodes, as LDS allows
            a.sets = 0;
            a.hash_bits = 11;
            while (a.hash_bits < (a.grid == 8 ? 15 : 14) && (1 << a.hash_bits) < 80 * a.Leff) ++a.hash_bits;
            if (ix->n + 64 * (kMaxWide + 1) > (3ll << a.hash_bits) / 4) {
                if (hipMallocAsync(&ws, (size_t)nq * a.bm_words * 4, st) != hipSuccess) {
                    return no_memory("rg_search: out of device memory for visited bitmaps");
                }
                a.bitmap = static_cast<uint32_t *>(ws);
            }
        }
        rc = launch_search_wide(a, st);
        if (ws && hipFreeAsync(ws, st) != hipSuccess && !rc) {
            set_error("rg_search: device call failed");
            rc = RG_EDEVICE;
        }
        return rc;
    }
    if (bits) {
        // a small base: its bitmap fits in 4 KB of LDS, without the atomics'
        // way to device memory and back at every expansion (10k x 64, 1,000
        // queries, L = 50: 431 -> 360 us)
        a.hash_bits = 6;
        while ((32ll << a.hash_bits) < ix->n) ++a.hash_bits;
        return launch_search_bits(a, st);
    }
    if (!counts) {
        // the search waits on memory latency: a small visited table in LDS (no
        // device atomics) is faster even though it forgets and rescores some
        // rows (same results)
        rc = choose_table(a, cus);
        return rc ? rc : launch_search(a, st);
    }
    // persistent grid: as many resident workgroups as the chip holds, each
    // with its own visited bitmap (bounded to 8 GiB in total)
    int per_cu = 0;
    rc = search_occupancy(a, &per_cu);
    if (rc) return rc;
    int64_t grid = (int64_t)std::max(1, per_cu) * std::max(1, cus);
    grid = std::min<int64_t>(grid, nq);
    grid = std::min<int64_t>(grid, std::max<int64_t>(1, (8ll << 30) / (a.bm_words * 4)));
    a.grid = (int32_t)grid;
    void *ws = nullptr;
    const size_t bytes = (size_t)grid * a.bm_words * 4 + 256;
    if (hipMallocAsync(&ws, bytes, st) != hipSuccess) {
        return no_memory("rg_search: out of device memory for visited bitmaps");
    }
    a.work = static_cast<uint32_t *>(ws);
    a.bitmap = reinterpret_cast<uint32_t *>(static_cast<char *>(ws) + 256);
    rc = hipMemsetAsync(a.work, 0, 4, st) == hipSuccess ? RG_OK : RG_EDEVICE;
    if (!rc) rc = launch_search_persistent(a, st);
    if (hipFreeAsync(ws, st) != hipSuccess && !rc) rc = RG_EDEVICE;
    if (rc == RG_EDEVICE) set_error("rg_search: device call failed");
    return rc;
}

int rg_search_noalloc(const rg_index *ix, const float *queries, int64_t nq, int32_t k, int32_t L, uint32_t *ids,
                      float *dists, uint32_t *hops, uint32_t *evals, void *stream) {
    if (!ix || nq < 0 || (nq > 0 && (!queries || !ids || !dists)) || k < 1 || L < 1 || k > kMaxSearchL ||
        L > kMaxSearchL || nq >= (1ll << 31)) {
        set_error("rg_search_noalloc: invalid argument (need 1 <= k, L <= 1024)");
        return RG_EINVAL;
    }
    if (!ix->d_base) {
        set_error("rg_search_noalloc: index has no device data (built by rg_build_from_knn)");
        return RG_EINVAL;
    }
    SearchArgs a = search_args(ix, queries, nq, k, L, ids, dists, hops, evals);
    a.bm_words = ((ix->n + 31) / 32 + 63) / 64 * 64;
    const int64_t fit = ((int64_t)kNoAllocScratchBytes - 256) / (a.bm_words * 4);
    if (fit < 1) {
        set_error("rg_search_noalloc: one visited bitmap of " + std::to_string(a.bm_words * 4) +
                  " bytes does not fit the " + std::to_string(kNoAllocScratchBytes) + "-byte scratch");
        return RG_EINVAL;
    }
    if (nq == 0) return RG_OK;
    hipStream_t st = (hipStream_t)stream;
    uint32_t *ptr = nullptr;
    int rc = noalloc_scratch(ix->device, &ptr);
    if (rc) return rc;
    int per_cu = 0, cus = 0;
    rc = search_occupancy(a, &per_cu);
    if (rc) return rc;
    RG_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ix->device));
    int64_t grid = (int64_t)std::max(1, per_cu) * std::max(1, cus);
    grid = std::min<int64_t>(std::min<int64_t>(grid, nq), fit);
    a.grid = (int32_t)grid;
    a.work = ptr;
    a.bitmap = ptr + 64;
    rc = launch_zero_words(a.work, 64, st);
    if (!rc) rc = launch_search_persistent(a, st);
    return rc;
}

// Same as rg_search with an explicit visited-table size (2^hash_bits
// entries, 8..15); used to check that the table size never changes results.
int rg_search_hashbits(const rg_index *ix, const float *queries, int64_t nq, int32_t k, int32_t L, uint32_t *ids,
                       float *dists, uint32_t *hops, uint32_t *evals, int32_t hash_bits, void *stream) {
    if (hash_bits < 8 || hash_bits > 15) {
        set_error("rg_search_hashbits: hash_bits must be in [8, 15]");
        return RG_EINVAL;
    }
    if (!ix || nq < 0 || (nq > 0 && (!queries || !ids || !dists)) || k < 1 || L < 1 || k > kMaxSearchL ||
        L > kMaxSearchL) {
        set_error("rg_search_hashbits: invalid argument");
        return RG_EINVAL;
    }
    if (!ix->d_base) {
        set_error("rg_search_hashbits: index has no device data");
        return RG_EINVAL;
    }
    const int width = ix->d_adj_off ? kMaxEll : ix->ell;  // ids inserted per batch
    if ((1 << hash_bits) < 2 * width + 2) {
        set_error("rg_search_hashbits: table too small for the row width");
        return RG_EINVAL;
    }
    SearchArgs a = search_args(ix, queries, nq, k, L, ids, dists, hops, evals);
    set_table(a, hash_bits);
    return launch_search(a, (hipStream_t)stream);
}

int rg_save(const rg_index *ix, const char *path) {
    if (!ix || !path || !ix->d_base) {
        set_error("rg_save: invalid argument");
        return RG_EINVAL;
    }
    // the padded device rows come back in plain copies of up to 16k rows,
    // and lose their padding on the host
    std::vector<float> base((size_t)ix->n * ix->d);
    {
        const int64_t chunk = 16384;
        std::vector<float> pad((size_t)std::min<int64_t>(chunk, ix->n) * ix->pitch);
        for (int64_t r0 = 0; r0 < ix->n; r0 += chunk) {
            const int64_t m = std::min<int64_t>(chunk, ix->n - r0);
            RG_HIP(hipMemcpy(pad.data(), ix->d_base + (size_t)r0 * ix->pitch, sizeof(float) * (size_t)m * ix->pitch,
                             hipMemcpyDeviceToHost));
            for (int64_t r = 0; r < m; ++r)
                std::memcpy(base.data() + (size_t)(r0 + r) * ix->d, pad.data() + (size_t)r * ix->pitch,
                            sizeof(float) * ix->d);
        }
    }
    FILE *f = std::fopen(path, "wb");
    if (!f) {
        set_error(std::string("rg_save: cannot open ") + path);
        return RG_EINVAL;
    }
    uint64_t h = 1469598103934665603ull;
    auto put = [&](const void *p, size_t nb) {
        h = fnv1a(h, p, nb);
        return std::fwrite(p, 1, nb, f) == nb;
    };
    const char magic[8] = {'R', 'G', 'I', 'D', 'X', 0, 0, 1};
    const int64_t nnz = ix->offsets[ix->n];
    const int32_t hdr[8] = {ix->d, ix->metric, (int32_t)ix->entry, ix->Nq, ix->M, ix->L_build, ix->m_pj, ix->m_ce};
    bool ok = put(magic, 8) && put(&ix->n, 8) && put(hdr, sizeof(hdr)) && put(&ix->repairs, 8) && put(&nnz, 8) &&
              put(ix->offsets.data(), sizeof(int64_t) * ix->offsets.size()) &&
              put(ix->indices.data(), sizeof(uint32_t) * ix->indices.size()) &&
              put(base.data(), sizeof(float) * base.size());
    ok = ok && std::fwrite(&h, 1, 8, f) == 8;
    ok = (std::fclose(f) == 0) && ok;
    if (!ok) {
        set_error("rg_save: write failed");
        return RG_EINVAL;
    }
    return RG_OK;
}

int rg_load(const char *path, void *stream, rg_index **out) {
    if (!path || !out) {
        set_error("rg_load: invalid argument");
        return RG_EINVAL;
    }
    *out = nullptr;
    FILE *f = std::fopen(path, "rb");
    if (!f) {
        set_error(std::string("rg_load: cannot open ") + path);
        return RG_EINVAL;
    }
    uint64_t h = 1469598103934665603ull;
    auto get = [&](void *p, size_t nb) {
        if (std::fread(p, 1, nb, f) != nb) return false;
        h = fnv1a(h, p, nb);
        return true;
    };
    char magic[8];
    int64_t n = 0, repairs = 0, nnz = 0;
    int32_t hdr[8];
    const char want[8] = {'R', 'G', 'I', 'D', 'X', 0, 0, 1};
    bool ok = get(magic, 8) && std::memcmp(magic, want, 8) == 0 && get(&n, 8) && get(hdr, sizeof(hdr)) &&
              get(&repairs, 8) && get(&nnz, 8) && n >= 1 && n < (1ll << 31) && hdr[0] >= 1 && nnz >= 0 &&
              nnz < (1ll << 40);
    rg_index *ix = nullptr;
    std::vector<float> base;
    if (ok) {
        ix = new rg_index();
        ix->n = n;
        ix->d = hdr[0];
        ix->metric = hdr[1];
        ix->entry = (uint32_t)hdr[2];
        ix->Nq = hdr[3];
        ix->M = hdr[4];
        ix->L_build = hdr[5];
        ix->m_pj = hdr[6];
        ix->m_ce = hdr[7];
        ix->repairs = repairs;
        ix->offsets.resize((size_t)n + 1);
        ix->indices.resize((size_t)nnz);
        base.resize((size_t)n * ix->d);
        ok = get(ix->offsets.data(), sizeof(int64_t) * (size_t)(n + 1)) &&
             get(ix->indices.data(), sizeof(uint32_t) * (size_t)nnz) && get(base.data(), sizeof(float) * base.size());
    }
    uint64_t stored = 0;
    const uint64_t computed = h;
    ok = ok && std::fread(&stored, 1, 8, f) == 8 && stored == computed;
    std::fclose(f);
    if (!ok || ix->offsets[n] != nnz || check_csr(n, ix->offsets.data(), ix->indices.data(), ix->entry)) {
        delete ix;
        set_error("rg_load: corrupt index file");
        return RG_ECORRUPT;
    }
    hipStream_t st = (hipStream_t)stream;
    DevBuf tmp;
    int rc = tmp.alloc(sizeof(float) * base.size());
    if (!rc && hipMemcpyAsync(tmp.p, base.data(), sizeof(float) * base.size(), hipMemcpyHostToDevice, st) != hipSuccess)
        rc = RG_EDEVICE;
    (void)hipGetDevice(&ix->device);
    if (!rc) rc = upload_index(ix, tmp.as<float>(), st);
    if (rc) {
        free_index_device(ix);
        delete ix;
        return rc;
    }
    *out = ix;
    return RG_OK;
}

int rg_device_copy(void *dst, const void *src, int64_t bytes, void *stream) {
    if (!dst || !src || bytes < 0) {
        set_error("rg_device_copy: invalid argument");
        return RG_EINVAL;
    }
    return launch_copy_probe(dst, src, bytes, (hipStream_t)stream);
}

int rg_measure_peaks(double *hbm_read_gbs, double *f16_tflops, double *f32_tflops, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    int dev = 0, cus = 0;
    RG_HIP(hipGetDevice(&dev));
    RG_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    const int blocks = 8 * std::max(1, cus);  // 8 waves per SIMD
    const int64_t bytes = 4ll << 30;
    DevBuf buf, sink;
    int rc = buf.alloc((size_t)bytes);
    if (!rc) rc = sink.alloc(sizeof(float) * 256 * (size_t)std::max(blocks, 65536));
    if (rc) return rc;
    RG_HIP(hipMemsetAsync(buf.p, 1, (size_t)bytes, st));
    hipEvent_t e0, e1;
    RG_HIP(hipEventCreate(&e0));
    RG_HIP(hipEventCreate(&e1));
    auto timed = [&](auto &&launch, int reps, float *best) -> int {
        *best = 1e30f;
        for (int r = 0; r < reps + 1; ++r) {  // the first run warms up
            RG_HIP(hipEventRecord(e0, st));
            int rc2 = launch();
            if (rc2) return rc2;
            RG_HIP(hipEventRecord(e1, st));
            RG_HIP(hipEventSynchronize(e1));
            float ms = 0.f;
            RG_HIP(hipEventElapsedTime(&ms, e0, e1));
            if (r > 0) *best = std::min(*best, ms);
        }
        return RG_OK;
    };
    float ms = 0.f;
    double flop = 0.0;
    rc = timed([&]() { return launch_read_stream(buf.p, bytes, sink.p, 65536, st); }, 5, &ms);
    if (!rc && hbm_read_gbs) *hbm_read_gbs = (double)bytes / (ms * 1e-3) / 1e9;
    if (!rc) rc = timed([&]() { return launch_mfma_probe(0, 4096, sink.p, blocks, st, &flop); }, 3, &ms);
    if (!rc && f16_tflops) *f16_tflops = flop / (ms * 1e-3) / 1e12;
    if (!rc) rc = timed([&]() { return launch_mfma_probe(1, 1024, sink.p, blocks, st, &flop); }, 3, &ms);
    if (!rc && f32_tflops) *f32_tflops = flop / (ms * 1e-3) / 1e12;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return rc;
}

void rg_free(rg_index *ix) {
    if (!ix) return;
    free_index_device(ix);
    delete ix;
}

}  // extern "C"
