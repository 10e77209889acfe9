// Construction-time searches, selections and reverse updates with the
// canonical FP64 distance.
//
// Connectivity enhancement (Algorithm 1; Sec. 4.2.4) searches the projected
// graph once per base vector, with the base vector as the query and a queue
// of length L, uses the final queue as candidate neighbours, and lets every
// selected node reconsider its list.  All of it decides the graph, so it is
// computed with the same canonical distance the host uses everywhere in
// construction: delta(a, b) = -sum_i a_i b_i, accumulated in FP64 in
// increasing i.  On the GPU one lane computes one sum as a chain of FP64
// fused multiply-adds; the product of two floats is exact in FP64, so every
// step rounds exactly like the host's add, and the value is bit-identical.
//
// Such a chain is a lane's walk over a whole row, hundreds of dependent steps,
// and what decides is hardly ever its last bits.  So sums that many lanes
// share go first, with a bound on how far they can be from the canonical
// value, and only what the bound leaves open takes the chain: the searches
// compare FP64 sums, the selections FP32 ones.
#include "queue_ops.h"
#include "rg_internal.h"
#include "wave_ops.h"

#include <chrono>
#include <cstdio>
#include <cstdlib>

namespace rg {
namespace {

// -delta(q, row), q and row 16-byte aligned; the next 16 elements are loaded
// while the current ones are added
__device__ __forceinline__ double canon_sum(const float *q, const float *row, int d) {
    double s = 0.0;
    const float4 *q4 = reinterpret_cast<const float4 *>(q);
    const float4 *r4 = reinterpret_cast<const float4 *>(row);
    const int d4 = d >> 2, full = d4 & ~3;
    float4 nx[4];
    if (full > 0) {
#pragma unroll
        for (int t = 0; t < 4; ++t) nx[t] = r4[t];
    }
    for (int c = 0; c < full; c += 4) {
        float4 b[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) b[t] = nx[t];
        if (c + 4 < full) {
#pragma unroll
            for (int t = 0; t < 4; ++t) nx[t] = r4[c + 4 + t];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float4 a = q4[c + t];
            s = fma((double)a.x, (double)b[t].x, s);
            s = fma((double)a.y, (double)b[t].y, s);
            s = fma((double)a.z, (double)b[t].z, s);
            s = fma((double)a.w, (double)b[t].w, s);
        }
    }
    for (int i = full * 4; i < d; ++i) s = fma((double)q[i], (double)row[i], s);
    return s;
}

// delta(q, row).  A NaN counts as +inf: without a place in the order it would
// leave holes in a queue and gaps among ranks.
__device__ __forceinline__ double canon_delta(const float *q, const float *row, int d) {
    return __builtin_fmin(-canon_sum(q, row, d), __builtin_inf());
}

struct CanonArgs {
    const float *X;         // n x pitch (zero padded)
    const uint32_t *adj;    // n x ell
    uint32_t *out_ids;      // count x L
    double *out_d;          // count x L
    int32_t *out_n;         // count
    int64_t x0, count;
    int32_t d, pitch, ell, L, hash_bits, id_bits, cand, redo;
    uint32_t entry;
    const double *xmax2;    // the largest squared row norm
    double gam, gam32;      // |shared sum - canonical sum| <= gam |q| |x|; of FP32 sums
};

// LDS of one search; qd is 8-byte aligned
struct CanonLds {
    float *qrow;
    double *qd;
    uint32_t *htab;
    QueueLds<double> ql;
    __device__ __forceinline__ CanonLds(unsigned char *smem, const CanonArgs &a) {
        qrow = reinterpret_cast<float *>(smem);
        qd = reinterpret_cast<double *>(qrow + a.pitch);
        double *cd = qd + a.L, *sd = cd + a.cand;
        uint32_t *ci = reinterpret_cast<uint32_t *>(sd + a.cand), *si = ci + a.cand;
        int32_t *slb = reinterpret_cast<int32_t *>(si + a.cand);
        htab = reinterpret_cast<uint32_t *>(slb + a.cand);  // cand is even: 8-byte aligned
        ql = QueueLds<double>{qd, htab + (1 << a.hash_bits), cd, ci, sd, si, slb};
    }
};
size_t canon_lds_bytes(const CanonArgs &a) {
    return (size_t)a.pitch * 4 + (size_t)a.L * 12 + (size_t)a.cand * 28 + ((size_t)4 << a.hash_bits);
}

// delta of q and each of the rows ids[0..cnt), up to gam |q| |x| (T = double)
// or gam32 |q| |x| (float): 16 lanes per row, each adding the products of every
// 16th 4-element piece, then a tree; the value depends on the two rows alone.
// R rows per group in flight.
template <typename T, int R>
__device__ __forceinline__ void shared_sums(const CanonArgs &a, const float *q, const uint32_t *ids, int cnt, T *out) {
    constexpr int G = 16, NG = 4;
    const int g = lane_id() / G, j = lane_id() % G, nch = a.pitch >> 2;
    const float4 *q4 = reinterpret_cast<const float4 *>(q);
    for (int p = 0; p < cnt; p += NG * R) {
        const float4 *row[R];
        T s[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = p + r * NG + g;
            row[r] = reinterpret_cast<const float4 *>(a.X + (size_t)ids[i < cnt ? i : 0] * a.pitch);
            s[r] = (T)0;
        }
#pragma unroll 4
        for (int c = j; c < nch; c += G) {
            const float4 x = q4[c];
            const T x0 = (T)x.x, x1 = (T)x.y, x2 = (T)x.z, x3 = (T)x.w;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float4 y = row[r][c];
                s[r] = fma(x0, (T)y.x, s[r]);
                s[r] = fma(x1, (T)y.y, s[r]);
                s[r] = fma(x2, (T)y.z, s[r]);
                s[r] = fma(x3, (T)y.w, s[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            s[r] = group_sum<G>(s[r]);
            const int i = p + r * NG + g;
            if (j == 0 && i < cnt) out[i] = -s[r];
        }
    }
}

// One wavefront per searched node; the queue (FP64 keys), candidate batch and
// visited table live in LDS.  The expansion rule, the forgetting visited
// table and the merge are those of the query-time search, so the final queue
// equals the host searcher's.
//
// NEAR: the keys are shared sums.  They decide while no two that are compared
// lie within twice their error (2.5e-14 |q| |x| at d = 200) of each other; then
// the queue is the canonical one, and its distances are computed at the end,
// one lane per entry.  While the queue is full most candidates are far beyond
// its last entry: FP32 sums with their own bound turn those away, unless |q|
// times the longest row's norm is near FP32's largest value.  A search that
// meets two closer keys (copies of a row, say) gives up, and a second launch
// (redo) runs it with a canonical chain for every candidate, as all searches
// did before.  60k rows of 200, L = 500 (about 550 expansions and
// 16k rows scored each): 69.5 ms against 210; before the merge was short,
// shared FP64 sums for every row took 117 (their conversions keep the VALU
// busy), FP32 sums with chains for what they leave open 129, this form 83.
template <class VIS, bool NEAR>
__global__ __launch_bounds__(64) void k_canon_search(CanonArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = lane_id();
    const int L = a.L, ell = a.ell, d = a.d;
    const int64_t b = blockIdx.x;
    const int64_t x = a.x0 + b;
    if (!NEAR && a.redo && a.out_n[b] >= 0) return;
    const CanonLds s(smem, a);
    float *qrow = s.qrow;
    double *qd = s.qd, *cd = s.ql.cd;
    uint32_t *qi = s.ql.qi, *ci = s.ql.ci;
    VIS vis(s.htab, a.hash_bits, a.id_bits);

    double n2 = 0.0;
    for (int i = lane; i < a.pitch; i += 64) {
        const float v = a.X[x * a.pitch + i];
        qrow[i] = v;
        n2 = fma((double)v, (double)v, n2);
    }
    vis.clear();
    double tol = 0.0, tol32 = 0.0;
    int when = -1;  // the queue length at which FP32 sums turn candidates away
    if constexpr (NEAR) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
        const double nn = sqrt(n2 * *a.xmax2) * (1.0 + 1e-9);
        tol = 2.0 * a.gam * nn;
        // and what underflow may lose; an FP32 sum that can overflow bounds nothing
        tol32 = (a.gam + a.gam32) * nn + 1e-30;
        when = __builtin_amdgcn_readfirstlane(nn < 1e38 ? L : -1);
    }
    wave_sync();
    if (NEAR) {
        if (lane == 0) ci[0] = a.entry;
        wave_sync();
        shared_sums<double, 1>(a, qrow, ci, 1, qd);
    } else if (lane == 0) {
        qd[0] = canon_delta(qrow, a.X + (size_t)a.entry * a.pitch, d);
    }
    if (lane == 0) {
        qi[0] = a.entry;
        vis.mark_entry(a.entry);
    }
    vis.added(1);
    int qn = 1, ptr = 0;
    wave_sync();
    for (;;) {
        int sel = -1;
        for (int bb = ptr; bb < qn; bb += 64) {
            const int i = bb + lane;
            const uint64_t m = ballot64(i < qn && !(qi[i] & kExpanded));
            if (m) {
                sel = bb + (int)__builtin_ctzll(m);
                break;
            }
        }
        if (sel < 0) break;
        ptr = sel;
        const uint32_t v = qi[sel];
        wave_sync();
        if (lane == 0) qi[sel] = v | kExpanded;
        vis.begin_hop(ell);
        int nnew = 0;
        for (int e0 = 0; e0 < ell; e0 += 64) {
            const int e = e0 + lane;
            const uint32_t u = e < ell ? a.adj[(size_t)v * ell + e] : kNone;
            const bool fresh = u != kNone && vis.insert(u);
            const uint64_t m = ballot64(fresh);
            if (fresh) ci[nnew + lanes_below(m)] = u;
            nnew += (int)__popcll(m);
        }
        vis.added(nnew);
        wave_sync();
        if (nnew == 0) continue;
        if constexpr (NEAR) {
            if (qn == when) {
                float *fd = reinterpret_cast<float *>(s.ql.sd);
                shared_sums<float, 4>(a, qrow, ci, nnew, fd);
                wave_sync();
                const double bar = qd[L - 1] + tol32;
                const uint32_t u = ci[lane];
                const bool keep = lane < nnew && !((double)fd[lane] > bar);
                const uint64_t m = ballot64(keep);
                nnew = (int)__popcll(m);
                if (nnew == 0) continue;
                wave_sync();
                if (keep) ci[lanes_below(m)] = u;
                wave_sync();
            }
            if (nnew <= 4)
                shared_sums<double, 1>(a, qrow, ci, nnew, cd);
            else
                shared_sums<double, 4>(a, qrow, ci, nnew, cd);
            wave_sync();
            if (!merge_batch<1, double, kMaxL / 64, true>(s.ql, nnew, L, qn, ptr, tol)) {
                if (lane == 0) a.out_n[b] = -1;
                return;
            }
        } else {
            for (int j = lane; j < nnew; j += 64) cd[j] = canon_delta(qrow, a.X + (size_t)ci[j] * a.pitch, d);
            wave_sync();
            if (nnew <= 64)
                merge_batch<1, double>(s.ql, nnew, L, qn, ptr);
            else
                merge_batch<2, double>(s.ql, nnew, L, qn, ptr);
        }
        wave_sync();
    }
    for (int i = lane; i < qn; i += 64) {
        const uint32_t u = qi[i] & ~kExpanded;
        a.out_ids[b * L + i] = u;
        a.out_d[b * L + i] = NEAR ? canon_delta(qrow, a.X + (size_t)u * a.pitch, d) : qd[i];
    }
    if (lane == 0) a.out_n[b] = qn;
}

// The largest squared row norm (the sums' own rounding is in the callers'
// margin); *out starts at 0.  A NaN norm counts as infinite: nothing is then
// far enough apart.
__global__ __launch_bounds__(256) void k_max_norm(const float *X, int64_t n, int pitch, double *out) {
    const int lane = lane_id();
    double best = 0.0;
    for (int64_t r = blockIdx.x * 4 + (threadIdx.x >> 6); r < n; r += (int64_t)gridDim.x * 4) {
        double s = 0.0;
        for (int i = lane; i < pitch; i += 64) {
            const float v = X[r * pitch + i];
            s = fma((double)v, (double)v, s);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        best = s != s ? __builtin_inf() : fmax(best, s);
    }
    // the bits of values that are not negative order like the values
    if (lane == 0) atomicMax(reinterpret_cast<unsigned long long *>(out), (unsigned long long)__double_as_longlong(best));
}

// Candidates of the projection (Algorithm 2): of each pivot x, the entries of
// the kNN lists of its bridges (ascending; the list without its first entry, x
// itself) until a whole list brings their number to L or more, each once, with
// their canonical distances, in (delta, id) order, the first L of them.  One
// wavefront per pivot: a hash set in LDS keeps each id once, a lane walks a
// chain per candidate, the wavefront sorts.  Pivots differ in their work (one
// bridge or hundreds) and run side by side; loads bound it.  8,033 pivots of
// 60k rows of 200, L = 500: 0.43 ms, and 2.3 ms for their selections; on 16
// host threads both took 55.
struct CandArgs {
    const float *X;          // n x pitch
    int32_t d, pitch;
    const uint32_t *nodes;   // the pivots
    const uint32_t *lists;   // nt x Nq
    const int64_t *boff;     // n + 1: the bridges of each node
    const uint32_t *bidx;
    int32_t Nq, L, hash_bits, cap;  // cap: a power of two, room for L + Nq
    uint32_t *ids;           // count x L
    double *dists;
    int32_t *counts;
};

template <int E>
__device__ __forceinline__ void rank_candidates(const CandArgs &a, const float *xrow, const uint32_t *cid, int cnt,
                                                int64_t b) {
    const int lane = lane_id();
    double key[E];
    uint32_t id[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = e * 64 + lane;  // any assignment of candidates to lanes will do
        id[e] = j < cnt ? cid[j] : kNone;
        key[e] = j < cnt ? canon_delta(xrow, a.X + (size_t)id[e] * a.pitch, a.d) : INFINITY;
    }
    wave_sort<E, double>(key, id);
    const int nk = min(cnt, a.L);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = lane * E + e;
        if (j < nk) {
            a.ids[b * a.L + j] = id[e];
            a.dists[b * a.L + j] = key[e];
        }
    }
    if (lane == 0) a.counts[b] = nk;
}

__global__ __launch_bounds__(64) void k_project_cands(CandArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *xrow = reinterpret_cast<float *>(smem);
    uint32_t *cid = reinterpret_cast<uint32_t *>(xrow + a.pitch);
    uint32_t *set = cid + a.cap;
    const int lane = lane_id();
    const int64_t b = blockIdx.x;
    const uint32_t x = a.nodes[b], mask = (1u << a.hash_bits) - 1u;
    for (int i = lane; i < a.pitch; i += 64) xrow[i] = a.X[(size_t)x * a.pitch + i];
    for (uint32_t i = lane; i <= mask; i += 64) set[i] = kNone;
    wave_sync();
    int cnt = 0;
    for (int64_t e = a.boff[x]; e < a.boff[x + 1] && cnt < a.L; ++e) {
        const uint32_t *lst = a.lists + (int64_t)a.bidx[e] * a.Nq;
        for (int j0 = 1; j0 < a.Nq; j0 += 64) {
            const uint32_t c = j0 + lane < a.Nq ? lst[j0 + lane] : kNone;
            bool fresh = false;
            if (c != kNone && c != x) {
                uint32_t h = (c * 2654435761u) >> (32 - a.hash_bits);
                // at most half the slots are ever taken, so a free one comes
                for (;;) {
                    const uint32_t was = atomicCAS(&set[h], kNone, c);
                    fresh = was == kNone;
                    if (fresh || was == c) break;
                    h = (h + 1) & mask;
                }
            }
            const uint64_t fm = ballot64(fresh);
            const int to = cnt + lanes_below(fm);
            if (fresh && to < a.cap) cid[to] = c;  // to < cap holds: cnt < L before each list of Nq - 1
            cnt += (int)__popcll(fm);
        }
    }
    cnt = min(cnt, a.cap);
    wave_sync();
    if (cnt <= 128)
        rank_candidates<2>(a, xrow, cid, cnt, b);
    else if (cnt <= 256)
        rank_candidates<4>(a, xrow, cid, cnt, b);
    else if (cnt <= 512)
        rank_candidates<8>(a, xrow, cid, cnt, b);
    else
        rank_candidates<16>(a, xrow, cid, cnt, b);
}

// AcquireNeighbors (Algorithm 3) for a node's ranked candidates, on the
// device: those of the projection, with the fill, or the node's final queue
// (without the node itself), without it.  They stand in (delta, id) order; a
// candidate is kept iff delta(x, c) < delta(c, p) for every kept p (strict),
// until m are kept; the fill adds the others in order up to m.  One
// lane per candidate, 64 at a time in rank order.  FP32 sums (16 kept rows in
// one pass over the candidate's row) settle what lies outside their bound,
// gam |c| |p|; the rest takes the host's FP64 chain, so every decision is the
// host's.  The kept rows sit in LDS when they fit.  60k queues of 500 rows of
// 200, m = 31: 22 ms against 71 with a chain for every pair.
struct SelectArgs {
    const float *X;          // n x pitch
    int32_t d, pitch;
    const uint32_t *ids;     // count x L search output
    const double *dists;
    const int32_t *counts;
    int32_t L, m, head_len;
    int64_t x0;
    const uint32_t *nodes;   // the nodes, or null: x0, x0 + 1, ...
    uint32_t *sel_ids;       // rows of m, of nodes sel0, sel0 + 1, ...
    double *sel_d;
    int32_t *sel_n;
    int64_t sel0;
    uint32_t *head;          // count x head_len: the first candidates
    int32_t *head_n;         // candidates per node (without the node), or null
    float gam;
    float floor2;            // what squares that underflow can add up to
};

constexpr int KG = 16;

// FP32 sums of this lane's candidate row with kept rows r0 .. r0 + nk, and
// the candidate's squared norm.  kr(t) is kept row r0 + t.
template <class KR>
__device__ __forceinline__ void near_kept(const float *crow, KR kr, int nch, int nk, float (&acc)[KG], float &norm2) {
    const float4 *kp[KG];
    norm2 = 0.f;
#pragma unroll
    for (int t = 0; t < KG; ++t) {
        acc[t] = 0.f;
        kp[t] = reinterpret_cast<const float4 *>(t < nk ? kr(t) : kr(0));
    }
    const float4 *c4 = reinterpret_cast<const float4 *>(crow);
#pragma unroll 2
    for (int i = 0; i < nch; ++i) {
        const float4 c = c4[i];
        norm2 = fmaf(c.x, c.x, fmaf(c.y, c.y, fmaf(c.z, c.z, fmaf(c.w, c.w, norm2))));
#pragma unroll
        for (int t = 0; t < KG; ++t)
            if (t < nk) {
                const float4 k = kp[t][i];
                acc[t] = fmaf(c.x, k.x, acc[t]);
                acc[t] = fmaf(c.y, k.y, acc[t]);
                acc[t] = fmaf(c.z, k.z, acc[t]);
                acc[t] = fmaf(c.w, k.w, acc[t]);
            }
    }
}

// At least the norm of a row whose FP32 sum of squares is n2.  Squares below
// FP32's smallest normal number may have counted as zero: floor2 is what they
// can add up to.  The 1.01 makes it infinite, and with it the bound, before
// the product of two norms, and so a sum of two rows, can overflow.
__device__ __forceinline__ float norm_above(float n2, const SelectArgs &a) {
    return sqrtf(fmaf(n2, 1.01f, a.floor2)) * (1.0001f + a.gam);
}

template <bool KEPT_IN_LDS, bool FILL>
__global__ __launch_bounds__(64) void k_canon_select(SelectArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint64_t kept_of[kMaxL / 64];              // per 64 candidates (for the fill)
    uint32_t *kid = reinterpret_cast<uint32_t *>(smem);   // m kept ids
    float *kn = reinterpret_cast<float *>(smem) + ((a.m + 3) & ~3);  // their norms (rounded up)
    float *K = kn + ((a.m + 3) & ~3);                     // m x pitch kept rows (if they fit)
    const int lane = lane_id(), nch = a.pitch >> 2;
    const int64_t b = blockIdx.x;
    const uint32_t x = a.nodes ? a.nodes[b] : (uint32_t)(a.x0 + b);
    const int64_t at = (int64_t)x - a.sel0;
    uint32_t *sel_ids = a.sel_ids + at * a.m;
    double *sel_d = a.sel_d + at * a.m;
    const uint32_t *cid = a.ids + b * a.L;
    const double *cdd = a.dists + b * a.L;
    const int qn = a.counts[b];
    int nr = 0, hn = 0;
    auto kept_row = [&](int r) -> const float * {
        if constexpr (KEPT_IN_LDS) return K + (size_t)r * a.pitch;
        return a.X + (size_t)kid[r] * a.pitch;
    };
    for (int j0 = 0; j0 < qn; j0 += 64) {
        const int j = j0 + lane;
        const uint32_t c = j < qn ? cid[j] : kNone;
        const bool valid = j < qn && c != x;
        const uint64_t vm = ballot64(valid);
        const int pos = hn + lanes_below(vm);
        if (valid && pos < a.head_len) a.head[b * a.head_len + pos] = c;
        hn += (int)__popcll(vm);
        if (nr >= a.m) {
            if (FILL) break;
            continue;
        }
        uint64_t kept = 0;
        const double dxc = valid ? cdd[j] : 0.0;
        const float *crow = a.X + (size_t)(valid ? c : 0u) * a.pitch;
        bool alive = valid;
        float cnorm = 0.f;
        // this lane's candidate against kept rows r0 .. r0 + nk
        auto against = [&](int r0, int nk) {
            float acc[KG];
            uint32_t open = 0;
            if (alive) {
                float n2;
                near_kept(crow, [&](int t) { return kept_row(r0 + t); }, nch, nk, acc, n2);
                cnorm = norm_above(n2, a);
#pragma unroll
                for (int t = 0; t < KG; ++t)
                    if (t < nk) {
                        const double dcp = -(double)acc[t], tau = (double)fmaf(a.gam * cnorm, kn[r0 + t], 1e-30f);
                        if (dxc >= dcp + tau)
                            alive = false;
                        else if (!(dxc < dcp - tau))
                            open |= 1u << t;
                    }
                if (!alive) open = 0;
            }
            while (ballot64(open != 0)) {
                if (open) {
                    const int t = __builtin_ctz(open);
                    open &= open - 1;
                    if (!(dxc < canon_delta(crow, kept_row(r0 + t), a.d))) {
                        alive = false;
                        open = 0;
                    }
                }
            }
        };
        // rejected by a row kept before this batch?
        for (int r0 = 0; r0 < nr && ballot64(alive) != 0; r0 += KG) against(r0, min(KG, nr - r0));
        // in rank order: the lowest surviving candidate is kept, and the
        // later survivors are checked against it
        for (;;) {
            const uint64_t am = ballot64(alive);
            if (am == 0 || nr >= a.m) break;
            const int js = (int)__builtin_ctzll(am);
            const uint32_t cs = (uint32_t)__builtin_amdgcn_readlane((int)c, js);
            const double ds = __shfl(dxc, js);
            float n2 = 0.f;
            for (int i = lane; i < a.pitch; i += 64) {
                const float y = a.X[(size_t)cs * a.pitch + i];
                if (KEPT_IN_LDS) K[(size_t)nr * a.pitch + i] = y;
                n2 = fmaf(y, y, n2);
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
            if (lane == 0) {
                kid[nr] = cs;
                kn[nr] = norm_above(n2, a);
                sel_ids[nr] = cs;
                sel_d[nr] = ds;
            }
            ++nr;
            kept |= 1ull << js;
            wave_sync();
            if (lane == js) alive = false;
            against(nr - 1, 1);
        }
        if (FILL && lane == 0) kept_of[j0 >> 6] = kept;
    }
    if constexpr (FILL) {
        wave_sync();
        for (int j0 = 0; j0 < qn && nr < a.m; j0 += 64) {
            const int j = j0 + lane;
            const uint32_t c = j < qn ? cid[j] : kNone;
            const bool rest = j < qn && c != x && !((kept_of[j0 >> 6] >> lane) & 1ull);
            const uint64_t rm = ballot64(rest);
            const int to = nr + lanes_below(rm);
            if (rest && to < a.m) {
                sel_ids[to] = c;
                sel_d[to] = cdd[j];
            }
            nr = min(a.m, nr + (int)__popcll(rm));
        }
    }
    if (lane == 0) {
        a.sel_n[at] = nr;
        if (a.head_n) a.head_n[b] = hn;
    }
}

// Reverse updates.  Node p's list starts as its own selection; every later
// node x that selected p asks it, in ascending x, to take x in: p's list
// becomes AcquireNeighbors (without fill) of the list and x.  The list is the
// outcome of such a selection, so its entries stand in rank order and each is
// nearer to p than to all before it.  Then x, of rank r, is kept iff it is
// nearer to p than to the r entries before it; if not (or if r = m) nothing
// changes; if so, the entries behind it stay iff they are nearer to p than to
// x, as far as m go.  That takes the canonical distances of x to p and to the
// entries only: one lane each.  One wavefront per list; lists of updates are
// short (at most 189 where 20k nodes made 535k).  60k rows of 200, m = 31: 3.4
// ms; on 16 host threads it took 260.
struct ReplayArgs {
    const float *X;
    int32_t d, pitch, m;
    const uint32_t *sel_ids;  // n x m
    const double *sel_d;
    const int32_t *sel_n;
    const int64_t *off;       // n + 1: the nodes that selected p
    const uint32_t *src;      // ascending per p where they are more than 64
    uint32_t *out;            // n x out_pitch
    int32_t *out_n;
    int32_t out_pitch;
    const int64_t *boff;      // k_replay_fill: the bridges of each node, none if it is no pivot
    int64_t p0;               // the first workgroup's node
};

__global__ __launch_bounds__(64) void k_replay(ReplayArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *xrow = reinterpret_cast<float *>(smem);
    double *cd = reinterpret_cast<double *>(xrow + a.pitch);
    uint32_t *ci = reinterpret_cast<uint32_t *>(cd + a.m + 1);
    const int lane = lane_id();
    const int64_t p = a.p0 + blockIdx.x;
    int nc = a.sel_n[p];
    for (int j = lane; j < nc; j += 64) {
        ci[j] = a.sel_ids[p * a.m + j];
        cd[j] = a.sel_d[p * a.m + j];
    }
    const int64_t e0 = a.off[p], ne = a.off[p + 1] - e0;
    uint32_t ev[1] = {lane < ne ? a.src[e0 + lane] : kNone}, id[1] = {0};
    if (ne <= 64) wave_sort<1, uint32_t>(ev, id);
    wave_sync();
    for (int64_t e = 0; e < ne; ++e) {
        if (e > 0 && (e & 63) == 0) ev[0] = e + lane < ne ? a.src[e0 + e + lane] : kNone;
        const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)ev[0], (int)(e & 63));
        if ((int64_t)x < p) continue;  // before p's own selection, which replaced it
        bool there = false;
        for (int j = lane; j < nc; j += 64) there |= ci[j] == x;
        if (ballot64(there)) continue;
        for (int i = lane; i < a.pitch; i += 64) xrow[i] = a.X[(size_t)x * a.pitch + i];
        wave_sync();
        // entry j (j == nc: p itself) in slot j / 64 of lane j % 64
        double dj[2] = {0.0, 0.0}, key[2] = {0.0, 0.0};
        uint32_t c[2] = {0, 0};
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int j = lane + 64 * s;
            if (j <= nc) {
                if (j < nc) {
                    c[s] = ci[j];
                    key[s] = cd[j];
                } else {
                    c[s] = (uint32_t)p;
                }
                dj[s] = canon_delta(xrow, a.X + (size_t)c[s] * a.pitch, a.d);
            }
        }
        const double d0 = __shfl(dj[0], nc & 63), d1 = __shfl(dj[1], nc & 63);
        const double dx = nc < 64 ? d0 : d1;
        bool before[2], occ[2], stay[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int j = lane + 64 * s;
            before[s] = j < nc && kless(key[s], c[s], dx, x);
            occ[s] = before[s] && !(dx < dj[s]);
            stay[s] = j < nc && !before[s] && key[s] < dj[s];
        }
        const int r = (int)__popcll(ballot64(before[0])) + (int)__popcll(ballot64(before[1]));
        if (ballot64(occ[0] || occ[1]) || r >= a.m) continue;
        const uint64_t s0 = ballot64(stay[0]), s1 = ballot64(stay[1]);
        wave_sync();
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int to = r + 1 + (s == 0 ? lanes_below(s0) : (int)__popcll(s0) + lanes_below(s1));
            if (stay[s] && to < a.m) {
                ci[to] = c[s];
                cd[to] = key[s];
            }
        }
        if (lane == 0) {
            ci[r] = x;
            cd[r] = dx;
        }
        nc = min(a.m, r + 1 + (int)__popcll(s0) + (int)__popcll(s1));
        wave_sync();
    }
    for (int j = lane; j < nc; j += 64) a.out[p * a.out_pitch + j] = ci[j];
    if (lane == 0) a.out_n[p] = nc;
}

// Reverse updates of the projection (Algorithm 2), which fills: the list of p
// starts as its own selection (a pivot) or empty, and takes each later node x
// that selected p, ascending, while it has room.  A full list of m and x are m
// + 1 candidates for m places, so AcquireNeighbors with the fill drops exactly
// one: the last in rank that is not kept, or the last of all if every one is.
// So the list is kept as slots, one per lane (SL of them for m >= 64), each
// with its rank and a mask of the slots that rank before it and are no farther
// from it than p is: those that keep it out if they are kept.  x brings one
// distance per slot, a lane each, and the kept ones follow from the masks in a
// few ballots: a slot is out if a kept one keeps it out, and kept once all
// that could are out; the lowest rank still open is settled in every round.
// The masks of the slots filled before are made when the list first overflows.
// A lane's chain over a row of L2 and its loads bound a step.  257k updates of
// 60k rows of 200 (at most 217 in a list), m = 32: 1.2 ms; on 16 host threads
// 28.
template <int SL>
__global__ __launch_bounds__(64) void k_replay_fill(ReplayArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *xrow = reinterpret_cast<float *>(smem);
    const int lane = lane_id();
    const int64_t p = a.p0 + blockIdx.x;
    const bool own = a.boff[p] != a.boff[p + 1];  // a pivot: its selection replaced what came before
    int nc = own ? a.sel_n[p] : 0;
    uint32_t id[SL], rank[SL];
    double key[SL];
    uint64_t out_by[SL][SL];  // the slots that keep slot s of this lane out
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        const int j = lane + 64 * s;
        id[s] = j < nc ? a.sel_ids[p * a.m + j] : kNone;
        key[s] = 0.0;
        rank[s] = 0;
#pragma unroll
        for (int t = 0; t < SL; ++t) out_by[s][t] = 0;
    }
    auto load_row = [&](uint32_t x) {
        wave_sync();
        for (int i = lane; i < a.pitch; i += 64) xrow[i] = a.X[(size_t)x * a.pitch + i];
        wave_sync();
    };
    auto id_of = [&](int slot) {
        const int l = slot & 63;
        uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)id[0], l);
        if constexpr (SL > 1) {
            const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)id[SL - 1], l);
            v = slot < 64 ? v : w;
        }
        return v;
    };
    auto key_of = [&](int slot) {
        double v = __shfl(key[0], slot & 63);
        if constexpr (SL > 1) {
            const double w = __shfl(key[SL - 1], slot & 63);
            v = slot < 64 ? v : w;
        }
        return v;
    };
    int open = -1;  // the one free slot of a list that has overflowed, or -1
    const int64_t e0 = a.off[p], ne = a.off[p + 1] - e0;
    uint32_t ev[1] = {lane < ne ? a.src[e0 + lane] : kNone}, tag[1] = {0};
    if (ne <= 64) wave_sort<1, uint32_t>(ev, tag);
    for (int64_t e = 0; e < ne; ++e) {
        if (e > 0 && (e & 63) == 0) ev[0] = e + lane < ne ? a.src[e0 + e + lane] : kNone;
        const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)ev[0], (int)(e & 63));
        if (own && (int64_t)x < p) continue;
        bool there = false;
#pragma unroll
        for (int s = 0; s < SL; ++s) there |= id[s] == x;
        if (ballot64(there)) continue;
        if (nc < a.m) {
#pragma unroll
            for (int s = 0; s < SL; ++s)
                if (lane + 64 * s == nc) id[s] = x;
            ++nc;
            continue;
        }
        if (open < 0) {
            // keys, ranks and masks of the m slots
            open = a.m;
            load_row((uint32_t)p);
#pragma unroll
            for (int s = 0; s < SL; ++s)
                if (id[s] != kNone) key[s] = canon_delta(xrow, a.X + (size_t)id[s] * a.pitch, a.d);
            for (int r = 0; r < a.m; ++r) {
                const uint32_t ir = id_of(r);
                const double kr = key_of(r);
                load_row(ir);
#pragma unroll
                for (int s = 0; s < SL; ++s)
                    if (id[s] != kNone && kless(kr, ir, key[s], id[s])) {
                        ++rank[s];
                        const double dj = canon_delta(xrow, a.X + (size_t)id[s] * a.pitch, a.d);
                        if (!(key[s] < dj)) {
#pragma unroll
                            for (int t = 0; t < SL; ++t)
                                if (r >> 6 == t) out_by[s][t] |= 1ull << (r & 63);
                        }
                    }
            }
        }
        // distances of x to the slots, and to p in the free slot's lane
        load_row(x);
        double dj[SL];
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const bool here = lane + 64 * s == open;
            dj[s] = here || id[s] != kNone
                        ? canon_delta(xrow, a.X + (size_t)(here ? (uint32_t)p : id[s]) * a.pitch, a.d)
                        : 0.0;
        }
        double dx = __shfl(dj[0], open & 63);
        if constexpr (SL > 1) {
            const double w = __shfl(dj[SL - 1], open & 63);
            dx = open < 64 ? dx : w;
        }
        uint64_t ob[SL];
        uint32_t rx = 0;
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const bool used = id[s] != kNone;
            const bool before = used && kless(key[s], id[s], dx, x);
            ob[s] = ballot64(before && !(dx < dj[s]));
            rx += (uint32_t)__popcll(ballot64(before));
            if (used) {
                const bool by_x = !before && !(key[s] < dj[s]);
#pragma unroll
                for (int t = 0; t < SL; ++t)
                    if (open >> 6 == t) {
                        const uint64_t bit = 1ull << (open & 63);
                        out_by[s][t] = by_x ? out_by[s][t] | bit : out_by[s][t] & ~bit;
                    }
                if (!before) ++rank[s];
            }
        }
#pragma unroll
        for (int s = 0; s < SL; ++s)
            if (lane + 64 * s == open) {
                id[s] = x;
                key[s] = dx;
                rank[s] = rx;
#pragma unroll
                for (int t = 0; t < SL; ++t) out_by[s][t] = ob[t];
            }
        // who is kept
        uint64_t kept[SL] = {}, outm[SL] = {};
        bool undecided[SL];
#pragma unroll
        for (int s = 0; s < SL; ++s) undecided[s] = id[s] != kNone;
        for (;;) {
            bool k[SL], o[SL];
#pragma unroll
            for (int s = 0; s < SL; ++s) {
                uint64_t by_kept = 0, by_open = 0;
#pragma unroll
                for (int t = 0; t < SL; ++t) {
                    by_kept |= out_by[s][t] & kept[t];
                    by_open |= out_by[s][t] & ~outm[t];
                }
                o[s] = undecided[s] && by_kept != 0;
                k[s] = undecided[s] && by_open == 0;
                if (o[s] || k[s]) undecided[s] = false;
            }
            uint64_t settled = 0;
            bool any = false;
#pragma unroll
            for (int s = 0; s < SL; ++s) {
                const uint64_t km = ballot64(k[s]), om = ballot64(o[s]);
                kept[s] |= km;
                outm[s] |= om;
                settled |= km | om;
                any |= undecided[s];
            }
            if (ballot64(any) == 0 || settled == 0) break;  // (every round settles the lowest rank still open)
        }
        // the highest rank of those out, or of all
        bool none_out = true;
#pragma unroll
        for (int s = 0; s < SL; ++s) none_out &= outm[s] == 0;
        bool cand[SL];
#pragma unroll
        for (int s = 0; s < SL; ++s)
            cand[s] = id[s] != kNone && (none_out || ((outm[s] >> lane) & 1ull));
        for (int bit = 6; bit >= 0; --bit) {
            uint64_t any = 0;
#pragma unroll
            for (int s = 0; s < SL; ++s) any |= ballot64(cand[s] && ((rank[s] >> bit) & 1u));
            if (any) {
#pragma unroll
                for (int s = 0; s < SL; ++s) cand[s] = cand[s] && ((rank[s] >> bit) & 1u);
            }
        }
        uint32_t rd = 0;
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const uint64_t cm = ballot64(cand[s]);
            if (cm) {
                open = 64 * s + (int)__builtin_ctzll(cm);
                rd = (uint32_t)__builtin_amdgcn_readlane((int)rank[s], (int)__builtin_ctzll(cm));
            }
        }
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            if (lane + 64 * s == open)
                id[s] = kNone;
            else if (rank[s] > rd)
                --rank[s];
        }
    }
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        const int j = lane + 64 * s, to = open >= 0 && j > open ? j - 1 : j;
        if (id[s] != kNone) a.out[p * a.out_pitch + to] = id[s];
        if (j >= nc && j < a.out_pitch) a.out[p * a.out_pitch + j] = kNone;
    }
    if (lane == 0) a.out_n[p] = nc;
}

__global__ __launch_bounds__(256) void k_first_of_lists(const uint32_t *lists, int64_t nt, int Nq, uint32_t *out) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < nt; t += (int64_t)gridDim.x * blockDim.x)
        out[t] = lists[t * Nq];
}

// The nodes that selected each node: counts, then places (in any order).
__global__ __launch_bounds__(256) void k_count_events(const uint32_t *sel, const int32_t *sel_n, int64_t n, int m,
                                                     uint32_t *cnt) {
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x)
        for (int j = 0; j < sel_n[x]; ++j) atomicAdd(&cnt[sel[x * m + j]], 1u);
}

__global__ __launch_bounds__(256) void k_place_events(const uint32_t *sel, const int32_t *sel_n, int64_t n, int m,
                                                     const int64_t *off, uint32_t *cnt, uint32_t *src) {
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x)
        for (int j = 0; j < sel_n[x]; ++j) {
            const uint32_t t = sel[x * m + j];
            src[off[t] + (int64_t)atomicSub(&cnt[t], 1u) - 1] = (uint32_t)x;
        }
}

// Ascending order of the lists longer than 64 (shorter ones are sorted by the
// wavefront that replays them): a bitonic network whose comparators all point
// the same way, so that a length that is no power of two needs no padding.
__global__ __launch_bounds__(256) void k_sort_events(const int64_t *off, uint32_t *src, int64_t p0) {
    const int64_t p = p0 + blockIdx.x;
    const int64_t n = off[p + 1] - off[p];
    if (n <= 64) return;
    uint32_t *a = src + off[p];
    const uint32_t ne = (uint32_t)n;  // fewer than nodes
    int top = 7;
    while ((1u << top) < ne) ++top;
    for (int k = 1; k <= top; ++k)
        for (int j = k - 1; j >= 0; --j) {
            for (uint32_t i = threadIdx.x; i < 1u << (top - 1); i += blockDim.x) {
                // the lower element of pair i, and its partner: mirrored in its
                // block of 2^k at first, then 2^j apart
                const uint32_t lo = ((i >> j) << (j + 1)) | (i & ((1u << j) - 1u));
                const uint32_t hi = j == k - 1 ? lo ^ ((1u << k) - 1u) : lo + (1u << j);
                if (hi < ne && a[hi] < a[lo]) {
                    const uint32_t t = a[lo];
                    a[lo] = a[hi];
                    a[hi] = t;
                }
            }
            __syncthreads();
        }
}

__global__ __launch_bounds__(256) void k_zero32(uint32_t *p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// How far an FP32 sum of `steps` fused steps and additions per term may be
// from the exact one, as a share of the sum of magnitudes, with room for the
// rounding of that sum, of the bound itself and of the canonical sum.
float sum_bound(int d, int steps) {
    const double u = 1.0 / 16777216.0;
    return (float)((steps * u / (1.0 - steps * u) + (d + 1) * 0x1p-53) * (1.0 + 2.0 * steps * u) * 1.0001);
}

struct Dev {
    void *p = nullptr;
    Dev() = default;
    Dev(const Dev &) = delete;
    Dev &operator=(const Dev &) = delete;
    ~Dev() { release(); }
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr;
    }
    bool alloc(size_t bytes) {
        release();
        if (hipMalloc(&p, bytes ? bytes : 1) == hipSuccess) return true;
        p = nullptr;
        (void)hipGetLastError();  // callers may go on without it
        return false;
    }
    template <class T>
    T *as() const {
        return static_cast<T *>(p);
    }
};

// launch(first, count) over n workgroups, at most 2^18 at a time: a HIP grid
// holds fewer than 2^32 threads, which one workgroup of 256 per node passes at
// 2^24 nodes.  A launch of 2^18 is 32 rounds of workgroups or more, so its end
// costs little.
template <class F>
int in_grids(int64_t n, F &&launch) {
    constexpr int64_t most = 1 << 18;
    for (int64_t p0 = 0; p0 < n; p0 += most) {
        launch(p0, (unsigned)std::min(most, n - p0));
        RG_HIP(hipGetLastError());
    }
    return RG_OK;
}

unsigned blocks_for(int64_t items) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(65536, (items + 255) / 256)); }

}  // namespace

int launch_max_norm(const float *X, int64_t n, int32_t pitch, double *xmax2, hipStream_t stream) {
    hipLaunchKernelGGL(k_zero32, dim3(1), dim3(256), 0, stream, reinterpret_cast<uint32_t *>(xmax2), (int64_t)2);
    hipLaunchKernelGGL(k_max_norm, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(512, (n + 3) / 4))), dim3(256),
                       0, stream, X, n, pitch, xmax2);
    RG_HIP(hipGetLastError());
    return RG_OK;
}

int launch_canon_search(const float *X, int64_t n, int32_t d, int32_t pitch, const uint32_t *adj, int32_t ell,
                        uint32_t entry, int32_t L, int64_t x0, int64_t count, const double *xmax2, uint32_t *ids,
                        double *dists, int32_t *counts, hipStream_t stream) {
    if (count == 0) return RG_OK;
    if (L < 1 || L > kMaxL || ell > kMaxEll || pitch % 4 != 0) {
        set_error("canon search: unsupported L, row width or pitch");
        return RG_EINVAL;
    }
    CanonArgs a{};
    a.X = X;
    a.adj = adj;
    a.out_ids = ids;
    a.out_d = dists;
    a.out_n = counts;
    a.x0 = x0;
    a.count = count;
    a.d = d;
    a.pitch = pitch;
    a.ell = ell;
    a.L = L;
    a.cand = ell <= 64 ? 64 : 128;
    a.entry = entry;
    a.xmax2 = xmax2;
    // both sums err by at most d + 8 roundings' worth of sum |q_i x_i|
    a.gam = 2.0 * (d + 8) * 0x1p-53 * 1.01;
    a.gam32 = sum_bound(d, (pitch + 63) / 64 * 4 + 6);
    // the table bounds work, not results: sets of 16-bit entries in 2 KB, or
    // ids in 8 KB
    SearchArgs t{};
    t.n_rows = n;
    t.ell = ell;
    set_table(t, 9);
    auto run = [&](auto kernel) -> int {
        const size_t lds = canon_lds_bytes(a);
        if (lds > (64u << 10))
            RG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(kernel, dim3((unsigned)count), dim3(64), lds, stream, a);
        RG_HIP(hipGetLastError());
        return RG_OK;
    };
    if (t.sets) {
        a.hash_bits = t.hash_bits;
        a.id_bits = t.id_bits;
        a.redo = 1;
        const int rc = run(k_canon_search<VisitSets, true>);
        return rc ? rc : run(k_canon_search<VisitSets, false>);
    }
    a.hash_bits = 11;
    return run(k_canon_search<VisitLds, false>);
}

namespace {

// The nodes that selected each node, off (n + 1) and src, ascending where they
// are more than 64.  selected() is called once the selections are done.
template <class F>
int selected_by(const SelectArgs &s, int64_t n, Dev &d_off, Dev &d_src, hipStream_t st, F &&selected) {
    Dev d_cnt;
    if (!d_cnt.alloc(sizeof(uint32_t) * n) || !d_off.alloc(sizeof(int64_t) * (n + 1))) {
        set_error("build: out of memory for reverse updates");
        return RG_ENOMEM;
    }
    hipLaunchKernelGGL(k_zero32, dim3(blocks_for(n)), dim3(256), 0, st, d_cnt.as<uint32_t>(), n);
    hipLaunchKernelGGL(k_count_events, dim3(blocks_for(n)), dim3(256), 0, st, s.sel_ids, s.sel_n, n, s.m,
                       d_cnt.as<uint32_t>());
    RG_HIP(hipGetLastError());
    std::vector<uint32_t> cnt((size_t)n);
    RG_HIP(hipMemcpyAsync(cnt.data(), d_cnt.p, sizeof(uint32_t) * n, hipMemcpyDeviceToHost, st));
    RG_HIP(hipStreamSynchronize(st));
    selected();
    std::vector<int64_t> off((size_t)n + 1, 0);
    for (int64_t i = 0; i < n; ++i) off[i + 1] = off[i] + cnt[i];
    if (!d_src.alloc(sizeof(uint32_t) * (size_t)off[n])) {
        set_error("build: out of memory for reverse updates");
        return RG_ENOMEM;
    }
    RG_HIP(hipMemcpyAsync(d_off.p, off.data(), sizeof(int64_t) * (n + 1), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_place_events, dim3(blocks_for(n)), dim3(256), 0, st, s.sel_ids, s.sel_n, n, s.m,
                       d_off.as<int64_t>(), d_cnt.as<uint32_t>(), d_src.as<uint32_t>());
    RG_HIP(hipGetLastError());
    const int rc = in_grids(n, [&](int64_t p0, unsigned cnt) {
        hipLaunchKernelGGL(k_sort_events, dim3(cnt), dim3(256), 0, st, d_off.as<int64_t>(), d_src.as<uint32_t>(), p0);
    });
    if (rc) return rc;
    // before the counts and offsets go
    RG_HIP(hipStreamSynchronize(st));
    return RG_OK;
}

// LDS of k_canon_select without and with the kept rows
size_t select_lds(const GpuCtx &gpu, int m, bool *rows) {
    const size_t ids = 2 * (size_t)((m + 3) & ~3) * sizeof(uint32_t), kept = (size_t)m * gpu.pitch * sizeof(float);
    *rows = ids + kept <= (48u << 10);
    return ids + (*rows ? kept : 0);
}

}  // namespace

int canon_pivots(const GpuCtx &gpu, int64_t nt, int32_t Nq, uint32_t *out) {
    Dev d_out;
    if (!d_out.alloc(sizeof(uint32_t) * nt)) {
        set_error("build: out of memory for the pivots");
        return RG_ENOMEM;
    }
    hipLaunchKernelGGL(k_first_of_lists, dim3(blocks_for(nt)), dim3(256), 0, gpu.stream, gpu.lists, nt, Nq,
                       d_out.as<uint32_t>());
    RG_HIP(hipGetLastError());
    RG_HIP(hipMemcpyAsync(out, d_out.p, sizeof(uint32_t) * nt, hipMemcpyDeviceToHost, gpu.stream));
    RG_HIP(hipStreamSynchronize(gpu.stream));
    return RG_OK;
}

int canon_lists(const GpuCtx &gpu, int64_t words, uint32_t *out) {
    RG_HIP(hipMemcpyAsync(out, gpu.lists, sizeof(uint32_t) * words, hipMemcpyDeviceToHost, gpu.stream));
    RG_HIP(hipStreamSynchronize(gpu.stream));
    return RG_OK;
}

// Pivots in batches (the candidates are the large buffers).  RG_ENOMEM: a
// buffer did not fit, nothing was written.
int canon_project(const GpuCtx &gpu, int64_t n, int32_t d, int64_t nt, int32_t Nq, const std::vector<int64_t> &boff,
                  const std::vector<uint32_t> &bidx, int32_t L, int32_t m, int32_t ell, std::vector<uint32_t> *pj,
                  std::vector<int32_t> *pj_n) {
    hipStream_t st = gpu.stream;
    if (!gpu.lists) return RG_ENOMEM;
    if (L > kMaxL || m < 1 || m >= kMaxEll || Nq > 512 || ell < m) return RG_ENOMEM;  // no room in the kernels
    std::vector<uint32_t> piv;
    for (int64_t x = 0; x < n; ++x)
        if (boff[x] != boff[x + 1]) piv.push_back((uint32_t)x);
    const int64_t np = (int64_t)piv.size(), B = std::max<int64_t>(1, std::min<int64_t>(np, 1 << 15));
    CandArgs c{};
    c.cap = 256;
    while (c.cap < L + Nq) c.cap *= 2;
    c.hash_bits = 1;
    while ((1 << c.hash_bits) < 2 * c.cap) ++c.hash_bits;
    const size_t cand_lds = (size_t)gpu.pitch * 4 + (size_t)c.cap * 4 + ((size_t)4 << c.hash_bits);
    if (cand_lds > (64u << 10) || (size_t)gpu.pitch * 4 > (64u << 10)) return RG_ENOMEM;
    Dev d_piv, d_boff, d_bidx, d_c, d_cd, d_cn, d_sid, d_sd, d_sn, d_out, d_on, d_off, d_src;
    if (!d_piv.alloc(sizeof(uint32_t) * np) || !d_boff.alloc(sizeof(int64_t) * (n + 1)) ||
        !d_bidx.alloc(sizeof(uint32_t) * nt) || !d_c.alloc(sizeof(uint32_t) * B * L) ||
        !d_cd.alloc(sizeof(double) * B * L) || !d_cn.alloc(sizeof(int32_t) * B) ||
        !d_sid.alloc(sizeof(uint32_t) * n * m) || !d_sd.alloc(sizeof(double) * n * m) ||
        !d_sn.alloc(sizeof(int32_t) * n) || !d_out.alloc(sizeof(uint32_t) * n * ell) ||
        !d_on.alloc(sizeof(int32_t) * n))
        return RG_ENOMEM;
    RG_HIP(hipMemcpyAsync(d_piv.p, piv.data(), sizeof(uint32_t) * np, hipMemcpyHostToDevice, st));
    RG_HIP(hipMemcpyAsync(d_boff.p, boff.data(), sizeof(int64_t) * (n + 1), hipMemcpyHostToDevice, st));
    RG_HIP(hipMemcpyAsync(d_bidx.p, bidx.data(), sizeof(uint32_t) * nt, hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_zero32, dim3(blocks_for(n)), dim3(256), 0, st, d_sn.as<uint32_t>(), n);
    c.X = gpu.X;
    c.d = d;
    c.pitch = gpu.pitch;
    c.lists = gpu.lists;
    c.boff = d_boff.as<int64_t>();
    c.bidx = d_bidx.as<uint32_t>();
    c.Nq = Nq;
    c.L = L;
    c.ids = d_c.as<uint32_t>();
    c.dists = d_cd.as<double>();
    c.counts = d_cn.as<int32_t>();
    SelectArgs s{};
    s.X = gpu.X;
    s.d = d;
    s.pitch = gpu.pitch;
    s.ids = c.ids;
    s.dists = c.dists;
    s.counts = c.counts;
    s.L = L;
    s.m = m;
    s.sel_ids = d_sid.as<uint32_t>();
    s.sel_d = d_sd.as<double>();
    s.sel_n = d_sn.as<int32_t>();
    s.gam = sum_bound(d, gpu.pitch + 8);
    s.floor2 = (float)gpu.pitch * 1.2e-38f;
    bool rows;
    const size_t lds = select_lds(gpu, m, &rows);
    auto k_select = rows ? k_canon_select<true, true> : k_canon_select<false, true>;
    for (int64_t b0 = 0; b0 < np; b0 += B) {
        const unsigned cnt = (unsigned)std::min(B, np - b0);
        c.nodes = s.nodes = d_piv.as<uint32_t>() + b0;
        hipLaunchKernelGGL(k_project_cands, dim3(cnt), dim3(64), cand_lds, st, c);
        hipLaunchKernelGGL(k_select, dim3(cnt), dim3(64), lds, st, s);
        RG_HIP(hipGetLastError());
    }
    int rc = selected_by(s, n, d_off, d_src, st, [] {});
    if (rc) return rc;
    ReplayArgs r{};
    r.X = gpu.X;
    r.d = d;
    r.pitch = gpu.pitch;
    r.m = m;
    r.sel_ids = s.sel_ids;
    r.sel_d = s.sel_d;
    r.sel_n = s.sel_n;
    r.off = d_off.as<int64_t>();
    r.src = d_src.as<uint32_t>();
    r.out = d_out.as<uint32_t>();
    r.out_n = d_on.as<int32_t>();
    r.out_pitch = ell;
    r.boff = c.boff;
    auto k_fill = m < 64 ? k_replay_fill<1> : k_replay_fill<2>;
    rc = in_grids(n, [&](int64_t p0, unsigned cnt) {
        r.p0 = p0;
        hipLaunchKernelGGL(k_fill, dim3(cnt), dim3(64), (size_t)gpu.pitch * 4, st, r);
    });
    if (rc) return rc;
    pj->resize((size_t)n * ell);
    pj_n->resize((size_t)n);
    RG_HIP(hipMemcpyAsync(pj->data(), d_out.p, sizeof(uint32_t) * n * ell, hipMemcpyDeviceToHost, st));
    RG_HIP(hipMemcpyAsync(pj_n->data(), d_on.p, sizeof(int32_t) * n, hipMemcpyDeviceToHost, st));
    RG_HIP(hipStreamSynchronize(st));
    return RG_OK;
}

// The searches and selections run in batches (their queues are the large
// buffers); selections, reverse updates and the lists stay on the device.
// Where those of all nodes do not fit, the selections of each batch go to the
// host.
int canon_enhance(const GpuCtx &gpu, int64_t n, int32_t d, const std::vector<uint32_t> &adj, int32_t ell,
                  uint32_t entry, int32_t L, int32_t m, int32_t head_len, std::vector<uint32_t> *ce,
                  std::vector<int32_t> *ce_n, Selections *sel, uint32_t *head, int32_t *head_n, double *t_search) {
    if (m < 1 || m >= kMaxEll || L < 1) {
        set_error("build: bad list bound");
        return RG_EINVAL;
    }
    using Clock = std::chrono::steady_clock;
    const auto t0 = Clock::now();
    const bool log = std::getenv("RG_LOG") != nullptr;
    hipStream_t st = gpu.stream;
    const int64_t B = std::min<int64_t>(n, 1 << 15);
    Dev d_adj, d_q, d_qd, d_qn, d_sid, d_sd, d_sn, d_hd, d_hn, d_max;
    // the selections and first candidates of this many nodes
    auto room_for = [&](int64_t rows) {
        if (d_sid.alloc(sizeof(uint32_t) * rows * m) && d_sd.alloc(sizeof(double) * rows * m) &&
            d_sn.alloc(sizeof(int32_t) * rows) && d_hd.alloc(sizeof(uint32_t) * rows * head_len) &&
            d_hn.alloc(sizeof(int32_t) * rows))
            return true;
        for (Dev *b : {&d_sid, &d_sd, &d_sn, &d_hd, &d_hn}) b->release();
        return false;
    };
    if (!d_max.alloc(8) || !d_adj.alloc(sizeof(uint32_t) * adj.size()) || !d_q.alloc(sizeof(uint32_t) * B * L) ||
        !d_qd.alloc(sizeof(double) * B * L) || !d_qn.alloc(sizeof(int32_t) * B)) {
        set_error("build: out of memory for enhancement searches");
        return RG_ENOMEM;
    }
    const bool whole = room_for(n);
    if (!whole && !room_for(B)) {
        set_error("build: out of memory for enhancement searches");
        return RG_ENOMEM;
    }
    // nodes x0 .. x0 + cnt of what room_for holds, to the host
    auto selections_to_host = [&](int64_t x0, int64_t cnt) -> int {
        if (sel->counts.empty()) {
            sel->ids.resize((size_t)n * m);
            sel->dists.resize((size_t)n * m);
            sel->counts.resize((size_t)n);
        }
        RG_HIP(hipMemcpyAsync(sel->ids.data() + x0 * m, d_sid.p, sizeof(uint32_t) * cnt * m, hipMemcpyDeviceToHost, st));
        RG_HIP(hipMemcpyAsync(sel->dists.data() + x0 * m, d_sd.p, sizeof(double) * cnt * m, hipMemcpyDeviceToHost, st));
        RG_HIP(hipMemcpyAsync(sel->counts.data() + x0, d_sn.p, sizeof(int32_t) * cnt, hipMemcpyDeviceToHost, st));
        RG_HIP(hipStreamSynchronize(st));
        return RG_OK;
    };
    auto head_to_host = [&](int64_t x0, int64_t cnt) -> int {
        RG_HIP(hipMemcpyAsync(head + x0 * head_len, d_hd.p, sizeof(uint32_t) * cnt * head_len, hipMemcpyDeviceToHost, st));
        RG_HIP(hipMemcpyAsync(head_n + x0, d_hn.p, sizeof(int32_t) * cnt, hipMemcpyDeviceToHost, st));
        return RG_OK;
    };
    RG_HIP(hipMemcpyAsync(d_adj.p, adj.data(), sizeof(uint32_t) * adj.size(), hipMemcpyHostToDevice, st));
    int rc = launch_max_norm(gpu.X, n, gpu.pitch, d_max.as<double>(), st);
    if (rc) return rc;
    SelectArgs s{};
    s.X = gpu.X;
    s.d = d;
    s.pitch = gpu.pitch;
    s.ids = d_q.as<uint32_t>();
    s.dists = d_qd.as<double>();
    s.counts = d_qn.as<int32_t>();
    s.L = L;
    s.m = m;
    s.head_len = head_len;
    s.sel_ids = d_sid.as<uint32_t>();
    s.sel_d = d_sd.as<double>();
    s.sel_n = d_sn.as<int32_t>();
    // a lane's chain over the whole row, and the norms' own rounding
    s.gam = sum_bound(d, gpu.pitch + 8);
    s.floor2 = (float)gpu.pitch * 1.2e-38f;
    bool kept_in_lds;
    const size_t lds = select_lds(gpu, m, &kept_in_lds);
    auto k_select = kept_in_lds ? k_canon_select<true, false> : k_canon_select<false, false>;
    const int64_t step = std::max<int64_t>(B, (n / 10 + B - 1) / B * B);
    for (int64_t x0 = 0; x0 < n; x0 += B) {
        const int64_t cnt = std::min(B, n - x0);
        rc = launch_canon_search(gpu.X, n, d, gpu.pitch, d_adj.as<uint32_t>(), ell, entry, L, x0, cnt,
                                 d_max.as<double>(), d_q.as<uint32_t>(), d_qd.as<double>(), d_qn.as<int32_t>(), st);
        if (rc) return rc;
        s.x0 = x0;
        s.sel0 = whole ? 0 : x0;
        s.head = d_hd.as<uint32_t>() + (x0 - s.sel0) * head_len;
        s.head_n = d_hn.as<int32_t>() + (x0 - s.sel0);
        hipLaunchKernelGGL(k_select, dim3((unsigned)cnt), dim3(64), lds, st, s);
        RG_HIP(hipGetLastError());
        if (!whole) {
            rc = head_to_host(x0, cnt);
            if (!rc) rc = selections_to_host(x0, cnt);
            if (rc) return rc;
        }
        if (log && ((x0 + cnt) % step == 0 || x0 + cnt == n)) {  // progress (waits for the batches)
            RG_HIP(hipStreamSynchronize(st));
            std::fprintf(stderr, "[rg] enhancement searches %lld / %lld nodes\n", (long long)(x0 + cnt), (long long)n);
        }
    }
    if (!whole) {
        *t_search = std::chrono::duration<double>(Clock::now() - t0).count();
        return RG_OK;
    }
    rc = head_to_host(0, n);
    if (rc) return rc;
    Dev d_off, d_src, d_out, d_on;
    rc = selected_by(s, n, d_off, d_src, st, [&] { *t_search = std::chrono::duration<double>(Clock::now() - t0).count(); });
    if (!rc && (!d_out.alloc(sizeof(uint32_t) * n * m) || !d_on.alloc(sizeof(int32_t) * n))) rc = RG_ENOMEM;
    if (rc == RG_ENOMEM) {
        rc = selections_to_host(0, n);
        *t_search = std::chrono::duration<double>(Clock::now() - t0).count();
        return rc;
    }
    if (rc) return rc;
    ReplayArgs r{};
    r.X = gpu.X;
    r.d = d;
    r.pitch = gpu.pitch;
    r.m = m;
    r.sel_ids = s.sel_ids;
    r.sel_d = s.sel_d;
    r.sel_n = s.sel_n;
    r.off = d_off.as<int64_t>();
    r.src = d_src.as<uint32_t>();
    r.out = d_out.as<uint32_t>();
    r.out_n = d_on.as<int32_t>();
    r.out_pitch = m;
    rc = in_grids(n, [&](int64_t p0, unsigned cnt) {
        r.p0 = p0;
        hipLaunchKernelGGL(k_replay, dim3(cnt), dim3(64), (size_t)gpu.pitch * 4 + (size_t)(m + 1) * 12 + 8, st, r);
    });
    if (rc) return rc;
    ce->resize((size_t)n * m);
    ce_n->resize((size_t)n);
    RG_HIP(hipMemcpyAsync(ce->data(), d_out.p, sizeof(uint32_t) * n * m, hipMemcpyDeviceToHost, st));
    RG_HIP(hipMemcpyAsync(ce_n->data(), d_on.p, sizeof(int32_t) * n, hipMemcpyDeviceToHost, st));
    RG_HIP(hipStreamSynchronize(st));
    if (log)
        std::fprintf(stderr, "[rg] enhancement on the device: searches and selections %.3f s, reverse updates %.3f s\n",
                     *t_search, std::chrono::duration<double>(Clock::now() - t0).count() - *t_search);
    return RG_OK;
}

}  // namespace rg
