// Batched beam search over the RoarGraph index (Sec. 4.3), one 64-lane
// wavefront (= one workgroup) per query on gfx950.
//
// Per query, in LDS:
//   * the queue: the best L_eff (delta, id) pairs seen, sorted ascending, the
//     id's top bit marking "expanded";
//   * a visited table that forgets: sets of 16-bit entries that drop their
//     oldest, or an open-addressing table of node ids that is cleared when it
//     passes half load.  A forgotten node seen again is scored again and
//     dropped at the merge if it is already queued.  Because the queue's last
//     key only decreases once the queue is full, a forgotten node that was
//     rejected or evicted is rejected again, so forgetting changes only the
//     work done, never the result;
//   * the candidate batch of the current expansion.
// Per expansion: pick the first unexpanded queue entry, read its adjacency
// row (ELL, one id per lane; or a CSR row of any length, 128 ids at a time),
// filter through the visited set, gather the
// new neighbours' rows (G lanes per row, 16-byte loads, R rows per group in
// flight), reduce the FP32 dot products inside each G-lane group (DPP lane
// moves), order the survivors, and merge the entries that beat the queue's
// last key.  The search stops when every queue entry is expanded.
//
// Rows are read in 16-byte chunks of EPC elements (4 FP32, 8 BF16 or 16
// E4M3 values).  Lane j of a group accumulates, with fused multiply-adds in
// order, the elements of chunks c = j, j+G, j+2G, ...; then the G partial
// sums are added by a log2(G)-level xor tree (times the row's scale for
// E4M3).  A distance is therefore a fixed function of (query, row)
// whichever group computes it.
#include "rg_internal.h"
#include "queue_ops.h"
#include "wave_ops.h"

#include <climits>
#include <mutex>

// The build compiles this file in parts, side by side: per storage form
// (RG_BEAM_STORAGE = RG_STORE_*) the search with a visited table of ids
// (RG_BEAM_PART 0) or of 16-bit entries (1), the persistent search and the
// serving step (2) and the search of few queries (3), and once without them
// the dispatch and the rest.
namespace rg {

// the launches of one storage form
template <int ST>
struct BeamOps {
    static int search_ids(const SearchArgs &a, hipStream_t s);   // visited table of ids
    static int search_sets(const SearchArgs &a, hipStream_t s);  // visited table of 16-bit entries
    static int search_bits(const SearchArgs &a, hipStream_t s);  // one bit per node (FP32 rows)
    static int ids_occupancy(const SearchArgs &a);
    static int sets_occupancy(const SearchArgs &a);
    static int wide(const SearchArgs &a, hipStream_t s);         // several wavefronts per query
    static int persistent(const SearchArgs &a, hipStream_t s);
    static int persistent_occupancy(const SearchArgs &a);
    static int serve_step(const SlotArgs &a, hipStream_t s);
    static int serve_occupancy(const SlotArgs &a);
};

#ifdef RG_BEAM_STORAGE
namespace {


struct Lds {
    float *qs;      // the query, zero padded to the row pitch
    float *qd;
    uint32_t *qi;
    float *cd;
    uint32_t *ci;
    float *sd;
    uint32_t *si;
    int32_t *slb;
    uint32_t *htab;
};

// cand = the candidate-batch capacity of this launch (64 or 128)
__device__ __forceinline__ Lds carve(unsigned char *p, int Leff, int pitch, int cand) {
    Lds s;
    s.qs = reinterpret_cast<float *>(p);
    s.qd = s.qs + pitch;
    s.qi = reinterpret_cast<uint32_t *>(s.qd + Leff);
    s.cd = reinterpret_cast<float *>(s.qi + Leff);
    s.ci = reinterpret_cast<uint32_t *>(s.cd + cand);
    s.sd = reinterpret_cast<float *>(s.ci + cand);
    s.si = reinterpret_cast<uint32_t *>(s.sd + cand);
    s.slb = reinterpret_cast<int32_t *>(s.si + cand);
    // 8-byte aligned: qpad and cand are even and L_eff counts twice
    s.htab = reinterpret_cast<uint32_t *>(s.slb + cand);
    return s;
}

typedef float f32x2 __attribute__((ext_vector_type(2)));


// Storage formats: 16-byte chunks of EPC elements.
template <int ST>
struct Fmt {
    static constexpr int EPC = ST == RG_STORE_FP32 ? 4 : ST == RG_STORE_BF16 ? 8 : 16;
};

// Lane shape per dimension class (d <= 64, 128, 224, 256, 512, 1024) and
// storage: G lanes per row and NCH chunks per lane, G * NCH * EPC >= d; R rows
// per group whose loads are in flight together.
constexpr int kClassMaxD[6] = {64, 128, 224, 256, 512, 1024};
constexpr int shape_g(int st, int cls) {
    constexpr int g32[6] = {16, 16, 8, 16, 16, 32}, g16[6] = {8, 16, 8, 8, 16, 32}, g8[6] = {4, 8, 8, 8, 16, 32};
    return st == RG_STORE_FP32 ? g32[cls] : st == RG_STORE_BF16 ? g16[cls] : g8[cls];
}
// E4M3 rows also hold their scale after the codes (up to d + 7 bytes), so
// each E4M3 shape covers the class's largest d plus 8 bytes.
constexpr int shape_nch(int st, int cls) {
    constexpr int n32[6] = {1, 2, 7, 4, 8, 8}, n16[6] = {1, 1, 4, 4, 4, 4}, n8[6] = {2, 2, 2, 3, 3, 3};
    return st == RG_STORE_FP32 ? n32[cls] : st == RG_STORE_BF16 ? n16[cls] : n8[cls];
}
// R: what the registers hold beside the chunks; a wavefront waits once per
// round of rows.  Two rows -> R, ms for 10,000 queries at the same visited
// set: FP32 1M x 64 L = 200 4.86 -> 4.55, 1M x 96 L = 100 2.95 -> 2.84 (eight
// rows 3.12), 1M x 250 L = 200 12.96 -> 12.77; BF16 1M x 64 L = 200 3.86 ->
// 3.58, 1M x 100 L = 200 4.74 -> 4.46 (four rows 4.58), 1M x 200 L = 409
// unchanged by three; E4M3 1M x 256 L = 300 11.0 -> 10.6 with three.  With four
// the BF16 and E4M3 shapes of d > 256 need the registers of 4 wavefronts per
// SIMD instead of 5 and are faster all the same: E4M3 2M x 512 L = 409 33.6 ->
// 29.4, 1M x 512 L = 150 11.9 -> 11.1; BF16 1M x 512 L = 805 55.2 -> 54.1.  At
// d <= 256 the fifth wavefront is worth more (E4M3 1M x 256 L = 409, 1 KB:
// 14.7 -> 17.8).
constexpr int shape_r(int st, int cls) {
    constexpr int r32[6] = {8, 4, 2, 4, 2, 2}, r16[6] = {8, 8, 2, 2, 4, 4}, r8[6] = {4, 4, 4, 3, 4, 4};
    return st == RG_STORE_FP32 ? r32[cls] : st == RG_STORE_BF16 ? r16[cls] : r8[cls];
}

// Copy the query into LDS, zero padded to qpad (every element a row chunk
// can reach, so bytes past d meet a zero).
__device__ __forceinline__ void load_query(const float *q, int d, int qpad, float *qs) {
    for (int i = lane_id(); i < qpad; i += 64) qs[i] = i < d ? q[i] : 0.f;
    wave_sync();
}

// Chunks of a stored row the search reads: the d elements, and for E4M3 rows
// the scale that follows the codes.
template <int ST>
__device__ __forceinline__ int row_chunk_count(int d) {
    if constexpr (ST == RG_STORE_FP8E4M3) return (((d + 3) & ~3) + 4 + 15) >> 4;
    return (d + Fmt<ST>::EPC - 1) / Fmt<ST>::EPC;
}

template <int ST>
__device__ __forceinline__ const uint4 *row_chunks(const SearchArgs &a, uint32_t u) {
    if constexpr (ST == RG_STORE_FP32) return reinterpret_cast<const uint4 *>(a.base + (size_t)u * a.pitch);
    if constexpr (ST == RG_STORE_BF16) return reinterpret_cast<const uint4 *>(a.base_bf16 + (size_t)u * a.pitch);
    return reinterpret_cast<const uint4 *>(a.base_fp8 + (size_t)u * a.pitch8);
}

// acc += q . chunk c, in element order; q is read from LDS
template <int ST>
__device__ __forceinline__ float fma_chunk(const float *qs, int c, uint4 x, float acc) {
    constexpr int EPC = Fmt<ST>::EPC;
    const float4 *q4 = reinterpret_cast<const float4 *>(qs + c * EPC);
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
    if constexpr (ST == RG_STORE_FP32) {
        const float4 q = q4[0];
        acc = fmaf(q.x, __uint_as_float(w[0]), acc);
        acc = fmaf(q.y, __uint_as_float(w[1]), acc);
        acc = fmaf(q.z, __uint_as_float(w[2]), acc);
        acc = fmaf(q.w, __uint_as_float(w[3]), acc);
    } else if constexpr (ST == RG_STORE_BF16) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float4 q = q4[i];
            acc = fmaf(q.x, __uint_as_float(w[2 * i] << 16), acc);
            acc = fmaf(q.y, __uint_as_float(w[2 * i] & 0xFFFF0000u), acc);
            acc = fmaf(q.z, __uint_as_float(w[2 * i + 1] << 16), acc);
            acc = fmaf(q.w, __uint_as_float(w[2 * i + 1] & 0xFFFF0000u), acc);
        }
    } else {
        // bytes at and past d (the scale, padding) decode to finite values and
        // meet zero query elements; the scale is taken separately
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // gfx950 converts OCP E4M3 pairs exactly (every code is a float)
            const float4 q = q4[i];
            const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[i], false);
            const f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[i], true);
            acc = fmaf(q.x, lo[0], acc);
            acc = fmaf(q.y, lo[1], acc);
            acc = fmaf(q.z, hi[0], acc);
            acc = fmaf(q.w, hi[1], acc);
        }
    }
    return acc;
}

// This lane's partial dot products with rows u[0..R) (kNone -> 0); all loads
// are issued before the first multiply.
// sc[r] receives the E4M3 row scale in the lane whose chunk holds it (0
// elsewhere), so a group sum yields it.
template <int ST, int G, int NCH, int R>
__device__ __forceinline__ void dot_rows(const SearchArgs &a, const uint32_t (&u)[R], const float *qs, int nch,
                                         float (&acc)[R], float (&sc)[R]) {
    const int j = lane_id() % G;
    uint4 raw[R][NCH];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint4 *row = row_chunks<ST>(a, u[r] != kNone ? u[r] : 0u);
#pragma unroll
        for (int t = 0; t < NCH; ++t) {
            const int c = j + G * t;
            raw[r][t] = (u[r] != kNone && c < nch) ? row[c] : make_uint4(0u, 0u, 0u, 0u);
        }
    }
    const int s_off = (a.d + 3) & ~3, s_chunk = s_off >> 4, s_word = (s_off & 15) >> 2;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        acc[r] = 0.f;
        sc[r] = 0.f;
#pragma unroll
        for (int t = 0; t < NCH; ++t) {
            const int c = j + G * t;
            if (c < nch) acc[r] = fma_chunk<ST>(qs, c, raw[r][t], acc[r]);
            if constexpr (ST == RG_STORE_FP8E4M3) {
                if (c == s_chunk) {
                    const uint32_t w = s_word == 0 ? raw[r][t].x : s_word == 1 ? raw[r][t].y
                                     : s_word == 2 ? raw[r][t].z : raw[r][t].w;
                    sc[r] = __uint_as_float(w);
                }
            }
        }
    }
}

// delta of this group's row from its group-summed dot product (and, for
// E4M3, the row's power-of-two scale: the product is exact).  A NaN would have
// no place in the queue's order (every merge would put it elsewhere): it counts
// as +inf, behind all that are nearer, and restore_nans returns it.
template <int ST>
__device__ __forceinline__ float finish_delta(float sum, float scale) {
    // one instruction with the sign: v_min_f32 returns the operand that is a number
    return __builtin_fminf(ST == RG_STORE_FP8E4M3 ? -(scale * sum) : -sum, __builtin_inff());
}

// Score ids[0..cnt) (LDS) into dout[0..cnt) (LDS); R rows per group in flight.
template <int ST, int G, int NCH, int R>
__device__ __forceinline__ void score_batch(const SearchArgs &a, const float *qs, int nch, const uint32_t *ids,
                                            uint32_t idmask, float *dout, int cnt) {
    constexpr int NG = 64 / G;
    const int g = lane_id() / G, j = lane_id() % G;
    for (int p = 0; p < cnt; p += NG * R) {
        uint32_t u[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int sl = p + r * NG + g;
            u[r] = sl < cnt ? (ids[sl] & idmask) : kNone;
        }
        float acc[R], sc[R];
        dot_rows<ST, G, NCH, R>(a, u, qs, nch, acc, sc);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            acc[r] = group_sum<G>(acc[r]);
            if constexpr (ST == RG_STORE_FP8E4M3) sc[r] = group_sum<G>(sc[r]);
            acc[r] = finish_delta<ST>(acc[r], sc[r]);
        }
        if (j == 0) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int sl = p + r * NG + g;
                if (sl < cnt) dout[sl] = acc[r];
            }
        }
    }
}

// Exact visited set of a small base: one bit per node in LDS, 32 per
// word of the table.
struct VisitBits {
    uint32_t *bits;
    int words;
    __device__ __forceinline__ VisitBits(uint32_t *t, int hash_bits, int) : bits(t), words(1 << hash_bits) {}
    __device__ __forceinline__ void clear() {
        for (int i = lane_id(); i < words; i += 64) bits[i] = 0u;
    }
    __device__ __forceinline__ void mark_entry(uint32_t u) { (void)insert(u); }
    __device__ __forceinline__ void begin_hop(int) {}
    __device__ __forceinline__ bool insert(uint32_t u) {
        const uint32_t bit = 1u << (u & 31u);
        return (atomicOr(&bits[u >> 5], bit) & bit) == 0u;
    }
    __device__ __forceinline__ void added(int) {}
};

// Exact visited set: one bit per base node in device memory, owned by the
// workgroup for the query it is running; test-and-set with vector atomics.
struct VisitBitmap {
    uint32_t *bm;
    int64_t words;  // multiple of 4
    __device__ __forceinline__ void clear() {
        uint4 *b4 = reinterpret_cast<uint4 *>(bm);
        const uint4 z = make_uint4(0u, 0u, 0u, 0u);
        for (int64_t i = lane_id(); i < (words >> 2); i += 64) b4[i] = z;
        __threadfence();
    }
    __device__ __forceinline__ void mark_entry(uint32_t u) { atomicOr(&bm[u >> 5], 1u << (u & 31u)); }
    __device__ __forceinline__ void begin_hop(int) {}
    __device__ __forceinline__ bool insert(uint32_t u) {
        const uint32_t bit = 1u << (u & 31u);
        return (atomicOr(&bm[u >> 5], bit) & bit) == 0u;
    }
    __device__ __forceinline__ void added(int) {}
};

// Expansions until done or `budget` expansions were made; the queue holds
// up to 64 * QR entries.
template <int ST, int CLS, int QR, class VIS>
__device__ __forceinline__ void run_search(const SearchArgs &a, const Lds &s, VIS &vis,
                                           int &qn, int &ptr, uint32_t &hops, uint32_t &evals, int budget,
                                           bool &done) {
    constexpr int G = shape_g(ST, CLS), NCH = shape_nch(ST, CLS), R = shape_r(ST, CLS);
    const int lane = lane_id();
    const int Leff = a.Leff, ell = a.ell, nch = row_chunk_count<ST>(a.d);
    done = false;
    for (; budget > 0; --budget) {
        int sel = -1;
        for (int b = ptr; b < qn; b += 64) {
            const int i = b + lane;
            const bool un = i < qn && !(s.qi[i] & kExpanded);
            const uint64_t m = ballot64(un);
            if (m) {
                sel = b + (int)__builtin_ctzll(m);
                break;
            }
        }
        if (sel < 0) {
            done = true;
            break;
        }
        ptr = sel;
        const uint32_t v = s.qi[sel];
        wave_sync();
        if (lane == 0) s.qi[sel] = v | kExpanded;
        ++hops;
        // ELL row (width ell), or a CSR row of any length taken a.cand ids
        // at a time; each chunk is scored and merged before the next, which
        // ends in the same queue as one merge of the whole row.
        int64_t row = (int64_t)v * ell;
        int deg = ell;
        if (a.adj_off) {
            row = a.adj_off[v];
            deg = (int)(a.adj_off[v + 1] - row);
        }
        for (int c0 = 0; c0 < deg; c0 += a.cand) {
            const int cl = min(a.cand, deg - c0);
            const uint32_t *ids = a.adj + row + c0;
            vis.begin_hop(cl);
            const uint32_t r0 = lane < cl ? ids[lane] : kNone;
            const uint32_t r1 = lane + 64 < cl ? ids[lane + 64] : kNone;
            int nnew = 0;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if (half == 1 && cl <= 64) break;
                const uint32_t u = half == 0 ? r0 : r1;
                const bool fresh = u != kNone && vis.insert(u);
                const uint64_t m = ballot64(fresh);
                if (fresh) s.ci[nnew + lanes_below(m)] = u;
                nnew += (int)__popcll(m);
            }
            vis.added(nnew);
            evals += (uint32_t)nnew;
            wave_sync();
            if (nnew == 0) continue;
            score_batch<ST, G, NCH, R>(a, s.qs, nch, s.ci, 0xFFFFFFFFu, s.cd, nnew);
            wave_sync();
            const QueueLds<float> ql{s.qd, s.qi, s.cd, s.ci, s.sd, s.si, s.slb};
            if (nnew <= 64)
                merge_batch<1, float, QR>(ql, nnew, Leff, qn, ptr);
            else
                merge_batch<2, float, QR>(ql, nnew, Leff, qn, ptr);
            wave_sync();
        }
    }
}

// Queue = [entry]; the visited set is cleared and holds the entry.
template <int ST, int CLS, class VIS>
__device__ __forceinline__ void init_state(const SearchArgs &a, const Lds &s, VIS &vis, int &qn, int &ptr,
                                           uint32_t &hops, uint32_t &evals) {
    constexpr int G = shape_g(ST, CLS), NCH = shape_nch(ST, CLS);
    const int lane = lane_id();
    vis.clear();
    const uint32_t u[1] = {lane < G ? a.entry : kNone};
    float acc[1], sc[1];
    dot_rows<ST, G, NCH, 1>(a, u, s.qs, row_chunk_count<ST>(a.d), acc, sc);
    acc[0] = group_sum<G>(acc[0]);
    if constexpr (ST == RG_STORE_FP8E4M3) sc[0] = group_sum<G>(sc[0]);
    wave_sync();
    if (lane == 0) {
        s.qd[0] = finish_delta<ST>(acc[0], sc[0]);
        s.qi[0] = a.entry;
        vis.mark_entry(a.entry);
    }
    vis.added(1);
    qn = 1;
    ptr = 0;
    hops = 0;
    evals = 1;
    wave_sync();
}

// Rescore the final queue (at most 64 * QR entries) against FP32 rows and
// sort it (reduced-precision storage).
template <int CLS, int QR>
__device__ __forceinline__ void rerank_queue(const SearchArgs &a, const Lds &s, int qn) {
    constexpr int G = shape_g(RG_STORE_FP32, CLS), NCH = shape_nch(RG_STORE_FP32, CLS);
    score_batch<RG_STORE_FP32, G, NCH, 2>(a, s.qs, (a.d + 3) >> 2, s.qi, ~kExpanded, s.qd, qn);
    wave_sync();
    constexpr int E = QR;
    const int lane = lane_id();
    float k[E];
    uint32_t id[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = lane * E + e;
        k[e] = i < qn ? s.qd[i] : __builtin_inff();
        id[e] = i < qn ? (s.qi[i] & ~kExpanded) : kNone;
    }
    wave_sort<E>(k, id);
    wave_sync();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = lane * E + e;
        if (i < qn) {
            s.qd[i] = k[e];
            s.qi[i] = id[e];
        }
    }
    wave_sync();
}

// Where a key of +inf stands for a NaN: the NaN again.
__device__ __forceinline__ void restore_nans(const SearchArgs &a, const Lds &s, int qn) {
    // the last entry has the largest key
    if (!(s.qd[qn - 1] == __builtin_inff())) return;
    for (int i = lane_id(); i < qn; i += 64) {
        if (!(s.qd[i] == __builtin_inff())) continue;
        const float *row = a.base + (size_t)(s.qi[i] & ~kExpanded) * a.pitch;
        float sum = 0.f;
        for (int j = 0; j < a.d; ++j) sum = fmaf(s.qs[j], row[j], sum);
        if (sum != sum) s.qd[i] = sum;
    }
    wave_sync();
}

// The k results: the first k entries of the final queue that are not
// deleted (a tombstoned node still routes the search but is never
// returned), padded with kNone / +inf.
__device__ __forceinline__ void emit_topk(const SearchArgs &a, const Lds &s, int qn, uint32_t *ids, float *ds) {
    const int lane = lane_id();
    restore_nans(a, s, qn);
    if (!a.tomb) {
        for (int i = lane; i < a.k; i += 64) {
            ids[i] = i < qn ? (s.qi[i] & ~kExpanded) : kNone;
            ds[i] = i < qn ? s.qd[i] : __builtin_inff();
        }
        return;
    }
    int w = 0;
    for (int b0 = 0; b0 < qn && w < a.k; b0 += 64) {
        const int i = b0 + lane;
        uint32_t u = kNone;
        bool alive = false;
        if (i < qn) {
            u = s.qi[i] & ~kExpanded;
            alive = ((a.tomb[u >> 5] >> (u & 31u)) & 1u) == 0u;
        }
        const uint64_t m = ballot64(alive);
        const int pos = w + lanes_below(m);
        if (alive && pos < a.k) {
            ids[pos] = u;
            ds[pos] = s.qd[i];
        }
        w += (int)__popcll(m);
    }
    for (int i = min(w, a.k) + lane; i < a.k; i += 64) {
        ids[i] = kNone;
        ds[i] = __builtin_inff();
    }
}

__device__ __forceinline__ void write_result(const SearchArgs &a, const Lds &s, int64_t q, int qn, uint32_t hops,
                                             uint32_t evals) {
    const int lane = lane_id();
    emit_topk(a, s, qn, a.out_ids + q * a.k, a.out_d + q * a.k);
    if (lane == 0) {
        if (a.out_hops) a.out_hops[q] = hops;
        if (a.out_evals) a.out_evals[q] = evals;
    }
}

// One query per workgroup, visited set in LDS.  Five resident wavefronts per
// SIMD (<= 102 VGPRs) measured fastest for the BF16/FP8 searches, which wait
// on memory latency more than on bandwidth; six or more spill.  FP32 rows
// (more chunks in flight per row) take four, which keeps them out of
// scratch: 4.6% faster on a 10M-row graph.
// QR = queue capacity / 64: kMaxL / 64, or kMaxSearchL / 64 for L_eff above
// kMaxL, where twice the queue entries per lane in the merge and the rerank
// take four resident wavefronts per SIMD for every storage form.
// VIS: VisitSets, or VisitLds (rg_search_hashbits, wide rows, huge bases).
template <int ST, int CLS, int QR, class VIS>
__global__ __launch_bounds__(64)
__attribute__((amdgpu_waves_per_eu(ST == RG_STORE_FP32 || QR > kMaxL / 64 || CLS >= 4 ? 4 : 5))) void k_search(SearchArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t q = blockIdx.x;
    const Lds s = carve(smem, a.Leff, a.qpad, a.cand);
    VIS vis(s.htab, a.hash_bits, a.id_bits);
    load_query(a.queries + q * a.d, a.d, a.qpad, s.qs);
    int qn, ptr;
    uint32_t hops, evals;
    bool done;
    init_state<ST, CLS>(a, s, vis, qn, ptr, hops, evals);
    run_search<ST, CLS, QR>(a, s, vis, qn, ptr, hops, evals, INT_MAX, done);
    if constexpr (ST != RG_STORE_FP32) rerank_queue<CLS, QR>(a, s, qn);
    write_result(a, s, q, qn, hops, evals);
}

// Persistent grid: each workgroup stays resident, takes queries from a
// device counter until none are left, and keeps an exact visited bitmap
// (one bit per base node) in device memory, so LDS holds only the queue and
// the candidate batch and many more queries are in flight per CU.
// Four resident wavefronts per SIMD (<= 128 VGPRs) measured fastest for all
// storage forms, ahead of fewer waves with more registers.
// QR as for k_search.
template <int ST, int CLS, int QR>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_search_persistent(SearchArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Lds s = carve(smem, a.Leff, a.qpad, a.cand);
    VisitBitmap vis{a.bitmap + (size_t)blockIdx.x * a.bm_words, a.bm_words};
    const int lane = lane_id();
    for (;;) {
        int q = 0;
        if (lane == 0) q = (int)atomicAdd(a.work, 1u);
        q = __shfl(q, 0);
        if ((int64_t)q >= a.nq) break;
        load_query(a.queries + (int64_t)q * a.d, a.d, a.qpad, s.qs);
        int qn, ptr;
        uint32_t hops, evals;
        bool done;
        init_state<ST, CLS>(a, s, vis, qn, ptr, hops, evals);
        run_search<ST, CLS, QR>(a, s, vis, qn, ptr, hops, evals, INT_MAX, done);
        if constexpr (ST != RG_STORE_FP32) rerank_queue<CLS, QR>(a, s, qn);
        write_result(a, s, q, qn, hops, evals);
        wave_sync();
    }
}

// One scheduler step of the serving loop: advance each listed slot by up to
// hops_budget expansions, keeping its whole state in device memory.  Five
// resident wavefronts per SIMD where the registers hold the rows in flight:
// the step is latency-bound.
// Slot state word 0: 0 = admitted, not started; > 0 = queue length of a
// search in progress; -1 = finished (its record written; the slot is
// skipped until the host admits a new request into it).
template <int ST, int CLS, class VIS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(ST == RG_STORE_FP32 || CLS >= 3 ? 4 : 5)))
void k_serve_step(SlotArgs sa) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int slot = sa.active[blockIdx.x];
    if (sa.slot_state[(size_t)slot * 8] < 0) return;
    SearchArgs a = sa.s;
    a.k = sa.slot_k[slot];
    a.Leff = max(sa.slot_L[slot], a.k);
    const Lds s = carve(smem, a.Leff, a.qpad, a.cand);
    const int lane = lane_id();
    const int H = 1 << a.hash_bits;
    load_query(sa.slot_q + (size_t)slot * a.d, a.d, a.qpad, s.qs);
    int32_t *st = sa.slot_state + (size_t)slot * 8;
    float *gqd = sa.slot_qd + (size_t)slot * kMaxL;
    uint32_t *gqi = sa.slot_qi + (size_t)slot * kMaxL;
    uint32_t *gh = sa.slot_hash + ((size_t)slot << a.hash_bits);
    int qn, ptr;
    uint32_t hops, evals;
    VIS vis(s.htab, a.hash_bits, a.id_bits);
    if (st[0] == 0) {
        init_state<ST, CLS>(a, s, vis, qn, ptr, hops, evals);
    } else {
        qn = st[0];
        ptr = st[1];
        vis.restore(st[2]);
        hops = (uint32_t)st[3];
        evals = (uint32_t)st[4];
        for (int i = lane; i < qn; i += 64) {
            s.qd[i] = gqd[i];
            s.qi[i] = gqi[i];
        }
        for (int i = lane; i < H; i += 64) s.htab[i] = gh[i];
        wave_sync();
    }
    bool done;
    run_search<ST, CLS, kMaxL / 64>(a, s, vis, qn, ptr, hops, evals, sa.hops_budget, done);
    if (done) {
        if constexpr (ST != RG_STORE_FP32) rerank_queue<CLS, kMaxL / 64>(a, s, qn);
        int pos = 0;
        if (lane == 0) pos = (int)atomicAdd(sa.out_count, 1u);
        pos = __shfl(pos, 0);
        ServeRecord *r = sa.out_rec + pos;
        emit_topk(a, s, qn, r->ids, r->d);
        if (lane == 0) {
            r->slot = slot;
            r->qn = qn;
            r->hops = hops;
            r->evals = evals;
            st[0] = -1;
        }
    } else {
        for (int i = lane; i < qn; i += 64) {
            gqd[i] = s.qd[i];
            gqi[i] = s.qi[i];
        }
        for (int i = lane; i < H; i += 64) gh[i] = s.htab[i];
        if (lane == 0) {
            st[0] = qn;
            st[1] = ptr;
            st[2] = vis.count();
            st[3] = (int32_t)hops;
            st[4] = (int32_t)evals;
        }
    }
}

// ---------------------------------------------------------------------------
// Few queries: several wavefronts per query.
//
// With fewer queries than the chip holds wavefronts an expansion is a chain
// of waits (the adjacency row, the visited set, two or three rounds of rows,
// the merge: 7 us on FP32 d = 200, 13 us on BF16 d = 512), and the rest of
// the chip idles.  Here a workgroup runs one query, in rounds of three parts:
//   * prepare, all wavefronts, P to each of the first W unexpanded queue
//     entries that are not prepared yet: read the adjacency row and score the
//     neighbours that are not visited;
//   * commit, wavefront 0: while the first unexpanded entry is a prepared one,
//     mark it expanded and merge what was scored.  It stops at an entry that
//     is not prepared (a merge brought a closer one); what was prepared stays
//     until it is committed or its place is needed;
//   * visit, the last wavefront, while the others wait for their adjacency
//     rows: mark the committed entries' neighbours visited, in commit order,
//     and count the new ones.
// The results are the sequential search's: distances do not depend on when
// they are computed, expansions are committed in its order, and a node that
// is scored although a commit in between has visited it is dropped at the
// merge (it is queued, or it was rejected or evicted against a last key that
// has only decreased since).  Rows prepared and never committed are extra
// work; the counts are those of the visits, which happen as they would in
// sequence.
//
// The visited set is VisitSets, or VisitSpill: exact, node ids in a large LDS
// table that is written out to the query's bitmap in device memory when it is
// three quarters full.  What has been prepared is then dropped, so that every
// later preparation sees all that was written out.
// ---------------------------------------------------------------------------
struct VisitSpill {
    static constexpr bool kExact [[maybe_unused]] = true;
    uint32_t *htab, *bm;
    int hb;
    __device__ __forceinline__ VisitSpill(uint32_t *t, const SearchArgs &a, int64_t q)
        : htab(t), bm(a.bitmap ? a.bitmap + q * a.bm_words : nullptr), hb(a.hash_bits) {}
    __device__ __forceinline__ bool seen(uint32_t u, bool spilled) const {
        const uint32_t hmask = (1u << hb) - 1u;
        for (uint32_t h = hslot(u, hb);; h = (h + 1u) & hmask) {  // a quarter of the table is free
            const uint32_t x = htab[h];
            if (x == u) return true;
            if (x == kEmpty) break;
        }
        return spilled && ((__hip_atomic_load(&bm[u >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> (u & 31u)) & 1u);
    }
    __device__ __forceinline__ bool insert(uint32_t u) {
        const uint32_t hmask = (1u << hb) - 1u;
        for (uint32_t h = hslot(u, hb);; h = (h + 1u) & hmask) {
            const uint32_t old = atomicCAS(&htab[h], kEmpty, u);
            if (old == kEmpty) return true;
            if (old == u) return false;
        }
    }
    // whether count ids and one row more may fill the table too far
    __device__ __forceinline__ bool full(int count) const { return count + 64 > (3 << hb) / 4; }
    // all threads; the table's ids move to the bitmap (cleared the first time)
    __device__ __forceinline__ void spill(int64_t words, bool first) {
        if (first) {
            uint4 *b4 = reinterpret_cast<uint4 *>(bm);
            for (int64_t i = threadIdx.x; i < (words >> 2); i += blockDim.x) b4[i] = make_uint4(0u, 0u, 0u, 0u);
            __threadfence();
            __syncthreads();
        }
        for (int i = threadIdx.x; i < (1 << hb); i += blockDim.x) {
            const uint32_t u = htab[i];
            if (u != kEmpty) atomicOr(&bm[u >> 5], 1u << (u & 31u));
            htab[i] = kEmpty;
        }
        __threadfence();
    }
};

struct VisitSetsWide : VisitSets {
    static constexpr bool kExact [[maybe_unused]] = false;
    __device__ __forceinline__ VisitSetsWide(uint32_t *t, const SearchArgs &a, int64_t)
        : VisitSets(t, a.hash_bits, a.id_bits) {}
    __device__ __forceinline__ bool seen(uint32_t u, bool) const { return holds(u); }
    __device__ __forceinline__ bool full(int) const { return false; }
    __device__ __forceinline__ void spill(int64_t, bool) {}
};

// Merge one candidate per lane (cand: it takes part) into the sorted queue of
// up to 64 * QR entries by counting, for two entries per lane: each survivor
// is read out of its lane and compared with every entry, which gives its place
// and the entries' moves without a look into LDS; three ballots or more each.
// A candidate that is queued, or that stands earlier in the batch, is dropped.
// One query, 300k x 200 L = 100: 525 us against 560 with merge_held; at more
// entries per lane merge_held wins (16 queries BF16 200k x 512 L = 200 1,400 ->
// 1,190 us, 500 queries 500k x 512 L = 800 7,500 -> 6,420).
template <int QR>
__device__ __forceinline__ void merge_lanes(float *qd, uint32_t *qi, int Leff, int &qn, int &ptr, float kc, uint32_t ic,
                                            bool cand) {
    const int lane = lane_id();
    bool sv = cand;
    if (qn == Leff) sv = cand && kless(kc, ic, qd[Leff - 1], qi[Leff - 1] & ~kExpanded);
    const uint64_t all = ballot64(sv);
    if (all == 0) return;
    int sh[QR];  // candidates ahead of entry 64 r + lane
    float k[QR];
    uint32_t v[QR];
#pragma unroll
    for (int r = 0; r < QR; ++r) {
        const int i = r * 64 + lane;
        sh[r] = 0;
        k[r] = __builtin_inff();
        v[r] = kNone;
        if (i < qn) {
            k[r] = qd[i];
            v[r] = qi[i];
        }
    }
    int lb = 0, ahead = 0, total = 0, lbmin = INT_MAX;
    for (uint64_t m = all; m; m &= m - 1) {
        const int src = (int)__builtin_ctzll(m);
        const float ks = lane_value(kc, src);
        const uint32_t is = lane_value(ic, src);
        uint64_t drop = ballot64(sv && ic == is && lane < src);
        int ls = 0;
        bool less[QR];
#pragma unroll
        for (int r = 0; r < QR; ++r) {
            const uint32_t id = v[r] & ~kExpanded;
            less[r] = kless(k[r], id, ks, is);
            ls += (int)__popcll(ballot64(less[r]));
            drop |= ballot64(id == is);
        }
        if (drop) {
            if (lane == src) sv = false;
            continue;
        }
#pragma unroll
        for (int r = 0; r < QR; ++r) sh[r] += less[r] ? 0 : 1;
        if (lane == src) lb = ls;
        ahead += kless(ks, is, kc, ic) ? 1 : 0;
        lbmin = min(lbmin, ls);
        ++total;
    }
    if (total == 0) return;
    wave_sync();
#pragma unroll
    for (int r = 0; r < QR; ++r)
        if (r * 64 + 63 >= lbmin) {
            const int i = r * 64 + lane, p = i + sh[r];
            if (i < qn && sh[r] > 0 && p < Leff) {
                qd[p] = k[r];
                qi[p] = v[r];
            }
        }
    if (sv && lb + ahead < Leff) {
        qd[lb + ahead] = kc;
        qi[lb + ahead] = ic;
    }
    qn = min(Leff, qn + total);
    ptr = min(ptr, lbmin);
    wave_sync();
}

constexpr int kWide = kMaxWide;  // most wavefronts per query
enum { kRun = 0, kDone = 1, kSpill = 2 };
struct alignas(16) WideLds {
    uint32_t id[kWide][64];  // a preparation: the adjacency row,
    float cd[kWide][64];     // the distances of what was scored, in row order,
    uint64_t mask[kWide];    // and which of the row that is
    uint32_t ci[kWide][64];
    uint32_t node[kWide], next[kWide], tgt[kWide];
    int done[kWide];         // preparations committed in the last round, in order
    int n_done, state, qn, count;
    uint32_t hops, evals;
    int pad[2];
    uint32_t bits[kMaxSearchL / 32];  // of the merge
};
// rows in flight per group: 32 chunks per lane, 4 to 8 rows
constexpr int wide_r(int nch) { return nch >= 8 ? 4 : nch * 8 <= 32 ? 8 : 32 / nch; }

template <int ST, int CLS, int QR, class VIS>
__global__ __launch_bounds__(64 * kWide) __attribute__((amdgpu_waves_per_eu(2))) void k_search_wide(SearchArgs a) {
    constexpr int G = shape_g(ST, CLS), NCH = shape_nch(ST, CLS), R = wide_r(NCH);
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, nthr = blockDim.x, w = tid >> 6, lane = lane_id();
    // P wavefronts per preparation, W preparations at a time
    constexpr int P = kPrep;
    const int W = (nthr >> 6) / P, slot_w = w / P, part = w % P;
    const int64_t q = blockIdx.x;
    const int Leff = a.Leff, nch = row_chunk_count<ST>(a.d);
    WideLds &s = *reinterpret_cast<WideLds *>(smem);
    float *qs = reinterpret_cast<float *>(smem + sizeof(WideLds));
    float *qd = qs + a.qpad;
    uint32_t *qi = reinterpret_cast<uint32_t *>(qd + Leff);
    uint32_t *htab = qi + Leff;
    VIS vis(htab, a, q);

    for (int i = tid; i < a.qpad; i += nthr) qs[i] = i < a.d ? a.queries[q * a.d + i] : 0.f;
    for (int i = tid; i < (1 << a.hash_bits); i += nthr) htab[i] = kEmpty;
    // no queue place ever holds anything but a node
    for (int i = tid; i < Leff; i += nthr) {
        qd[i] = __builtin_inff();
        qi[i] = a.entry | kExpanded;
    }
    if (tid < kWide) s.node[tid] = kNone;
    if (tid == 0) {
        s.n_done = 0;
        s.count = 1;
    }
    __syncthreads();

    // state of wavefront 0
    int qn = 1, ptr = 0;
    uint32_t hops = 0;
    // of the last wavefront
    const bool last = w == (nthr >> 6) - 1;
    int count = 1;
    uint32_t evals = 1;
    bool spilled = false;
    // the first W unexpanded entries that are not prepared, one to each
    // preparation that is not among them (wavefront 0)
    auto plan = [&]() {
        int nt = 0;
        for (int b = ptr; b < qn && nt < W; b += 64) {
            const int i = b + lane;
            const uint32_t x = i < qn ? qi[i] : kExpanded;
            const bool un = !(x & kExpanded);
            const uint64_t m = ballot64(un);
            const int k = nt + lanes_below(m);
            if (un && k < W) s.tgt[k] = x;
            nt += (int)__popcll(m);
        }
        nt = min(nt, W);
        wave_sync();
        const uint32_t tv = lane < nt ? s.tgt[lane] : kNone, sv = lane < W ? s.node[lane] : kNone;
        bool have = false, keep = false;
        for (int i = 0; i < W; ++i) {
            const uint32_t si = (uint32_t)__builtin_amdgcn_readlane((int)sv, i);
            const uint32_t ti = (uint32_t)__builtin_amdgcn_readlane((int)tv, i);
            have |= tv == si;
            keep |= sv == ti && ti != kNone;
        }
        const uint64_t need = ballot64(lane < nt && !have), fre = ballot64(lane < W && !keep);
        wave_sync();
        if ((need >> lane) & 1u) s.tgt[lanes_below(need)] = tv;
        wave_sync();
        if (lane < W) {
            const int r = lanes_below(fre);
            s.next[lane] = ((fre >> lane) & 1u) && r < (int)__popcll(need) ? s.tgt[r] : kNone;
        }
        if (lane == 0) s.state = kRun;
    };

    if (w == 0) {
        const uint32_t u[1] = {lane < G ? a.entry : kNone};
        float acc[1], sc[1];
        dot_rows<ST, G, NCH, 1>(a, u, qs, nch, acc, sc);
        acc[0] = group_sum<G>(acc[0]);
        if constexpr (ST == RG_STORE_FP8E4M3) sc[0] = group_sum<G>(sc[0]);
        if (lane == 0) {
            qd[0] = finish_delta<ST>(acc[0], sc[0]);
            qi[0] = a.entry;
            (void)vis.insert(a.entry);
        }
        wave_sync();
        plan();
    }
    for (;;) {
        __syncthreads();
        const int state = s.state;
        const uint32_t mine = state == kRun ? s.next[slot_w] : kNone;
        uint32_t u = kNone;
        if (mine != kNone && lane < a.ell) u = a.adj[(int64_t)mine * a.ell + lane];
        if (last) {
            const int nd = s.n_done;
            for (int i = 0; i < nd; ++i) {
                const int c = s.done[i];
                const uint32_t x = s.id[c][lane];
                // exact: what was not scored is visited; sets: it may be forgotten
                bool fresh = false;
                if (x != kNone && (!VIS::kExact || ((s.mask[c] >> lane) & 1u))) fresh = vis.insert(x);
                const int nf = (int)__popcll(ballot64(fresh));
                evals += (uint32_t)nf;
                count += nf;
            }
            if (lane == 0) {
                s.count = count;
                s.evals = evals;
            }
        }
        __syncthreads();
        if (state == kDone) break;
        if (state == kSpill) {
            vis.spill(a.bm_words, !spilled);
            spilled = true;
            count = 0;
            if (tid < kWide) s.node[tid] = kNone;
            __syncthreads();
            if (w == 0) {
                if (lane == 0) {
                    s.n_done = 0;
                    s.count = 0;
                }
                plan();
            }
            continue;
        }
        if (mine != kNone) {
            const bool fresh = u != kNone && !vis.seen(u, spilled);
            const uint64_t m = ballot64(fresh);
            const int cnt = (int)__popcll(m), r0 = cnt * part / P, r1 = cnt * (part + 1) / P;
            if (fresh) s.ci[w][lanes_below(m)] = u;
            wave_sync();
            score_batch<ST, G, NCH, R>(a, qs, nch, s.ci[w] + r0, 0xFFFFFFFFu, s.cd[slot_w] + r0, r1 - r0);
            if (part == 0) {
                s.id[slot_w][lane] = u;
                if (lane == 0) {
                    s.mask[slot_w] = m;
                    s.node[slot_w] = mine;
                }
            }
        }
        __syncthreads();
        if (w != 0) continue;
        // at most W commits (each uses a preparation up), so done[] holds them
        int nd = 0, seen = s.count;
        for (;;) {
            int sel = -1;
            for (int b = ptr; b < qn; b += 64) {
                const int i = b + lane;
                const uint64_t m = ballot64(i < qn && !(qi[i] & kExpanded));
                if (m) {
                    sel = b + (int)__builtin_ctzll(m);
                    break;
                }
            }
            if (sel < 0) {
                if (lane == 0) {
                    s.state = kDone;
                    s.qn = qn;
                    s.hops = hops;
                }
                break;
            }
            ptr = sel;
            const uint32_t v = qi[sel];
            const uint64_t at = ballot64(lane < W && s.node[lane & (kWide - 1)] == v);
            if (at == 0) {
                plan();
                break;
            }
            if (vis.full(seen)) {
                if (lane == 0) s.state = kSpill;
                break;
            }
            const int slot = (int)__builtin_ctzll(at);
            const uint64_t m = s.mask[slot];
            const uint32_t x = s.id[slot][lane];
            const bool scored = (m >> lane) & 1u;
            const float kc = scored ? s.cd[slot][lanes_below(m)] : __builtin_inff();
            wave_sync();
            if (lane == 0) {
                qi[sel] = v | kExpanded;
                s.node[slot] = kNone;
                s.done[nd] = slot;
            }
            wave_sync();
            ++nd;
            ++hops;
            seen += (int)__popcll(m);
            if constexpr (QR <= 2)
                merge_lanes<QR>(qd, qi, Leff, qn, ptr, kc, x, scored);
            else
                merge_held<float, false, true>(qd, qi, s.bits, Leff, qn, ptr, kc, scored ? x : kNone, 0.f);
        }
        if (lane == 0) s.n_done = nd;
    }
    const int n = s.qn;
    if constexpr (ST != RG_STORE_FP32) {
        // the final queue by its FP32 distances: every wavefront rescores a
        // part, then every entry's place is the number of entries before it
        constexpr int G32 = shape_g(RG_STORE_FP32, CLS), N32 = shape_nch(RG_STORE_FP32, CLS);
        const int nw = nthr >> 6, per = (n + nw - 1) / nw, r0 = min(n, w * per), r1 = min(n, r0 + per);
        score_batch<RG_STORE_FP32, G32, N32, 4>(a, qs, (a.d + 3) >> 2, qi + r0, ~kExpanded, qd + r0, r1 - r0);
        __syncthreads();
        constexpr int E = QR / 2;  // entries per thread, two wavefronts at least
        float k[E];
        uint32_t id[E];
        int rank[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = e * nthr + tid;
            k[e] = i < n ? qd[i] : 0.f;
            id[e] = i < n ? qi[i] & ~kExpanded : 0u;
            rank[e] = 0;
        }
        for (int j = 0; j < n; ++j) {
            const float kj = qd[j];
            const uint32_t ij = qi[j] & ~kExpanded;
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (e * nthr < n) rank[e] += kless(kj, ij, k[e], id[e]) ? 1 : 0;
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = e * nthr + tid;
            if (i < n) {
                qd[rank[e]] = k[e];
                qi[rank[e]] = id[e];
            }
        }
        __syncthreads();
    }
    if (w == 0) {
        Lds out{};
        out.qs = qs;
        out.qd = qd;
        out.qi = qi;
        write_result(a, out, q, n, s.hops, s.evals);
    }
}

// The kernels for a queue of L_eff entries: kMaxL or fewer, or up to kMaxSearchL.
template <int ST, int CLS, class VIS>
void (*table_kernel(int Leff))(SearchArgs) {
    return Leff > kMaxL ? k_search<ST, CLS, kMaxSearchL / 64, VIS> : k_search<ST, CLS, kMaxL / 64, VIS>;
}
template <int ST, int CLS>
void (*persistent_kernel(int Leff))(SearchArgs) {
    return Leff > kMaxL ? k_search_persistent<ST, CLS, kMaxSearchL / 64> : k_search_persistent<ST, CLS, kMaxL / 64>;
}

template <int ST, int CLS, class VIS>
int launch_table(const SearchArgs &a, hipStream_t stream) {
    const size_t lds = search_lds_bytes(a.Leff, a.qpad, a.hash_bits, a.cand);
    // one wavefront per query: a HIP grid holds fewer than 2^32 threads
    constexpr int64_t most = 1 << 25;
    for (int64_t q0 = 0; q0 < a.nq; q0 += most) {
        SearchArgs b = a;
        b.nq = std::min(most, a.nq - q0);
        b.queries += q0 * a.d;
        b.out_ids += q0 * a.k;
        b.out_d += q0 * a.k;
        if (a.out_hops) b.out_hops += q0;
        if (a.out_evals) b.out_evals += q0;
        hipLaunchKernelGGL((table_kernel<ST, CLS, VIS>(a.Leff)), dim3((unsigned)b.nq), dim3(64), lds, stream, b);
        RG_HIP(hipGetLastError());
    }
    return RG_OK;
}

template <int ST, int CLS>
int launch_persistent(const SearchArgs &a, hipStream_t stream) {
    const size_t lds = search_lds_bytes(a.Leff, a.qpad, 0, a.cand);
    if (a.Leff > kMaxL)
        hipLaunchKernelGGL((k_search_persistent<ST, CLS, kMaxSearchL / 64>), dim3((unsigned)a.grid), dim3(64), lds,
                           stream, a);
    else
        hipLaunchKernelGGL((k_search_persistent<ST, CLS, kMaxL / 64>), dim3((unsigned)a.grid), dim3(64), lds, stream,
                           a);
    RG_HIP(hipGetLastError());
    return RG_OK;
}

template <int ST, int CLS>
int occupancy_of(int Leff, int pitch, int cand, int *blocks_per_cu) {
    const size_t lds = search_lds_bytes(Leff, pitch, 0, cand);
    RG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, persistent_kernel<ST, CLS>(Leff), 64, lds));
    return RG_OK;
}

template <int ST, int CLS>
void (*step_kernel(const SearchArgs &a))(SlotArgs) {
    return a.sets ? k_serve_step<ST, CLS, VisitSets> : k_serve_step<ST, CLS, VisitLds>;
}

template <int ST, int CLS, int QR>
void (*wide_kernel(bool sets))(SearchArgs) {
    if constexpr (ST == RG_STORE_FP32) {
        if (!sets) return k_search_wide<ST, CLS, QR, VisitSpill>;
    }
    return k_search_wide<ST, CLS, QR, VisitSetsWide>;
}

template <int ST, int CLS>
struct WideLaunch {
    static int run(const SearchArgs &a, hipStream_t stream) {
        const size_t lds = sizeof(WideLds) + (size_t)a.qpad * 4 + (size_t)a.Leff * 8 + ((size_t)4 << a.hash_bits);
        auto k = a.Leff <= 128     ? wide_kernel<ST, CLS, 2>(a.sets)
                 : a.Leff <= kMaxL ? wide_kernel<ST, CLS, kMaxL / 64>(a.sets)
                                   : wide_kernel<ST, CLS, kMaxSearchL / 64>(a.sets);
        if (lds > (64u << 10))
            RG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds));
        hipLaunchKernelGGL(k, dim3((unsigned)a.nq), dim3(64 * (unsigned)a.grid), lds, stream, a);
        RG_HIP(hipGetLastError());
        return RG_OK;
    }
};

template <int ST, int CLS>
int launch_step(const SlotArgs &sa, hipStream_t stream) {
    const size_t lds = search_lds_bytes(kMaxL, sa.s.qpad, sa.s.hash_bits, sa.s.cand);
    hipLaunchKernelGGL((step_kernel<ST, CLS>(sa.s)), dim3((unsigned)sa.n_active), dim3(64), lds, stream, sa);
    RG_HIP(hipGetLastError());
    return RG_OK;
}

// dimension class of d (see kClassMaxD)
template <template <int, int> class F, int ST, typename Arg>
int dispatch_dim(int d, const Arg &a, hipStream_t stream) {
    if (d <= kClassMaxD[0]) return F<ST, 0>::run(a, stream);
    if (d <= kClassMaxD[1]) return F<ST, 1>::run(a, stream);
    if (d <= kClassMaxD[2]) return F<ST, 2>::run(a, stream);
    if (d <= kClassMaxD[3]) return F<ST, 3>::run(a, stream);
    if (d <= kClassMaxD[4]) return F<ST, 4>::run(a, stream);
    if (d <= kClassMaxD[5]) return F<ST, 5>::run(a, stream);
    set_error("search: d > 1024 is not supported");
    return RG_EINVAL;
}

template <class VIS>
struct Table {
    template <int ST, int CLS>
    struct Launch {
        static int run(const SearchArgs &a, hipStream_t s) { return launch_table<ST, CLS, VIS>(a, s); }
    };
    template <int ST, int CLS>
    struct Occ {
        static int run(const SearchArgs &a, hipStream_t) {
            const size_t lds = search_lds_bytes(a.Leff, a.qpad, a.hash_bits, a.cand);
            RG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(a.occ_out, table_kernel<ST, CLS, VIS>(a.Leff), 64, lds));
            return RG_OK;
        }
    };
};
template <int ST, int CLS>
struct PersistentLaunch {
    static int run(const SearchArgs &a, hipStream_t s) { return launch_persistent<ST, CLS>(a, s); }
};
template <int ST, int CLS>
struct OccLaunch {
    static int run(const SearchArgs &a, hipStream_t) {
        return occupancy_of<ST, CLS>(a.Leff, a.qpad, a.cand, a.occ_out);
    }
};
template <int ST, int CLS>
struct StepLaunch {
    static int run(const SlotArgs &a, hipStream_t s) { return launch_step<ST, CLS>(a, s); }
};
template <int ST, int CLS>
struct StepOcc {
    static int run(const SlotArgs &a, hipStream_t) {
        const size_t lds = search_lds_bytes(kMaxL, a.s.qpad, a.s.hash_bits, a.s.cand);
        RG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(a.s.occ_out, step_kernel<ST, CLS>(a.s), 64, lds));
        return RG_OK;
    }
};

}  // namespace

constexpr int kST = RG_BEAM_STORAGE;
#if RG_BEAM_PART == 0
template <>
int BeamOps<kST>::search_ids(const SearchArgs &a, hipStream_t s) {
    return dispatch_dim<Table<VisitLds>::Launch, kST>(a.d, a, s);
}
#if RG_BEAM_STORAGE == 0
template <>
int BeamOps<kST>::search_bits(const SearchArgs &a, hipStream_t s) {
    return dispatch_dim<Table<VisitBits>::Launch, kST>(a.d, a, s);
}
#endif
template <>
int BeamOps<kST>::ids_occupancy(const SearchArgs &a) {
    return dispatch_dim<Table<VisitLds>::Occ, kST>(a.d, a, nullptr);
}
#elif RG_BEAM_PART == 1
template <>
int BeamOps<kST>::search_sets(const SearchArgs &a, hipStream_t s) {
    return dispatch_dim<Table<VisitSets>::Launch, kST>(a.d, a, s);
}
template <>
int BeamOps<kST>::sets_occupancy(const SearchArgs &a) {
    return dispatch_dim<Table<VisitSets>::Occ, kST>(a.d, a, nullptr);
}
#elif RG_BEAM_PART == 3
template <>
int BeamOps<kST>::wide(const SearchArgs &a, hipStream_t s) {
    return dispatch_dim<WideLaunch, kST>(a.d, a, s);
}
#else
template <>
int BeamOps<kST>::persistent(const SearchArgs &a, hipStream_t s) {
    return dispatch_dim<PersistentLaunch, kST>(a.d, a, s);
}
template <>
int BeamOps<kST>::persistent_occupancy(const SearchArgs &a) {
    return dispatch_dim<OccLaunch, kST>(a.d, a, nullptr);
}
template <>
int BeamOps<kST>::serve_step(const SlotArgs &a, hipStream_t s) {
    return dispatch_dim<StepLaunch, kST>(a.s.d, a, s);
}
template <>
int BeamOps<kST>::serve_occupancy(const SlotArgs &a) {
    return dispatch_dim<StepOcc, kST>(a.s.d, a, nullptr);
}
#endif

#else  // !RG_BEAM_STORAGE
namespace {

constexpr int kCand = 128;  // largest candidate batch (the widest ELL row, a CSR chunk)

__global__ __launch_bounds__(64) void k_serve_admit(int32_t n, const int32_t *slots, const float *q,
                                                   const int32_t *k, const int32_t *L, int32_t d, float *slot_q,
                                                   int32_t *slot_k, int32_t *slot_L, int32_t *slot_state) {
    const int i = blockIdx.x;
    const int s = slots[i];
    for (int j = threadIdx.x; j < d; j += 64) slot_q[(size_t)s * d + j] = q[(size_t)i * d + j];
    if (threadIdx.x < 8) slot_state[(size_t)s * 8 + threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        slot_k[s] = k[i];
        slot_L[s] = L[i];
    }
}

// f(BeamOps of the storage form)
template <class F>
int with_storage(int storage, const char *who, F &&f) {
    switch (storage) {
    case RG_STORE_FP32: return f(BeamOps<RG_STORE_FP32>());
    case RG_STORE_BF16: return f(BeamOps<RG_STORE_BF16>());
    case RG_STORE_FP8E4M3: return f(BeamOps<RG_STORE_FP8E4M3>());
    default: set_error(std::string(who) + ": unknown storage"); return RG_EINVAL;
    }
}

}  // namespace

size_t search_lds_bytes(int Leff, int pitch, int hash_bits, int cand) {
    return (size_t)pitch * 4 + (size_t)Leff * 8 + (size_t)cand * 20 + (hash_bits > 0 ? ((size_t)4 << hash_bits) : 0);
}

int cand_capacity(int ell, bool csr) { return csr || ell > 64 ? kCand : 64; }

int launch_search(const SearchArgs &a, hipStream_t stream) {
    if (a.nq == 0) return RG_OK;
    return with_storage(a.storage, "search", [&](auto ops) { return a.sets ? ops.search_sets(a, stream) : ops.search_ids(a, stream); });
}

int launch_search_bits(const SearchArgs &a, hipStream_t stream) {
    if (a.nq == 0) return RG_OK;
    if (a.storage != RG_STORE_FP32 || a.n_rows > (32ll << a.hash_bits)) {
        set_error("search: bad arguments for the visited bits in LDS");
        return RG_EINTERNAL;
    }
    return BeamOps<RG_STORE_FP32>::search_bits(a, stream);
}

int launch_search_wide(const SearchArgs &a, hipStream_t stream) {
    if (a.nq == 0) return RG_OK;
    if (a.adj_off || a.ell > 64 || a.Leff > kMaxSearchL || a.grid < 2 || a.grid > kMaxWide ||
        a.grid % kPrep != 0 ||
        (!a.sets && (a.storage != RG_STORE_FP32 || (!a.bitmap && a.n_rows + 64 * (kMaxWide + 1) > (3ll << a.hash_bits) / 4)))) {
        set_error("search: bad arguments for several wavefronts per query");
        return RG_EINTERNAL;
    }
    return with_storage(a.storage, "search", [&](auto ops) { return ops.wide(a, stream); });
}

int launch_search_persistent(const SearchArgs &a, hipStream_t stream) {
    if (a.nq == 0) return RG_OK;
    return with_storage(a.storage, "search", [&](auto ops) { return ops.persistent(a, stream); });
}

int search_occupancy(const SearchArgs &a, int *blocks_per_cu) {
    SearchArgs b = a;
    b.occ_out = blocks_per_cu;
    return with_storage(a.storage, "search", [&](auto ops) { return ops.persistent_occupancy(b); });
}

int table_search_occupancy(const SearchArgs &a, int *blocks_per_cu) {
    SearchArgs b = a;
    b.occ_out = blocks_per_cu;
    return with_storage(a.storage, "search", [&](auto ops) { return b.sets ? ops.sets_occupancy(b) : ops.ids_occupancy(b); });
}

int launch_serve_admit(int32_t n, const int32_t *slots, const float *q, const int32_t *k, const int32_t *L,
                       int32_t d, float *slot_q, int32_t *slot_k, int32_t *slot_L, int32_t *slot_state,
                       hipStream_t stream) {
    if (n == 0) return RG_OK;
    hipLaunchKernelGGL(k_serve_admit, dim3((unsigned)n), dim3(64), 0, stream, n, slots, q, k, L, d, slot_q, slot_k,
                       slot_L, slot_state);
    RG_HIP(hipGetLastError());
    return RG_OK;
}

int launch_serve_step(const SlotArgs &sa, hipStream_t stream) {
    if (sa.n_active == 0) return RG_OK;
    return with_storage(sa.s.storage, "serve", [&](auto ops) { return ops.serve_step(sa, stream); });
}

int serve_step_occupancy(const SlotArgs &a, int *blocks_per_cu) {
    SlotArgs b = a;
    b.s.occ_out = blocks_per_cu;
    return with_storage(a.s.storage, "serve", [&](auto ops) { return ops.serve_occupancy(b); });
}

// ---------------------------------------------------------------------------
// Device scratch of the allocation-free search (rg_search_noalloc): the
// persistent search's work counter (first 256 bytes) and one visited bitmap
// per resident workgroup.  Each device holds its own copy of this array from
// the library's first use on it until the process ends.  In host code the
// array's name is not a device address: the address comes from
// hipGetSymbolAddress, taken once per device with that device current.
// ---------------------------------------------------------------------------
namespace {

__device__ __align__(256) uint32_t scratch[kNoAllocScratchBytes / 4];

__global__ void k_zero_words(uint32_t *p, int n) {
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0u;
}

}  // namespace

int noalloc_scratch(int device, uint32_t **out) {
    static std::mutex mu;
    static uint32_t *ptr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices) {
        set_error("search_noalloc: device index out of range");
        return RG_EINVAL;
    }
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[device]) {
        int cur = -1;
        RG_HIP(hipGetDevice(&cur));
        if (cur != device) {
            set_error("search_noalloc: the index's device must be the current device");
            return RG_EINVAL;
        }
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_error(std::string("search_noalloc: hipGetSymbolAddress: ") + hipGetErrorString(e));
            return RG_EDEVICE;
        }
        ptr[device] = static_cast<uint32_t *>(p);
    }
    *out = ptr[device];
    return RG_OK;
}

// a fill kernel rather than a memset, so callers may capture the search in a graph
int launch_zero_words(uint32_t *p, int n, hipStream_t stream) {
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, stream, p, n);
    RG_HIP(hipGetLastError());
    return RG_OK;
}

#endif  // RG_BEAM_STORAGE

}  // namespace rg
