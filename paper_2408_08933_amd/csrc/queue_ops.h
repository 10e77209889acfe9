// Visited tables and the sorted-queue merge shared by the search kernels (FP32 keys) and the
// construction-time canonical search (FP64 keys).  One wavefront owns the
// queue; all arrays live in LDS, so wave_sync orders its steps.
#pragma once

#include <climits>

#include "rg_internal.h"
#include "wave_ops.h"

namespace rg {

constexpr uint32_t kEmpty = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t hslot(uint32_t u, int hb) { return (u * 2654435761u) >> (32 - hb); }

// Visited set kept in LDS: open addressing, cleared when it passes half load
// (clearing only costs re-scoring; see the file comment).
struct VisitLds {
    uint32_t *htab;
    int hb, H, hcount;
    __device__ __forceinline__ VisitLds(uint32_t *t, int hash_bits, int) : htab(t), hb(hash_bits), H(1 << hb), hcount(0) {}
    __device__ __forceinline__ void clear() {
        for (int i = lane_id(); i < H; i += 64) htab[i] = kEmpty;
        hcount = 0;
    }
    __device__ __forceinline__ void mark_entry(uint32_t u) {  // lane 0, table just cleared
        htab[hslot(u, hb)] = u;
    }
    __device__ __forceinline__ void begin_hop(int ell) {
        if (hcount + ell > (H >> 1)) {
            clear();
            wave_sync();
        }
    }
    __device__ __forceinline__ bool insert(uint32_t u) {
        const uint32_t hmask = (uint32_t)H - 1u;
        uint32_t h = hslot(u, hb);
        for (int probe = 0; probe < H; ++probe) {
            const uint32_t old = atomicCAS(&htab[h], kEmpty, u);
            if (old == kEmpty) return true;
            if (old == u) return false;
            h = (h + 1u) & hmask;
        }
        return false;
    }
    __device__ __forceinline__ void added(int k) { hcount += k; }
    // what a resumed search needs beside the table's words
    __device__ __forceinline__ int count() const { return hcount; }
    __device__ __forceinline__ void restore(int c) { hcount = c; }
};

// Visited set kept in LDS that forgets one node at a time: 2^set_bits sets of
// four 16-bit entries, the newest first; a new node pushes its set's oldest
// one out.  A node's bits are spread by an odd multiplier (a bijection of the
// id_bits-bit numbers); the product's top set_bits bits name the set and the
// rest, which must fit 16 bits, is the entry, so an entry is one node and no
// other.  Half the bytes of an id per node, and never cleared: at any time it
// holds the last 4 * 2^set_bits nodes (up to uneven sets), where a table
// cleared at half load holds a quarter of its ids on average.  Rows scored
// per query, 10k queries a launch: 2M x 512 E4M3 at L = 409 26,160 -> 20,400
// (2 KB; 16,560 distinct) and 40.0 -> 34.1 ms, 500k x 200 BF16 at L = 805,
// 3,001 queries, 44,310 -> 33,200 (26,890) and 11.1 -> 8.8 ms, 700k x 100
// FP32 at L = 32, 4,096 queries, 2,190 -> 1,713 (1,704) and 0.83 -> 0.69 ms.
//
// Lanes of one expansion that meet in a set take turns: each turn one lane's
// compare-and-swap succeeds and the others look at the set again, so a node
// that stands twice in an adjacency row is taken once.  That needs the row in
// one turn (at most 64 ids).  The entry 0xFFFF marks a free place; the one
// node per set that would have it (16-bit entries only) is never remembered,
// and copies of it within a row are told apart by a vote.
struct VisitSets {
    unsigned long long *tab;
    int set_bits, rest_bits;
    uint32_t idmask;
    __device__ __forceinline__ VisitSets(uint32_t *t, int hash_bits, int id_bits)
        : tab(reinterpret_cast<unsigned long long *>(t)), set_bits(hash_bits - 1), rest_bits(id_bits - hash_bits + 1),
          idmask(id_bits >= 32 ? 0xFFFFFFFFu : (1u << id_bits) - 1u) {}
    __device__ __forceinline__ void clear() {
        for (int i = lane_id(); i < (1 << set_bits); i += 64) tab[i] = ~0ull;
    }
    __device__ __forceinline__ void mark_entry(uint32_t u) { (void)insert(u); }
    __device__ __forceinline__ void begin_hop(int) {}
    __device__ __forceinline__ void added(int) {}
    __device__ __forceinline__ int count() const { return 0; }
    __device__ __forceinline__ void restore(int) {}
    // whether one of a set's four entries is rest (twice = rest * 0x10001): a
    // 16-bit half of the difference is zero
    static __device__ __forceinline__ bool among(unsigned long long set, uint32_t twice) {
        const uint32_t a = (uint32_t)set ^ twice, b = (uint32_t)(set >> 32) ^ twice;
        return ((((a - 0x10001u) & ~a) | ((b - 0x10001u) & ~b)) & 0x80008000u) != 0u;
    }
    __device__ __forceinline__ bool holds(uint32_t u) const {
        const uint32_t h = (u * 2654435761u) & idmask, rest = h & ((1u << rest_bits) - 1u);
        return rest != 0xFFFFu && among(tab[h >> rest_bits], rest * 0x10001u);
    }
    __device__ __forceinline__ bool insert(uint32_t u) {
        const uint32_t h = (u * 2654435761u) & idmask;
        const uint32_t rest = h & ((1u << rest_bits) - 1u), twice = rest * 0x10001u;
        unsigned long long *p = tab + (h >> rest_bits);
        bool fresh = true;
        for (uint64_t m = ballot64(rest == 0xFFFFu); m; m &= m - 1) {
            const int src = (int)__builtin_ctzll(m);
            // readlane: the lanes after src compare with it, whichever are active
            const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)u, src);
            if (u == first && lane_id() > src) fresh = false;
        }
        if (rest == 0xFFFFu) return fresh;
        unsigned long long old = *p;
        for (;;) {
            if (among(old, twice)) return false;
            const unsigned long long got = atomicCAS(p, old, (old << 16) | rest);
            if (got == old) return true;
            old = got;
        }
    }
};

template <typename K>
struct QueueLds {
    K *qd;          // queue keys, ascending
    uint32_t *qi;   // queue ids, top bit = expanded
    K *cd;          // candidate batch keys
    uint32_t *ci;   // candidate batch ids
    K *sd;          // survivors (scratch)
    uint32_t *si;
    int32_t *slb;
};

template <typename K>
__device__ __forceinline__ int lower_bound_q(const K *qd, const uint32_t *qi, int qn, K kd, uint32_t kid) {
    int lo = 0, hi = qn;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (kless(qd[mid], qi[mid] & ~kExpanded, kd, kid))
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// #{t < S : slb[t] <= i}, slb non-decreasing
__device__ __forceinline__ int count_le(const int32_t *slb, int S, int i) {
    int lo = 0, hi = S;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (slb[mid] <= i)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Merge the candidate batch s.cd/s.ci[0..cnt) into the queue s.qd/s.qi[0..qn):
// keep the entries that beat the queue's last key (all, if the queue is not
// full) and are not already queued, order them, then move queue entries and
// survivors to their merged places, truncating at Leff.  The result is the
// best Leff of queue u batch, whatever the batch order.
//
// QR = queue capacity / 64: each lane holds QR of the entries that move.
// NEAR (E = 1): the keys are only known to within tol / 2; returns false, with
// the queue in any state, where two keys that a decision compares are within
// tol of each other (a batch that holds a queued node again, with its very
// key, is no such case).  Otherwise returns true.
//
// Up to 64 candidates (E = 1), one per lane: an expansion waits for each LDS
// access in turn, so what counts is how many follow one another.  The place in
// the queue takes one access per factor of four (three probes at once), the
// place among the survivors none (each is read out of its lane), and the
// merged places one bitmap: its bits are the survivors' places, and what lies
// at another place is the queue entry as many places earlier as there are bits
// before it.  Entries only move up, so they move in place from the end.  An
// expansion brings 37 candidates, of which 4 or 5 stay: a sort or binary
// searches took 4,400 to 8,200 cycles of its 11,000 to 40,000.  us before and
// after: FP32 10k x 64 L = 50, 1,000 queries 360 -> 315; E4M3 1M x 100 L = 200,
// 10,000 queries 4,290 -> 4,110; BF16 300k x 200 L = 200, 1,500 queries 2,200 ->
// 2,050.
// bits: kMaxSearchL / 32 words of LDS.  DUPS: a candidate may stand in several
// lanes; all but the first are dropped.
template <typename K, bool NEAR, bool DUPS>
__device__ __forceinline__ bool merge_held(K *qd, uint32_t *qi, uint32_t *bits, int Leff, int &qn, int &ptr, K kc,
                                           uint32_t ic, K tol) {
    static_assert(!DUPS || sizeof(K) == 4, "");
    int lane = lane_id();
    asm volatile("" : "+v"(lane));  // places per lane are cheaper to make than to keep in registers
    const bool full = qn == Leff;
    const K lastd = qd[qn - 1];
    const uint32_t lasti = qi[qn - 1] & ~kExpanded;
    bool sv = ic != kNone && (!full || kless(kc, ic, lastd, lasti));
    bool close = false;
    if constexpr (NEAR) close = full && ic != kNone && !(fabs(kc - lastd) > tol) && ic != lasti;
    if (ballot64(sv) == 0) {
        if constexpr (NEAR) return ballot64(close) == 0;
        return true;
    }
    int lb = 0;  // queue entries before this candidate
    // at most 1,023: a full queue of 1,024 has an entry behind every survivor
    for (int st = qn >= 256 ? 256 : qn >= 64 ? 64 : qn >= 16 ? 16 : qn >= 4 ? 4 : 1; st > 0; st >>= 2) {
        K k[3];
        uint32_t v[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int i = min(lb + (j + 1) * st, qn) - 1;
            k[j] = qd[i];
            v[j] = qi[i] & ~kExpanded;
        }
        int c = 0;
#pragma unroll
        for (int j = 0; j < 3; ++j) c += lb + (j + 1) * st <= qn && kless(k[j], v[j], kc, ic) ? 1 : 0;
        lb += c * st;
    }
    const int at = min(lb, qn - 1);
    if (sv) sv = lb >= qn || (qi[at] & ~kExpanded) != ic;  // not queued already
    if constexpr (NEAR) {
        const K ka = qd[at], kb = qd[max(lb - 1, 0)];
        close |= sv && ((lb > 0 && !(kc - kb > tol)) || (lb < qn && !(ka - kc > tol)));
        if (ballot64(close)) return false;
    }
    uint64_t all = ballot64(sv);
    if (all == 0) return true;
    int ahead = 0;
    if constexpr (sizeof(K) == 4) {
        // keys that order like (key, id)
        const uint32_t f = __float_as_uint(kc + 0.f), o = f ^ ((uint32_t)((int32_t)f >> 31) | 0x80000000u);
        const uint64_t mine = ((uint64_t)o << 32) | ic;
        for (;;) {
            bool dup = false;
            for (uint64_t m = all; m; m &= m - 1) {
                const int src = (int)__builtin_ctzll(m);
                const uint64_t other = ((uint64_t)lane_value(o, src) << 32) | lane_value(ic, src);
                ahead += other < mine ? 1 : 0;
                if constexpr (DUPS) dup |= sv && other == mine && src < lane;
            }
            if (!DUPS || ballot64(dup) == 0) break;
            sv = sv && !dup;
            all = ballot64(sv);
            ahead = 0;
        }
    } else {
        for (uint64_t m = all; m; m &= m - 1) {
            const int src = (int)__builtin_ctzll(m);
            const K ks = lane_value(kc, src);
            ahead += kless(ks, lane_value(ic, src), kc, ic) ? 1 : 0;
            if constexpr (NEAR) close |= sv && lane != src && !(fabs(ks - kc) > tol);
        }
    }
    if constexpr (NEAR) {
        if (ballot64(close)) return false;
    }
    const uint64_t head = ballot64(sv && ahead == 0);
    const int lbmin = head ? (int)lane_value((uint32_t)lb, (int)__builtin_ctzll(head)) : 0;
    const int to = lb + ahead, qn2 = min(Leff, qn + (int)__popcll(all));
    const bool stays = sv && to < Leff;
    // the bitmap of the survivors' places
    if (lane < kMaxSearchL / 32) bits[lane] = 0u;
    wave_sync();
    if (stays) atomicOr(&bits[to >> 5], 1u << (to & 31));
    wave_sync();
    const uint32_t word = lane < kMaxSearchL / 32 ? bits[lane] : 0u;
    int before = (int)__popcll(ballot64(stays));
    for (int r = (qn2 - 1) >> 6; r >= lbmin >> 6; --r) {
        const uint64_t w = ((uint64_t)lane_value(word, 2 * r + 1) << 32) | lane_value(word, 2 * r);
        before -= (int)__popcll(w);
        const int p = 64 * r + lane;
        const int i = max(0, min(p - before - lanes_below(w), qn - 1));  // (a lane past the queue reads an entry)
        const K md = qd[i];
        const uint32_t mi = qi[i];
        wave_sync();
        if (p >= lbmin && p < qn2 && !((w >> lane) & 1ull)) {
            qd[p] = md;
            qi[p] = mi;
        }
        wave_sync();
    }
    if (stays) {
        qd[to] = kc;
        qi[to] = ic;
    }
    qn = qn2;
    ptr = min(ptr, lbmin);
    wave_sync();
    return true;
}

template <typename K, bool NEAR>
__device__ __forceinline__ bool merge_one(const QueueLds<K> &s, int cnt, int Leff, int &qn, int &ptr, K tol) {
    const int lane = lane_id();
    const K kc = s.cd[lane];
    const uint32_t ic = lane < cnt ? s.ci[lane] : kNone;
    return merge_held<K, NEAR, false>(s.qd, s.qi, s.si, Leff, qn, ptr, kc, ic, tol);
}

template <int E, typename K, int QR = kMaxL / 64, bool NEAR = false>
__device__ __forceinline__ bool merge_batch(const QueueLds<K> &s, int cnt, int Leff, int &qn, int &ptr, K tol = (K)0) {
    static_assert(!NEAR || E == 1, "");
    if constexpr (E == 1) return merge_one<K, NEAR>(s, cnt, Leff, qn, ptr, tol);
    const int lane = lane_id();
    const bool full = qn == Leff;
    const K lastd = full ? s.qd[Leff - 1] : (K)0;
    const uint32_t lasti = full ? (s.qi[Leff - 1] & ~kExpanded) : 0u;
    int total = 0;
    if (full) {  // nothing to do unless some candidate beats the last entry
        bool any = false;
        for (int i = lane; i < cnt; i += 64) any |= kless(s.cd[i], s.ci[i], lastd, lasti);
        if (ballot64(any) == 0) return true;
    }
    {
        K k[E];
        uint32_t id[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = lane * E + e;
            k[e] = i < cnt ? s.cd[i] : (K)__builtin_inf();
            id[e] = i < cnt ? s.ci[i] : kNone;
        }
        wave_sort<E, K>(k, id);
        int lb[E];
        bool sv[E];
        int mine = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            sv[e] = id[e] != kNone && (!full || kless(k[e], id[e], lastd, lasti));
            lb[e] = 0;
            if (sv[e]) {
                lb[e] = lower_bound_q(s.qd, s.qi, qn, k[e], id[e]);
                if (lb[e] < qn && (s.qi[lb[e]] & ~kExpanded) == id[e]) sv[e] = false;  // already queued
            }
            mine += sv[e] ? 1 : 0;
        }
        // order-preserving compaction: exclusive prefix of per-lane counts
        int incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        total = __shfl(incl, 63);
        int w = incl - mine;
        wave_sync();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (sv[e]) {
                s.sd[w] = k[e];
                s.si[w] = id[e];
                s.slb[w] = lb[e];
                ++w;
            }
        }
        wave_sync();
        if (total == 0) return true;
    }
    const int lbmin = s.slb[0];
    // entries of the queue that move, and their new places
    constexpr int R = QR;
    K md[R];
    uint32_t mi[R];
    int mp[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = lbmin + lane + 64 * r;
        mp[r] = INT_MAX;
        if (i < qn) {
            md[r] = s.qd[i];
            mi[r] = s.qi[i];
            mp[r] = i + count_le(s.slb, total, i);
        }
    }
    K pd[2];
    uint32_t pi[2];
    int pp[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int t = lane + 64 * r;
        pp[r] = INT_MAX;
        if (t < total) {
            pd[r] = s.sd[t];
            pi[r] = s.si[t];
            pp[r] = s.slb[t] + t;
        }
    }
    wave_sync();
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (mp[r] < Leff) {
            s.qd[mp[r]] = md[r];
            s.qi[mp[r]] = mi[r];
        }
#pragma unroll
    for (int r = 0; r < 2; ++r)
        if (pp[r] < Leff) {
            s.qd[pp[r]] = pd[r];
            s.qi[pp[r]] = pi[r];
        }
    qn = min(Leff, qn + total);
    ptr = min(ptr, lbmin);
    wave_sync();
    return true;
}

}  // namespace rg
