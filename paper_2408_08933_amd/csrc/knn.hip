// Exact-kNN candidates on gfx950: S = Q X^T with FP32 MFMA
// (v_mfma_f32_16x16x4_f32), fused with a streaming top-K per query row, so
// the nq x n score matrix is never written.  This is the preprocessing step
// of index construction (the training queries' nearest base vectors,
// Algorithm 1 input) and the ground truth of recall@k (Def. 1).
//
// Workgroup = 4 wavefronts, a 128-query x 128-base output tile per step,
// each wavefront owning a 64 x 64 quarter as 4 x 4 MFMA blocks (64
// accumulator registers).  Operands are staged through LDS in 32-wide
// slices of the coordinate axis, row-major with a 4-float pad (16-byte
// writes and reads, conflict free for 16 lanes).  The contraction order is
// free, so in the slice's k-step t lane l supplies coordinate 8*(l/16) + t:
// each lane reads its 8 coordinates of a row with two 16-byte LDS loads.  A
// last slice shorter than 32 is stored permuted so that its data meet the
// first k-steps, and only ceil(rem / 4) k-steps run on it.
//
// Top-K: every query row of the tile keeps, in global memory, a buffer of up
// to CAP (score, id) pairs and in LDS an admission threshold (the K-th best
// score after the last compaction; -inf before).  Each score >= threshold is
// appended; a row whose buffer could overflow on the next tile is compacted
// by one wavefront (in-register bitonic sort of CAP pairs, keep K).  After a
// workgroup has swept its share of the base it sorts each row once more and
// writes the K best by (score desc, id asc).  When the base is split across
// workgroups, a merge kernel combines the per-split lists the same way.
#include "rg_internal.h"
#include "wave_ops.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>

namespace rg {
namespace {

typedef float fx4 __attribute__((ext_vector_type(4)));

constexpr int BQ = 128, BX = 128, KC = 32, KCP = KC + 4;
constexpr int CAP = 512;        // per-row candidate buffer
constexpr int CE = CAP / 64;    // pairs per lane when sorting a buffer

struct KnnArgs {
    const void *Q;  // FP32 rows (k_knn) or FP16 rows padded to whole tiles (k_knn16)
    const void *X;
    float *buf_sc;
    uint32_t *buf_id;
    float *out_sc;
    uint32_t *out_id;
    int64_t nq, n;
    int64_t q_tile0;
    int64_t xtiles, xtiles_per_split;
    int32_t ldq, ldx, d, K, splits;
    int32_t vec_q, vec_x;
};

__device__ __forceinline__ float4 ld4(const float *M, int64_t rows, int ld, int d, int64_t r, int k, bool vec) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (r >= rows) return v;
    const float *p = M + r * (int64_t)ld + k;
    if (vec && k + 3 < d) return *reinterpret_cast<const float4 *>(p);
    if (k + 0 < d) v.x = p[0];
    if (k + 1 < d) v.y = p[1];
    if (k + 2 < d) v.z = p[2];
    if (k + 3 < d) v.w = p[3];
    return v;
}

// Sort the row's buffer (count c) by (score desc, id asc) and keep K.
// Returns the new count; thr receives the K-th best score when c >= K.
__device__ __forceinline__ int compact_row(float *bsc, uint32_t *bid, int c, int K, float &thr) {
    const int lane = lane_id();
    float key[CE];
    uint32_t id[CE];
#pragma unroll
    for (int e = 0; e < CE; ++e) {
        const int i = lane * CE + e;
        key[e] = i < c ? -bsc[i] : __builtin_inff();
        id[e] = i < c ? bid[i] : kNone;
    }
    wave_sort<CE>(key, id);
#pragma unroll
    for (int e = 0; e < CE; ++e) {
        const int i = lane * CE + e;
        if (i < K && i < c) {
            bsc[i] = -key[e];
            bid[i] = id[e];
        }
    }
    const int src = (K - 1) / CE, se = (K - 1) % CE;
    float kth = 0.f;
#pragma unroll
    for (int e = 0; e < CE; ++e)
        if (e == se) kth = key[e];
    kth = __shfl(kth, src);
    if (c >= K) thr = -kth;
    return c < K ? c : K;
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_knn(KnnArgs a) {
    // two LDS buffers per operand: the MFMAs read one slice while the next is
    // stored into the other, one barrier per slice (73.7 KB per workgroup,
    // two workgroups per CU)
    __shared__ __align__(16) float As[2][BQ * KCP];
    __shared__ __align__(16) float Bs[2][BX * KCP];
    __shared__ float thr[BQ];
    __shared__ int cnt[BQ];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wr = w >> 1, wc = w & 1;
    const int64_t qt = a.q_tile0 + blockIdx.x;
    const int sp = blockIdx.y;
    const int64_t q0 = qt * BQ;
    const int64_t slot = (int64_t)blockIdx.x * a.splits + sp;
    float *bsc = a.buf_sc + slot * BQ * CAP;
    uint32_t *bid = a.buf_id + slot * BQ * CAP;
    const bool vq = a.vec_q != 0, vx = a.vec_x != 0;

    if (tid < BQ) {
        thr[tid] = -__builtin_inff();
        cnt[tid] = 0;
    }
    const int64_t xt0 = (int64_t)sp * a.xtiles_per_split;
    const int64_t xt1 = min(a.xtiles, xt0 + a.xtiles_per_split);
    const int lr = tid >> 3, lk = (tid & 7) * 4;
    const int kq = (lane >> 4) * 8;  // this lane's coordinates within a slice
    const int nsl = (a.d + KC - 1) / KC;
    float4 va[4], vb[4];
    // interior tiles and full slices load without bounds checks
    const float *Qf = static_cast<const float *>(a.Q), *Xf = static_cast<const float *>(a.X);
    const bool q_in = vq && q0 + BQ <= a.nq;
    const float *qrow = Qf + (q0 + lr) * (int64_t)a.ldq + lk;
    auto load_slice = [&](int64_t xt, int k0) {
        const int64_t x0 = xt * BX;
        if (q_in && vx && x0 + BX <= a.n && k0 + KC <= a.d) {
            const float *xrow = Xf + (x0 + lr) * (int64_t)a.ldx + lk + k0;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                va[p] = *reinterpret_cast<const float4 *>(qrow + (int64_t)p * 32 * a.ldq + k0);
                vb[p] = *reinterpret_cast<const float4 *>(xrow + (int64_t)p * 32 * a.ldx);
            }
            return;
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            va[p] = ld4(Qf, a.nq, a.ldq, a.d, q0 + p * 32 + lr, k0 + lk, vq);
            vb[p] = ld4(Xf, a.n, a.ldx, a.d, x0 + p * 32 + lr, k0 + lk, vx);
        }
    };
    // A partial last slice is stored permuted: coordinate c at position
    // 8 (c % 4) + c / 4, where k-step s of lane group g reads 8 g + s, so
    // step s meets coordinates 4 s .. 4 s + 3 and the steps past the data
    // can be skipped.
    auto store_slice = [&](int buf, bool tail) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int r = p * 32 + lr;
            if (!tail) {
                *reinterpret_cast<float4 *>(&As[buf][r * KCP + lk]) = va[p];
                *reinterpret_cast<float4 *>(&Bs[buf][r * KCP + lk]) = vb[p];
            } else {
                float *pa = &As[buf][r * KCP + (lk >> 2)], *pb = &Bs[buf][r * KCP + (lk >> 2)];
                pa[0] = va[p].x;
                pa[8] = va[p].y;
                pa[16] = va[p].z;
                pa[24] = va[p].w;
                pb[0] = vb[p].x;
                pb[8] = vb[p].y;
                pb[16] = vb[p].z;
                pb[24] = vb[p].w;
            }
        }
    };
    // The slices of consecutive tiles form one pipeline: the buffer parity
    // runs on across tiles, and the next tile's first slice is loaded while
    // the current tile's last slice is multiplied.
    int gsl = 0;
    if (xt0 < xt1) {
        load_slice(xt0, 0);
        store_slice(0, KC > a.d);
    }
    __syncthreads();
    for (int64_t xt = xt0; xt < xt1; ++xt) {
        const int64_t x0 = xt * BX;
        fx4 acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = fx4{0.f, 0.f, 0.f, 0.f};
        for (int sl = 0; sl < nsl; ++sl, ++gsl) {
            const int buf = gsl & 1;
            // the slice stored next: (xt, sl + 1), else the next tile's first
            const bool more = sl + 1 < nsl || xt + 1 < xt1;
            const bool more_tail = sl + 1 < nsl ? (sl + 2) * KC > a.d : KC > a.d;
            if (sl + 1 < nsl)
                load_slice(xt, (sl + 1) * KC);
            else if (xt + 1 < xt1)
                load_slice(xt + 1, 0);
            // k-steps of this slice: 8, or ceil(rem / 4) for a partial last one
            const int ns = (sl + 1) * KC <= a.d ? 8 : (a.d - sl * KC + 3) >> 2;
#pragma unroll 1
            for (int h = 0; h < 2 && 4 * h < ns; ++h) {
                float4 af[4], bf[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    af[i] = *reinterpret_cast<const float4 *>(
                        &As[buf][(wr * 64 + i * 16 + (lane & 15)) * KCP + kq + 4 * h]);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    bf[j] = *reinterpret_cast<const float4 *>(
                        &Bs[buf][(wc * 64 + j * 16 + (lane & 15)) * KCP + kq + 4 * h]);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (4 * h + t >= ns) break;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i][t], bf[j][t], acc[i][j], 0, 0, 0);
                }
            }
            if (more) store_slice(buf ^ 1, more_tail);
            __syncthreads();
        }
        // filter: accumulator element r of block (i, j) is row 4*(lane/16)+r, column lane%16
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = wr * 64 + i * 16 + 4 * (lane >> 4) + r;
                const float t = thr[row];
                const bool rok = q0 + row < a.nq;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t gx = x0 + wc * 64 + j * 16 + (lane & 15);
                    const float s = acc[i][j][r];
                    if (rok && gx < a.n && s >= t) {
                        const int pos = atomicAdd(&cnt[row], 1);
                        bsc[(int64_t)row * CAP + pos] = s;
                        bid[(int64_t)row * CAP + pos] = (uint32_t)gx;
                    }
                }
            }
        }
        __syncthreads();
        for (int row = w; row < BQ; row += 4) {
            const int c = cnt[row];
            if (c > CAP - BX) {
                float t = thr[row];
                const int nc = compact_row(bsc + (int64_t)row * CAP, bid + (int64_t)row * CAP, c, a.K, t);
                if (lane == 0) {
                    cnt[row] = nc;
                    thr[row] = t;
                }
            }
        }
        __syncthreads();
    }
    for (int row = w; row < BQ; row += 4) {
        const int64_t gq = q0 + row;
        if (gq >= a.nq) continue;
        float t = thr[row];
        float *rs = bsc + (int64_t)row * CAP;
        uint32_t *ri = bid + (int64_t)row * CAP;
        const int c = compact_row(rs, ri, cnt[row], a.K, t);
        float *os = a.out_sc + ((int64_t)sp * a.nq + gq) * a.K;
        uint32_t *oi = a.out_id + ((int64_t)sp * a.nq + gq) * a.K;
        for (int i = lane; i < a.K; i += 64) {
            os[i] = i < c ? rs[i] : -__builtin_inff();
            oi[i] = i < c ? ri[i] : kNone;
        }
    }
}

// ---------------------------------------------------------------------------
// FP16 candidate pass (v_mfma_f32_16x16x32_f16, FP32 accumulation).
//
// The rows arrive rounded to FP16 (round to nearest even) and packed by
// k_pack16 into blocks of 16 rows x 32 coordinates (1 KB, consecutive; a row
// block's coordinate blocks follow one another), zero padded to a multiple of
// 32 coordinates and to whole 128-row tiles.  Inside a block row j's 16-byte
// chunk c sits at 64 j + 16 (c ^ ((j >> 2) & 3)), so that the 16 lanes of a
// quarter-wave that read one chunk of 16 rows hit distinct LDS banks, and one
// global_load_lds moves a block from 1 KB of consecutive memory to 1 KB of
// consecutive LDS (row-major rows gave it 16 separate 64-byte pieces).
//
// In an MFMA k-step lane l supplies, for row (or column) l % 16, the 8
// coordinates 8 * (l / 16) .. + 7 of the block, the same coordinates for both
// operands.  The scores are FP32 sums of exact products of the rounded
// inputs; how far they may be from the exact ones is bounded in the
// certification (knn_exact).
//
// Two kernels find the K best rows of each query:
//   * k_scan16 (below) sweeps the base once against a threshold per query
//     that a sample of the base has given, and only collects what passes;
//   * k_knn16 keeps a running top-K instead, and serves the queries whose
//     threshold turned out wrong, and small bases.
//
// k_knn16: a workgroup owns 128 query rows and sweeps 128-row tiles of the
// base; its four wavefronts each hold a 64 x 64 quarter of the tile as 4 x 4
// blocks of 16 x 16 (64 accumulator registers).  At the FP16 matrix rate one
// 32-coordinate stage of a tile is only ~256 cycles of MFMA work per
// wavefront, far less than a load's latency, so the operands go straight from
// global memory into a ring of NST16 LDS stages (no registers involved): the
// loads of stage s + NST16 - 1 are issued while stage s is multiplied.  The
// filter and the per-row candidate buffers are those of k_knn above.
// ---------------------------------------------------------------------------
typedef _Float16 hx8 __attribute__((ext_vector_type(8)));

constexpr int BQ16 = 128, BX16 = 128, KS16 = 32, NST16 = 4;
constexpr int BLK16 = 16 * KS16;               // halves per packed block
constexpr int STAGE16 = (BQ16 + BX16) * KS16;  // halves per stage: A blocks, then B blocks

// s_waitcnt immediates: vmcnt [3:0] and [15:14], expcnt [6:4], lgkmcnt
// [11:8]; a field at its maximum does not wait.
constexpr int kWaitLgkm0 = 0xC07F;                       // LDS done, memory ops may be outstanding
__device__ __forceinline__ void wait_vm(int n) {         // at most n (0, 4 or 8) vector-memory ops outstanding
    if (n >= 8)
        __builtin_amdgcn_s_waitcnt(0x0F78);
    else if (n >= 4)
        __builtin_amdgcn_s_waitcnt(0x0F74);
    else
        __builtin_amdgcn_s_waitcnt(0x0F70);
}

// The LDS reads that follow the ring's loads are written as one asm block
// each, which waits for its own results: the compiler cannot tell which ring
// slot a global_load_lds writes and would otherwise wait for every load in
// flight before any LDS read, emptying the ring at each stage.  The stage
// loads are waited for by wait_vm above, before the barrier.
__device__ __forceinline__ void lds_frags(uint32_t a_addr, uint32_t b_addr, hx8 &a0, hx8 &a1, hx8 &a2, hx8 &a3,
                                          hx8 &b0, hx8 &b1, hx8 &b2, hx8 &b3) {
    asm volatile(
        "ds_read_b128 %0, %8\n\t"
        "ds_read_b128 %1, %8 offset:1024\n\t"
        "ds_read_b128 %2, %8 offset:2048\n\t"
        "ds_read_b128 %3, %8 offset:3072\n\t"
        "ds_read_b128 %4, %9\n\t"
        "ds_read_b128 %5, %9 offset:1024\n\t"
        "ds_read_b128 %6, %9 offset:2048\n\t"
        "ds_read_b128 %7, %9 offset:3072\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(a0), "=&v"(a1), "=&v"(a2), "=&v"(a3), "=&v"(b0), "=&v"(b1), "=&v"(b2), "=&v"(b3)
        : "v"(a_addr), "v"(b_addr)
        : "memory");
}

__device__ __forceinline__ fx4 lds_f4(uint32_t addr) {
    fx4 v;
    asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(addr) : "memory");
    return v;
}

__device__ __forceinline__ int lds_i32(uint32_t addr) {
    int v;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(addr) : "memory");
    return v;
}

__device__ __forceinline__ uint32_t lds_addr(const void *p) { return (uint32_t)(uintptr_t)p; }

// LDS append operations that leave the ring's loads in flight (see lds_frags)
__device__ __forceinline__ int lds_add(uint32_t addr, int v) {
    int old;
    asm volatile("ds_add_rtn_u32 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=&v"(old) : "v"(addr), "v"(v) : "memory");
    return old;
}

__device__ __forceinline__ void lds_store(uint32_t addr, uint32_t v) {
    asm volatile("ds_write_b32 %0, %1" : : "v"(addr), "v"(v) : "memory");
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_knn16(KnnArgs a) {
    __shared__ __align__(1024) _Float16 ring[NST16 * STAGE16];
    __shared__ __align__(16) float thr[BQ16];
    __shared__ int cnt[BQ16];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wr = w >> 1, wc = w & 1;
    const int64_t qt = a.q_tile0 + blockIdx.x;
    const int sp = blockIdx.y;
    const int64_t q0 = qt * BQ16;
    const int64_t slot = (int64_t)blockIdx.x * a.splits + sp;
    float *bsc = a.buf_sc + slot * BQ16 * CAP;
    uint32_t *bid = a.buf_id + slot * BQ16 * CAP;
    const _Float16 *Qh = static_cast<const _Float16 *>(a.Q), *Xh = static_cast<const _Float16 *>(a.X);

    if (tid < BQ16) {
        thr[tid] = -__builtin_inff();
        cnt[tid] = 0;
    }
    __syncthreads();
    const int64_t xt0 = (int64_t)sp * a.xtiles_per_split;
    const int64_t xt1 = min(a.xtiles, xt0 + a.xtiles_per_split);
    const int nks = a.d / KS16;  // d is the padded width here
    const int64_t nstage = (xt1 > xt0 ? xt1 - xt0 : 0) * nks;
    // wave w moves blocks 2w and 2w + 1 of both operands (rows 32 w .. 32 w + 31)
    const int64_t rb = (int64_t)nks * BLK16;  // halves of a row block
    const _Float16 *qsrc = Qh + (q0 / 16 + 2 * w) * rb + lane * 8;
    const _Float16 *xsrc = Xh + 2 * w * rb + lane * 8;
    // the next stage to load: block offset ik of the tile at xs, ring slot islot
    int ik = 0, islot = 0;
    const int64_t xtile = (BX16 / 16) * rb;
    const _Float16 *xs = xsrc + xt0 * xtile;
    auto issue = [&]() {
        _Float16 *dst = ring + islot * STAGE16 + 2 * w * BLK16;
        __builtin_amdgcn_global_load_lds(qsrc + ik, dst, 16, 0, 0);
        __builtin_amdgcn_global_load_lds(qsrc + ik + rb, dst + BLK16, 16, 0, 0);
        __builtin_amdgcn_global_load_lds(xs + ik, dst + BQ16 * KS16, 16, 0, 0);
        __builtin_amdgcn_global_load_lds(xs + ik + rb, dst + BQ16 * KS16 + BLK16, 16, 0, 0);
        islot = islot + 1 == NST16 ? 0 : islot + 1;
        ik += BLK16;
        if (ik == rb) {
            ik = 0;
            xs += xtile;
        }
    };
    for (int64_t g = 0; g < NST16 - 1 && g < nstage; ++g) issue();
    // fragment reads: block row fr of the wave's blocks, chunk fg (k-group)
    const int fr = lane & 15, fg = lane >> 4;
    const int foff = fr * 32 + ((fg ^ ((fr >> 2) & 3)) * 8);
    const uint32_t ring_a = lds_addr(ring + wr * 4 * 512 + foff);
    const uint32_t ring_b = lds_addr(ring + BQ16 * KS16 + wc * 4 * 512 + foff);
    int64_t g = 0;
    int cslot = 0;  // ring slot of stage g
    for (int64_t xt = xt0; xt < xt1; ++xt) {
        const int64_t x0 = xt * BX16;
        fx4 acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = fx4{0.f, 0.f, 0.f, 0.f};
        for (int ks = 0; ks < nks; ++ks, ++g) {
            // stage g has landed once at most the later stages' loads (4 per
            // stage) are outstanding; the barrier then also tells every wave
            // that all waves are done with slot (g - 1) % NST16
            wait_vm(4 * (int)min<int64_t>(NST16 - 2, nstage - 1 - g));
            __builtin_amdgcn_s_barrier();
            if (g + NST16 - 1 < nstage) issue();
            const uint32_t so = (uint32_t)cslot * STAGE16 * 2;
            cslot = cslot + 1 == NST16 ? 0 : cslot + 1;
            hx8 af[4], bf[4];
            lds_frags(ring_a + so, ring_b + so, af[0], af[1], af[2], af[3], bf[0], bf[1], bf[2], bf[3]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[i], bf[j], acc[i][j], 0, 0, 0);
        }
        // filter: accumulator element r of block (i, j) is query row
        // 16 i + 4 (lane / 16) + r of the wave's half, base column lane % 16
        bool stored = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int rb = wr * 64 + i * 16 + 4 * (lane >> 4);
            const fx4 t4 = lds_f4(lds_addr(&thr[rb]));
            bool hit = false;
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < 4; ++j) hit |= acc[i][j][r] >= t4[r];
            if (!__builtin_amdgcn_ballot_w64(hit)) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = rb + r;
                const bool rok = q0 + row < a.nq;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int64_t gx = x0 + wc * 64 + j * 16 + fr;
                    const float sc = acc[i][j][r];
                    if (rok && gx < a.n && sc >= t4[r]) {
                        const int pos = atomicAdd(&cnt[row], 1);
                        bsc[(int64_t)row * CAP + pos] = sc;
                        bid[(int64_t)row * CAP + pos] = (uint32_t)gx;
                        stored = true;
                    }
                }
            }
        }
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        __builtin_amdgcn_s_barrier();
        // rows w, w + 4, ..: lane l < 32 looks at row w + 4 l; compaction of a
        // row whose buffer could overflow on the next tile (rare)
        const int myc = lane < BQ16 / 4 ? lds_i32(lds_addr(&cnt[w + 4 * lane])) : 0;
        uint64_t full = __builtin_amdgcn_ballot_w64(myc > CAP - BX16);
        while (full) {
            const int l = __builtin_ctzll(full);
            full &= full - 1;
            const int row = w + 4 * l;
            float t = thr[row];
            const int nc = compact_row(bsc + (int64_t)row * CAP, bid + (int64_t)row * CAP, cnt[row], a.K, t);
            stored = true;
            if (lane == 0) {
                cnt[row] = nc;
                thr[row] = t;
            }
        }
        // the candidate stores count in the same counter as the stage
        // loads; drain them so the waits above keep their meaning.  The
        // kernel issues no other vector-memory operation (no register
        // spills; the build checks that it uses no scratch)
        if (__builtin_amdgcn_ballot_w64(stored)) __builtin_amdgcn_s_waitcnt(0x0F70);
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        __builtin_amdgcn_s_barrier();
    }
    __syncthreads();
    for (int row = w; row < BQ16; row += 4) {
        const int64_t gq = q0 + row;
        if (gq >= a.nq) continue;
        float t = thr[row];
        float *rs = bsc + (int64_t)row * CAP;
        uint32_t *ri = bid + (int64_t)row * CAP;
        const int c = compact_row(rs, ri, cnt[row], a.K, t);
        float *os = a.out_sc + ((int64_t)sp * a.nq + gq) * a.K;
        uint32_t *oi = a.out_id + ((int64_t)sp * a.nq + gq) * a.K;
        for (int i = lane; i < a.K; i += 64) {
            os[i] = i < c ? rs[i] : -__builtin_inff();
            oi[i] = i < c ? ri[i] : kNone;
        }
    }
}

// s_waitcnt vmcnt(N): at most N vector-memory operations outstanding
template <int N>
__device__ __forceinline__ void wait_vm_const() {
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// LDS reads of one operand's four blocks, one asm block for the reason given
// at lds_frags.
__device__ __forceinline__ void lds_frags4(uint32_t addr, hx8 &b0, hx8 &b1, hx8 &b2, hx8 &b3) {
    asm volatile(
        "ds_read_b128 %0, %4\n\t"
        "ds_read_b128 %1, %4 offset:1024\n\t"
        "ds_read_b128 %2, %4 offset:2048\n\t"
        "ds_read_b128 %3, %4 offset:3072\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(b0), "=&v"(b1), "=&v"(b2), "=&v"(b3)
        : "v"(addr)
        : "memory");
}

// ---------------------------------------------------------------------------
// One sweep of the base against known thresholds.
//
// A running top-K costs far more than the products it sorts: each split of
// the base starts from nothing, admits about K (1 + ln(rows / K)) rows per
// query, sorts the row's buffer every CAP - K of them, and every store makes
// the wave drain its load ring.  On 10k x 1M x 200 (K = 200) k_knn16 took 53
// ms, 44 us per 128 x 128 tile, of which the products are 1.5.  So the
// threshold is found first, from the scores of every s-th base row (s = K /
// 12, 6% of the products at K = 200): the r-th best of the sample, r = E + 5
// sqrt(E) + 4 with E = K / s, is passed by the K best rows of the base except
// with a chance of about 1e-6 for rows in no particular order, and by about r
// s rows in all.  The sweep then only compares, which needs neither sorts nor
// stores until something passes: what passes goes to a queue in LDS and from
// there to the query's buffer in batches.  k_pick16 sorts each buffer and
// keeps the K best; a query with fewer than K or more than SCAP entries goes
// to k_knn16, so the result never depends on the sample.
//
// 10k x 1M x 200: 6.4 ms for the sweep (700 TFLOP/s on the padded 224
// coordinates) + 0.32 sample + 0.04 thresholds + 0.29 k_pick16, against 53 ms.
//
// Because the thresholds stay, the base can be split freely: workgroups are
// cut to fill the chip (choose_splits).  For d <= 224 the query fragments of
// a wavefront (64 rows) stay in registers for the whole sweep (NKS * 16
// registers) and only the base goes through LDS, which halves the LDS reads
// (with both operands in LDS they need the full LDS rate at the full matrix
// rate); NKS = 0 is the kernel for any width, both operands in the ring
// (at 256 coordinates the fragments no longer fit beside the accumulators).
//
// SAMPLE: no threshold; each lane keeps the best score of each of its query
// rows over T tiles of the sample (a group of 4 T sample rows) and writes it
// to gm.  The r-th largest group maximum is a lower bound of the r-th largest
// score, and close to it: the r best rows seldom share a group.
// ---------------------------------------------------------------------------
constexpr int NSTS = 8;              // ring stages when only the base is staged (8 KB each)
constexpr int SQ = 1024;             // entries of the LDS queue
constexpr int SCAP = 2048;           // entries of a query's buffer

struct ScanArgs {
    const _Float16 *Q;   // packed rows
    const _Float16 *X;   // packed rows of the base, or of the sample
    const float *thr;    // per query row (whole tiles; +inf past nq)
    float *buf_sc;       // row x SCAP
    uint32_t *buf_id;
    uint32_t *cnt;       // per query row: entries that passed (may exceed SCAP)
    float *gm;           // SAMPLE: row x ngroups
    int64_t n;           // rows of X
    int64_t units, units_per_split;  // tiles of X, or (SAMPLE) groups of T tiles
    int32_t qtiles, nks, T, ngroups;
};

template <int NKS, bool SAMPLE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_scan16(ScanArgs a) {
    constexpr bool AREG = NKS > 0;                       // query fragments in registers
    constexpr int NST = AREG ? NSTS : NST16;             // ring stages
    constexpr int LPS = AREG ? 2 : 4;                    // loads per stage and wave
    constexpr int STG = AREG ? BX16 * KS16 : STAGE16;    // halves per stage
    __shared__ __align__(1024) _Float16 ring[NST * STG];
    __shared__ float q_sc[SAMPLE ? 1 : SQ];
    __shared__ uint32_t q_id[SAMPLE ? 1 : SQ], q_row[SAMPLE ? 1 : SQ];
    __shared__ int q_n;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wr = w >> 1, wc = w & 1;
    const int qt = (int)(blockIdx.x % (unsigned)a.qtiles);
    const int sp = (int)(blockIdx.x / (unsigned)a.qtiles);
    const int64_t q0 = (int64_t)qt * BQ16;
    const int nks = AREG ? NKS : a.nks;
    const int64_t rb = (int64_t)nks * BLK16;
    // n < 2^31: tile and stage counts of a split fit 32 and 64 bits
    const int xtiles = (int)((a.n + BX16 - 1) / BX16);
    const int per = (int)a.units_per_split * (SAMPLE ? a.T : 1);
    const int xt0 = sp * per, xt1 = min(xtiles, xt0 + per);
    const int64_t nstage = (int64_t)(xt1 > xt0 ? xt1 - xt0 : 0) * nks;
    const int fr = lane & 15, fg = lane >> 4;
    const int foff = fr * 32 + ((fg ^ ((fr >> 2) & 3)) * 8);  // this lane's chunk of a block

    if (tid == 0) q_n = 0;
    float thr[4][4];  // SAMPLE: the running maxima
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            thr[i][r] = SAMPLE ? -__builtin_inff() : a.thr[q0 + wr * 64 + i * 16 + 4 * fg + r];
    hx8 A[4][AREG ? NKS : 1];
    if constexpr (AREG) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
                A[i][ks] = *reinterpret_cast<const hx8 *>(a.Q + (q0 / 16 + wr * 4 + i) * rb + ks * BLK16 + foff);
    }
    __syncthreads();  // q_n; the plain loads above are done before the ring starts

    const _Float16 *qsrc = a.Q + (q0 / 16 + 2 * w) * rb + lane * 8;
    int ik = 0, islot = 0;
    const int64_t xtile = (BX16 / 16) * rb;
    const _Float16 *xs = a.X + xt0 * xtile + 2 * w * rb + lane * 8;
    int64_t issued = 0;
    auto issue = [&]() {
        _Float16 *dst = ring + islot * STG + 2 * w * BLK16;
        if constexpr (!AREG) {
            __builtin_amdgcn_global_load_lds(qsrc + ik, dst, 16, 0, 0);
            __builtin_amdgcn_global_load_lds(qsrc + ik + rb, dst + BLK16, 16, 0, 0);
            dst += BQ16 * KS16;
        }
        __builtin_amdgcn_global_load_lds(xs + ik, dst, 16, 0, 0);
        __builtin_amdgcn_global_load_lds(xs + ik + rb, dst + BLK16, 16, 0, 0);
        islot = islot + 1 == NST ? 0 : islot + 1;
        ++issued;
        ik += BLK16;
        if (ik == rb) {
            ik = 0;
            xs += xtile;
        }
    };
    wait_vm_const<0>();
    for (int g = 0; g < NST - 1 && g < nstage; ++g) issue();
    const uint32_t ring_a = lds_addr(ring + wr * 4 * BLK16 + foff);
    const uint32_t ring_b = lds_addr(ring + (AREG ? 0 : BQ16 * KS16) + wc * 4 * BLK16 + foff);
    int64_t g = 0;
    int cslot = 0;
    // stage g has landed when at most the later stages' loads are outstanding;
    // the barrier then also tells every wave that all are done with the slot
    // that the next issue fills
    auto next_stage = [&]() -> uint32_t {
        if (issued - g >= NST - 1)
            wait_vm_const<LPS *(NST - 2)>();
        else
            wait_vm_const<0>();
        __builtin_amdgcn_s_barrier();
        if (issued < nstage) issue();
        const uint32_t so = (uint32_t)cslot * STG * 2;
        cslot = cslot + 1 == NST ? 0 : cslot + 1;
        ++g;
        return so;
    };
    // empty the LDS queue into the queries' buffers (all waves)
    auto flush = [&](int n) {
        n = min(n, SQ);
        for (int e = tid; e < n; e += 256) {
            const int64_t row = q0 + q_row[e];
            const uint32_t pos = atomicAdd(&a.cnt[row], 1u);
            if (pos < SCAP) {
                a.buf_sc[row * SCAP + pos] = q_sc[e];
                a.buf_id[row * SCAP + pos] = q_id[e];
            }
        }
        wait_vm_const<0>();  // stores and atomics count in the ring's counter
        __syncthreads();
        if (tid == 0) q_n = 0;
        __syncthreads();
    };
    for (int xt = xt0; xt < xt1; ++xt) {
        const int64_t x0 = (int64_t)xt * BX16;
        fx4 acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = fx4{0.f, 0.f, 0.f, 0.f};
        auto step = [&](const hx8(&af)[4], const hx8(&bf)[4]) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[i], bf[j], acc[i][j], 0, 0, 0);
        };
        if constexpr (AREG) {
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                const uint32_t so = next_stage();
                if (ks == 0 && !SAMPLE) {
                    // the barrier of this stage follows every append of the last
                    // tile, and another barrier follows before the next append
                    const int qn = lds_i32(lds_addr(&q_n));
                    if constexpr (NKS == 1) __builtin_amdgcn_s_barrier();
                    if (qn >= SQ / 2) flush(qn);
                }
                hx8 bf[4];
                lds_frags4(ring_b + so, bf[0], bf[1], bf[2], bf[3]);
                const hx8 af[4] = {A[0][ks], A[1][ks], A[2][ks], A[3][ks]};
                step(af, bf);
            }
        } else {
            for (int ks = 0; ks < nks; ++ks) {
                const uint32_t so = next_stage();
                if (ks == 0 && !SAMPLE) {
                    const int qn = lds_i32(lds_addr(&q_n));  // nks > 7 here: a barrier follows
                    if (qn >= SQ / 2) flush(qn);
                }
                hx8 af[4], bf[4];
                lds_frags(ring_a + so, ring_b + so, af[0], af[1], af[2], af[3], bf[0], bf[1], bf[2], bf[3]);
                step(af, bf);
            }
        }
        // accumulator element r of block (i, j) is query row 16 i + 4 (lane / 16)
        // + r of the wave's half, base column lane % 16 of its block
        if constexpr (SAMPLE) {
            const int rows = (int)std::min<int64_t>(a.n - x0, BX16);
            int col0 = wc * 64 + fr;
            asm volatile("" : "+v"(col0));  // no column kept over the sweep
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool ok = col0 + j * 16 < rows;
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) thr[i][r] = fmaxf(thr[i][r], ok ? acc[i][j][r] : -__builtin_inff());
            }
            if ((xt + 1) % a.T == 0 || xt + 1 == xt1) {
                int row0 = wr * 64 + 4 * fg;
                asm volatile("" : "+v"(row0));  // no address kept over the sweep
                int grp = wc * 16 + fr;
                asm volatile("" : "+v"(grp));
                grp += xt / a.T * 32;
                float *g0 = a.gm + (q0 + row0) * a.ngroups + grp;
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        *g0 = thr[i][r];
                        thr[i][r] = -__builtin_inff();
                        g0 += r < 3 ? a.ngroups : 13 * a.ngroups;
                        asm volatile("" : "+v"(g0));  // one address at a time
                    }
                wait_vm_const<0>();
            }
        } else {
            bool any = false;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    any |= fmaxf(fmaxf(acc[i][0][r], acc[i][1][r]), fmaxf(acc[i][2][r], acc[i][3][r])) >= thr[i][r];
            if (__builtin_amdgcn_ballot_w64(any)) {
                bool direct = false;
                // opaque to the compiler, which would otherwise compute the
                // addresses of all 64 appends ahead of the sweep and spill
                int row0 = wr * 64 + 4 * fg, col0 = wc * 64 + fr;
                asm volatile("" : "+v"(row0), "+v"(col0));
                const uint32_t gx0 = (uint32_t)xt * BX16 + (uint32_t)col0, nx = (uint32_t)a.n;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = row0 + i * 16 + r;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const uint32_t gx = gx0 + j * 16;
                            const float sc = acc[i][j][r];
                            if (sc >= thr[i][r] && gx < nx) {
                                const int pos = lds_add(lds_addr(&q_n), 1);
                                if (pos < SQ) {
                                    lds_store(lds_addr(&q_sc[pos]), __float_as_uint(sc));
                                    lds_store(lds_addr(&q_id[pos]), gx);
                                    lds_store(lds_addr(&q_row[pos]), (uint32_t)row);
                                } else {  // the queue is full: straight to the buffer
                                    const uint32_t p = atomicAdd(&a.cnt[q0 + row], 1u);
                                    if (p < SCAP) {
                                        a.buf_sc[(q0 + row) * SCAP + p] = sc;
                                        a.buf_id[(q0 + row) * SCAP + p] = gx;
                                    }
                                    direct = true;
                                }
                            }
                        }
                    }
                }
                if (__builtin_amdgcn_ballot_w64(direct)) wait_vm_const<0>();
                __builtin_amdgcn_s_waitcnt(kWaitLgkm0);  // appends done before the next barrier
            }
        }
    }
    if constexpr (!SAMPLE) {
        __syncthreads();
        flush(q_n);
    }
}

// The threshold of each query row: the r-th largest of its G group maxima
// (at most 64 * KTH_E), found bit by bit on an order-preserving integer form;
// the lowest 8 bits are left clear (a slightly lower threshold).  Rows past nq
// get +inf.  One wavefront per row.
constexpr int KTH_E = 32;
__global__ __launch_bounds__(64) void k_kth16(const float *gm, int G, int r, int64_t nq, float *thr) {
    const int64_t q = blockIdx.x;
    const int lane = lane_id();
    if (q >= nq) {
        if (lane == 0) thr[q] = __builtin_inff();
        return;
    }
    uint32_t u[KTH_E];
#pragma unroll
    for (int e = 0; e < KTH_E; ++e) {
        const int i = e * 64 + lane;
        const uint32_t b = i < G ? __float_as_uint(gm[q * G + i]) : 0xFF800000u;
        u[e] = b ^ ((b & 0x80000000u) ? 0xFFFFFFFFu : 0x80000000u);
    }
    uint32_t t = 0;
    for (int bit = 31; bit >= 8; --bit) {
        const uint32_t c = t | (1u << bit);
        int have = 0;
#pragma unroll
        for (int e = 0; e < KTH_E; ++e) have += (int)__popcll(ballot64(u[e] >= c));
        if (have >= r) t = c;
    }
    if (lane == 0) {
        const uint32_t b = (t & 0x80000000u) ? t ^ 0x80000000u : ~t;
        // fewer than r finite groups (t at or below the form of -inf): no threshold
        thr[q] = t <= 0x007FFFFFu ? -__builtin_inff() : __uint_as_float(b);
    }
}

// The K best entries of each query's buffer by (score desc, id asc); a query
// whose buffer holds fewer than K entries or overflowed is listed in fail.
// One wavefront per row.
template <int E>
__device__ __forceinline__ void pick_sorted(const float *bsc, const uint32_t *bid, int c, int K, float *os,
                                            uint32_t *oi) {
    const int lane = lane_id();
    float key[E];
    uint32_t id[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = e * 64 + lane;  // the sort takes any placement
        key[e] = i < c ? -bsc[i] : __builtin_inff();
        id[e] = i < c ? bid[i] : kNone;
    }
    wave_sort<E>(key, id);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = lane * E + e;
        if (i < K) {
            os[i] = -key[e];
            oi[i] = id[e];
        }
    }
}

__global__ __launch_bounds__(64) void k_pick16(const float *buf_sc, const uint32_t *buf_id, const uint32_t *cnt,
                                              int64_t row0, int K, float *out_sc, uint32_t *out_id, uint32_t *fail,
                                              uint32_t *n_fail) {
    const int64_t q = blockIdx.x;
    const uint32_t c = cnt[q];
    if (c < (uint32_t)K || c > (uint32_t)SCAP) {
        if (lane_id() == 0) fail[atomicAdd(n_fail, 1u)] = (uint32_t)(row0 + q);
        return;
    }
    const float *bsc = buf_sc + q * SCAP;
    const uint32_t *bid = buf_id + q * SCAP;
    float *os = out_sc + (row0 + q) * K;
    uint32_t *oi = out_id + (row0 + q) * K;
    if (c <= 512)
        pick_sorted<8>(bsc, bid, (int)c, K, os, oi);
    else if (c <= 1024)
        pick_sorted<16>(bsc, bid, (int)c, K, os, oi);
    else
        pick_sorted<32>(bsc, bid, (int)c, K, os, oi);
}

// Packed rows list[0..m) of src into dst (rows of dp coordinates, rows past
// m zero); one workgroup per packed row block of dst.
__global__ __launch_bounds__(256) void k_gather16(const _Float16 *src, const uint32_t *list, int64_t m, int nks,
                                                 _Float16 *dst) {
    const int64_t b = blockIdx.x;
    for (int i = threadIdx.x; i < nks * 64; i += 256) {
        const int ks = i >> 6, l = i & 63, j = l >> 2, c = (l & 3) ^ ((j >> 2) & 3);
        const int64_t r = b * 16 + j;
        hx8 v = {};
        if (r < m) {
            const int64_t s = list[r];
            const int sj = (int)(s & 15);
            v = *reinterpret_cast<const hx8 *>(src + ((s >> 4) * nks + ks) * BLK16 +
                                               (sj * 4 + (c ^ ((sj >> 2) & 3))) * 8);
        }
        *reinterpret_cast<hx8 *>(dst + (b * nks + ks) * BLK16 + l * 8) = v;
    }
}

// Lists of the rows list[0..m) (m x K) back to their places.
__global__ __launch_bounds__(64) void k_scatter_lists(const uint32_t *list, int K, const float *sc,
                                                     const uint32_t *id, float *out_sc, uint32_t *out_id) {
    const int64_t r = blockIdx.x, q = list[r];
    for (int i = lane_id(); i < K; i += 64) {
        out_sc[q * K + i] = sc[r * K + i];
        out_id[q * K + i] = id[r * K + i];
    }
}

__global__ __launch_bounds__(64) void k_gather_rows(const float *src, const uint32_t *list, int32_t d, float *dst) {
    const int64_t r = blockIdx.x, q = list[r];
    for (int i = lane_id(); i < d; i += 64) dst[r * d + i] = src[q * d + i];
}

__global__ void k_fill_words(uint32_t *p, int64_t n, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// FP32 rows -> packed FP16 (round to nearest even), zeros past (rows, d) up
// to rows_pad x 32 nks (dst; null: none), and in the same pass over the rows
// what the choice of pass and the certificate need: the largest |element|, the
// largest squared row norm (FP64), whether some element is not below 2^15 in
// magnitude (a NaN included), and whether row 0's norm is a NaN.  Every s-th row is also
// written to the sample, packed the same way (dst_s, when s > 0).  Sixteen
// threads per row, each 8 coordinates at a time; bound by memory: 0.30 ms for
// 1M x 200 (1.28 GB moved, 4.3 TB/s).
__global__ __launch_bounds__(256) void k_pack16(const float *src, int64_t rows, int32_t d, int64_t ld, bool vec,
                                               _Float16 *dst, int64_t rows_pad, int32_t nks, _Float16 *dst_s,
                                               int32_t s, PackStats *st) {
    __shared__ double sh_n[16];
    __shared__ float sh_a[16];
    const int j = threadIdx.x >> 4, t = threadIdx.x & 15;
    double best = 0.0;
    float amax = 0.f;
    bool bad = false, nan0 = false;
    for (int64_t b = blockIdx.x; b * 16 < rows_pad; b += gridDim.x) {
        const int64_t r = b * 16 + j;
        const bool live = r < rows;
        const float *p = src + (live ? r : 0) * ld;
        double n2 = 0.0;
        const bool samp = s > 0 && live && r % s == 0;
        const int64_t rs = samp ? r / s : 0;
        for (int c = t; c < nks * 4; c += 16) {
            float v[8];
            if (live && vec && 8 * c + 8 <= d) {
                const float4 x = *reinterpret_cast<const float4 *>(p + 8 * c);
                const float4 y = *reinterpret_cast<const float4 *>(p + 8 * c + 4);
                v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
                v[4] = y.x, v[5] = y.y, v[6] = y.z, v[7] = y.w;
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = live && 8 * c + i < d ? p[8 * c + i] : 0.f;
            }
            hx8 h;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                h[i] = (_Float16)v[i];
                n2 = fma((double)v[i], (double)v[i], n2);
                amax = fmaxf(amax, fabsf(v[i]));
                bad |= !(fabsf(v[i]) < 32768.f);
            }
            if (dst)
                *reinterpret_cast<hx8 *>(dst + (b * nks + (c >> 2)) * BLK16 + (4 * j + ((c & 3) ^ ((j >> 2) & 3))) * 8) = h;
            if (samp) {
                const int sj = (int)(rs & 15);
                *reinterpret_cast<hx8 *>(dst_s + ((rs >> 4) * nks + (c >> 2)) * BLK16 +
                                         (4 * sj + ((c & 3) ^ ((sj >> 2) & 3))) * 8) = h;
            }
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
        if (r == 0 && n2 != n2) nan0 = true;
        best = fmax(best, n2);  // a NaN norm is passed over
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        best = fmax(best, __shfl_xor(best, o));
        amax = fmaxf(amax, __shfl_xor(amax, o));
    }
    const uint64_t bm = ballot64(bad), nm = ballot64(nan0);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sh_n[w] = best;
        sh_a[w] = amax;
        if (bm) atomicOr(&st->bad, 1u);
        if (nm) atomicOr(&st->nan0, 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < 4; ++i) {
            best = fmax(best, sh_n[i]);
            amax = fmaxf(amax, sh_a[i]);
        }
        // the bits of values that are not negative order like the values
        atomicMax(&st->norm2, (unsigned long long)__double_as_longlong(best));
        atomicMax(&st->amax, __float_as_uint(amax));
    }
}

// Merge per-split top-K lists into one (one wavefront per query row).
__global__ __launch_bounds__(64) void k_knn_merge(const float *sc, const uint32_t *id, int64_t nq, int K,
                                                  int splits, float *out_sc, uint32_t *out_id) {
    const int64_t q = blockIdx.x;
    const int lane = lane_id();
    float key[CE];
    uint32_t v[CE];
    // running list occupies slots [0, K); the next split's list [K, 2K)
#pragma unroll
    for (int e = 0; e < CE; ++e) {
        const int i = lane * CE + e;
        key[e] = i < K ? -sc[q * K + i] : __builtin_inff();
        v[e] = i < K ? id[q * K + i] : kNone;
    }
    for (int s = 1; s < splits; ++s) {
        const float *ss = sc + ((int64_t)s * nq + q) * K;
        const uint32_t *si = id + ((int64_t)s * nq + q) * K;
#pragma unroll
        for (int e = 0; e < CE; ++e) {
            const int i = lane * CE + e;
            if (i >= K) {
                key[e] = i < 2 * K ? -ss[i - K] : __builtin_inff();
                v[e] = i < 2 * K ? si[i - K] : kNone;
            }
        }
        wave_sort<CE>(key, v);
    }
#pragma unroll
    for (int e = 0; e < CE; ++e) {
        const int i = lane * CE + e;
        if (i < K) {
            out_sc[q * K + i] = -key[e];
            out_id[q * K + i] = v[e];
        }
    }
}

// Certification of the exact k nearest rows from the FP32 candidates (one
// wavefront per query row).  Each lane rescores its candidates with the
// canonical distance delta = -sum_i q_i x_i, a chain of FP64 fused
// multiply-adds in increasing i (the products of floats are exact in FP64,
// so every step rounds like a plain FP64 add and the value equals the host's
// sum bit for bit), the wave sorts (delta, id) ascending, and the row is
// certified when the K-th candidate's FP32 score plus the error bound of
// both sums is below the k-th canonical score: no row outside the candidate
// list can then be among the k nearest.
constexpr int CERT_E = 4;  // candidates per lane (K <= 256)

struct CertArgs {
    const float *Q;
    const float *X;
    const uint32_t *cid;  // m x K, FP32 score descending
    const float *csc;
    const uint32_t *map;  // row r's place in the outputs, or null: r
    uint32_t *out_id;     // rows of k
    float *out_d;         // rows of k (the FP64 distance rounded), or null
    uint32_t *fail;       // places of the rows not certified
    uint32_t *n_fail;
    int64_t m, n, ldq, ldx;
    int32_t d, K, k;
    double gsum, xmax;  // relative error bound factor of the candidate scores (and the canonical sum), max row norm
    double eta, abs0;   // absolute part of that bound: eta * (|t| + xmax) + abs0 (FP16 underflow)
};

__device__ __forceinline__ double canon_dot(const float *qs, const float *row, int d) {
    double s = 0.0;
    for (int i = 0; i < d; ++i) s = fma((double)qs[i], (double)row[i], s);
    return s;
}

__global__ __launch_bounds__(64) void k_knn_certify(CertArgs a) {
    extern __shared__ float qs[];
    const int64_t r = blockIdx.x;
    const int lane = lane_id();
    const float *q = a.Q + r * a.ldq;
    for (int i = lane; i < a.d; i += 64) qs[i] = q[i];
    __syncthreads();
    // candidate c = lane + 64 e (the sort takes any placement)
    double key[CERT_E];
    uint32_t id[CERT_E];
    int valid = 0;
#pragma unroll
    for (int e = 0; e < CERT_E; ++e) {
        const int c = lane + 64 * e;
        key[e] = __builtin_inf();
        id[e] = kNone;
        if (c < a.K) {
            const uint32_t u = a.cid[r * a.K + c];
            if (u != kNone) {
                id[e] = u;
                key[e] = -canon_dot(qs, a.X + (int64_t)u * a.ldx, a.d);
                ++valid;
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) valid += __shfl_xor(valid, o);
    wave_sort<CERT_E, double>(key, id);
    bool certified = (int64_t)a.K >= a.n;
    if (!certified && valid >= a.k) {
        double tn = 0.0;
        for (int i = 0; i < a.d; ++i) tn = fma((double)qs[i], (double)qs[i], tn);
        const double tnorm = sqrt(tn) * (1.0 + 1e-12);
        const double tau = a.gsum * tnorm * a.xmax + a.eta * (tnorm + a.xmax) + a.abs0;
        const double sigma = (double)a.csc[r * a.K + a.K - 1];
        const int src = (a.k - 1) / CERT_E, se = (a.k - 1) % CERT_E;
        double kth = 0.0;
#pragma unroll
        for (int e = 0; e < CERT_E; ++e)
            if (e == se) kth = key[e];
        kth = __shfl(kth, src);
        certified = sigma + tau < -kth;
    }
    const int64_t to = a.map ? a.map[r] : r;
    if (!certified) {
        if (lane == 0) a.fail[atomicAdd(a.n_fail, 1u)] = (uint32_t)to;
        return;
    }
#pragma unroll
    for (int e = 0; e < CERT_E; ++e) {
        const int j = lane * CERT_E + e;
        if (j < a.k) {
            a.out_id[to * a.k + j] = j < valid ? id[e] : kNone;
            if (a.out_d) a.out_d[to * a.k + j] = j < valid ? (float)key[e] : __builtin_inff();
        }
    }
}

}  // namespace

namespace {

// One device allocation handed out in 256-byte aligned parts.
struct DevMem {
    char *p = nullptr;
    size_t at = 0;
    DevMem() = default;
    DevMem(const DevMem &) = delete;
    DevMem &operator=(const DevMem &) = delete;
    ~DevMem() {
        if (p) (void)hipFree(p);
    }
    int alloc(size_t bytes) {
        if (hipMalloc(&p, bytes) != hipSuccess) {
            p = nullptr;
            return no_memory("knn: out of device memory (" + std::to_string(bytes) + " bytes)");
        }
        return RG_OK;
    }
    template <class T>
    T *take(size_t n) {
        T *r = reinterpret_cast<T *>(p + at);
        at += (n * sizeof(T) + 255) / 256 * 256;
        return r;
    }
};

// One kernel of the candidate pass: the kernel, its query rows per
// workgroup and base rows per tile, and the byte size of a row element.
struct KnnKernel {
    void (*fn)(KnnArgs);
    int bq, bx, threads;
    size_t elem;
};

// Candidates of query rows [0, nq) of Q (one launch series, one split policy).
int knn_range(const KnnKernel &kk, const void *Q, int64_t nq, int32_t ldq, const void *X, int64_t n, int32_t ldx,
              int32_t d, int32_t K, uint32_t *ids, float *scores, bool vec_q, bool vec_x, hipStream_t stream) {
    if (nq == 0) return RG_OK;
    const int64_t qtiles = (nq + kk.bq - 1) / kk.bq;
    const int64_t xtiles = (n + kk.bx - 1) / kk.bx;
    // split the base when there are too few query tiles to fill the chip (a
    // few tiles further: their merge, one list after the other, stays short)
    int splits = (int)std::min<int64_t>(qtiles <= 8 ? 64 : 16, std::max<int64_t>(1, 1024 / qtiles));
    splits = (int)std::min<int64_t>(splits, xtiles);
    const int64_t per = (xtiles + splits - 1) / splits;
    splits = (int)((xtiles + per - 1) / per);
    const int64_t tiles_per_launch = std::max<int64_t>(1, 1024 / splits);
    const int64_t slots = std::min(qtiles, tiles_per_launch) * splits;

    float *buf_sc = nullptr, *tmp_sc = nullptr;
    uint32_t *buf_id = nullptr, *tmp_id = nullptr;
    auto cleanup = [&]() {
        if (buf_sc) (void)hipFree(buf_sc);
        if (buf_id) (void)hipFree(buf_id);
        if (tmp_sc) (void)hipFree(tmp_sc);
        if (tmp_id) (void)hipFree(tmp_id);
    };
    if (hipMalloc(&buf_sc, sizeof(float) * slots * kk.bq * CAP) != hipSuccess ||
        hipMalloc(&buf_id, sizeof(uint32_t) * slots * kk.bq * CAP) != hipSuccess) {
        cleanup();
        return no_memory("knn: out of device memory for candidate buffers");
    }
    if (splits > 1) {
        if (hipMalloc(&tmp_sc, sizeof(float) * splits * nq * K) != hipSuccess ||
            hipMalloc(&tmp_id, sizeof(uint32_t) * splits * nq * K) != hipSuccess) {
            cleanup();
            return no_memory("knn: out of device memory for split lists");
        }
    }
    KnnArgs a{};
    a.Q = Q;
    a.X = X;
    a.buf_sc = buf_sc;
    a.buf_id = buf_id;
    a.out_sc = splits > 1 ? tmp_sc : scores;
    a.out_id = splits > 1 ? tmp_id : ids;
    a.nq = nq;
    a.n = n;
    a.xtiles = xtiles;
    a.xtiles_per_split = per;
    a.ldq = ldq;
    a.ldx = ldx;
    a.d = d;
    a.K = K;
    a.splits = splits;
    a.vec_q = vec_q;
    a.vec_x = vec_x;
    const bool log = std::getenv("RG_LOG") != nullptr && qtiles > tiles_per_launch;
    for (int64_t t0 = 0; t0 < qtiles; t0 += tiles_per_launch) {
        a.q_tile0 = t0;
        const int64_t nt = std::min(tiles_per_launch, qtiles - t0);
        hipLaunchKernelGGL(kk.fn, dim3((unsigned)nt, (unsigned)splits), dim3(kk.threads), 0, stream, a);
        if (hipGetLastError() != hipSuccess) {
            cleanup();
            set_error("knn: kernel launch failed");
            return RG_EDEVICE;
        }
        if (log) {  // progress for long sweeps (waits for this launch)
            (void)hipStreamSynchronize(stream);
            std::fprintf(stderr, "[rg] knn tiles %lld / %lld\n", (long long)(t0 + nt), (long long)qtiles);
        }
    }
    if (splits > 1) {
        hipLaunchKernelGGL(k_knn_merge, dim3((unsigned)nq), dim3(64), 0, stream, tmp_sc, tmp_id, nq, K, splits,
                           scores, ids);
        if (hipGetLastError() != hipSuccess) {
            cleanup();
            set_error("knn: merge launch failed");
            return RG_EDEVICE;
        }
    }
    // buffers are freed only after the kernels that use them have finished
    if (hipStreamSynchronize(stream) != hipSuccess) {
        cleanup();
        set_error("knn: kernel failed");
        return RG_EDEVICE;
    }
    cleanup();
    return RG_OK;
}

// Each workgroup sweeps the base for one query tile.  When the tiles leave
// a thin last wave of workgroups (under half the device), its tiles run
// with the base split across workgroups instead, so the chip is not mostly
// idle for a whole sweep (same candidates).
int knn_series(const KnnKernel &kk, const void *Q, int64_t nq, int32_t ldq, const void *X, int64_t n, int32_t ldx,
               int32_t d, int32_t K, uint32_t *ids, float *scores, bool vec_q, bool vec_x, hipStream_t stream) {
    int per_cu = 0, cus = 0, dev = 0;
    RG_HIP(hipGetDevice(&dev));
    RG_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    RG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kk.fn, kk.threads, 0));
    const int64_t resident = (int64_t)std::max(1, per_cu) * std::max(1, cus);
    const int64_t qtiles = (nq + kk.bq - 1) / kk.bq;
    const int64_t rem = qtiles % resident;
    if (qtiles > resident && rem != 0 && rem < resident / 2) {
        const int64_t nq_main = (qtiles - rem) * kk.bq;
        const int rc = knn_range(kk, Q, nq_main, ldq, X, n, ldx, d, K, ids, scores, vec_q, vec_x, stream);
        if (rc) return rc;
        const void *Qr = static_cast<const char *>(Q) + (size_t)nq_main * ldq * kk.elem;
        return knn_range(kk, Qr, nq - nq_main, ldq, X, n, ldx, d, K, ids + nq_main * K, scores + nq_main * K,
                         vec_q, vec_x, stream);
    }
    return knn_range(kk, Q, nq, ldq, X, n, ldx, d, K, ids, scores, vec_q, vec_x, stream);
}

}  // namespace

int launch_knn_candidates(const float *Q, int64_t nq, int32_t ldq, const float *X, int64_t n, int32_t ldx,
                          int32_t d, int32_t K, uint32_t *ids, float *scores, hipStream_t stream) {
    if (K < 1 || K > CAP - BX || K > CAP / 2) {
        set_error("knn: K must be in [1, 256]");
        return RG_EINVAL;
    }
    const KnnKernel kk{k_knn, BQ, BX, 256, sizeof(float)};
    const bool vq = (ldq % 4 == 0) && ((uintptr_t)Q % 16 == 0);
    const bool vx = (ldx % 4 == 0) && ((uintptr_t)X % 16 == 0);
    return knn_series(kk, Q, nq, ldq, X, n, ldx, d, K, ids, scores, vq, vx, stream);
}

int64_t knn16_rows(int64_t rows) { return (rows + BQ16 - 1) / BQ16 * BQ16; }

int32_t knn16_width(int32_t d) { return (d + KS16 - 1) / KS16 * KS16; }

// Base rows per sample row for lists of K: about 12 of the K best rows fall
// into the sample, few enough that it costs 12 / K of the sweep and enough
// that the threshold's spread stays small (see k_scan16).  0: no sample, the
// running top-K.  Below 4,096 rows a sweep is a few tiles and the extra
// launches cost more than they save.
int32_t knn16_sample(int64_t n, int32_t K) { return n < 4096 ? 0 : std::max(2, K / 12); }

int launch_pack16(const float *src, int64_t rows, int32_t d, int64_t ld, void *dst, int64_t rows_pad, int32_t dp,
                  void *dst_s, int32_t s, PackStats *st, hipStream_t stream) {
    if (rows_pad % 16 != 0 || dp % KS16 != 0 || d < 1 || d > dp) {
        set_error("knn16: bad shape");
        return RG_EINVAL;
    }
    hipLaunchKernelGGL(k_fill_words, dim3(1), dim3(64), 0, stream, reinterpret_cast<uint32_t *>(st),
                       (int64_t)(sizeof(PackStats) / 4), 0u);
    RG_HIP(hipGetLastError());
    if (rows_pad == 0) return RG_OK;
    const bool vec = ld % 4 == 0 && (uintptr_t)src % 16 == 0;
    const unsigned blocks = (unsigned)std::min<int64_t>(8192, rows_pad / 16);
    hipLaunchKernelGGL(k_pack16, dim3(blocks), dim3(256), 0, stream, src, rows, d, ld, vec,
                       static_cast<_Float16 *>(dst), rows_pad, dp / KS16, static_cast<_Float16 *>(dst_s), s, st);
    RG_HIP(hipGetLastError());
    return RG_OK;
}

namespace {

template <bool SAMPLE>
void (*scan_kernel(int nks))(ScanArgs) {
    switch (nks) {
    case 1: return k_scan16<1, SAMPLE>;
    case 2: return k_scan16<2, SAMPLE>;
    case 3: return k_scan16<3, SAMPLE>;
    case 4: return k_scan16<4, SAMPLE>;
    case 5: return k_scan16<5, SAMPLE>;
    case 6: return k_scan16<6, SAMPLE>;
    case 7: return k_scan16<7, SAMPLE>;
    default: return k_scan16<0, SAMPLE>;
    }
}

// Units (tiles) per workgroup so that qtiles x splits workgroups fill the
// chip evenly: the fewest tile times over all rounds of workgroups, a
// workgroup's start counted as two tiles.
int64_t choose_splits(int64_t qtiles, int64_t units, int64_t resident) {
    int64_t best = units;
    double best_cost = 1e300;
    for (int64_t s = 1; s <= units && s <= 4 * resident; ++s) {
        const int64_t per = (units + s - 1) / s;
        const int64_t got = (units + per - 1) / per;
        const double cost = (double)((qtiles * got + resident - 1) / resident) * (double)(per + 2);
        if (cost < best_cost) {
            best_cost = cost;
            best = per;
        }
    }
    return best;
}

int running_topk(const void *Q16, int64_t nq, const void *X16, int64_t n, int32_t dp, int32_t K, uint32_t *ids,
                 float *scores, hipStream_t stream) {
    const KnnKernel kk{k_knn16, BQ16, BX16, 256, sizeof(_Float16)};
    return knn_series(kk, Q16, nq, dp, X16, n, dp, dp, K, ids, scores, true, true, stream);
}

}  // namespace

int launch_knn16_candidates(const void *Q16, int64_t nq, const void *X16, int64_t n, int32_t d, int32_t dp,
                            const void *S16, int32_t s, int32_t K, uint32_t *ids, float *scores,
                            hipStream_t stream) {
    if (K < 1 || K > CAP - BX16 || K > CAP / 2 || dp % KS16 != 0 || d < 1 || d > dp) {
        set_error("knn16: K must be in [1, 256] and the width a multiple of 32");
        return RG_EINVAL;
    }
    if (nq == 0) return RG_OK;
    if (s <= 0) return running_topk(Q16, nq, X16, n, dp, K, ids, scores, stream);
    const int nks = dp / KS16;
    const int64_t ns = (n + s - 1) / s;
    const int64_t xtiles = (n + BX16 - 1) / BX16, stiles = (ns + BX16 - 1) / BX16;
    // groups of 4 T sample rows: at most 64 * KTH_E of them per query
    const int32_t T = (int32_t)((stiles + 2 * KTH_E - 1) / (2 * KTH_E));
    const int64_t gunits = (stiles + T - 1) / T;
    const int32_t G = (int32_t)gunits * 32;
    const double E = (double)K / s;
    const int r = (int)std::ceil(E + 5.0 * std::sqrt(E) + 4.0);
    int per_cu = 0, cus = 0, dev = 0;
    RG_HIP(hipGetDevice(&dev));
    RG_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    auto ksample = scan_kernel<true>(nks);
    auto kscan = scan_kernel<false>(nks);
    RG_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kscan, 256, 0));
    const int64_t resident = (int64_t)std::max(1, per_cu) * std::max(1, cus);
    // queries of one launch series: whole rounds of workgroups, and buffers
    // of at most 131,072 rows (2.2 GB)
    const int64_t chunk = std::min<int64_t>(knn16_rows(nq), 1024 * BQ16);

    DevMem mem;
    float *gm, *thr, *buf_sc;
    uint32_t *buf_id, *cnt, *fail;
    const size_t bytes = sizeof(float) * chunk * (size_t)G + 8 * (size_t)chunk * SCAP + 8 * (size_t)chunk +
                         4 * (size_t)nq + 8 * 256;
    // no room for the buffers: the running top-K needs less
    if (mem.alloc(bytes)) return running_topk(Q16, nq, X16, n, dp, K, ids, scores, stream);
    gm = mem.take<float>(chunk * (size_t)G);
    thr = mem.take<float>(chunk);
    buf_sc = mem.take<float>(chunk * (size_t)SCAP);
    buf_id = mem.take<uint32_t>(chunk * (size_t)SCAP);
    cnt = mem.take<uint32_t>(chunk);
    fail = mem.take<uint32_t>(nq);
    uint32_t *n_fail = mem.take<uint32_t>(1);
    hipLaunchKernelGGL(k_fill_words, dim3(1), dim3(64), 0, stream, n_fail, (int64_t)1, 0u);
    ScanArgs a{};
    a.thr = thr;
    a.buf_sc = buf_sc;
    a.buf_id = buf_id;
    a.cnt = cnt;
    a.gm = gm;
    a.nks = nks;
    a.T = T;
    a.ngroups = G;
    const bool log = std::getenv("RG_LOG") != nullptr && nq > chunk;
    for (int64_t r0 = 0; r0 < nq; r0 += chunk) {
        const int64_t m = std::min(chunk, nq - r0), mp = knn16_rows(m);
        a.Q = static_cast<const _Float16 *>(Q16) + r0 * dp;
        a.qtiles = (int32_t)(mp / BQ16);
        hipLaunchKernelGGL(k_fill_words, dim3((unsigned)std::min<int64_t>(1024, (mp + 255) / 256)), dim3(256), 0, stream,
                           cnt, mp, 0u);
        a.X = static_cast<const _Float16 *>(S16);
        a.n = ns;
        a.units = gunits;
        a.units_per_split = choose_splits(a.qtiles, gunits, resident);
        const int64_t gs = (gunits + a.units_per_split - 1) / a.units_per_split;
        hipLaunchKernelGGL(ksample, dim3((unsigned)(a.qtiles * gs)), dim3(256), 0, stream, a);
        hipLaunchKernelGGL(k_kth16, dim3((unsigned)mp), dim3(64), 0, stream, gm, G, r, m, thr);
        a.X = static_cast<const _Float16 *>(X16);
        a.n = n;
        a.units = xtiles;
        a.units_per_split = choose_splits(a.qtiles, xtiles, resident);
        const int64_t xs = (xtiles + a.units_per_split - 1) / a.units_per_split;
        hipLaunchKernelGGL(kscan, dim3((unsigned)(a.qtiles * xs)), dim3(256), 0, stream, a);
        hipLaunchKernelGGL(k_pick16, dim3((unsigned)m), dim3(64), 0, stream, buf_sc, buf_id, cnt, r0, K, scores, ids,
                           fail, n_fail);
        RG_HIP(hipGetLastError());
        if (log) {  // progress for long sweeps (waits for this series)
            RG_HIP(hipStreamSynchronize(stream));
            std::fprintf(stderr, "[rg] knn rows %lld / %lld\n", (long long)(r0 + m), (long long)nq);
        }
    }
    uint32_t nf = 0;
    RG_HIP(hipMemcpyAsync(&nf, n_fail, 4, hipMemcpyDeviceToHost, stream));
    RG_HIP(hipStreamSynchronize(stream));
    if (nf == 0) return RG_OK;
    // queries whose threshold was wrong: the running top-K
    if (std::getenv("RG_LOG")) std::fprintf(stderr, "[rg] knn: %u rows by the running top-K\n", nf);
    const int64_t fp = knn16_rows(nf);
    DevMem sub;
    int rc = sub.alloc(2 * (size_t)fp * dp + 8 * (size_t)nf * K + 4 * 256);
    if (rc) return rc;
    _Float16 *qs = sub.take<_Float16>((size_t)fp * dp);
    float *fsc = sub.take<float>((size_t)nf * K);
    uint32_t *fid = sub.take<uint32_t>((size_t)nf * K);
    hipLaunchKernelGGL(k_gather16, dim3((unsigned)(fp / 16)), dim3(256), 0, stream,
                       static_cast<const _Float16 *>(Q16), fail, (int64_t)nf, nks, qs);
    RG_HIP(hipGetLastError());
    rc = running_topk(qs, nf, X16, n, dp, K, fid, fsc, stream);
    if (rc) return rc;
    hipLaunchKernelGGL(k_scatter_lists, dim3(nf), dim3(64), 0, stream, fail, K, fsc, fid, scores, ids);
    RG_HIP(hipGetLastError());
    RG_HIP(hipStreamSynchronize(stream));
    return RG_OK;
}

int launch_knn_certify(const float *Q, int64_t m, int64_t ldq, const float *X, int64_t n, int64_t ldx, int32_t d,
                       const uint32_t *cid, const float *csc, int32_t K, int32_t k, double gsum, double xmax,
                       double eta, double abs0, const uint32_t *map, uint32_t *out_id, float *out_d, uint32_t *fail,
                       uint32_t *n_fail, hipStream_t stream) {
    if (K < k || K > 64 * CERT_E || k < 1 || d < 1 || d > 16384) {
        set_error("knn certify: bad candidate count or dimension");
        return RG_EINVAL;
    }
    hipLaunchKernelGGL(k_fill_words, dim3(1), dim3(64), 0, stream, n_fail, (int64_t)1, 0u);
    RG_HIP(hipGetLastError());
    if (m == 0) return RG_OK;
    CertArgs a{};
    a.Q = Q;
    a.X = X;
    a.cid = cid;
    a.csc = csc;
    a.map = map;
    a.out_id = out_id;
    a.out_d = out_d;
    a.fail = fail;
    a.n_fail = n_fail;
    a.m = m;
    a.n = n;
    a.ldq = ldq;
    a.ldx = ldx;
    a.d = d;
    a.K = K;
    a.k = k;
    a.gsum = gsum;
    a.xmax = xmax;
    a.eta = eta;
    a.abs0 = abs0;
    hipLaunchKernelGGL(k_knn_certify, dim3((unsigned)m), dim3(64), sizeof(float) * (size_t)d, stream, a);
    RG_HIP(hipGetLastError());
    return RG_OK;
}

// Rows list[0..m) of src (rows of d floats) to dst.
int launch_gather_rows(const float *src, const uint32_t *list, int64_t m, int32_t d, float *dst, hipStream_t stream) {
    if (m == 0) return RG_OK;
    hipLaunchKernelGGL(k_gather_rows, dim3((unsigned)m), dim3(64), 0, stream, src, list, d, dst);
    RG_HIP(hipGetLastError());
    return RG_OK;
}

}  // namespace rg
