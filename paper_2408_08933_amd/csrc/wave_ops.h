// Wavefront (64-lane) helpers for gfx950 kernels: ballot/prefix helpers and
// an in-register bitonic sort of (key, id) pairs held E per lane.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace rg {

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ uint64_t ballot64(bool p) { return __ballot(p); }

// Orders a wavefront's LDS accesses across its lanes.  The LDS serves one
// wavefront's operations in order, so this only keeps the compiler from
// moving them; a workgroup barrier, even where a workgroup is one wavefront,
// also waits for every outstanding load and store.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// number of set bits of m below this lane
__device__ __forceinline__ int lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// lane l reads lane l + n of its 16-lane row (row shift left) or lane
// l ^ 2 / l ^ 1 (quad permutes); lanes past the row read 0
template <int CTRL>
__device__ __forceinline__ float dpp_read(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

template <int CTRL>
__device__ __forceinline__ double dpp_read(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (uint32_t)lo);
}

// v of lane src (the same for all lanes), whichever lanes are active
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int src) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, src);
}
__device__ __forceinline__ float lane_value(float v, int src) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}
__device__ __forceinline__ double lane_value(double v, int src) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, src), hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | (uint32_t)lo);
}

// Sum of the G lanes of each group, valid in the group's first lane.  The
// steps are those of an xor butterfly with the largest offset first, as
// seen from the first lane, so the value is the butterfly's bit for bit;
// inside a 16-lane row they use DPP (no LDS round trip), across rows
// (G = 32) a shuffle.
template <int G, typename T>
__device__ __forceinline__ T group_sum(T v) {
    if constexpr (G >= 32) v += __shfl_down(v, 16);
    if constexpr (G >= 16) v += dpp_read<0x108>(v);  // row_shl:8: lane + 8
    if constexpr (G >= 8) v += dpp_read<0x104>(v);   // row_shl:4: lane + 4
    if constexpr (G >= 4) v += dpp_read<0x4E>(v);    // quad_perm [2,3,0,1]: lane ^ 2
    if constexpr (G >= 2) v += dpp_read<0xB1>(v);    // quad_perm [1,0,3,2]: lane ^ 1
    return v;
}

// (key, id) strict order: smaller key first, then smaller id
template <typename K>
__device__ __forceinline__ bool kless(K ka, uint32_t ia, K kb, uint32_t ib) {
    return ka < kb || (ka == kb && ia < ib);
}

__device__ __forceinline__ float wave_min(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o));
    return v;
}

__device__ __forceinline__ int wave_min_i(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        int w = __shfl_xor(v, o);
        v = w < v ? w : v;
    }
    return v;
}

// One compare-exchange stage of a bitonic network over 64*E pairs held E
// per lane (element i = lane*E + e); SIZE and STRIDE are compile-time so
// every register index is static.
template <int E, int SIZE, int STRIDE, typename K>
__device__ __forceinline__ void bitonic_stage(K (&k)[E], uint32_t (&v)[E]) {
    const int lane = lane_id();
    if constexpr (STRIDE >= E) {
        constexpr int lx = STRIDE / E;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = lane * E + e;
            const K ok = __shfl_xor(k[e], lx);
            const uint32_t ov = __shfl_xor(v[e], lx);
            const bool up = (i & SIZE) == 0;
            const bool lower = (i & STRIDE) == 0;
            const bool keep_min = (lower == up);
            const bool take = keep_min ? kless(ok, ov, k[e], v[e]) : kless(k[e], v[e], ok, ov);
            if (take) {
                k[e] = ok;
                v[e] = ov;
            }
        }
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if ((e & STRIDE) == 0) {
                const int p = e | STRIDE;
                const int i = lane * E + e;
                const bool up = (i & SIZE) == 0;
                const bool sw = up ? kless(k[p], v[p], k[e], v[e]) : kless(k[e], v[e], k[p], v[p]);
                const K ka = k[e], kb = k[p];
                const uint32_t va = v[e], vb = v[p];
                k[e] = sw ? kb : ka;
                k[p] = sw ? ka : kb;
                v[e] = sw ? vb : va;
                v[p] = sw ? va : vb;
            }
        }
    }
}

template <int E, int SIZE, int STRIDE, typename K>
__device__ __forceinline__ void bitonic_merge_steps(K (&k)[E], uint32_t (&v)[E]) {
    bitonic_stage<E, SIZE, STRIDE, K>(k, v);
    if constexpr (STRIDE > 1) bitonic_merge_steps<E, SIZE, STRIDE / 2, K>(k, v);
}

template <int E, int SIZE, typename K>
__device__ __forceinline__ void bitonic_sizes(K (&k)[E], uint32_t (&v)[E]) {
    bitonic_merge_steps<E, SIZE, SIZE / 2, K>(k, v);
    if constexpr (SIZE < 64 * E) bitonic_sizes<E, SIZE * 2, K>(k, v);
}

// Ascending bitonic sort of 64*E (key, id) pairs; element i = lane*E + e.
template <int E, typename K>
__device__ __forceinline__ void wave_sort(K (&k)[E], uint32_t (&v)[E]) {
    bitonic_sizes<E, 2, K>(k, v);
}

}  // namespace rg
