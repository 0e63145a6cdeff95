// Device-side building blocks shared by the kernels: 64-lane wavefront
// reductions and scans, block reductions, the XCD-aware block remap and the
// deterministic re-summation of per-block partials.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rp_internal.hpp"

namespace rp {

// ---- wavefront (64 lanes) ------------------------------------------------
// the value another lane of the 16-lane row holds (DPP control word), and the
// value of lane l, for 4- and 8-byte types
template <int CTRL, typename T>
__device__ __forceinline__ T dpp_row(T v) {
    constexpr int N = sizeof(T) / 4;
    int32_t w[N];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = __builtin_amdgcn_mov_dpp(w[i], CTRL, 0xF, 0xF, true);
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}
template <typename T>
__device__ __forceinline__ T lane_value(T v, int l) {
    constexpr int N = sizeof(T) / 4;
    int32_t w[N];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = __builtin_amdgcn_readlane(w[i], l);
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

// Sum over the wave, in every lane (all 64 lanes active): pairs of lanes,
// quads, eights and rows of 16 by DPP (the mirrors meet the other half, whose
// lanes all hold its sum), then the four rows' sums.  Register moves instead
// of six trips through LDS: a reduction's latency, which small kernels and
// the starts of all solver kernels wait for, is a few times shorter.
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma clang fp contract(off)
    v += dpp_row<0xB1>(v);    // quad_perm [1, 0, 3, 2]
    v += dpp_row<0x4E>(v);    // quad_perm [2, 3, 0, 1]
    v += dpp_row<0x141>(v);   // row_half_mirror
    v += dpp_row<0x140>(v);   // row_mirror
    const T a = lane_value(v, 0) + lane_value(v, 16);
    const T b = lane_value(v, 32) + lane_value(v, 48);
    return a + b;
}

__device__ __forceinline__ int32_t wave_incl_scan(int32_t v) {
    // within rows of 16 lanes, then the last lane of a row into the next rows;
    // lanes without a source add 0
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // from 1 lane below
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // rows 0, 2 -> 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // lane 31 -> rows 2, 3
    return v;
}

// Sum over a block of BLOCK threads, result valid in thread 0.  `red` holds
// BLOCK/64 values of shared memory.  Fixed shape, so the rounding is fixed.
template <typename T, int BLOCK>
__device__ __forceinline__ T block_sum(T v, T* red) {
#pragma clang fp contract(off)
    constexpr int NW = BLOCK / 64;
    __syncthreads();  // `red` may still be read from a previous call
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) red[w] = v;
    __syncthreads();
    T s = T(0);
    if (threadIdx.x == 0) {
        for (int i = 0; i < NW; ++i) s += red[i];
    }
    return s;
}

// Barrier for hand-offs through LDS only.  __syncthreads fences global
// memory too, which makes every wave wait for all of its outstanding global
// loads at the barrier; this one waits only for the wave's LDS (and scalar)
// accesses, so global loads issued before it stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- XCD-aware block order -----------------------------------------------
// Workgroups are handed to the 8 XCDs round-robin (block b -> XCD b % 8).
// Remapping b to (b % 8) * per + b / 8 makes the logical blocks of one XCD
// consecutive, so neighbouring row groups (and the x entries they share) are
// worked on by one XCD and its L2.  gridDim.x must be a multiple of 8.
__device__ __forceinline__ int32_t xcd_block() {
    const int32_t per = (int32_t)(gridDim.x / N_XCD);
    return (int32_t)(blockIdx.x % N_XCD) * per + (int32_t)(blockIdx.x / N_XCD);
}

// Sum of partials[0..n), computed identically by every block of a kernel:
// thread t adds t, t + BLOCK, ... in order, then the fixed block tree.  The
// result is returned to every thread.  The partials come from an earlier
// kernel, so plain loads see them.
template <typename T, int BLOCK>
__device__ __forceinline__ T sum_partials_all(const T* partials, int32_t n, T* red) {
#pragma clang fp contract(off)
    __shared__ T bcast;
    T s = T(0);
    for (int32_t i = threadIdx.x; i < n; i += BLOCK) s += partials[i];
    const T b = block_sum<T, BLOCK>(s, red);
    if (threadIdx.x == 0) bcast = b;
    __syncthreads();
    return bcast;
}

}  // namespace rp
