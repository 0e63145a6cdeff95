// Exchange of values between the workgroups of one running kernel (the CG
// loops that keep every workgroup resident), without barriers and fences.
//
// What is exchanged is stored and loaded by agent-scope relaxed atomics, which
// pass the die's L2 by, so nothing is written back or invalidated; and every
// value is its own flag: its slot holds EMPTY (a NaN no value is stored as)
// until it is stored, and a reader loads until it is not.  Slots rotate through
// RES_SETS sets.  Waits are bounded: after so many loads the reader gives up,
// and a reader that finds the abort word set gives up too.  A workgroup that gives
// up publishes nothing more, so all do; the host goes on with launched kernels.
#pragma once

#include "device_util.hpp"

namespace rp {

constexpr int RES_SETS = 4;
// Loads of one wait at most, some tenths of a second: what it can wait for
// beside values on their way is a workgroup that has no place yet, behind another
// stream's or process's kernels.
constexpr uint32_t WAIT_SPINS = 1u << 18;
inline uint32_t wait_spins(const rp_plan* p) { return p->loop_spins ? p->loop_spins : WAIT_SPINS; }

__device__ __forceinline__ uint32_t load_relaxed(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// a value as the word it is exchanged as
template <typename T>
struct Word;
template <>
struct Word<double> {
    typedef uint64_t type;
    static constexpr type EMPTY = ~0ull;
    static __device__ __forceinline__ type of(double v) {
        return v == v ? (type)__double_as_longlong(v) : 0x7FF8000000000000ull;
    }
    static __device__ __forceinline__ double value(type u) { return __longlong_as_double((long long)u); }
};
template <>
struct Word<float> {
    typedef uint32_t type;
    static constexpr type EMPTY = ~0u;
    static __device__ __forceinline__ type of(float v) { return v == v ? __float_as_uint(v) : 0x7FC00000u; }
    static __device__ __forceinline__ float value(type u) { return __uint_as_float(u); }
};

template <typename V>
__device__ __forceinline__ V agent_load(const V* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// from a byte offset to a base that is the same in every lane (one address register)
template <typename V>
__device__ __forceinline__ V agent_load_at(const V* base, uint32_t bytes) {
    return agent_load(reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + bytes));
}
template <typename V>
__device__ __forceinline__ void agent_store(V* p, V v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the bound of a launch's waits
struct Wait {
    uint32_t* bar;    // abort word
    uint32_t most;    // loads
};

// spins of one wait: true = give up (too many, or another block gave up)
__device__ __forceinline__ bool wait_over(uint32_t& spins, const Wait& wait) {
    return ++spins > wait.most || (spins % 256 == 0 && load_relaxed(wait.bar) != 0u);
}

// The sums of N values per group once no slot of slots[0 .. N ng) is empty
// (value j of group m at N m + j), added up as sum_partials_all does it with
// SPMV_BLOCK threads: thread t adds groups t, t + 256, ...; the wave sums go
// to red[j][0 .. 4).  False: the wait was abandoned.
template <typename T, int N>
__device__ __forceinline__ bool gather_slots(const typename Word<T>::type* slots, int32_t ng, int32_t t,
                                             const Wait& wait, T (*red)[SPMV_BLOCK / 64]) {
#pragma clang fp contract(off)
    T s[N];
#pragma unroll
    for (int j = 0; j < N; ++j) s[j] = T(0);
    bool good = true;
    for (int32_t m = t; m < ng; m += SPMV_BLOCK) {
        typename Word<T>::type u[N];
        for (uint32_t spins = 0;;) {
            bool empty = false;
#pragma unroll
            for (int j = 0; j < N; ++j) u[j] = agent_load(slots + N * m + j);
#pragma unroll
            for (int j = 0; j < N; ++j) empty |= u[j] == Word<T>::EMPTY;
            if (!empty) break;
            if (wait_over(spins, wait)) {
                good = false;
                break;
            }
        }
#pragma unroll
        for (int j = 0; j < N; ++j) s[j] += Word<T>::value(u[j]);
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        s[j] = wave_sum(s[j]);
        if ((t & 63) == 0) red[j][t >> 6] = s[j];
    }
    return good;
}

template <typename T>
__device__ __forceinline__ T sum_red(const T* red) {
#pragma clang fp contract(off)
    T s = T(0);
    for (int w = 0; w < SPMV_BLOCK / 64; ++w) s += red[w];
    return s;
}

}  // namespace rp
