// Tiles of a plan's rows for the loops that keep a system on the chip for a
// whole launch (cg_tile.hip, bi_tile.hip): their shape, how a kernel addresses
// them, and what the host builds once per plan.
#pragma once

#include <algorithm>

#include "exchange.hpp"

namespace rp {

constexpr int TT = 512;                 // threads per block: 8 wavefronts, 256 registers each
constexpr int U = 7;                    // entries per row at most: a cell and its six faces
constexpr int BI_NR_MAX = 10;           // rows per thread at most: BiCGStab's vectors in half of the registers
template <typename T>
constexpr int nr_max() { return sizeof(T) == 8 ? 16 : 32; }   // CG's x, r, z and M^-1
constexpr int HALO_PER_THREAD = 16;
constexpr int HALO_MAX = HALO_PER_THREAD * TT;

// words of p (tile and halo) in LDS
template <typename T>
constexpr int lds_words() { return sizeof(T) == 8 ? 18432 : 36864; }   // 144 KB

struct __align__(16) Places {
    uint32_t w[4];   // entry 2 i in the low half of w[i], the next one in the high half
};

constexpr int TILE_VECS = 6;            // vectors gathered to the positions of an order, at most

__device__ __forceinline__ uint32_t place(const Places& pl, int u) {
    return u % 2 == 0 ? pl.w[u / 2] & 0xFFFFu : pl.w[u / 2] >> 16;
}

// A pointer that is the same in every lane, hidden from the compiler: what is
// loaded from it in a loop stays in the loop, and it is an address in scalar
// registers to which every lane adds the same offset of its own.  (Left to
// itself the compiler keeps an address per row and entry, or the values
// themselves, for all iterations, and spills them.)
template <typename P>
__device__ __forceinline__ __attribute__((address_space(1))) P* hidden(P* p) {
    __attribute__((address_space(1))) P* q = (__attribute__((address_space(1))) P*)p;
    asm volatile("" : "+s"(q));
    return q;
}

// sum over the block's TT threads, in every thread; red: TT / 64 words
template <typename T>
__device__ __forceinline__ T tile_sum(const T* red) {
#pragma clang fp contract(off)
    T s = T(0);
    for (int w = 0; w < TT / 64; ++w) s += red[w];
    return s;
}

// cg_tile.hip
int tile_setup(rp_plan* p, hipStream_t s);
template <typename T>
bool tile_room(rp_plan* p);
template <typename T>
int tile_slices(rp_plan* p, const T* src, bool transposed, hipStream_t s, const T** val);

}  // namespace rp
