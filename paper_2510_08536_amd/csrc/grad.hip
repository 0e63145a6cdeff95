// Adjoint value gradient: for A x = b and lambda = A^-T dL/dx, the gradient
// of L with respect to the coefficient in slot k, at matrix position
// (row, col), is -lambda[row] * x[col].  Computed in slot order, so the
// caller receives it in the LDU order it supplied the values in and every
// read of the addressing and write of g is coalesced.  A rank's slots are its
// cells (position (c, c)), its upper faces (owner, neighbour), its lower
// faces (neighbour, owner) and its interface faces; rank s's cell c is row
// row0[s] + c.  An interface slot's column is read from the CSR pattern and
// its row is the column of its transposed partner (the partner rank's
// matching interface slot).
//
// A face's two slots are one work item: the addressing is read once and the
// four gathers (lambda and x of both cells) serve both products.
#include "device_util.hpp"

namespace rp {

namespace {

// first work item of rank s: its slots without the lower faces
struct Items {
    const int32_t* slot_off;
    const int32_t* face_off;
    __device__ __forceinline__ int32_t operator()(int32_t s) const { return slot_off[s] - face_off[s]; }
};

constexpr int GU = 4;                      // items per thread, loads first
constexpr int GCHUNK = GU * VEC_BLOCK;     // items per block

// One contiguous chunk of the items per block, taken rank by rank and region
// by region, so a trip's items are of one kind and the rank's tables are the
// same in every lane.  The chunks in flight on a die are neighbours
// (xcd_block), so the cells a plane away are in its L2; small chunks keep that
// window short.  Bound by the stream of g and the addressing (8 bytes written
// per slot, 8 read per face): 200 x 190 x 210 cells 378 -> 194 us (180 on the same
// inputs again, 4.2 TB/s), 60 x 61 x 65 cells 58 -> 11, numbered at random 130 x 140
// x 150 333 -> 114.
// With blocks on the dies in turn 224 and 223 us; with 8192 items per block
// 236 and 138 us.
__global__ void __launch_bounds__(VEC_BLOCK)
value_grad_kernel(int32_t n_items, int32_t alpha, Items items, const int32_t* __restrict__ row0,
                  const int32_t* __restrict__ nf, const int32_t* __restrict__ owner, const int32_t* __restrict__ nbr,
                  const int32_t* __restrict__ iface_off, const int32_t* __restrict__ partner,
                  const int32_t* __restrict__ perm, const int32_t* __restrict__ col,
                  const double* __restrict__ lambda, const double* __restrict__ x, double* __restrict__ g) {
    const int32_t t = threadIdx.x;
    const int64_t a64 = (int64_t)xcd_block() * GCHUNK;
    if (a64 >= n_items) return;
    const int32_t k0 = (int32_t)a64;
    const int32_t k1 = (int32_t)(a64 + GCHUNK < n_items ? a64 + GCHUNK : n_items);
    int32_t s = 0;
    for (int32_t b = alpha; b - s > 1;) {   // largest s with items(s) <= k0
        const int32_t m = (s + b) >> 1;
        if (items(m) <= k0) s = m; else b = m;
    }
    for (; s < alpha; ++s) {
        const int32_t i0 = items(s);
        if (i0 >= k1) break;
        const int32_t r0 = row0[s], nc = row0[s + 1] - r0, f = nf[s], fo = items.face_off[s];
        const int32_t io = iface_off[s], ni = iface_off[s + 1] - io;
        double* const gs = g + items.slot_off[s];
        // the chunk's part of the rank's cells, faces and interfaces
        const int32_t a = max(k0 - i0, 0), e = k1 - i0;
        {
            const int32_t c1 = min(e, nc);
            const double* const lr = lambda + r0;
            const double* const xr = x + r0;
            int32_t c = a + t;
            for (; c + (GU - 1) * VEC_BLOCK < c1; c += GU * VEC_BLOCK) {
                double l[GU], v[GU];
#pragma unroll
                for (int u = 0; u < GU; ++u) {
                    l[u] = lr[c + u * VEC_BLOCK];
                    v[u] = xr[c + u * VEC_BLOCK];
                }
#pragma unroll
                for (int u = 0; u < GU; ++u) __builtin_nontemporal_store(-l[u] * v[u], gs + c + u * VEC_BLOCK);
            }
            for (; c < c1; c += VEC_BLOCK) __builtin_nontemporal_store(-lr[c] * xr[c], gs + c);
        }
        {
            const int32_t q1 = min(e - nc, f);
            const double* const lr = lambda + r0;
            const double* const xr = x + r0;
            double* const up = gs + nc;
            double* const lo = up + f;
            int32_t q = max(a - nc, 0) + t;
            for (; q + (GU - 1) * VEC_BLOCK < q1; q += GU * VEC_BLOCK) {
                int32_t o[GU], n[GU];
                double l_o[GU], l_n[GU], x_o[GU], x_n[GU];
#pragma unroll
                for (int u = 0; u < GU; ++u) {
                    o[u] = __builtin_nontemporal_load(owner + fo + q + u * VEC_BLOCK);
                    n[u] = __builtin_nontemporal_load(nbr + fo + q + u * VEC_BLOCK);
                }
#pragma unroll
                for (int u = 0; u < GU; ++u) {
                    l_o[u] = lr[o[u]];
                    x_n[u] = xr[n[u]];
                    l_n[u] = lr[n[u]];
                    x_o[u] = xr[o[u]];
                }
#pragma unroll
                for (int u = 0; u < GU; ++u) {
                    __builtin_nontemporal_store(-l_o[u] * x_n[u], up + q + u * VEC_BLOCK);
                    __builtin_nontemporal_store(-l_n[u] * x_o[u], lo + q + u * VEC_BLOCK);
                }
            }
            for (; q < q1; q += VEC_BLOCK) {
                const int32_t o = owner[fo + q], n = nbr[fo + q];
                __builtin_nontemporal_store(-lr[o] * xr[n], up + q);
                __builtin_nontemporal_store(-lr[n] * xr[o], lo + q);
            }
        }
        {
            const int32_t q1 = min(e - nc - f, ni);
            double* const gi = gs + nc + 2 * f;
            const int32_t k = items.slot_off[s] + nc + 2 * f;   // slot of the rank's first interface
            for (int32_t q = max(a - nc - f, 0) + t; q < q1; q += VEC_BLOCK) {
                const int32_t kp = partner[io + q];
                // a coupling outside the share has no local position
                gi[q] = kp < 0 ? 0.0 : -lambda[col[perm[kp]]] * x[col[perm[k + q]]];
            }
        }
    }
}

}  // namespace

int launch_value_grad(rp_plan* p, const double* lambda, const double* x, double* g, hipStream_t s) {
    if (p->n_slots == 0) return RP_OK;
    int64_t faces = 0;
    for (int32_t f : p->n_faces) faces += f;
    const int64_t items = p->n_slots - faces;
    int64_t blocks = (items + GCHUNK - 1) / GCHUNK;
    blocks = (blocks + N_XCD - 1) / N_XCD * N_XCD;   // xcd_block
    hipLaunchKernelGGL(value_grad_kernel, dim3((int)blocks), dim3(VEC_BLOCK), 0, s,
                       (int32_t)items, p->alpha, Items{p->d_slot_off, p->d_face_off}, p->d_row0, p->d_nf, p->d_owner,
                       p->d_nbr, p->d_iface_off, p->d_iface_partner, p->d_perm, p->d_col, lambda, x, g);
    RP_HIP_TRY(hipGetLastError());
    return RP_OK;
}

}  // namespace rp
