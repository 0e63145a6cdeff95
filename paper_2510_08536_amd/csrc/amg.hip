// Aggregation multigrid preconditioner (rp_solve_opts.precond =
// RP_PRECOND_AMG), the multigrid option of the outlook in Sec. 5.
//
// Hierarchy (built once from the values at hand, rp_plan_amg_setup or the
// first solve that asks for it; the aggregates and patterns are then kept,
// and every later value update refreshes only the coarse values):
//  * pairwise matching in rounds on the negative couplings: every unmatched
//    row picks its strongest coupling to an unmatched row, rows that picked
//    each other pair up; a row left over joins the pair of its strongest
//    coupling to a matched row, else stays alone.  Strength: the value's
//    magnitude, ties broken by a hash of the row pair (MurmurHash3's 32-bit
//    finaliser), then by the smaller pair.  Aggregates are numbered by their
//    leaders (a pair's smaller row), ascending.
//  * Galerkin coarse matrix A_c = P^T A P, P the aggregate indicator: each
//    coarse entry sums its fine entries in ascending fine CSR position.  The
//    plan keeps, per coarse entry, the list of those positions, so a value
//    refresh is a gather-sum through a fixed map (like the update by P).
//  * coarsest level (at most AMG_COARSE_MAX rows): dense Gauss-Jordan
//    inverse without pivoting in the textbook order, one workgroup.
// V-cycle y = V_l(r): even levels smooth with one damped-Jacobi sweep from
// zero, restrict the residual, add the prolonged coarse correction and
// smooth again; odd levels only restrict and prolong (two pairwise passes
// per smoothed level); the coarsest level multiplies by the dense inverse.
// Every product and sum is one rounding in the order the definition states
// (row sums in column order, aggregate sums over the members ascending), so
// the hierarchy and one V-cycle are bit-exact against the serial definition.
// The levels from the first one with at most AMG_TAIL_ROWS rows down run in
// one workgroup (amg_tail), with the same operations in the same order.
//
// Setup runs on the device: matching rounds (the host reads one counter per
// round), scans for the numbering, per-coarse-row key lists (aggregate of the
// column, fine position) sorted in place for the patterns and the
// contribution lists.
#include "spmv.hpp"

namespace rp {

int scan_i32(const int32_t* in, int64_t n, int32_t* out, int32_t* total, hipStream_t s);
int64_t scan_i32_scratch(int64_t n);
int scan_i32_enqueue(const int32_t* in, int64_t n, int32_t* out, int32_t* scratch, hipStream_t s);

namespace {

constexpr int AB = 256;   // threads per block of the setup and vector kernels

int grid_of(int64_t n) {
    int64_t g = (n + AB - 1) / AB;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, 16384));
}

// ---- coupling strength -----------------------------------------------------
__device__ __forceinline__ uint32_t fmix32(uint32_t x) {
    x ^= x >> 16;
    x *= 0x85EBCA6Bu;
    x ^= x >> 13;
    x *= 0xC2B2AE35u;
    x ^= x >> 16;
    return x;
}

// strongest negative coupling of row i to a row whose matched state is
// `matched`; -1 if none.  The comparison is one boolean expression and the
// running best is updated by selects: the form with nested branches was
// compiled (hipcc, gfx950) into code that kept the first candidate's weight.
__device__ int32_t strongest(int32_t i, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                             const double* __restrict__ val, const int32_t* __restrict__ mate, bool matched) {
    int32_t best = -1, blo = 0, bhi = 0;
    double bw = 0.0;
    uint32_t bh = 0u;
    for (int32_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p) {
        const int32_t j = col[p];
        const double a = val[p];
        const bool cand = j != i && a < 0.0 && ((mate[j] >= 0) == matched);
        const double w = -a;
        const int32_t lo = min(i, j), hi = max(i, j);
        const uint32_t h = fmix32((uint32_t)lo * 0x9E3779B1u + (uint32_t)hi);
        const bool better = (w > bw) | ((w == bw) & ((h > bh) | ((h == bh) & ((lo < blo) | ((lo == blo) & (hi < bhi))))));
        const bool take = cand & ((best < 0) | better);
        best = take ? j : best;
        bw = take ? w : bw;
        bh = take ? h : bh;
        blo = take ? lo : blo;
        bhi = take ? hi : bhi;
    }
    return best;
}

// ---- setup kernels -----------------------------------------------------------
__global__ void amg_fill(int32_t n, int32_t v, int32_t* a) {
    for (int32_t i = blockIdx.x * AB + threadIdx.x; i < n; i += gridDim.x * AB) a[i] = v;
}

__global__ void __launch_bounds__(AB)
amg_pick(int32_t n, const int32_t* row_ptr, const int32_t* col, const double* val, const int32_t* mate,
         int32_t* pick) {
    for (int32_t i = blockIdx.x * AB + threadIdx.x; i < n; i += gridDim.x * AB)
        pick[i] = mate[i] >= 0 ? -1 : strongest(i, row_ptr, col, val, mate, false);
}

// rows that picked each other pair up; count[0] += pairs (two rows each)
__global__ void __launch_bounds__(AB)
amg_pair(int32_t n, const int32_t* pick, int32_t* mate, uint32_t* count) {
    __shared__ uint32_t red[AB / 64];
    uint32_t c = 0;
    for (int32_t i = blockIdx.x * AB + threadIdx.x; i < n; i += gridDim.x * AB) {
        const int32_t j = pick[i];
        if (j >= 0 && pick[j] == i) {
            mate[i] = j;
            ++c;
        }
    }
    // one add per block: an add per thread made every round wait on one word
    c = block_sum<uint32_t, AB>(c, red);
    if (threadIdx.x == 0 && c) atomicAdd(count, c);
}

__global__ void __launch_bounds__(AB)
amg_leader(int32_t n, const int32_t* row_ptr, const int32_t* col, const double* val, const int32_t* mate,
           int32_t* leader, int32_t* is_leader) {
    for (int32_t i = blockIdx.x * AB + threadIdx.x; i < n; i += gridDim.x * AB) {
        int32_t l;
        if (mate[i] >= 0) {
            l = min(i, mate[i]);
        } else {
            const int32_t j = strongest(i, row_ptr, col, val, mate, true);
            l = j >= 0 ? min(j, mate[j]) : i;
        }
        leader[i] = l;
        is_leader[i] = l == i ? 1 : 0;
    }
}

// agg[i] = number of leaders below leader[i]; members counted per aggregate
__global__ void __launch_bounds__(AB)
amg_number(int32_t n, const int32_t* leader, const int32_t* lead_id, int32_t* agg, int32_t* cnt) {
    for (int32_t i = blockIdx.x * AB + threadIdx.x; i < n; i += gridDim.x * AB) {
        const int32_t a = lead_id[leader[i]];
        agg[i] = a;
        atomicAdd(cnt + a, 1);
    }
}

__global__ void __launch_bounds__(AB)
amg_members(int32_t n, const int32_t* agg, const int32_t* mem_ptr, int32_t* fill, int32_t* mem) {
    for (int32_t i = blockIdx.x * AB + threadIdx.x; i < n; i += gridDim.x * AB) {
        const int32_t a = agg[i];
        mem[mem_ptr[a] + atomicAdd(fill + a, 1)] = i;
    }
}

// per aggregate: members ascending (insertion sort, aggregates are small);
// keys of the coarse row counted
__global__ void __launch_bounds__(AB)
amg_sort_members(int32_t nc, const int32_t* mem_ptr, int32_t* mem, const int32_t* row_ptr, int32_t* kcnt) {
    for (int32_t I = blockIdx.x * AB + threadIdx.x; I < nc; I += gridDim.x * AB) {
        const int32_t a0 = mem_ptr[I], a1 = mem_ptr[I + 1];
        int32_t k = 0;
        for (int32_t a = a0; a < a1; ++a) {
            const int32_t v = mem[a];
            int32_t b = a;
            while (b > a0 && mem[b - 1] > v) {
                mem[b] = mem[b - 1];
                --b;
            }
            mem[b] = v;
            k += row_ptr[v + 1] - row_ptr[v];
        }
        kcnt[I] = k;
    }
}

// keys (aggregate of the column << 32 | fine position) of coarse row I,
// sorted; the number of distinct coarse columns into ucnt[I]
__global__ void __launch_bounds__(AB)
amg_keys(int32_t nc, const int32_t* mem_ptr, const int32_t* mem, const int32_t* row_ptr, const int32_t* col,
         const int32_t* agg, const int32_t* kstart, uint64_t* keys, int32_t* ucnt) {
    for (int32_t I = blockIdx.x * AB + threadIdx.x; I < nc; I += gridDim.x * AB) {
        const int32_t k0 = kstart[I];
        int32_t k = k0;
        for (int32_t m = mem_ptr[I]; m < mem_ptr[I + 1]; ++m) {
            const int32_t i = mem[m];
            for (int32_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p)
                keys[k++] = ((uint64_t)(uint32_t)agg[col[p]] << 32) | (uint32_t)p;
        }
        for (int32_t a = k0 + 1; a < k; ++a) {
            const uint64_t v = keys[a];
            int32_t b = a;
            while (b > k0 && keys[b - 1] > v) {
                keys[b] = keys[b - 1];
                --b;
            }
            keys[b] = v;
        }
        int32_t u = 0;
        for (int32_t a = k0; a < k; ++a)
            if (a == k0 || (keys[a] >> 32) != (keys[a - 1] >> 32)) ++u;
        ucnt[I] = u;
    }
}

// coarse columns, diagonal positions, contribution ranges and positions
__global__ void __launch_bounds__(AB)
amg_cfill(int32_t nc, const int32_t* kstart, const uint64_t* keys, const int32_t* c_row_ptr, int32_t* c_col,
          int32_t* c_diag, int32_t* cptr, int32_t* cpos) {
    for (int32_t I = blockIdx.x * AB + threadIdx.x; I < nc; I += gridDim.x * AB) {
        int32_t e = c_row_ptr[I];
        int32_t diag = -1;
        for (int32_t a = kstart[I]; a < kstart[I + 1]; ++a) {
            const int32_t J = (int32_t)(keys[a] >> 32);
            if (a == kstart[I] || J != (int32_t)(keys[a - 1] >> 32)) {
                cptr[e] = a;
                c_col[e] = J;
                if (J == I) diag = e;
                ++e;
            }
            cpos[a] = (int32_t)(keys[a] & 0xFFFFFFFFu);
        }
        c_diag[I] = diag;
        if (I == nc - 1) cptr[e] = kstart[nc];
    }
}

// ---- two aggregations composed (AmgLevel::map, ::rows) -----------------------
// fine rows of the k-th entry of the middle level's member list
__global__ void __launch_bounds__(AB)
amg_link_count(int32_t nm, const int32_t* mid_mem, const int32_t* mem_ptr, int32_t* cnt) {
    for (int32_t k = blockIdx.x * AB + threadIdx.x; k < nm; k += gridDim.x * AB) {
        const int32_t m = mid_mem[k];
        cnt[k] = mem_ptr[m + 1] - mem_ptr[m];
    }
}

__global__ void __launch_bounds__(AB)
amg_link_rows(int32_t nm, const int32_t* mid_mem, const int32_t* mem_ptr, const int32_t* mem, const int32_t* pos,
              int32_t* rows) {
    for (int32_t k = blockIdx.x * AB + threadIdx.x; k < nm; k += gridDim.x * AB) {
        const int32_t m = mid_mem[k], a0 = mem_ptr[m], len = mem_ptr[m + 1] - a0;
        for (int32_t j = 0; j < len; ++j) rows[pos[k] + j] = mem[a0 + j] | (j == 0 ? INT32_MIN : 0);
    }
}

__global__ void __launch_bounds__(AB)
amg_link_ptr(int32_t nc, const int32_t* mid_mem_ptr, const int32_t* pos, int32_t* rows_ptr) {
    for (int32_t I = blockIdx.x * AB + threadIdx.x; I <= nc; I += gridDim.x * AB) rows_ptr[I] = pos[mid_mem_ptr[I]];
}

__global__ void __launch_bounds__(AB)
amg_link_map(int32_t n, const int32_t* agg, const int32_t* mid_agg, int32_t* map) {
    for (int32_t i = blockIdx.x * AB + threadIdx.x; i < n; i += gridDim.x * AB) map[i] = mid_agg[agg[i]];
}

// ---- value refresh -----------------------------------------------------------
__global__ void __launch_bounds__(AB)
amg_gvals(int32_t nnz_c, const int32_t* cptr, const int32_t* cpos, const double* fine, double* c64, float* c32) {
#pragma clang fp contract(off)
    for (int32_t e = blockIdx.x * AB + threadIdx.x; e < nnz_c; e += gridDim.x * AB) {
        double s = 0.0;
        for (int32_t t = cptr[e]; t < cptr[e + 1]; ++t) s += fine[cpos[t]];
        c64[e] = s;
        c32[e] = (float)s;
    }
}

__global__ void __launch_bounds__(AB)
amg_gdiag(int32_t nc, const int32_t* c_diag, const double* c64, double* dinv64, float* dinv32, uint32_t* flag) {
    for (int32_t I = blockIdx.x * AB + threadIdx.x; I < nc; I += gridDim.x * AB) {
        const int32_t e = c_diag[I];
        const double d = e >= 0 ? c64[e] : 0.0;
        if (!(d > 0.0) || !isfinite(d)) atomicOr(flag, 1u);
        const double v = 1.0 / d;
        dinv64[I] = v;
        dinv32[I] = (float)v;
    }
}

// dense Gauss-Jordan inverse of the n x n coarsest matrix (n <= AMG_COARSE_MAX),
// one workgroup: pivot row divided, multipliers of column k read, then every
// other row updated; the same single roundings in the same order as the
// serial elimination.  W: n*n work, Z: the inverse.
constexpr int GJ_THREADS = 1024;

__global__ void __launch_bounds__(GJ_THREADS)
amg_dense_inverse(int32_t n, const int32_t* row_ptr, const int32_t* col, const double* val, double* W, double* Z,
                  float* Z32, uint32_t* flag) {
#pragma clang fp contract(off)
    __shared__ double f[AMG_COARSE_MAX];
    __shared__ double piv_s;
    const int32_t t = threadIdx.x, nn = n * n;
    for (int32_t e = t; e < nn; e += GJ_THREADS) {
        W[e] = 0.0;
        Z[e] = (e / n == e % n) ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int32_t i = t; i < n; i += GJ_THREADS)
        for (int32_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p) W[i * n + col[p]] = val[p];
    __syncthreads();
    for (int32_t k = 0; k < n; ++k) {
        if (t == 0) piv_s = W[k * n + k];
        __syncthreads();
        const double piv = piv_s;
        if (!(piv > 0.0) || !isfinite(piv)) {
            if (t == 0) atomicOr(flag, 2u);
            return;
        }
        for (int32_t j = t; j < n; j += GJ_THREADS) {
            W[k * n + j] = W[k * n + j] / piv;
            Z[k * n + j] = Z[k * n + j] / piv;
        }
        __syncthreads();
        for (int32_t i = t; i < n; i += GJ_THREADS) f[i] = W[i * n + k];
        __syncthreads();
        for (int32_t e = t; e < nn; e += GJ_THREADS) {
            const int32_t i = e / n, j = e - i * n;
            if (i == k) continue;
            W[e] = W[e] - f[i] * W[k * n + j];
            Z[e] = Z[e] - f[i] * Z[k * n + j];
        }
        __syncthreads();
    }
    for (int32_t e = t; e < nn; e += GJ_THREADS) Z32[e] = (float)Z[e];
}

// ---- V-cycle kernels -----------------------------------------------------------
// gate: the solve's K2-written iteration word; < 0 means K2 did no update
// this iteration and the cycle's result is not used, so every kernel returns

// x = omega (dinv r)
template <typename T>
__global__ void __launch_bounds__(AB)
amg_pre(int32_t n, const T* __restrict__ r, const T* __restrict__ dinv, T* __restrict__ x, T omega,
        const int32_t* gate) {
#pragma clang fp contract(off)
    if (gate && *gate < 0) return;
    for (int32_t i = blockIdx.x * AB + threadIdx.x; i < n; i += gridDim.x * AB) x[i] = omega * (dinv[i] * r[i]);
}

// t = r - A x
template <typename T>
__global__ void __launch_bounds__(SPMV_BLOCK)
amg_resid(int32_t n, SpmvIdx ix, const T* __restrict__ val, const T* __restrict__ x, const T* __restrict__ r,
          T* __restrict__ t, const int32_t* gate) {
#pragma clang fp contract(off)
    __shared__ __align__(16) T lds[SPMV_CAP];
    __shared__ T xs[1];
    if (gate && *gate < 0) return;
    const XWin w{{0, 0}};
    GroupRange gr = block_groups(ix, n);
    for (int32_t g = gr.g0; g < gr.n_groups; g += gr.step) {
        const int32_t r0 = g * SPMV_BLOCK;
        const int32_t nr = min(SPMV_BLOCK, n - r0);
        const GroupRow<T> row = spmv_group_row<T, -1>(ix, val, x, n, g, nr, w, xs, lds, gr);
        if ((int32_t)threadIdx.x < nr) {
            const int32_t i = r0 + threadIdx.x;
            t[i] = r[i] - row.s;
        }
    }
}

// Coarse levels (plain CSR, 10 to 30 entries per row): one wavefront per
// block, chunks of CR consecutive rows (64, or 32 on levels with more than
// 12 entries per row).  The wave forms the chunk's products val * x together
// (coalesced over the entries, every load of a lane issued before the first
// product) into LDS, then each lane sums its row's products in column order
// from 0: the same single roundings as the serial row sum.  A chunk with
// more than wcap() entries is summed straight from memory, a lane per row.
constexpr int WB = 64;            // threads per block: one wavefront

// staged products per chunk of CR rows (16 or 24 per row; more fall back to memory)
template <int CR>
constexpr int wcap() { return CR == 64 ? 1024 : 768; }

// x of the level, and x with the coarse correction e added on the fly
template <typename T>
struct PlainX {
    const T* x;
    __device__ __forceinline__ T operator()(int32_t i) const { return x[i]; }
};
template <typename T>
struct CorrectedX {
    const T* x;
    const T* e;
    const int32_t* map;
    __device__ __forceinline__ T operator()(int32_t i) const {
#pragma clang fp contract(off)
        return x[i] + e[map[i]];
    }
};

// sum of p[0 .. n) from 0, ascending; four reads of LDS in flight
template <typename T>
__device__ __forceinline__ T serial_sum(const T* p, int32_t n) {
#pragma clang fp contract(off)
    T s = T(0);
    int32_t j = 0;
    for (; j + 4 <= n; j += 4) {
        const T a = p[j], b = p[j + 1], c = p[j + 2], d = p[j + 3];
        s += a;
        s += b;
        s += c;
        s += d;
    }
    for (; j < n; ++j) s += p[j];
    return s;
}

template <typename T, int CR, typename X>
__device__ __forceinline__ T wave_row_sum(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                          const T* __restrict__ val, const X& x, int32_t r0, int32_t nr, T* prod) {
#pragma clang fp contract(off)
    constexpr int WU = wcap<CR>() / WB;   // loads per lane
    const int32_t t = threadIdx.x;
    const int32_t e0 = row_ptr[r0], e1 = row_ptr[r0 + nr];
    int32_t rs = 0, re = 0;
    if (t < nr) {
        rs = row_ptr[r0 + t];
        re = row_ptr[r0 + t + 1];
    }
    T s = T(0);
    if (e1 - e0 <= wcap<CR>()) {
        // lanes past the chunk load its last entry again (a row has its diagonal,
        // so there is one): a branch per load kept the loads from leaving together
        // (a V-cycle 421 -> 408 us at 160^3, 263 -> 246 at 131 x 117 x 142)
        int32_t cv[WU];
        T vv[WU], xv[WU];
#pragma unroll
        for (int u = 0; u < WU; ++u) {
            const int32_t e = e0 + t + u * WB;
            const int32_t ec = min(e, e1 - 1);
            cv[u] = col[ec];
            vv[u] = val[ec];
        }
#pragma unroll
        for (int u = 0; u < WU; ++u) xv[u] = x(cv[u]);
#pragma unroll
        for (int u = 0; u < WU; ++u) {
            const int32_t e = e0 + t + u * WB;
            if (e < e1) prod[e - e0] = vv[u] * xv[u];
        }
        __syncthreads();   // one wave: orders its LDS writes before the reads
        s = serial_sum(prod + (rs - e0), re - rs);
        __syncthreads();   // prod is refilled by the next chunk
    } else {
        for (int32_t e = rs; e < re; ++e) s += val[e] * x(col[e]);
    }
    return s;
}

// t = r - A x on a coarse level
template <typename T, int CR>
__global__ void __launch_bounds__(WB)
amg_csr_resid(int32_t n, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
              const T* __restrict__ val, const T* __restrict__ x, const T* __restrict__ r, T* __restrict__ t,
              const int32_t* gate) {
#pragma clang fp contract(off)
    __shared__ T prod[wcap<CR>()];
    if (gate && *gate < 0) return;
    const int32_t nch = (n + CR - 1) / CR;
    for (int32_t c = xcd_block(); c < nch; c += gridDim.x) {
        const int32_t r0 = c * CR, nr = min(CR, n - r0);
        const T s = wave_row_sum<T, CR>(row_ptr, col, val, PlainX<T>{x}, r0, nr, prod);
        if ((int32_t)threadIdx.x < nr) {
            const int32_t i = r0 + threadIdx.x;
            t[i] = r[i] - s;
        }
    }
}

// y = x' + omega (dinv (r - A x')) on a coarse level; x' = x, or with the
// coarse correction (X = CorrectedX: x + e[map], formed at every use)
template <typename T, int CR, typename X>
__global__ void __launch_bounds__(WB)
amg_csr_post(int32_t n, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
             const T* __restrict__ val, X x, const T* __restrict__ r, const T* __restrict__ dinv, T omega,
             T* __restrict__ y, const int32_t* gate) {
#pragma clang fp contract(off)
    __shared__ T prod[wcap<CR>()];
    if (gate && *gate < 0) return;
    const int32_t nch = (n + CR - 1) / CR;
    for (int32_t c = xcd_block(); c < nch; c += gridDim.x) {
        const int32_t r0 = c * CR, nr = min(CR, n - r0);
        const T s = wave_row_sum<T, CR>(row_ptr, col, val, x, r0, nr, prod);
        if ((int32_t)threadIdx.x < nr) {
            const int32_t i = r0 + threadIdx.x;
            y[i] = x(i) + omega * (dinv[i] * (r[i] - s));
        }
    }
}

// chunk rows of a level: 64, or 32 where rows average more than 12 entries
int chunk_rows(const AmgLevel& L) { return L.nnz > 12 * L.n ? 32 : 64; }

// grid of the chunked kernels: a multiple of 8 (xcd_block), one chunk per
// block (at most 16384 blocks a V-cycle took 430 us at 160^3 and 1463 at 256^3
// where this takes 421 and 1385)
int chunk_grid(int64_t n, int cr) {
    int64_t g = (n + cr - 1) / cr;
    g = ((g + N_XCD - 1) / N_XCD) * N_XCD;
    return (int)std::max<int64_t>(N_XCD, g);
}

// rc[I] = the restricted v of coarse row I (its rows in the list's order, see
// AmgLevel::rows); xc (nullable): the first sweep of the coarse level,
// xc = omega (dinv_c rc).  A block takes RI coarse rows; its threads gather
// the listed rows' values together into LDS (each fine row is read once, a
// lane per row), then a thread per coarse row adds its own.
constexpr int RI = 192;          // coarse rows per block
constexpr int RU = 4;            // gathers per thread and pass
constexpr int RCAP = RU * AB;    // listed rows per pass (4.6 per coarse row on average)

template <typename T>
__global__ void __launch_bounds__(AB)
amg_restrict(int32_t nc, const int32_t* __restrict__ rows_ptr, const int32_t* __restrict__ rows,
             const T* __restrict__ v, T* __restrict__ rc, const T* __restrict__ dinv_c, T omega,
             T* __restrict__ xc, const int32_t* gate) {
#pragma clang fp contract(off)
    __shared__ T tv[RCAP];
    __shared__ uint8_t tn[RCAP];
    if (gate && *gate < 0) return;
    const int32_t t = threadIdx.x;
    const int32_t nb = (nc + RI - 1) / RI;
    for (int32_t c = xcd_block(); c < nb; c += gridDim.x) {
        const int32_t I0 = c * RI, nI = min(RI, nc - I0);
        const int32_t f0 = rows_ptr[I0], f1 = rows_ptr[I0 + nI];
        int32_t fa = 0, fb = 0;
        if (t < nI) {
            fa = rows_ptr[I0 + t];
            fb = rows_ptr[I0 + t + 1];
        }
        T s = T(0), s1 = T(0);
        for (int32_t base = f0; base < f1; base += RCAP) {
            int32_t k[RU];
            T vv[RU];
            // past the list: its last row again, as in wave_row_sum
#pragma unroll
            for (int u = 0; u < RU; ++u) k[u] = rows[min(base + t + u * AB, f1 - 1)];
#pragma unroll
            for (int u = 0; u < RU; ++u) vv[u] = v[k[u] & INT32_MAX];
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                tv[t + u * AB] = vv[u];
                tn[t + u * AB] = k[u] < 0;
            }
            __syncthreads();
            for (int32_t f = max(fa, base); f < min(fb, base + RCAP); ++f) {
                if (tn[f - base]) {
                    s += s1;
                    s1 = T(0);
                }
                s1 += tv[f - base];
            }
            __syncthreads();
        }
        if (t < nI) {
            s += s1;
            rc[I0 + t] = s;
            if (xc) xc[I0 + t] = omega * (dinv_c[I0 + t] * s);
        }
    }
}

// x += e[map]
template <typename T>
__global__ void __launch_bounds__(AB)
amg_prolong(int32_t n, const int32_t* __restrict__ map, const T* __restrict__ e, T* __restrict__ x,
            const int32_t* gate) {
#pragma clang fp contract(off)
    if (gate && *gate < 0) return;
    for (int32_t i = blockIdx.x * AB + threadIdx.x; i < n; i += gridDim.x * AB) x[i] = x[i] + e[map[i]];
}

// y = x + omega (dinv (r - A x)); PART: partials of (r, y) -> PART_RZ and,
// RR, of (r, r) -> PART_RR, one per block at xcd_block()
template <typename T, bool PART, bool RR>
__global__ void __launch_bounds__(SPMV_BLOCK)
amg_post(int32_t n, SpmvIdx ix, const T* __restrict__ val, const T* __restrict__ x, const T* __restrict__ r,
         const T* __restrict__ dinv, T omega, T* __restrict__ y, T* __restrict__ part, const int32_t* gate) {
#pragma clang fp contract(off)
    __shared__ __align__(16) T lds[SPMV_CAP];
    __shared__ T xs[1];
    __shared__ T red[SPMV_BLOCK / 64];
    if (gate && *gate < 0) return;
    const XWin w{{0, 0}};
    T prz = T(0), prr = T(0);
    GroupRange gr = block_groups(ix, n);
    for (int32_t g = gr.g0; g < gr.n_groups; g += gr.step) {
        const int32_t r0 = g * SPMV_BLOCK;
        const int32_t nr = min(SPMV_BLOCK, n - r0);
        const GroupRow<T> row = spmv_group_row<T, -1>(ix, val, x, n, g, nr, w, xs, lds, gr);
        if ((int32_t)threadIdx.x < nr) {
            const int32_t i = r0 + threadIdx.x;
            const T ri = r[i];
            const T yi = x[i] + omega * (dinv[i] * (ri - row.s));
            y[i] = yi;
            prz += ri * yi;
            prr += ri * ri;
        }
    }
    if (PART) {
        const T b1 = block_sum<T, SPMV_BLOCK>(prz, red);
        if (RR) {
            const T b2 = block_sum<T, SPMV_BLOCK>(prr, red);
            if (threadIdx.x == 0) part[PART_RR + xcd_block()] = b2;
        }
        if (threadIdx.x == 0) part[PART_RZ + xcd_block()] = b1;
    }
}

// y = Cinv r on the coarsest level (one block); PART as amg_post
template <typename T, bool PART, bool RR>
__global__ void __launch_bounds__(AB)
amg_coarse(int32_t n, const T* __restrict__ cinv, const T* __restrict__ r, T* __restrict__ y, T* __restrict__ part,
           int32_t n_part, const int32_t* gate) {
#pragma clang fp contract(off)
    __shared__ T rs[AMG_COARSE_MAX];
    __shared__ T red[AB / 64];
    if (gate && *gate < 0) return;
    for (int32_t j = threadIdx.x; j < n; j += AB) rs[j] = r[j];
    __syncthreads();
    T prz = T(0), prr = T(0);
    for (int32_t i = threadIdx.x; i < n; i += AB) {
        T s = T(0);
        for (int32_t j = 0; j < n; ++j) s += cinv[(int64_t)i * n + j] * rs[j];
        y[i] = s;
        prz += rs[i] * s;
        prr += rs[i] * rs[i];
    }
    if (PART) {
        // the solve sums n_part partials: this block's, then zeros
        const T b1 = block_sum<T, AB>(prz, red);
        const T b2 = RR ? block_sum<T, AB>(prr, red) : T(0);
        if (threadIdx.x == 0) {
            part[PART_RZ] = b1;
            if (RR) part[PART_RR] = b2;
        }
        for (int32_t q = 1 + threadIdx.x; q < n_part; q += AB) {
            part[PART_RZ + q] = T(0);
            if (RR) part[PART_RR + q] = T(0);
        }
    }
}

// ---------------------------------------------------------------------------
// The tail of the V-cycle: every level from the first one with at most
// AMG_TAIL_ROWS rows down to the coarsest, in one workgroup.  Each step is
// the corresponding kernel's above, row by row with the same operations in
// the same order (rows' products summed in column order from 0, listed rows
// in their order, the coarsest inverse times r with j ascending), and the
// workgroup barrier stands where the level kernels had a launch boundary.
// On the small levels a launch costs more than its work.
// ---------------------------------------------------------------------------
constexpr int64_t AMG_TAIL_ROWS = RP_AMG_TAIL_ROWS;
constexpr int TB = 1024;              // threads of the tail workgroup
// Rows of the tail's steps together, and words of their lists and row_ptr, at
// most for the form that keeps vectors and lists in LDS (64 KB in FP64).  Rows
// fall by four or more from step to step, so nearly every hierarchy fits; one
// that coarsens by a few rows a level (a chain of growing couplings) does not.
constexpr int TAIL_LDS_ROWS = 2048;
constexpr int TAIL_LDS_IDX = 6144;

// One level the tail stops at: its first level, then the even ones, then the
// coarsest.  A first level of odd number only restricts and prolongs.
template <typename T>
struct TailStep {
    int32_t n, nnz;
    int32_t smooth;           // even level above the coarsest
    int32_t at;               // first element of the level in the tail's vectors
    int32_t idx;              // first word of its lists in LDS
    const int32_t* row_ptr;
    const int32_t* col;
    const T* val;
    const T* dinv;
    const int32_t* rows_ptr;  // all steps but the coarsest, as in AmgLevel
    const int32_t* rows;
    const int32_t* map;
};

// row i of A x: U entries per trip, every load of a trip issued before its
// first product; the products are added in column order from 0
template <typename T>
__device__ __forceinline__ T tail_row_sum(const TailStep<T>& L, const int32_t* row_ptr, const T* x, int32_t i) {
#pragma clang fp contract(off)
    constexpr int U = 12;
    T s = T(0);
    const int32_t e0 = row_ptr[i], e1 = row_ptr[i + 1];
    for (int32_t eb = e0; eb < e1; eb += U) {
        int32_t c[U];
        T v[U], xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = eb + u < e1;
            c[u] = in ? L.col[eb + u] : 0;
            v[u] = in ? L.val[eb + u] : T(0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) xv[u] = x[c[u]];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (eb + u < e1) s += v[u] * xv[u];
    }
    return s;
}

// one load per 128-byte line of a[0 .. n), folded into h (so that it is not dropped)
template <typename E>
__device__ __forceinline__ void touch(const E* a, int32_t n, uint32_t& h) {
    constexpr int PER = 128 / sizeof(E);
    for (int32_t i = threadIdx.x * PER; i < n; i += TB * PER) h |= *reinterpret_cast<const uint32_t*>(a + i);
}

__device__ __forceinline__ void tail_copy(int32_t* dst, const int32_t* src, int32_t n) {
    for (int32_t i = threadIdx.x; i < n; i += TB) dst[i] = src[i];
}

// y0 = V_lt(r0) over the tail's ns steps.  LV: vectors and lists live in LDS,
// else in work and where the hierarchy has them.  By the time the tail runs,
// the larger levels have pushed its matrices out of the die's L2, and every
// step would wait for memory several times over; so the workgroup first
// touches all of them, together.  One workgroup is bound by the latency of
// its chain of steps: 55 us after a 160^3 fine level with everything in
// memory, 34 with the vectors in LDS and the touches, 29 with the lists too.
template <typename T, bool LV>
__global__ void __launch_bounds__(TB)
amg_tail(int32_t ns, const TailStep<T>* __restrict__ st, const T* __restrict__ cinv, T omega,
         const T* __restrict__ r0, T* __restrict__ y0, T* work, int32_t total, const int32_t* gate) {
#pragma clang fp contract(off)
    __shared__ T lds[LV ? 2 * TAIL_LDS_ROWS + AMG_TAIL_ROWS : 1];
    __shared__ int32_t idx[LV ? TAIL_LDS_IDX : 1];
    if (gate && *gate < 0) return;
    const int32_t t = threadIdx.x;
    const int32_t span = LV ? TAIL_LDS_ROWS : total;
    // right-hand sides (results on the way up), iterates; one step's residual
    T* const vr = LV ? lds : work;
    T* const vx = vr + span;
    T* const vt = vx + span;
    uint32_t h = 0;
    for (int32_t k = 0; k + 1 < ns; ++k) {
        const TailStep<T>& S = st[k];
        const int32_t nc = st[k + 1].n;
        if (S.smooth) {
            touch(S.col, S.nnz, h);
            touch(S.val, S.nnz, h);
            touch(S.dinv, S.n, h);
        }
        if (LV) {
            tail_copy(idx + S.idx, S.rows_ptr, nc + 1);
            tail_copy(idx + S.idx + nc + 1, S.rows, S.n);
            tail_copy(idx + S.idx + nc + 1 + S.n, S.map, S.n);
            if (S.smooth) tail_copy(idx + S.idx + nc + 1 + 2 * S.n, S.row_ptr, S.n + 1);
        }
    }
    touch(cinv, st[ns - 1].n * st[ns - 1].n, h);
    for (int32_t i = t; i < st[0].n; i += TB) {
        const T ri = r0[i];
        vr[i] = ri;
        if (st[0].smooth) vx[i] = omega * (st[0].dinv[i] * ri);
    }
    asm volatile("" ::"v"(h));
    __syncthreads();
    for (int32_t k = 0; k + 1 < ns; ++k) {
        const TailStep<T>& S = st[k];
        const TailStep<T>& C = st[k + 1];
        const int32_t* rows_ptr = LV ? idx + S.idx : S.rows_ptr;
        const int32_t* rows = LV ? rows_ptr + C.n + 1 : S.rows;
        const T* r = vr + S.at;
        const T* src = r;   // what restricts to the next step
        if (S.smooth) {
            const int32_t* row_ptr = LV ? rows + 2 * S.n : S.row_ptr;
            for (int32_t i = t; i < S.n; i += TB) vt[i] = r[i] - tail_row_sum(S, row_ptr, vx + S.at, i);
            __syncthreads();
            src = vt;
        }
        for (int32_t I = t; I < C.n; I += TB) {
            T s = T(0), s1 = T(0);
            for (int32_t f = rows_ptr[I]; f < rows_ptr[I + 1]; ++f) {
                const int32_t q = rows[f];
                if (q < 0) {
                    s += s1;
                    s1 = T(0);
                }
                s1 += src[q & INT32_MAX];
            }
            s += s1;
            vr[C.at + I] = s;
            if (C.smooth) vx[C.at + I] = omega * (C.dinv[I] * s);
        }
        __syncthreads();
    }
    {
        const TailStep<T>& L = st[ns - 1];
        const int32_t n = L.n;   // at most AMG_COARSE_MAX
        T* r = vr + L.at;
        T s = T(0);
        if (t < n)
            for (int32_t j = 0; j < n; ++j) s += cinv[(int64_t)t * n + j] * r[j];
        __syncthreads();
        if (t < n) r[t] = s;
        __syncthreads();
    }
    for (int32_t k = ns - 2; k >= 0; --k) {
        const TailStep<T>& S = st[k];
        const TailStep<T>& C = st[k + 1];
        const int32_t* map = LV ? idx + S.idx + C.n + 1 + S.n : S.map;
        const T* e = vr + C.at;
        T* r = vr + S.at;
        if (!S.smooth) {
            for (int32_t i = t; i < S.n; i += TB) r[i] = e[map[i]];
        } else {
            const int32_t* row_ptr = LV ? map + S.n : S.row_ptr;
            T* x = vx + S.at;
            for (int32_t i = t; i < S.n; i += TB) x[i] = x[i] + e[map[i]];
            __syncthreads();
            for (int32_t i = t; i < S.n; i += TB)
                r[i] = x[i] + omega * (S.dinv[i] * (r[i] - tail_row_sum(S, row_ptr, x, i)));
        }
        __syncthreads();
    }
    for (int32_t i = t; i < st[0].n; i += TB) y0[i] = vr[i];
}

// the level-0 system of a hierarchy: the fused pattern (with its
// offset-coded SpMV form) or the solve-order copy (plain CSR)
struct Src {
    int64_t nnz;
    const int32_t* row_ptr;
    const int32_t* col;
    const double* val64;
    const float* val32;
    const double* dinv64;
    const float* dinv32;
    SpmvIdx ix;
};

Src source(const rp_plan* p, bool ordered) {
    if (ordered)
        return Src{p->nnz, p->d_ro_row_ptr, p->d_ro_col, p->d_ro_val64, p->d_ro_val32, p->d_ro_dinv64,
                   p->d_ro_dinv32, SpmvIdx{p->d_ro_row_ptr, p->d_ro_col, nullptr, nullptr, nullptr,
                                       (int32_t)p->nnz}};
    return Src{p->nnz, p->d_row_ptr, p->d_col, p->d_val64, p->d_val32, p->d_dinv64, p->d_dinv32, spmv_idx(p)};
}

AmgHier*& hier(rp_plan* p, bool ordered) { return ordered ? p->amg_ro : p->amg; }

template <typename T>
struct Prec;
template <>
struct Prec<double> {
    static const double* val(const AmgLevel& L) { return L.val64; }
    static const double* dinv(const AmgLevel& L) { return L.dinv64; }
    static double** vec(AmgLevel& L) { return L.vec64; }
    static const double* cinv(const AmgHier& h) { return h.cinv64; }
    static void*& tail(AmgHier& h) { return h.tail64; }
    static double*& work(AmgHier& h) { return h.tail_work64; }
    static const double* val0(const Src& q) { return q.val64; }
    static const double* dinv0(const Src& q) { return q.dinv64; }
};
template <>
struct Prec<float> {
    static const float* val(const AmgLevel& L) { return L.val32; }
    static const float* dinv(const AmgLevel& L) { return L.dinv32; }
    static float** vec(AmgLevel& L) { return L.vec32; }
    static const float* cinv(const AmgHier& h) { return h.cinv32; }
    static void*& tail(AmgHier& h) { return h.tail32; }
    static float*& work(AmgHier& h) { return h.tail_work32; }
    static const float* val0(const Src& q) { return q.val32; }
    static const float* dinv0(const Src& q) { return q.dinv32; }
};

template <typename T>
int alloc_vectors(AmgHier& h) {
    for (int32_t l = 0; l < h.n_levels; ++l) {
        AmgLevel& L = h.lev[l];
        T** v = Prec<T>::vec(L);
        const size_t bytes = sizeof(T) * (size_t)std::max<int64_t>(L.n, 1);
        // in and out down to the tail's first level (level 0 uses the solve's
        // vectors); x and t above it; nothing on the odd levels above it,
        // which the cycle steps over.  Each one is allocated once, so a call
        // after a failed one completes the set.
        if (l > h.tail_level || (l % 2 == 1 && l < h.tail_level)) continue;
        for (int k = 0; k < 4; ++k) {
            const bool need = (k == 0 || k == 3) ? l > 0 : l < h.tail_level;
            if (need && !v[k]) RP_HIP_TRY(hipMalloc(&v[k], bytes));
        }
    }
    // the tail's steps
    void*& tab = Prec<T>::tail(h);
    if (h.tail_level > 0 && !tab) {
        std::vector<TailStep<T>> tl;
        int64_t at = 0, idx = 0;
        for (int32_t l = h.tail_level;; l = h.lev[l].target) {
            const AmgLevel& L = h.lev[l];
            const bool last = l == h.n_levels - 1;
            const bool smooth = !last && l % 2 == 0;
            tl.push_back(TailStep<T>{(int32_t)L.n, (int32_t)L.nnz, smooth, (int32_t)at, (int32_t)idx, L.row_ptr,
                                     L.col, Prec<T>::val(L), Prec<T>::dinv(L), L.rows_ptr, L.rows, L.map});
            at += L.n;
            if (last) break;
            idx += h.lev[L.target].n + 1 + 2 * L.n + (smooth ? L.n + 1 : 0);
        }
        h.tail_steps = (int32_t)tl.size();
        h.tail_rows = (int32_t)at;
        h.tail_in_lds = at <= TAIL_LDS_ROWS && idx <= TAIL_LDS_IDX;
        T*& w = Prec<T>::work(h);
        if (!h.tail_in_lds && !w) RP_HIP_TRY(hipMalloc(&w, sizeof(T) * (size_t)(2 * at + AMG_TAIL_ROWS)));
        void* d = nullptr;
        RP_HIP_TRY(hipMalloc(&d, sizeof(TailStep<T>) * tl.size()));
        const hipError_t e = hipMemcpy(d, tl.data(), sizeof(TailStep<T>) * tl.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            (void)hipFree(d);
            RP_HIP_TRY(e);
        }
        tab = d;
    }
    return RP_OK;
}

// Levels below level 0 with at most this many rows add the coarse correction
// where the post-smoothing reads x: two more gathers per entry, a launch less.
// Measured per level (FP64): 8.8 us against 4.9 + 4.7 at 24000 rows, even at
// 10^5, 13.4 against 5 + 6 with launches at 10^5 and slower beyond.  (The
// residual in the restriction's kernel, its rows in list order, was slower
// above 20000 rows and gained nothing below.)
constexpr int64_t AMG_FUSE_UP_ROWS = 1 << 16;

// from the right-hand side r of even level l: residual after one sweep from
// zero (x = omega (dinv r) is in v[1]) restricted to level L.target, with that
// level's first sweep
template <typename T>
int cycle_down(AmgHier& h, const Src& q, int32_t l, const T* r, const int32_t* gate, hipStream_t s) {
    AmgLevel& L = h.lev[l];
    AmgLevel& C = h.lev[L.target];
    const int32_t n = (int32_t)L.n, nc = (int32_t)C.n;
    const T omega = (T)RP_AMG_OMEGA;
    T** v = Prec<T>::vec(L);
    T** cv = Prec<T>::vec(C);
    T* xc = L.target < h.tail_level ? cv[1] : nullptr;   // the tail makes its own first sweep
    const T* dinv_c = Prec<T>::dinv(C);
    if (l == 0) {
        hipLaunchKernelGGL(amg_resid<T>, dim3(product_grid(n, q.nnz)), dim3(SPMV_BLOCK), 0, s, n, q.ix,
                           Prec<T>::val0(q), v[1], r, v[2], gate);
    } else {
        const int cr = chunk_rows(L), g = chunk_grid(n, cr);
        if (cr == 64)
            hipLaunchKernelGGL((amg_csr_resid<T, 64>), dim3(g), dim3(WB), 0, s, n, L.row_ptr, L.col,
                               Prec<T>::val(L), v[1], r, v[2], gate);
        else
            hipLaunchKernelGGL((amg_csr_resid<T, 32>), dim3(g), dim3(WB), 0, s, n, L.row_ptr, L.col,
                               Prec<T>::val(L), v[1], r, v[2], gate);
    }
    hipLaunchKernelGGL(amg_restrict<T>, dim3(chunk_grid(nc, RI)), dim3(AB), 0, s, nc, L.rows_ptr, L.rows, v[2], cv[0],
                       dinv_c, omega, xc, gate);
    RP_HIP_TRY(hipGetLastError());
    return RP_OK;
}

// level l > 0 on the way up: y (v[3]) from x (v[1]), the right-hand side
// (v[0]) and the correction e of level L.target
template <typename T>
int cycle_up(AmgHier& h, int32_t l, const int32_t* gate, hipStream_t s) {
    AmgLevel& L = h.lev[l];
    const int32_t n = (int32_t)L.n;
    const T omega = (T)RP_AMG_OMEGA;
    T** v = Prec<T>::vec(L);
    const T* e = Prec<T>::vec(h.lev[L.target])[3];
    const int cr = chunk_rows(L), g = chunk_grid(n, cr);
#define RP_LAUNCH(CR, X, x)                                                                                   \
    hipLaunchKernelGGL((amg_csr_post<T, CR, X>), dim3(g), dim3(WB), 0, s, n, L.row_ptr, L.col, Prec<T>::val(L), x, \
                       v[0], Prec<T>::dinv(L), omega, v[3], gate)
    if (n <= AMG_FUSE_UP_ROWS) {
        const CorrectedX<T> x{v[1], e, L.map};
        if (cr == 64) RP_LAUNCH(64, CorrectedX<T>, x);
        else RP_LAUNCH(32, CorrectedX<T>, x);
    } else {
        hipLaunchKernelGGL(amg_prolong<T>, dim3(grid_of(n)), dim3(AB), 0, s, n, L.map, e, v[1], gate);
        const PlainX<T> x{v[1]};
        if (cr == 64) RP_LAUNCH(64, PlainX<T>, x);
        else RP_LAUNCH(32, PlainX<T>, x);
    }
#undef RP_LAUNCH
    RP_HIP_TRY(hipGetLastError());
    return RP_OK;
}

// y = V_0(r) on stream s: down the even levels to the tail, the tail, and up
// again.  An odd level above the tail only restricts and prolongs, so the
// cycle steps over it through the composed lists (AmgLevel::rows, ::map): a
// small level's launch costs about 4.6 us whatever it does, and a large one's
// vectors a pass each.  With the odd levels as launches of their own, a first
// sweep per level and the tail's vectors in memory, a cycle took 355 us at
// 131 x 117 x 142 cells, 598 at 160^3 and 1799 at 256^3 (FP64, 40 launches);
// now 242, 401 and 1387 us (19 to 21 launches).  What is left is the fine
// level's two products (27 + 29 us of the 242, near the memory's rate) and,
// below about 10^5 rows, the launches.  swept: amg_first_sweep(h) already holds
// omega (dinv r).
template <typename T>
int vcycle(AmgHier& h, const Src& q, const T* r, T* y, T* part, int32_t n_part, bool rr, bool swept,
           const int32_t* gate, hipStream_t s) {
    AmgLevel& L0 = h.lev[0];
    const int32_t n = (int32_t)L0.n;
    const T omega = (T)RP_AMG_OMEGA;
    const bool want = part != nullptr;
    if (h.n_levels == 1) {
#define RP_LAUNCH(PT, RRF)                                                                                       \
    hipLaunchKernelGGL((amg_coarse<T, PT, RRF>), dim3(1), dim3(AB), 0, s, n, Prec<T>::cinv(h), r, y, part, n_part, \
                       gate)
        if (want && rr) RP_LAUNCH(true, true);
        else if (want) RP_LAUNCH(true, false);
        else RP_LAUNCH(false, false);
#undef RP_LAUNCH
        RP_HIP_TRY(hipGetLastError());
        return RP_OK;
    }
    T** v = Prec<T>::vec(L0);
    if (!swept)
        hipLaunchKernelGGL(amg_pre<T>, dim3(grid_of(n)), dim3(AB), 0, s, n, r, Prec<T>::dinv0(q), v[1], omega,
                           gate);
    for (int32_t l = 0; l < h.tail_level; l = h.lev[l].target)
        RP_TRY(cycle_down<T>(h, q, l, l == 0 ? r : Prec<T>::vec(h.lev[l])[0], gate, s));
    {
        T** tv = Prec<T>::vec(h.lev[h.tail_level]);
#define RP_LAUNCH(LV)                                                                                          \
    hipLaunchKernelGGL((amg_tail<T, LV>), dim3(1), dim3(TB), 0, s, h.tail_steps,               \
                       (const TailStep<T>*)Prec<T>::tail(h), Prec<T>::cinv(h), omega, (const T*)tv[0], tv[3], \
                       Prec<T>::work(h), h.tail_rows, gate)
        if (h.tail_in_lds) RP_LAUNCH(true);
        else RP_LAUNCH(false);
#undef RP_LAUNCH
    }
    RP_HIP_TRY(hipGetLastError());
    // the even levels above the tail, back to level 2
    for (int32_t l = (h.tail_level - 1) & ~1; l > 0; l -= 2) RP_TRY(cycle_up<T>(h, l, gate, s));
    hipLaunchKernelGGL(amg_prolong<T>, dim3(grid_of(n)), dim3(AB), 0, s, n, L0.map,
                       (const T*)Prec<T>::vec(h.lev[L0.target])[3], v[1], gate);
#define RP_LAUNCH(PT, RRF)                                                                                       \
    hipLaunchKernelGGL((amg_post<T, PT, RRF>), dim3(PT ? spmv_grid(n) : product_grid(n, q.nnz)), dim3(SPMV_BLOCK),    \
                       0, s, n, q.ix, Prec<T>::val0(q), v[1], r, Prec<T>::dinv0(q), omega, y, part, gate)
    if (want && rr) RP_LAUNCH(true, true);
    else if (want) RP_LAUNCH(true, false);
    else RP_LAUNCH(false, false);
#undef RP_LAUNCH
    RP_HIP_TRY(hipGetLastError());
    return RP_OK;
}

template <typename T>
T* dalloc(int64_t n) {
    T* q = nullptr;
    if (hipMalloc(&q, sizeof(T) * (size_t)std::max<int64_t>(n, 1)) != hipSuccess) return nullptr;
    return q;
}

#define RP_DALLOC(ptr, T, n)                                          \
    do {                                                              \
        (ptr) = dalloc<T>(n);                                         \
        if (!(ptr)) {                                                 \
            set_error("out of device memory building the multigrid"); \
            return RP_ERR_HIP;                                        \
        }                                                             \
    } while (0)

void free_level(AmgLevel& L) {
    void* q[] = {L.row_ptr, L.col, L.val64, L.val32, L.dinv64, L.dinv32, L.diag_pos, L.agg, L.mem_ptr, L.mem,
                 L.cptr, L.cpos, L.links, L.vec64[0], L.vec64[1], L.vec64[2], L.vec64[3], L.vec32[0], L.vec32[1],
                 L.vec32[2], L.vec32[3]};
    for (void* a : q)
        if (a) (void)hipFree(a);
    L = AmgLevel();
}

// level l + 1 from level l (its CSR: row_ptr, col, val64)
int coarsen(AmgHier& h, const Src& q, int32_t l, hipStream_t s) {
    AmgLevel& L = h.lev[l];
    const int32_t n = (int32_t)L.n;
    const int32_t* rp_ = l == 0 ? q.row_ptr : L.row_ptr;
    const int32_t* cl = l == 0 ? q.col : L.col;
    const double* vl = l == 0 ? q.val64 : L.val64;
    struct Tmp {   // work arrays of this call, freed on every return
        std::vector<void*> q;
        ~Tmp() {
            for (void* a : q)
                if (a) (void)hipFree(a);
        }
    } tmp;
    int32_t *mate = nullptr, *pick = nullptr, *leader = nullptr, *is_leader = nullptr, *lead_id = nullptr;
    RP_DALLOC(mate, int32_t, n);
    tmp.q.push_back(mate);
    RP_DALLOC(pick, int32_t, n);
    tmp.q.push_back(pick);
    RP_DALLOC(leader, int32_t, n);
    tmp.q.push_back(leader);
    RP_DALLOC(is_leader, int32_t, n);
    tmp.q.push_back(is_leader);
    RP_DALLOC(lead_id, int32_t, n + 1);
    tmp.q.push_back(lead_id);
    const int g = grid_of(n);
    hipLaunchKernelGGL(amg_fill, dim3(g), dim3(AB), 0, s, n, -1, mate);
    for (int round = 0; round < AMG_ROUNDS; ++round) {
        hipLaunchKernelGGL(amg_fill, dim3(1), dim3(AB), 0, s, 1, 0, (int32_t*)h.flag);
        hipLaunchKernelGGL(amg_pick, dim3(g), dim3(AB), 0, s, n, rp_, cl, vl, mate, pick);
        hipLaunchKernelGGL(amg_pair, dim3(g), dim3(AB), 0, s, n, pick, mate, h.flag);
        RP_HIP_TRY(hipGetLastError());
        uint32_t pairs = 0;
        RP_HIP_TRY(hipMemcpyAsync(&pairs, h.flag, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
        RP_HIP_TRY(hipStreamSynchronize(s));
        if (pairs == 0) break;
    }
    hipLaunchKernelGGL(amg_leader, dim3(g), dim3(AB), 0, s, n, rp_, cl, vl, mate, leader, is_leader);
    RP_HIP_TRY(hipGetLastError());
    int32_t nc = 0;
    RP_TRY(scan_i32(is_leader, n, lead_id, &nc, s));
    if (nc == n) {
        set_error("multigrid: no aggregate formed on level %d (%d rows without negative couplings)", l, n);
        return RP_ERR_UNSUPPORTED;
    }
    AmgLevel& C = h.lev[l + 1];
    C.n = nc;
    RP_DALLOC(L.agg, int32_t, n);
    RP_DALLOC(L.mem_ptr, int32_t, nc + 1);
    RP_DALLOC(L.mem, int32_t, n);
    int32_t *cnt = nullptr, *kstart = nullptr, *ucnt = nullptr;
    RP_DALLOC(cnt, int32_t, nc + 1);
    tmp.q.push_back(cnt);
    hipLaunchKernelGGL(amg_fill, dim3(grid_of(nc)), dim3(AB), 0, s, nc, 0, cnt);
    hipLaunchKernelGGL(amg_number, dim3(g), dim3(AB), 0, s, n, leader, lead_id, L.agg, cnt);
    RP_HIP_TRY(hipGetLastError());
    int32_t total = 0;
    RP_TRY(scan_i32(cnt, nc, L.mem_ptr, &total, s));
    hipLaunchKernelGGL(amg_fill, dim3(grid_of(nc)), dim3(AB), 0, s, nc, 0, cnt);
    hipLaunchKernelGGL(amg_members, dim3(g), dim3(AB), 0, s, n, L.agg, L.mem_ptr, cnt, L.mem);
    hipLaunchKernelGGL(amg_sort_members, dim3(grid_of(nc)), dim3(AB), 0, s, nc, L.mem_ptr, L.mem, rp_, cnt);
    RP_HIP_TRY(hipGetLastError());
    RP_DALLOC(kstart, int32_t, nc + 1);
    tmp.q.push_back(kstart);
    int32_t nkeys = 0;
    RP_TRY(scan_i32(cnt, nc, kstart, &nkeys, s));
    if ((int64_t)nkeys != L.nnz) {
        set_error("multigrid: %d coarse keys for %lld fine entries on level %d", nkeys, (long long)L.nnz, l);
        return RP_ERR_HIP;
    }
    uint64_t* keys = nullptr;
    RP_DALLOC(keys, uint64_t, L.nnz);
    tmp.q.push_back(keys);
    RP_DALLOC(ucnt, int32_t, nc + 1);
    tmp.q.push_back(ucnt);
    hipLaunchKernelGGL(amg_keys, dim3(grid_of(nc)), dim3(AB), 0, s, nc, L.mem_ptr, L.mem, rp_, cl, L.agg, kstart,
                       keys, ucnt);
    RP_HIP_TRY(hipGetLastError());
    RP_DALLOC(C.row_ptr, int32_t, nc + 1);
    int32_t nnz_c = 0;
    RP_TRY(scan_i32(ucnt, nc, C.row_ptr, &nnz_c, s));
    C.nnz = nnz_c;
    RP_DALLOC(C.col, int32_t, nnz_c + SPMV_PAD);
    RP_DALLOC(C.val64, double, nnz_c + SPMV_PAD);
    RP_DALLOC(C.val32, float, nnz_c + SPMV_PAD);
    RP_DALLOC(C.dinv64, double, nc);
    RP_DALLOC(C.dinv32, float, nc);
    RP_DALLOC(C.diag_pos, int32_t, nc);
    RP_DALLOC(L.cptr, int32_t, nnz_c + 1);
    RP_DALLOC(L.cpos, int32_t, L.nnz);
    RP_HIP_TRY(hipMemsetAsync(C.col + nnz_c, 0, sizeof(int32_t) * SPMV_PAD, s));
    RP_HIP_TRY(hipMemsetAsync(C.val64 + nnz_c, 0, sizeof(double) * SPMV_PAD, s));
    RP_HIP_TRY(hipMemsetAsync(C.val32 + nnz_c, 0, sizeof(float) * SPMV_PAD, s));
    hipLaunchKernelGGL(amg_cfill, dim3(grid_of(nc)), dim3(AB), 0, s, nc, kstart, keys, C.row_ptr, C.col, C.diag_pos,
                       L.cptr, L.cpos);
    RP_HIP_TRY(hipGetLastError());
    RP_HIP_TRY(hipStreamSynchronize(s));
    return RP_OK;
}

// Where the V-cycle's step at level l restricts to: the next level if the
// tail starts there, if it is the coarsest, or if l itself is an odd level
// (the tail's first); else past the odd level below l, whose aggregates are
// then composed with level l's.
int link_levels(AmgHier& h, hipStream_t s) {
    int32_t* tmp = nullptr;   // counts, positions and the scan's scratch, for the largest odd level
    struct Free {
        int32_t*& q;
        ~Free() {
            if (q) (void)hipFree(q);
        }
    } guard{tmp};
    for (int32_t l = 0; l < h.n_levels - 1; l = h.lev[l].target) {
        AmgLevel &L = h.lev[l], &M = h.lev[l + 1];
        if (l + 1 == h.tail_level || l + 1 == h.n_levels - 1 || l % 2 == 1) {
            L.target = l + 1;
            L.map = L.agg;
            L.rows = L.mem;
            L.rows_ptr = L.mem_ptr;
            continue;
        }
        L.target = l + 2;
        const int32_t n = (int32_t)L.n, nm = (int32_t)M.n, nc = (int32_t)h.lev[l + 2].n;
        if (!tmp) RP_DALLOC(tmp, int32_t, 2 * ((int64_t)nm + 1) + scan_i32_scratch(nm));
        int32_t *cnt = tmp, *pos = tmp + nm + 1, *scratch = pos + nm + 1;
        RP_DALLOC(L.links, int32_t, 2 * (int64_t)n + nc + 1);
        int32_t *map = L.links, *rows = map + n, *rows_ptr = rows + n;
        L.map = map;
        L.rows = rows;
        L.rows_ptr = rows_ptr;
        hipLaunchKernelGGL(amg_link_count, dim3(grid_of(nm)), dim3(AB), 0, s, nm, M.mem, L.mem_ptr, cnt);
        RP_TRY(scan_i32_enqueue(cnt, nm, pos, scratch, s));
        hipLaunchKernelGGL(amg_link_rows, dim3(grid_of(nm)), dim3(AB), 0, s, nm, M.mem, L.mem_ptr, L.mem, pos, rows);
        hipLaunchKernelGGL(amg_link_ptr, dim3(grid_of(nc + 1)), dim3(AB), 0, s, nc, M.mem_ptr, pos, rows_ptr);
        hipLaunchKernelGGL(amg_link_map, dim3(grid_of(n)), dim3(AB), 0, s, n, L.agg, M.agg, map);
        RP_HIP_TRY(hipGetLastError());
    }
    RP_HIP_TRY(hipStreamSynchronize(s));   // tmp is released
    return RP_OK;
}

// coarse values, diagonals and the coarsest inverse from the plan's values
int refresh(AmgHier& h, const Src& q, int64_t version, hipStream_t s) {
    hipLaunchKernelGGL(amg_fill, dim3(1), dim3(AB), 0, s, 1, 0, (int32_t*)h.flag);
    for (int32_t l = 0; l + 1 < h.n_levels; ++l) {
        AmgLevel &L = h.lev[l], &C = h.lev[l + 1];
        const double* fine = l == 0 ? q.val64 : L.val64;
        hipLaunchKernelGGL(amg_gvals, dim3(grid_of(C.nnz)), dim3(AB), 0, s, (int32_t)C.nnz, L.cptr, L.cpos, fine,
                           C.val64, C.val32);
        hipLaunchKernelGGL(amg_gdiag, dim3(grid_of(C.n)), dim3(AB), 0, s, (int32_t)C.n, C.diag_pos, C.val64, C.dinv64,
                           C.dinv32, h.flag);
        RP_HIP_TRY(hipGetLastError());
    }
    const AmgLevel& Lc = h.lev[h.n_levels - 1];
    const int32_t* rp_ = h.n_levels == 1 ? q.row_ptr : Lc.row_ptr;
    const int32_t* cl = h.n_levels == 1 ? q.col : Lc.col;
    const double* vl = h.n_levels == 1 ? q.val64 : Lc.val64;
    hipLaunchKernelGGL(amg_dense_inverse, dim3(1), dim3(GJ_THREADS), 0, s, (int32_t)Lc.n, rp_, cl, vl, h.cwork,
                       h.cinv64, h.cinv32, h.flag);
    RP_HIP_TRY(hipGetLastError());
    uint32_t bad = 0;
    RP_HIP_TRY(hipMemcpyAsync(&bad, h.flag, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    RP_HIP_TRY(hipStreamSynchronize(s));
    if (bad) {
        set_error("multigrid: a coarse diagonal or a pivot of the coarsest inverse is not positive");
        return RP_ERR_BREAKDOWN;
    }
    h.version = version;
    return RP_OK;
}

void free_hier(AmgHier*& hp) {
    if (!hp) return;
    AmgHier& h = *hp;
    // every level: a failed coarsening leaves arrays on the level it was building
    for (int32_t l = 0; l < AMG_MAX_LEVELS; ++l) free_level(h.lev[l]);
    for (void* a : {(void*)h.cinv64, (void*)h.cinv32, (void*)h.cwork, (void*)h.flag, h.tail64, h.tail32, (void*)h.tail_work64, (void*)h.tail_work32})
        if (a) (void)hipFree(a);
    delete hp;
    hp = nullptr;
}

}  // namespace

void amg_free(rp_plan* p) {
    free_hier(p->amg);
    free_hier(p->amg_ro);
}

int amg_setup(rp_plan* p, hipStream_t s, bool ordered) {
    if (p->nnz_nl > 0) {
        set_error("multigrid needs the whole system on the GPU (the share has a non-local block)");
        return RP_ERR_UNSUPPORTED;
    }
    AmgHier*& hp = hier(p, ordered);
    free_hier(hp);
    // a fused-order rebuild also retires the solve-order hierarchy: the next
    // multigrid solve in solve order builds it from the values then current
    if (!ordered) free_hier(p->amg_ro);
    hp = new AmgHier();
    AmgHier& h = *hp;
    const Src q = source(p, ordered);
    int rc = RP_OK;
    auto fail = [&](int code) {
        free_hier(hp);
        return code;
    };
    h.flag = dalloc<uint32_t>(2);
    if (!h.flag) return fail((set_error("out of device memory building the multigrid"), RP_ERR_HIP));
    h.lev[0].n = p->n_rows;
    h.lev[0].nnz = q.nnz;
    h.n_levels = 1;
    while (h.lev[h.n_levels - 1].n > AMG_COARSE_MAX) {
        if (h.n_levels == AMG_MAX_LEVELS) {
            set_error("multigrid: more than %d levels", AMG_MAX_LEVELS);
            return fail(RP_ERR_UNSUPPORTED);
        }
        if ((rc = coarsen(h, q, h.n_levels - 1, s)) != RP_OK) return fail(rc);
        h.n_levels += 1;
        // the coarse values now, so the next level's matching sees them
        AmgLevel &L = h.lev[h.n_levels - 2], &C = h.lev[h.n_levels - 1];
        const double* fine = h.n_levels == 2 ? q.val64 : L.val64;
        hipLaunchKernelGGL(amg_gvals, dim3(grid_of(C.nnz)), dim3(AB), 0, s, (int32_t)C.nnz, L.cptr, L.cpos, fine,
                           C.val64, C.val32);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return fail((set_error("launching amg_gvals failed: %s", hipGetErrorString(e)), RP_ERR_HIP));
    }
    // the first level below level 0 small enough for the one-workgroup tail
    for (int32_t l = 1; l < h.n_levels && h.tail_level == 0; ++l)
        if (h.lev[l].n <= AMG_TAIL_ROWS) h.tail_level = l;
    if ((rc = link_levels(h, s)) != RP_OK) return fail(rc);
    const int64_t nL = h.lev[h.n_levels - 1].n;
    h.cinv64 = dalloc<double>(nL * nL);
    h.cinv32 = dalloc<float>(nL * nL);
    h.cwork = dalloc<double>(nL * nL);
    if (!h.cinv64 || !h.cinv32 || !h.cwork)
        return fail((set_error("out of device memory building the multigrid"), RP_ERR_HIP));
    if ((rc = refresh(h, q, p->values_version, s)) != RP_OK) return fail(rc);
    return RP_OK;
}

int amg_prepare(rp_plan* p, bool fp32, hipStream_t s, bool ordered) {
    RP_TRY(alloc_z(p));
    AmgHier*& hp = hier(p, ordered);
    if (!hp) RP_TRY(amg_setup(p, s, ordered));
    if (hp->version != p->values_version) RP_TRY(refresh(*hp, source(p, ordered), p->values_version, s));
    if (fp32) RP_TRY(alloc_vectors<float>(*hp));
    else RP_TRY(alloc_vectors<double>(*hp));
    return RP_OK;
}

template <typename T>
T* amg_first_sweep(rp_plan* p, bool ordered) {
    return Prec<T>::vec(hier(p, ordered)->lev[0])[1];
}

template <typename T>
int amg_apply(rp_plan* p, const T* r, T* y, T* part, int32_t n_part, bool rr, bool swept, const int32_t* gate,
              hipStream_t s, bool ordered) {
    return vcycle<T>(*hier(p, ordered), source(p, ordered), r, y, part, n_part, rr, swept, gate, s);
}

template double* amg_first_sweep<double>(rp_plan*, bool);
template float* amg_first_sweep<float>(rp_plan*, bool);
template int amg_apply<double>(rp_plan*, const double*, double*, double*, int32_t, bool, bool, const int32_t*,
                               hipStream_t, bool);
template int amg_apply<float>(rp_plan*, const float*, float*, float*, int32_t, bool, bool, const int32_t*,
                              hipStream_t, bool);

}  // namespace rp
