// CG iterations on medium systems in one launch: one workgroup
// per compute unit, each owning a tile of consecutive rows for the whole
// launch.
//
// With three launches an iteration of a system of 10^6 rows spends some 13 us
// on launches and 10 n words on vectors.  Here x, r, z and M^-1 of a thread's
// rows stay in registers and p of the tile in LDS, together with p of its
// halo (the columns of its rows that other tiles own), so an iteration reads
// the matrix's values once, from the 256 MB memory-side cache where they fit
// it, and nothing else of size: the taps of the product come from LDS.  As in
// the resident loop for small systems (cg_loop.hip), an iteration exchanges
// z = M^-1 r and the three sums by value (exchange.hpp), in two exchanges:
//   (p, q) partials;   alpha, r, z;   z of the rows in other tiles' halos and
//   the (r, z), (r, r) partials;      stop tests, x, beta, p of tile and halo.
//
// The plan builds, once, each tile's halo (sorted) and, per row, the places in
// LDS of its columns (16-bit words, in column order); the values follow in
// slices of 64 rows, entry by entry, so that a wavefront's loads are whole
// lines.  They are refreshed by one pass when a solve finds them older than
// the last update.  Row sums run in column order from 0, every product and sum
// rounded once, so q is the SpMV's bit for bit; the dot products add a tile's
// rows first, so they differ from the launched kernels' by rounding.
//
// A plan fits if no row has more than U entries, the tiles hold its rows (16 per
// thread in FP64, 32 in FP32), and every tile's rows and halo fit LDS.  A mesh
// in a rank's natural order does as it is.  Where the numbering has no
// locality (an unstructured mesh) and a tile's halo would be nearly the whole
// rank, the tiles are cut from an order of their own (tile_order.hip): `order`
// gives the row at each position, the loop's private copies follow it and a
// launch's vectors are gathered before it and scattered after.
//
// Per iteration against three launches: FP64 26.3 -> 11.2 us at 80^3 rows, 36.8
// -> 16.4 at 96^3, 57.2 -> 23.6 at 110 x 108 x 112, 68.5 -> 38.2 at 128^3; FP32
// 20.6 -> 9.6, 28.1 -> 12.1, 44.5 -> 15.6, 46.7 -> 20.0, and 72.6 -> 50 at 160^3.
// Cells numbered at random, by the order: FP64 62 -> 16.6 us at 100 x 90 x 95
// (48 ranks), 130 -> 42 at 128^3; FP32 52 -> 13.1, 110 -> 22, and 235 -> 51 at
// 150 x 160 x 160; finding the order takes the first solve 7 and 16 ms more.
// About 7 us of it are the exchanges; the rest streams the values and, past
// some 10 rows per thread, the places and spilled registers: at 128^3 FP64 the
// counters have 185 MB read past the L2s and 32 MB written an iteration, of
// which values 117, places 34, and the spills of 16 rows a thread 27 each way.
// Non-temporal loads of the values made it slower (16.4 -> 18 us at 96^3: they
// come from the caches), more rows in flight no faster.
#include <algorithm>
#include <utility>
#include <vector>

#include "tile.hpp"

namespace rp {

// tile_order.hip
int tile_order(rp_plan* p, int64_t cap, int32_t* order, int32_t* inv, hipStream_t s, bool* ok, bool* memory);

namespace {

constexpr int LIST_MAX = 16384;   // halo entries with repeats, while building

// ---- structure ---------------------------------------------------------------
// One block per tile b, rows first[b] .. first[b + 1) (R at most): collect the
// columns outside the tile, sort them in LDS, drop repeats -> halo and its
// length (-1: does not fit); then the places, row l of tile b at b R + l.
// Rows and columns are positions; order and inv (nullptr: the identity)
// translate.
__global__ void __launch_bounds__(1024)
tile_build(int32_t R, const int32_t* __restrict__ first, const int32_t* __restrict__ order,
           const int32_t* __restrict__ inv, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
           int32_t* __restrict__ halo, int32_t* __restrict__ n_halo, Places* __restrict__ places) {
    __shared__ int32_t list[LIST_MAX];
    __shared__ int32_t uniq[HALO_MAX];
    __shared__ int32_t wtot[16];
    __shared__ int32_t count;
    const int32_t t = threadIdx.x, b = blockIdx.x;
    const int32_t base = first[b], rows = first[b + 1] - base;
    Places* const pb = places + (int64_t)b * R;
    if (t == 0) count = 0;
    __syncthreads();
    for (int32_t i = t; i < rows; i += 1024) {
        const int32_t row = order ? order[base + i] : base + i;
        for (int32_t e = row_ptr[row]; e < row_ptr[row + 1]; ++e) {
            const int32_t c = (inv ? inv[col[e]] : col[e]) - base;
            if (c < 0 || c >= rows) {
                const int32_t at = atomicAdd(&count, 1);
                if (at < LIST_MAX) list[at] = c + base;
            }
        }
    }
    __syncthreads();
    const int32_t m = count;
    if (m > LIST_MAX) {
        if (t == 0) n_halo[b] = -1;
        return;
    }
    int32_t P2 = 1;
    while (P2 < m) P2 *= 2;
    for (int32_t i = m + t; i < P2; i += 1024) list[i] = INT32_MAX;
    __syncthreads();
    for (int32_t k = 2; k <= P2; k *= 2)
        for (int32_t j = k / 2; j > 0; j /= 2) {
            for (int32_t i = t; i < P2; i += 1024) {
                const int32_t o = i ^ j;
                if (o > i) {
                    const int32_t x = list[i], y = list[o];
                    if ((x > y) == ((i & k) == 0)) {
                        list[i] = y;
                        list[o] = x;
                    }
                }
            }
            __syncthreads();
        }
    // each thread takes LIST_MAX / 1024 consecutive elements of the sorted list
    constexpr int PER = LIST_MAX / 1024;
    int32_t c = 0;
    for (int32_t i = t * PER; i < min(m, t * PER + PER); ++i) c += i == 0 || list[i] != list[i - 1];
    const int32_t inc = wave_incl_scan(c);
    if ((t & 63) == 63) wtot[t >> 6] = inc;
    __syncthreads();
    int32_t at = inc - c, H = 0;
    for (int q = 0; q < 16; ++q) {
        if (q < (t >> 6)) at += wtot[q];
        H += wtot[q];
    }
    if (H > HALO_MAX) {
        if (t == 0) n_halo[b] = -1;
        return;
    }
    for (int32_t i = t * PER; i < min(m, t * PER + PER); ++i)
        if (i == 0 || list[i] != list[i - 1]) uniq[at++] = list[i];
    __syncthreads();
    for (int32_t i = t; i < H; i += 1024) halo[(int64_t)b * HALO_MAX + i] = uniq[i];
    if (t == 0) n_halo[b] = H;
    for (int32_t i = t; i < rows; i += 1024) {
        const int32_t row = order ? order[base + i] : base + i;
        const int32_t e0 = row_ptr[row], len = row_ptr[row + 1] - e0;
        Places pl;
        for (int u = 0; u < 8; ++u) {
            uint32_t w = (uint32_t)i;   // a missing entry: its own row's place, times 0
            if (u < len) {
                const int32_t g = inv ? inv[col[e0 + u]] : col[e0 + u], cl = g - base;
                if (cl >= 0 && cl < rows) {
                    w = (uint32_t)cl;
                } else {
                    int32_t lo = 0, hi = H;
                    while (lo < hi) {
                        const int32_t mid = (lo + hi) >> 1;
                        if (uniq[mid] < g) lo = mid + 1;
                        else hi = mid;
                    }
                    w = (uint32_t)(R + lo);
                }
            }
            if (u % 2 == 0) pl.w[u / 2] = w;
            else pl.w[u / 2] |= w << 16;
        }
        pb[i] = pl;
    }
    // the places past the tile's rows: no entries
    for (int32_t i = rows + t; i < R; i += 1024) {
        const uint32_t w = (uint32_t)i | ((uint32_t)i << 16);
        pb[i] = Places{{w, w, w, w}};
    }
}

// values in slices of 64 rows: entry u of row l of tile b at
// ((b R + l) / 64 U + u) 64 + l % 64; zeros past the tile's rows
template <typename T>
__global__ void __launch_bounds__(256)
tile_values(int32_t R, const int32_t* __restrict__ first, const int32_t* __restrict__ order,
            const int32_t* __restrict__ row_ptr, const T* __restrict__ val, T* __restrict__ out) {
    const int32_t base = first[blockIdx.y], rows = first[blockIdx.y + 1] - base;
    const int32_t l = blockIdx.x * 256 + threadIdx.x;   // R is a multiple of 256
    int32_t e0 = 0, len = 0;
    if (l < rows) {
        const int32_t row = order ? order[base + l] : base + l;
        e0 = row_ptr[row];
        len = row_ptr[row + 1] - e0;
    }
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = u < len ? val[e0 + u] : T(0);
    T* o = out + (((int64_t)blockIdx.y * R + l) >> 6) * U * 64 + (l & 63);
#pragma unroll
    for (int u = 0; u < U; ++u) o[u * 64] = v[u];
}

__global__ void clear_words(uint32_t* w, int64_t words, uint32_t* bar) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (int64_t)gridDim.x * 256) w[i] = ~0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) bar[0] = 0u;
}

// the vectors of a launch from rows to positions, out[0 .. 4 n): x, r, p, M^-1;
// and x, r, p back.  (Translated inside cg_tile the index takes registers of
// every iteration: 128^3 FP64 38.7 -> 50.5 us.)
template <typename T>
__global__ void __launch_bounds__(256)
to_positions(int32_t n, const int32_t* __restrict__ order, const T* __restrict__ x, const T* __restrict__ r,
             const T* __restrict__ p, const T* __restrict__ dinv, T* __restrict__ out) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int32_t row = order[i];
    const int64_t m = n;
    out[i] = x[row];
    out[m + i] = r[row];
    out[2 * m + i] = p[row];
    out[3 * m + i] = dinv[row];
}

template <typename T>
__global__ void __launch_bounds__(256)
from_positions(int32_t n, const int32_t* __restrict__ inv, const T* __restrict__ in, T* __restrict__ x,
               T* __restrict__ r, T* __restrict__ p) {
    const int32_t row = blockIdx.x * 256 + threadIdx.x;
    if (row >= n) return;
    const int32_t i = inv[row];
    const int64_t m = n;
    x[row] = in[i];
    r[row] = in[m + i];
    p[row] = in[2 * m + i];
}

// ---- iterations ----------------------------------------------------------------
// NR rows per thread: tiles of at most R = NR TT rows
template <typename T, int NR>
__global__ void __launch_bounds__(TT)
cg_tile(int32_t n, const int32_t* __restrict__ first, const int32_t* __restrict__ halo, const int32_t* __restrict__ n_halo,
        const Places* __restrict__ places, const T* __restrict__ val, const T* __restrict__ dinv, T* __restrict__ x,
        T* __restrict__ r, T* __restrict__ p, CgState<T>* st, int32_t k0, int32_t k_end,
        typename Word<T>::type* slots, typename Word<T>::type* zs, Wait wait) {
#pragma clang fp contract(off)
    typedef typename Word<T>::type W;
    constexpr W EMPTY = Word<T>::EMPTY;
    constexpr int R = NR * TT;
    constexpr int D = sizeof(T) == 8 ? 2 : 3;   // rows whose loads are in flight (more: no gain)
    // rows whose places stay in registers, as many as these allow without
    // spilling; the others' are read every iteration
    constexpr int W32 = sizeof(T) / 4;
    constexpr int FREE = (256 - 4 * W32 * NR - D * U * W32 - (W32 == 2 ? 140 : 112)) / 4;   // the rest measured
    constexpr int KEEP = FREE < NR ? (FREE > 0 ? FREE : 0) : NR;
    __shared__ T P[lds_words<T>()];
    __shared__ T red1[TT / 64], red2[TT / 64];
    __shared__ T all[2][SPMV_BLOCK / 64];
    __shared__ int32_t bad;
    if (st->done != CG_RUNNING) return;
    const int32_t t = threadIdx.x, b = blockIdx.x, G = gridDim.x;
    const int32_t base = first[b], rows = first[b + 1] - base, H = n_halo[b];
    const int32_t k_stop = min(k_end, st->max_iter);
    const T thresh = st->thresh, pause_thresh = st->pause_thresh;
    T rz = st->rz[k0 & 3];
    T xv[NR], rv[NR], zv[NR], dv[NR];   // zv: q between the exchanges, then z
    Places pk[KEEP > 0 ? KEEP : 1];
    int32_t hid[HALO_PER_THREAD];       // byte offsets of the halo's rows, -1: none
    uint32_t remote = 0;                // rows in other tiles' halos, a bit each
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        const int32_t l = j * TT + t;
        xv[j] = rv[j] = zv[j] = dv[j] = T(0);
        if (l < rows) {
            const int32_t i = base + l;
            xv[j] = x[i];
            rv[j] = r[i];
            dv[j] = dinv[i];
            P[l] = p[i];
        } else {
            P[l] = T(0);
        }
        const Places pl = places[b * R + l];
        bool out = false;
#pragma unroll
        for (int u = 0; u < U; ++u) out |= place(pl, u) >= (uint32_t)R;
        remote |= (uint32_t)out << j;
        if (j < KEEP) pk[j < KEEP ? j : 0] = pl;
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int h = 0; h < HALO_PER_THREAD; ++h) {
        const int32_t l = h * TT + t;
        hid[h] = -1;
        if (l < H) {
            const int32_t c = halo[(int64_t)b * HALO_MAX + l];
            P[R + l] = p[c];
            hid[h] = c * (int32_t)sizeof(W);
        }
    }
    if (t == 0) bad = 0;
    __syncthreads();
    int32_t k = k0, stop = CG_RUNNING;
    T pq = T(0), a = T(0), beta = T(0), rr = T(0);
    bool given_up = false;
    const int32_t lane0 = (t >> 6) * U * 64 + (t & 63);
    for (; k < k_stop; ++k) {
        W* const s_pq = slots + (k % RES_SETS) * 3 * SPMV_BLOCK;
        W* const s_rr = s_pq + SPMV_BLOCK;   // (r, z) and (r, r), a pair per tile
        W* const z_k = zs + (int64_t)(k % RES_SETS) * n;
        // q = A p, partial of (p, q)
        T ppq = T(0);
        T v[D][U];
        Places pl[D];
#pragma unroll
        for (int j = 0; j < NR + D - 1; ++j) {
            if (j < NR) {
                const auto vj = hidden(val + ((int64_t)b * (R / 64) + j * (TT / 64)) * U * 64);
#pragma unroll
                for (int u = 0; u < U; ++u) v[j % D][u] = vj[u * 64 + lane0];
                if (j >= KEEP) pl[j % D] = *(const Places*)(hidden(places + b * R + j * TT) + t);
            }
            __builtin_amdgcn_sched_barrier(0);   // D rows ahead and no more
            if (j >= D - 1) {
                const int i = j - (D - 1);
                Places q_pl = i < KEEP ? pk[i < KEEP ? i : 0] : pl[i % D];
                // unpacked here, not once for all iterations (7 registers a row)
                if (i < KEEP)
                    asm volatile("" : "+v"(q_pl.w[0]), "+v"(q_pl.w[1]), "+v"(q_pl.w[2]), "+v"(q_pl.w[3]));
                T q = T(0);
#pragma unroll
                for (int u = 0; u < U; ++u) q += v[i % D][u] * P[place(q_pl, u)];
                zv[i] = q;
                ppq += P[i * TT + t] * q;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        T w1 = wave_sum(ppq);
        if ((t & 63) == 0) red1[t >> 6] = w1;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the slots emptied last time are
        __syncthreads();
        if (t == 0) agent_store(s_pq + b, Word<T>::of(tile_sum(red1)));
        if (t < SPMV_BLOCK && !gather_slots<T, 1>(s_pq, G, t, wait, all)) bad = 1;
        __syncthreads();
        if (bad) {
            given_up = true;
            break;
        }
        pq = sum_red(all[0]);
        if (!(pq > T(0)) || !isfinite(pq)) {
            stop = CG_BREAKDOWN;
            break;
        }
        a = rz / pq;
        // r -= alpha q; z = M^-1 r; partials of (r, z), (r, r)
        T prz = T(0), prr = T(0);
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            rv[j] = rv[j] - a * zv[j];
            const T zi = dv[j] * rv[j];
            zv[j] = zi;
            if (remote & (1u << j)) agent_store((W*)(hidden(z_k + (base + j * TT)) + t), Word<T>::of(zi));
            prz += rv[j] * zi;
            prr += rv[j] * rv[j];
            __builtin_amdgcn_sched_barrier(0);
        }
        w1 = wave_sum(prz);
        const T w2 = wave_sum(prr);
        if ((t & 63) == 0) {
            red1[t >> 6] = w1;
            red2[t >> 6] = w2;
        }
        __syncthreads();
        if (t == 0) {
            agent_store(s_rr + 2 * b, Word<T>::of(tile_sum(red1)));
            agent_store(s_rr + 2 * b + 1, Word<T>::of(tile_sum(red2)));
        }
        if (k > k0) {   // every tile is past iteration k - 1
            W* const zo = zs + (int64_t)((k - 1) % RES_SETS) * n + base;
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (remote & (1u << j)) agent_store((W*)(hidden(zo + j * TT) + t), EMPTY);
            if (t == 0) {
                W* const old = slots + ((k - 1) % RES_SETS) * 3 * SPMV_BLOCK;
                agent_store(old + b, EMPTY);
                agent_store(old + SPMV_BLOCK + 2 * b, EMPTY);
                agent_store(old + SPMV_BLOCK + 2 * b + 1, EMPTY);
            }
        }
        W zh[HALO_PER_THREAD];
#pragma unroll
        for (int h = 0; h < HALO_PER_THREAD; ++h)
            zh[h] = hid[h] >= 0 ? agent_load_at(z_k, (uint32_t)hid[h]) : W(0);
        if (t < SPMV_BLOCK && !gather_slots<T, 2>(s_rr, G, t, wait, all)) bad = 1;
        for (uint32_t spins = 0;;) {
            bool empty = false;
#pragma unroll
            for (int h = 0; h < HALO_PER_THREAD; ++h) empty |= zh[h] == EMPTY;
            if (!empty) break;
            if (wait_over(spins, wait)) {
                bad = 1;
                break;
            }
#pragma unroll
            for (int h = 0; h < HALO_PER_THREAD; ++h)
                if (zh[h] == EMPTY) zh[h] = agent_load_at(z_k, (uint32_t)hid[h]);
        }
        __syncthreads();
        if (bad) {
            given_up = true;
            break;
        }
        const T rzn = sum_red(all[0]);
        rr = sum_red(all[1]);
        // x += alpha p; stop tests; beta = rz_{k+1} / rz_k; p = z + beta p
        if (rr <= thresh) stop = CG_CONVERGED;
        else if (!(rzn > T(0)) || !isfinite(rzn)) stop = CG_BREAKDOWN;
        else if (rr <= pause_thresh) stop = CG_PAUSED;
        if (stop == CG_RUNNING) beta = rzn / rz;
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const int32_t l = j * TT + t;
            if (l < rows) {
                const T pi = P[l];
                xv[j] = xv[j] + a * pi;
                if (stop == CG_RUNNING) P[l] = zv[j] + beta * pi;
            }
        }
        if (stop != CG_RUNNING) {
            ++k;   // this iteration counts
            break;
        }
        rz = rzn;
#pragma unroll
        for (int h = 0; h < HALO_PER_THREAD; ++h)
            if (hid[h] >= 0) {
                const int32_t l = R + h * TT + t;
                P[l] = Word<T>::value(zh[h]) + beta * P[l];
            }
        __syncthreads();
    }
    if (given_up) {
        if (t == 0) atomicOr(wait.bar, 1u);
        return;
    }
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        const int32_t l = j * TT + t;
        if (l < rows) {
            x[base + l] = xv[j];
            r[base + l] = rv[j];
            p[base + l] = P[l];
        }
    }
    if (b == 0 && t == 0) {
        // rz_k of the last iteration that began, for a resumed direction: the
        // stop left rz alone, a finished iteration moved it on
        const int32_t at = stop == CG_RUNNING || (stop == CG_BREAKDOWN && !(pq > T(0) && isfinite(pq))) ? k : k - 1;
        st->rz[at & 3] = rz;
        st->pq = pq;
        st->alpha = a;
        st->beta = beta;
        if (k > k0) st->rr = rr;
        st->iter = k;
        st->kk = -1;
        st->done = stop;
    }
}

// the rows per thread of a tile (CG has kernels from 3 on: smaller systems take
// the resident loop)
constexpr int NRS[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 18, 20, 22, 24, 28, 32};

template <typename T, int... I>
const void* pick_kernel(int nr, std::integer_sequence<int, I...>) {
    const void* f = nullptr;
    ((nr == NRS[I] && NRS[I] >= 3 && NRS[I] <= nr_max<T>()
          ? (void)(f = (const void*)cg_tile<T, std::max(3, std::min(NRS[I], nr_max<T>()))>)
          : (void)0), ...);
    return f;
}
template <typename T>
const void* tile_kernel(int nr) {
    return pick_kernel<T>(nr, std::make_integer_sequence<int, (int)(sizeof(NRS) / sizeof(NRS[0]))>());
}

// Tiles of at most R rows over the plan's rows (or positions), at most `most`
// of them, none across two ranks (by_rank: such a tile's halo is that of two)
// or simply one after the other; empty if R is too small.
std::vector<int32_t> cut(const rp_plan* p, int64_t R, int most, bool by_rank) {
    std::vector<int32_t> first;
    auto run = [&](int64_t r0, int64_t rows) {   // even pieces of whole slices
        const int64_t t = (rows + R - 1) / R;
        const int64_t len = t > 0 ? ((rows + t - 1) / t + 63) / 64 * 64 : 0;
        for (int64_t a = 0; a < rows; a += len) first.push_back((int32_t)(r0 + a));
    };
    if (by_rank)
        for (int32_t s = 0; s < p->alpha; ++s) run(p->row0[s], p->n_cells[s]);
    else
        run(0, p->n_rows);
    if ((int)first.size() > most) return {};
    first.push_back((int32_t)p->n_rows);
    return first;
}

int tile_free(rp_plan* p) {
    auto& tl = p->tiles;
    for (void** q : {(void**)&tl.first, (void**)&tl.halo, (void**)&tl.n_halo, &tl.places}) {
        if (*q) RP_HIP_TRY(hipFree(*q));
        *q = nullptr;
    }
    tl.R = tl.G = tl.halo_most = 0;
    return RP_OK;
}

int order_free(rp_plan* p) {
    auto& tl = p->tiles;
    for (void** q : {(void**)&tl.order, (void**)&tl.inv, &tl.vec}) {
        if (*q) RP_HIP_TRY(hipFree(*q));
        *q = nullptr;
    }
    return RP_OK;
}

// the structure for one cut; *fits = false if a tile's halo is too long, or
// there is no memory for it (*memory = false)
int tile_try(rp_plan* p, int nr, const std::vector<int32_t>& first, hipStream_t s, bool* fits,
             bool* memory) {
    auto& tl = p->tiles;
    const int32_t G = (int32_t)first.size() - 1, R = nr * TT;
    RP_TRY(tile_free(p));
    *fits = false;
    if (!got(p, &tl.first, sizeof(int32_t) * first.size()) || !got(p, &tl.halo, sizeof(int32_t) * (size_t)G * HALO_MAX) ||
        !got(p, &tl.n_halo, sizeof(int32_t) * (size_t)G) || !got(p, &tl.places, sizeof(Places) * (size_t)G * R)) {
        *memory = false;
        return RP_OK;
    }
    RP_HIP_TRY(hipMemcpyAsync(tl.first, first.data(), sizeof(int32_t) * first.size(), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(tile_build, dim3(G), dim3(1024), 0, s, R, tl.first, tl.order, tl.inv, p->d_row_ptr, p->d_col,
                       tl.halo, tl.n_halo, (Places*)tl.places);
    RP_HIP_TRY(hipGetLastError());
    loop_host(p);
    std::vector<int32_t> h(G);
    RP_HIP_TRY(hipMemcpyAsync(h.data(), tl.n_halo, sizeof(int32_t) * (size_t)G, hipMemcpyDeviceToHost, s));
    RP_HIP_TRY(hipStreamSynchronize(s));
    const auto mm = std::minmax_element(h.begin(), h.end());
    *fits = *mm.first >= 0;
    if (*fits) {
        tl.R = R;
        tl.G = G;
        tl.halo_most = *mm.second;
    }
    return RP_OK;
}

int tile_find(rp_plan* p, hipStream_t s) {
    auto& tl = p->tiles;
    const int most = std::min(p->n_cus, SPMV_BLOCK);   // a thread per tile's sums
    // by rank where that costs at most a quarter more rows per thread, and no
    // solver the loop that the cut in one run has room for (128^3 rows in 3 x 3 x 3
    // ranks: 18 rows per thread against 16); else, or where a halo is too long,
    // the other one
    int nr[2] = {0, 0};
    loop_host(p);
    std::vector<int32_t> first[2];
    if (p->max_row <= U)
        for (int k = 0; k < 2; ++k)
            for (int v : NRS) {
                first[k] = cut(p, (int64_t)v * TT, most, k == 0);
                if (!first[k].empty()) {
                    nr[k] = v;
                    break;
                }
            }
    bool fits = false, memory = true;
    const bool by_rank = nr[0] > 0 && 4 * nr[0] <= 5 * nr[1];
    bool dear = false;
    for (int most_nr : {BI_NR_MAX, nr_max<double>(), nr_max<float>()}) dear |= nr[1] <= most_nr && most_nr < nr[0];
    if (by_rank && !dear) RP_TRY(tile_try(p, nr[0], first[0], s, &fits, &memory));
    if (!fits && nr[1] > 0) {
        RP_TRY(tile_try(p, nr[1], first[1], s, &fits, &memory));
        if (!fits && by_rank && dear) RP_TRY(tile_try(p, nr[0], first[0], s, &fits, &memory));
        if (!fits && memory) {
            bool ok = false;
            memory = got(p, &tl.order, sizeof(int32_t) * (size_t)p->n_rows) &&
                     got(p, &tl.inv, sizeof(int32_t) * (size_t)p->n_rows) &&
                     got(p, &tl.vec, TILE_VECS * sizeof(double) * (size_t)p->n_rows);
            if (memory) RP_TRY(tile_order(p, first[1][1], tl.order, tl.inv, s, &ok, &memory));
            if (ok) RP_TRY(tile_try(p, nr[1], first[1], s, &fits, &memory));
            if (!fits) RP_TRY(order_free(p));
        }
    }
    return fits ? RP_OK : tile_free(p);
}

}  // namespace

// the plan's tiles, or that it does not fit or has no memory for them
// (tiles.R = 0), found out once
int tile_setup(rp_plan* p, hipStream_t s) {
    if (p->tiles.asked) return RP_OK;
    try {
        RP_TRY(tile_find(p, s));
    } catch (const std::bad_alloc&) {   // no host memory: as without device memory
        RP_HIP_TRY(hipStreamSynchronize(s));
        RP_TRY(tile_free(p));
        RP_TRY(order_free(p));
    }
    // for good, also where memory was short: the values' slices are laid out by
    // these tables, and a search repeated by every solve costs more than it gives
    p->tiles.asked = true;
    return RP_OK;
}

namespace {

template <typename T>
struct TileVal;
template <>
struct TileVal<double> {
    static double*& val(rp_plan* p) { return p->tiles.val64; }
    static int64_t& version(rp_plan* p) { return p->tiles.version64; }
};
template <>
struct TileVal<float> {
    static float*& val(rp_plan* p) { return p->tiles.val32; }
    static int64_t& version(rp_plan* p) { return p->tiles.version32; }
};

}  // namespace

template <typename T>
bool tile_room(rp_plan* p) {
    return got(p, &TileVal<T>::val(p), sizeof(T) * (size_t)p->tiles.G * p->tiles.R * U);
}

// the slices of the values src: the matrix's, or (transposed) its transpose's
template <typename T>
int tile_slices(rp_plan* p, const T* src, bool transposed, hipStream_t s, const T** val) {
    auto& tl = p->tiles;
    *val = TileVal<T>::val(p);
    const int64_t version = 2 * p->values_version + transposed;
    if (TileVal<T>::version(p) == version) return RP_OK;
    hipLaunchKernelGGL(tile_values<T>, dim3(tl.R / 256, tl.G), dim3(256), 0, s, tl.R, tl.first, tl.order, p->d_row_ptr,
                       src, TileVal<T>::val(p));
    RP_HIP_TRY(hipGetLastError());
    TileVal<T>::version(p) = version;
    return RP_OK;
}

template bool tile_room<double>(rp_plan*);
template int tile_slices<double>(rp_plan*, const double*, bool, hipStream_t, const double**);

// whether the plan fits the tiled loop in this precision
template <typename T>
int tile_fits(rp_plan* p, hipStream_t s, bool* yes) {
    *yes = false;
    if (p->n_rows > (int64_t)SPMV_BLOCK * nr_max<T>() * TT) return RP_OK;
    RP_TRY(tile_setup(p, s));
    auto& tl = p->tiles;
    const int nr = tl.R / TT;
    if (tl.R == 0 || nr > nr_max<T>() || tl.R + tl.halo_most > lds_words<T>()) return RP_OK;
    int per_cu = 0;
    RP_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, tile_kernel<T>(nr), TT, 0));
    *yes = per_cu > 0 && tile_room<T>(p) &&
           got(p, &tl.slots, sizeof(uint64_t) * RES_SETS * (3 * SPMV_BLOCK + (size_t)p->n_rows)) &&
           got(p, &tl.bar, sizeof(uint32_t));
    return RP_OK;
}

// The iterations k0 .. min(k_end, budget) by the tiled loop, enqueued, on a
// plan that fits it.  See launch_loop.
template <typename T>
int launch_cg_tile(rp_plan* p, const T* src, const T* dinv, T* x, T* r, T* pv, CgState<T>* st, int32_t k0,
                   int32_t k_end, hipStream_t s) {
    auto& tl = p->tiles;
    int32_t n = (int32_t)p->n_rows;
    const T* val = nullptr;
    RP_TRY(tile_slices<T>(p, src, false, s, &val));
    typedef typename Word<T>::type W;
    const int64_t len = (int64_t)RES_SETS * (3 * SPMV_BLOCK + (int64_t)n);
    W* slots = (W*)tl.slots;
    W* zs = slots + RES_SETS * 3 * SPMV_BLOCK;
    uint32_t* bar = tl.bar;
    hipLaunchKernelGGL(clear_words, dim3(1024), dim3(256), 0, s, (uint32_t*)slots, len * (int64_t)(sizeof(W) / 4), bar);
    RP_HIP_TRY(hipGetLastError());
    const int32_t *first = tl.first, *halo = tl.halo, *n_halo = tl.n_halo;
    const Places* places = (const Places*)tl.places;
    T *tx = x, *tr = r, *tp = pv;
    const T* td = dinv;
    if (tl.order) {   // the vectors at the tiles' positions
        tx = (T*)tl.vec;
        tr = tx + n;
        tp = tr + n;
        td = tp + n;
        hipLaunchKernelGGL(to_positions<T>, dim3((n + 255) / 256), dim3(256), 0, s, n, tl.order, x, r, pv, dinv, tx);
        RP_HIP_TRY(hipGetLastError());
    }
    Wait wait{bar, wait_spins(p)};
    void* args[] = {&n, (void*)&first, (void*)&halo, (void*)&n_halo, (void*)&places, (void*)&val, (void*)&td, &tx, &tr,
                    &tp, &st, &k0, &k_end, &slots, &zs, &wait};
    RP_TRY(launch_loop(p, tile_kernel<T>(tl.R / TT), tl.G, TT, args, bar, s));
    if (tl.order) {
        hipLaunchKernelGGL(from_positions<T>, dim3((n + 255) / 256), dim3(256), 0, s, n, tl.inv, tx, x, r, pv);
        RP_HIP_TRY(hipGetLastError());
    }
    return RP_OK;
}

template int tile_fits<double>(rp_plan*, hipStream_t, bool*);
template int tile_fits<float>(rp_plan*, hipStream_t, bool*);
template int launch_cg_tile<double>(rp_plan*, const double*, const double*, double*, double*, double*,
                                    CgState<double>*, int32_t, int32_t, hipStream_t);
template int launch_cg_tile<float>(rp_plan*, const float*, const float*, float*, float*, float*, CgState<float>*,
                                   int32_t, int32_t, hipStream_t);

}  // namespace rp
