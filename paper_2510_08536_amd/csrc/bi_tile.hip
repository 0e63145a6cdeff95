// BiCGStab iterations in one launch: one workgroup per compute
// unit, each owning a tile of rows, as in the tiled CG loop (cg_tile.hip).
//
// Launched apart an iteration is five kernels that move 20 n words besides the
// matrix, twice.  Here r, r^, p, v, t and M^-1 of a thread's rows (and x, while
// the registers hold it) stay in registers and the product's operand, y and
// then z, in LDS; an iteration reads the values twice, from the memory-side
// cache where they fit it.  What tiles exchange goes by value (exchange.hpp):
//   p, y; v = A y, (r^, v);   alpha, s, z; t = A z, (s, s), (t, s), (t, t);
//   omega, x, r, (r^, r), (r, r);   stop tests, beta
// Of its halo a tile needs y and z.  With short halos (HK entries per thread)
// v goes with the first sums and t with the second, and a tile keeps r, p, v
// and M^-1 of its halo in registers and updates them as the owners do: three
// exchanges.  With longer ones y and z themselves are exchanged, five in all:
// keeping the halo's vectors in memory moved as much as the matrix (96^3: 50
// against 42 us).  The half-step test on (s, s) is made after t, whose product
// is then for nothing once a solve.
//
// Products and vector updates are the launched kernels' bit for bit; the dot
// products add a tile's rows first.
//
// Per iteration against the launched kernels, a solve's start and end included:
// 25 -> 9.5 us at 16^3 rows, 28 -> 11 at 32^3, 39 -> 17.5 at 64^3, 53 -> 24 at
// 80^3, 74 -> 42 at 96^3, 104 -> 58 at 110 x 108 x 100.
#include <algorithm>
#include <utility>

#include "tile.hpp"

namespace rp {

namespace {

constexpr int BI_SUMS = 6;          // slots of a tile per set: (r^, v); (s, s), (t, s), (t, t); (r^, r), (r, r)
constexpr int BI_NR[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10};
constexpr int BI_HK = 6, BI_HK_NR = 4;     // halo entries per thread kept in registers, rows per thread they have room beside

__global__ void __launch_bounds__(256) bi_clear(uint64_t* w, int64_t words, uint32_t* bar) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (int64_t)gridDim.x * 256) w[i] = ~0ull;
    if (blockIdx.x == 0 && threadIdx.x == 0) bar[0] = 0u;
}

// the vectors of a launch from rows to positions: x, r, p, v, r^, M^-1; and
// the first four back
__global__ void __launch_bounds__(256)
bi_to_positions(int32_t n, const int32_t* __restrict__ order, const double* __restrict__ x,
                const double* __restrict__ r, const double* __restrict__ p, const double* __restrict__ v,
                const double* __restrict__ rh, const double* __restrict__ dinv, double* __restrict__ out) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int32_t row = order[i];
    const int64_t m = n;
    out[i] = x[row];
    out[m + i] = r[row];
    out[2 * m + i] = p[row];
    out[3 * m + i] = v[row];
    out[4 * m + i] = rh[row];
    out[5 * m + i] = dinv[row];
}

__global__ void __launch_bounds__(256)
bi_from_positions(int32_t n, const int32_t* __restrict__ inv, const double* __restrict__ in, double* __restrict__ x,
                  double* __restrict__ r, double* __restrict__ p, double* __restrict__ v) {
    const int32_t row = blockIdx.x * 256 + threadIdx.x;
    if (row >= n) return;
    const int32_t i = inv[row];
    const int64_t m = n;
    x[row] = in[i];
    r[row] = in[m + i];
    p[row] = in[2 * m + i];
    v[row] = in[3 * m + i];
}

// row sums of the tile's NR rows per thread with the operand in P; done(i, q)
// takes the sum of row i.  D rows' loads are in flight.
template <int NR, int KEEP, typename F>
__device__ __forceinline__ void tile_product(const double* val, const Places* places, int32_t b, int32_t t,
                                             const double* P, const Places* pk, F done) {
#pragma clang fp contract(off)
    constexpr int R = NR * TT, D = 2;
    const int32_t lane0 = (t >> 6) * U * 64 + (t & 63);
    double v[D][U];
    Places pl[D];
#pragma unroll
    for (int j = 0; j < NR + D - 1; ++j) {
        if (j < NR) {
            const auto vj = hidden(val + ((int64_t)b * (R / 64) + j * (TT / 64)) * U * 64);
#pragma unroll
            for (int u = 0; u < U; ++u) v[j % D][u] = vj[u * 64 + lane0];
            if (j >= KEEP) pl[j % D] = *(const Places*)(hidden(places + b * R + j * TT) + t);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (j >= D - 1) {
            const int i = j - (D - 1);
            Places q_pl = i < KEEP ? pk[i < KEEP ? i : 0] : pl[i % D];
            if (i < KEEP) asm volatile("" : "+v"(q_pl.w[0]), "+v"(q_pl.w[1]), "+v"(q_pl.w[2]), "+v"(q_pl.w[3]));
            double q = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) q += v[i % D][u] * P[place(q_pl, u)];
            done(i, q);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// the values of N halo rows (byte offsets hid, -1: none), loaded until none is
// empty; false: given up
template <int N>
__device__ __forceinline__ void halo_load(const uint64_t* at, const int32_t* hid, uint64_t* w) {
#pragma unroll
    for (int h = 0; h < N; ++h) w[h] = hid[h] >= 0 ? agent_load_at(at, (uint32_t)hid[h]) : 0;
}
template <int N>
__device__ __forceinline__ bool halo_wait(const uint64_t* at, const int32_t* hid, uint64_t* w, const Wait& wait) {
    for (uint32_t spins = 0;;) {
        bool empty = false;
#pragma unroll
        for (int h = 0; h < N; ++h) empty |= w[h] == Word<double>::EMPTY;
        if (!empty) return true;
        if (wait_over(spins, wait)) return false;
#pragma unroll
        for (int h = 0; h < N; ++h)
            if (w[h] == Word<double>::EMPTY) w[h] = agent_load_at(at, (uint32_t)hid[h]);
    }
}

template <int NR, int HK>
__global__ void __launch_bounds__(TT)
bi_tile(int32_t n, const int32_t* __restrict__ first, const int32_t* __restrict__ halo,
        const int32_t* __restrict__ n_halo, const Places* __restrict__ places, const double* __restrict__ val,
        const double* __restrict__ dinv, double* __restrict__ x, double* __restrict__ r,
        const double* __restrict__ rh, double* __restrict__ p, double* __restrict__ v, BiState* st, int32_t k0,
        int32_t k_end, uint64_t* slots, uint64_t* vs, uint64_t* ts, Wait wait) {
#pragma clang fp contract(off)
    typedef Word<double> W;
    constexpr int R = NR * TT;
    constexpr bool DIRECT = HK == 0;
    constexpr bool XM = NR > 6;     // x stays in memory: read and written once an iteration
    constexpr int FREE = (256 - (XM ? 12 : 14) * NR - 28 - (DIRECT ? 116 : 100 + 10 * HK)) / 4;
    constexpr int HN = DIRECT ? HALO_PER_THREAD : HK;
    constexpr int KEEP = FREE < NR ? (FREE > 0 ? FREE : 0) : NR;
    __shared__ double P[lds_words<double>()];
    __shared__ double red[3][TT / 64];
    __shared__ double all[3][SPMV_BLOCK / 64];
    // a wait was given up; one word for every other check, so that none is set
    // again before every wave has read it
    __shared__ int32_t bad[2];
    if (st->done != CG_RUNNING) return;
    const int32_t t = threadIdx.x, b = blockIdx.x, G = gridDim.x;
    const int32_t base = first[b], rows = first[b + 1] - base, H = n_halo[b];
    const double thresh = st->thresh;
    double rho = st->rho[k0 & 3], rho_old = st->rho[(k0 + 3) & 3], alpha = st->alpha, omega = st->omega, rr = st->rr;
    double xv[XM ? 1 : NR], rv[NR], rhv[NR], pv[NR], vv[NR], tv[NR], dv[NR];
    Places pk[KEEP > 0 ? KEEP : 1];
    uint32_t remote = 0;            // rows in other tiles' halos, a bit each
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        const int32_t l = j * TT + t;
        rv[j] = rhv[j] = pv[j] = vv[j] = tv[j] = dv[j] = 0.0;
        if (!XM) xv[XM ? 0 : j] = 0.0;
        if (l < rows) {
            if (!XM) xv[XM ? 0 : j] = x[base + l];
            rv[j] = r[base + l];
            rhv[j] = rh[base + l];
            pv[j] = p[base + l];
            vv[j] = v[base + l];
            dv[j] = dinv[base + l];
        }
        const Places pl = places[b * R + l];
        bool out = false;
#pragma unroll
        for (int u = 0; u < U; ++u) out |= place(pl, u) >= (uint32_t)R;
        remote |= (uint32_t)out << j;
        if (j < KEEP) pk[j < KEEP ? j : 0] = pl;
        __builtin_amdgcn_sched_barrier(0);
    }
    int32_t hid[HN];
    double hr[DIRECT ? 1 : HN], hp[DIRECT ? 1 : HN], hv[DIRECT ? 1 : HN], hd[DIRECT ? 1 : HN];
#pragma unroll
    for (int h = 0; h < HN; ++h) {
        const int32_t l = h * TT + t;
        hid[h] = -1;
        if (!DIRECT) hr[DIRECT ? 0 : h] = hp[DIRECT ? 0 : h] = hv[DIRECT ? 0 : h] = hd[DIRECT ? 0 : h] = 0.0;
        if (l < H) {
            const int32_t c = halo[(int64_t)b * HALO_MAX + l];
            hid[h] = c * (int32_t)sizeof(uint64_t);
            if (!DIRECT) {
                hr[DIRECT ? 0 : h] = r[c];
                hp[DIRECT ? 0 : h] = p[c];
                hv[DIRECT ? 0 : h] = v[c];
                hd[DIRECT ? 0 : h] = dinv[c];
            }
        }
    }
    if (t < 2) bad[t] = 0;
    __syncthreads();
    const int32_t k_stop = k_end;
    int32_t k = k0, stop = CG_RUNNING;
    bool half = false, given_up = false;
    for (; k < k_stop; ++k) {
        if (rr <= thresh) stop = CG_CONVERGED;
        else if (rho == 0.0 || !isfinite(rho) || omega == 0.0) stop = CG_BREAKDOWN;
        if (stop != CG_RUNNING) break;
        uint64_t* const s_v = slots + (int64_t)(k % RES_SETS) * BI_SUMS * SPMV_BLOCK;
        uint64_t* const s_t = s_v + SPMV_BLOCK;
        uint64_t* const s_r = s_t + 3 * SPMV_BLOCK;
        uint64_t* const v_k = vs + (int64_t)(k % RES_SETS) * n;
        uint64_t* const t_k = ts + (int64_t)(k % RES_SETS) * n;
        // p = r + beta (p - omega v); y = M^-1 p
        const double beta = (rho / rho_old) * (alpha / omega);
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            pv[j] = rv[j] + beta * (pv[j] - omega * vv[j]);
            const double y = dv[j] * pv[j];
            P[j * TT + t] = y;
            if (DIRECT && (remote & (1u << j))) agent_store((uint64_t*)(hidden(v_k + (base + j * TT)) + t), W::of(y));
        }
        uint64_t w[HN];
        if (DIRECT) {
            halo_load<HN>(v_k, hid, w);
            if (!halo_wait<HN>(v_k, hid, w, wait)) bad[0] = 1;
        }
#pragma unroll
        for (int h = 0; h < HN; ++h) {
            if (DIRECT) {
                if (hid[h] >= 0) P[R + h * TT + t] = W::value(w[h]);
            } else {
                double &hph = hp[DIRECT ? 0 : h];
                hph = hr[DIRECT ? 0 : h] + beta * (hph - omega * hv[DIRECT ? 0 : h]);
                if (hid[h] >= 0) P[R + h * TT + t] = hd[DIRECT ? 0 : h] * hph;
            }
        }
        __syncthreads();
        // v = A y, (r^, v)
        double s1 = 0.0;
        tile_product<NR, KEEP>(val, places, b, t, P, pk, [&](int i, double q) {
            vv[i] = q;
            if (!DIRECT && (remote & (1u << i))) agent_store((uint64_t*)(hidden(v_k + (base + i * TT)) + t), W::of(q));
            s1 += rhv[i] * q;
        });
        s1 = wave_sum(s1);
        if ((t & 63) == 0) red[0][t >> 6] = s1;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the slots emptied last time are
        __syncthreads();
        if (t == 0) agent_store(s_v + b, W::of(tile_sum(red[0])));
        if (!DIRECT) halo_load<HN>(v_k, hid, w);
        if (t < SPMV_BLOCK && !gather_slots<double, 1>(s_v, G, t, wait, all)) bad[0] = 1;
        __syncthreads();
        if (bad[0]) {
            given_up = true;
            break;
        }
        if (k > k0) {   // every tile is past iteration k - 1
            const int64_t o = (k - 1) % RES_SETS;
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (remote & (1u << j)) {
                    agent_store((uint64_t*)(hidden(vs + o * n + (base + j * TT)) + t), W::EMPTY);
                    agent_store((uint64_t*)(hidden(ts + o * n + (base + j * TT)) + t), W::EMPTY);
                }
            uint64_t* const old = slots + o * BI_SUMS * SPMV_BLOCK;
            if (t < 1) agent_store(old + b, W::EMPTY);
            if (t < 3) agent_store(old + SPMV_BLOCK + 3 * b + t, W::EMPTY);
            if (t < 2) agent_store(old + 4 * SPMV_BLOCK + 2 * b + t, W::EMPTY);
        }
        const double sv = sum_red(all[0]);
        if (sv == 0.0 || !isfinite(sv)) {
            stop = CG_BREAKDOWN;
            break;
        }
        alpha = rho / sv;
        // s = r - alpha v (in r's registers); z = M^-1 s
        double s2 = 0.0, s3 = 0.0;
        s1 = 0.0;
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            rv[j] = rv[j] - alpha * vv[j];
            const double z = dv[j] * rv[j];
            P[j * TT + t] = z;
            if (DIRECT && (remote & (1u << j))) agent_store((uint64_t*)(hidden(t_k + (base + j * TT)) + t), W::of(z));
            s1 += rv[j] * rv[j];
        }
        if (DIRECT) halo_load<HN>(t_k, hid, w);
        if (!halo_wait<HN>(DIRECT ? t_k : v_k, hid, w, wait)) bad[1] = 1;
#pragma unroll
        for (int h = 0; h < HN; ++h) {
            if (DIRECT) {
                if (hid[h] >= 0) P[R + h * TT + t] = W::value(w[h]);
            } else {
                hv[DIRECT ? 0 : h] = W::value(w[h]);
                hr[DIRECT ? 0 : h] = hr[DIRECT ? 0 : h] - alpha * hv[DIRECT ? 0 : h];
                if (hid[h] >= 0) P[R + h * TT + t] = hd[DIRECT ? 0 : h] * hr[DIRECT ? 0 : h];
            }
        }
        __syncthreads();
        if (bad[1]) {
            given_up = true;
            break;
        }
        // t = A z, (s, s), (t, s), (t, t)
        tile_product<NR, KEEP>(val, places, b, t, P, pk, [&](int i, double q) {
            tv[i] = q;
            if (!DIRECT && (remote & (1u << i))) agent_store((uint64_t*)(hidden(t_k + (base + i * TT)) + t), W::of(q));
            s2 += q * rv[i];
            s3 += q * q;
        });
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        s3 = wave_sum(s3);
        if ((t & 63) == 0) {
            red[0][t >> 6] = s1;
            red[1][t >> 6] = s2;
            red[2][t >> 6] = s3;
        }
        __syncthreads();
        if (t < 3) agent_store(s_t + 3 * b + t, W::of(tile_sum(red[t])));
        if (!DIRECT) halo_load<HN>(t_k, hid, w);
        if (t < SPMV_BLOCK && !gather_slots<double, 3>(s_t, G, t, wait, all)) bad[0] = 1;
        __syncthreads();
        if (bad[0]) {
            given_up = true;
            break;
        }
        const double ss = sum_red(all[0]), st_ = sum_red(all[1]), tt = sum_red(all[2]);
        if (ss <= thresh) {
            rr = ss;
            half = true;
            break;
        }
        if (tt == 0.0 || !isfinite(tt)) {
            stop = CG_BREAKDOWN;
            ++k;
            break;
        }
        omega = st_ / tt;
        // x = (x + alpha y) + omega z; r = s - omega t; (r^, r), (r, r)
        s1 = s2 = 0.0;
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const int32_t l = j * TT + t;
            const double y = dv[j] * pv[j], z = dv[j] * rv[j];
            if (!XM) xv[XM ? 0 : j] = (xv[XM ? 0 : j] + alpha * y) + omega * z;
            else if (l < rows) x[base + l] = (x[base + l] + alpha * y) + omega * z;
            rv[j] = rv[j] - omega * tv[j];
            s1 += rhv[j] * rv[j];
            s2 += rv[j] * rv[j];
        }
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        if ((t & 63) == 0) {
            red[0][t >> 6] = s1;
            red[1][t >> 6] = s2;
        }
        __syncthreads();
        if (t < 2) agent_store(s_r + 2 * b + t, W::of(tile_sum(red[t])));
        if (!DIRECT) {
            if (!halo_wait<HN>(t_k, hid, w, wait)) bad[1] = 1;
#pragma unroll
            for (int h = 0; h < HN; ++h)
                hr[DIRECT ? 0 : h] = hr[DIRECT ? 0 : h] - omega * W::value(w[h]);
        }
        if (t < SPMV_BLOCK && !gather_slots<double, 2>(s_r, G, t, wait, all)) bad[1] = 1;
        __syncthreads();
        if (bad[1]) {
            given_up = true;
            break;
        }
        rho_old = rho;
        rho = sum_red(all[0]);
        rr = sum_red(all[1]);
    }
    if (given_up) {
        if (t == 0) atomicOr(wait.bar, 1u);
        return;
    }
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        const int32_t l = j * TT + t;
        if (l < rows) {
            if (half) {   // x += alpha y only
                const double y = dv[j] * pv[j];
                x[base + l] = (XM ? x[base + l] : xv[XM ? 0 : j]) + alpha * y;
            } else if (!XM) {
                x[base + l] = xv[XM ? 0 : j];
            }
            r[base + l] = rv[j];
            p[base + l] = pv[j];
            v[base + l] = vv[j];
        }
    }
    if (b == 0 && t == 0) {
        st->rho[(k + 3) & 3] = rho_old;
        st->rho[k & 3] = rho;
        st->alpha = alpha;
        st->omega = omega;
        st->rr = rr;
        st->half_k = k;
        st->iter = half ? k + 1 : k;
        st->done = half ? (int32_t)BI_HALF : stop;
    }
}

template <int... I>
const void* bi_kernel(int nr, int32_t halo_most, std::integer_sequence<int, I...>) {
    const void* f = nullptr;
    ((nr == BI_NR[I] ? (void)(f = halo_most <= BI_HK * TT && BI_NR[I] <= BI_HK_NR
                                      ? (const void*)bi_tile<std::min(BI_NR[I], BI_HK_NR), BI_HK>
                                      : (const void*)bi_tile<BI_NR[I], 0>)
                     : (void)0), ...);
    return f;
}
const void* bi_kernel(int nr, int32_t halo_most) {
    return bi_kernel(nr, halo_most, std::make_integer_sequence<int, (int)(sizeof(BI_NR) / sizeof(BI_NR[0]))>());
}

}  // namespace

// whether the plan fits the loop
int bi_tile_fits(rp_plan* p, hipStream_t s, bool* yes) {
    *yes = false;
    if (p->n_rows > (int64_t)SPMV_BLOCK * BI_NR_MAX * TT) return RP_OK;
    RP_TRY(tile_setup(p, s));
    auto& tl = p->tiles;
    const int nr = tl.R / TT;
    if (tl.R == 0 || nr > BI_NR_MAX || tl.R + tl.halo_most > lds_words<double>()) return RP_OK;
    int per_cu = 0;
    RP_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, bi_kernel(nr, tl.halo_most), TT, 0));
    *yes = per_cu > 0 && tile_room<double>(p) &&
           got(p, &tl.bi_slots, sizeof(uint64_t) * RES_SETS * (BI_SUMS * SPMV_BLOCK + 2 * (size_t)p->n_rows)) &&
           got(p, &tl.bar, sizeof(uint32_t));
    return RP_OK;
}

// The iterations k0 .. k_end, enqueued, on a plan that fits.  See
// launch_loop.
int launch_bi_tile(rp_plan* p, const double* src, bool transposed, const double* dinv, double* x, double* r,
                   const double* rh, double* pv, double* v, BiState* st, int32_t k0, int32_t k_end, hipStream_t s) {
    auto& tl = p->tiles;
    int32_t n = (int32_t)p->n_rows;
    const double* val = nullptr;
    RP_TRY(tile_slices<double>(p, src, transposed, s, &val));
    uint64_t* slots = tl.bi_slots;
    uint64_t* vs = slots + (int64_t)RES_SETS * BI_SUMS * SPMV_BLOCK;
    uint64_t* ts = vs + (int64_t)RES_SETS * n;
    uint32_t* bar = tl.bar;
    const int64_t len = (int64_t)RES_SETS * (BI_SUMS * SPMV_BLOCK + 2 * (int64_t)n);
    hipLaunchKernelGGL(bi_clear, dim3(1024), dim3(256), 0, s, slots, len, bar);
    RP_HIP_TRY(hipGetLastError());
    double *tx = x, *tr = r, *tp = pv, *tv = v;
    const double *trh = rh, *td = dinv;
    if (tl.order) {
        tx = (double*)tl.vec;
        tr = tx + n;
        tp = tr + n;
        tv = tp + n;
        trh = tv + n;
        td = trh + n;
        hipLaunchKernelGGL(bi_to_positions, dim3((n + 255) / 256), dim3(256), 0, s, n, tl.order, x, r, pv, v, rh, dinv,
                           tx);
        RP_HIP_TRY(hipGetLastError());
    }
    const int32_t *first = tl.first, *halo = tl.halo, *n_halo = tl.n_halo;
    const Places* places = (const Places*)tl.places;
    Wait wait{bar, wait_spins(p)};
    void* args[] = {&n,   (void*)&first, (void*)&halo, (void*)&n_halo, (void*)&places, (void*)&val, (void*)&td,
                    &tx,  &tr,           (void*)&trh,  &tp,            &tv,            &st,         &k0,
                    &k_end, &slots,      &vs,          &ts,            &wait};
    RP_TRY(launch_loop(p, bi_kernel(tl.R / TT, tl.halo_most), tl.G, TT, args, bar, s));
    if (tl.order) {
        hipLaunchKernelGGL(bi_from_positions, dim3((n + 255) / 256), dim3(256), 0, s, n, tl.inv, tx, x, r, pv, v);
        RP_HIP_TRY(hipGetLastError());
    }
    return RP_OK;
}

}  // namespace rp
