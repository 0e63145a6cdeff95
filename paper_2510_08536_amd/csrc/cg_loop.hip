// CG iterations in one launch (rp_solve_opts.fused_loop), in two forms: cg_loop
// (RP_LOOP_COOPERATIVE), for systems of any size, and cg_resident (RP_LOOP_AUTO
// on small systems), described further down; and what the one-launch loops
// share on the host (launch_loop).
//
// On small systems an iteration is bound by the gaps between its three
// dependent kernels, not by memory.  Here one launch, with every block
// resident at once (cooperative launch), runs the iterations itself: the
// three phases of an iteration (q = A p with (p, q); r -= alpha q with
// (r, M^-1 r) and (r, r); x and p updates with the stop tests) are separated
// by grid-wide barriers instead of kernel boundaries.  The arithmetic, the
// per-block partial sums and the device state are those of the three-kernel
// iteration in cg.hip (each phase re-sums the previous phase's partials in
// index order, every block the same scalars); every block takes every stop
// decision from the same sums, so all leave the loop together.
//
// The barrier: each block has a flag word of its own (one 128-byte line per
// block).  Arriving, the block's first thread publishes the block's writes
// (agent-scope release fence) and stores the barrier's sequence number into
// the block's flag; the first wave then polls every block's flag until all
// hold that number and takes an agent-scope acquire fence.  One release and
// one acquire per block and barrier: on this device they write back and
// invalidate the die's L2, so their count, not the polling, sets the cost of
// a barrier, and a grid of few blocks (several row groups per block) keeps it
// low.  The wait is bounded: after BAR_SPINS polls the block sets the abort
// word and leaves, and every block that sees the abort word leaves too; the
// host reports it.  The flags and the abort word are cleared by a kernel
// before each launch.
#include <condition_variable>
#include <mutex>

#include "exchange.hpp"
#include "spmv.hpp"

namespace rp {

namespace {

constexpr int FLAG_STRIDE = 32;            // words: one 128-byte line per block flag
constexpr int FLAG0 = FLAG_STRIDE;         // word 0: abort word; flags from line 1
constexpr int LOOP_GRID_MAX = 128;
constexpr uint32_t BAR_SPINS = 1u << 22;   // polls of a barrier at most: a few seconds

// all blocks of the grid; false when the wait was abandoned.  seq counts
// the barriers of this launch (the same in every block).
__device__ __forceinline__ bool grid_barrier(uint32_t* bar, uint32_t& seq) {
    __shared__ uint32_t ok;
    ++seq;
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __hip_atomic_store(bar + FLAG0 + FLAG_STRIDE * blockIdx.x, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (threadIdx.x < 64) {
        uint32_t good = 1, spins = 0;
        for (;;) {
            int pending = 0;
            for (int b = threadIdx.x; b < (int)gridDim.x; b += 64)
                pending |= load_relaxed(bar + FLAG0 + FLAG_STRIDE * b) < seq;
            if (!__any(pending)) break;
            // the abort word and the count are the same in every lane
            if (load_relaxed(bar) != 0u || ++spins > BAR_SPINS) {
                if (threadIdx.x == 0) atomicOr(bar, 1u);
                good = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (threadIdx.x == 0) ok = good;
    }
    __syncthreads();
    return ok != 0;
}

__global__ void clear_barrier(uint32_t* bar, int32_t words) {
    for (int32_t i = threadIdx.x; i < words; i += blockDim.x) bar[i] = 0u;
}

template <typename T>
__global__ void __launch_bounds__(SPMV_BLOCK)
cg_loop(int32_t n, SpmvIdx ix, const T* __restrict__ val, const T* __restrict__ dinv, T* x, T* r, T* p, T* q,
        T* part, CgState<T>* st, int32_t k0, int32_t k_end, uint32_t* bar) {
    // x, r, p, q and the partials are written by other blocks between
    // barriers: no __restrict__ on them
#pragma clang fp contract(off)
    __shared__ __align__(16) T lds[SPMV_CAP];
    __shared__ T xs[1];
    __shared__ T red[SPMV_BLOCK / 64];
    if (st->done != CG_RUNNING) return;
    const XWin w{{0, 0}};
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    const int32_t G = gridDim.x;
    const int32_t i0 = blockIdx.x * SPMV_BLOCK + threadIdx.x, di = G * SPMV_BLOCK;
    const int32_t k_stop = min(k_end, st->max_iter);
    uint32_t seq = 0;
    for (int32_t k = k0; k < k_stop; ++k) {
        // q = A p, partials of (p, q)
        T ppq = T(0);
        GroupRange gr = block_groups(ix, n);
        for (int32_t g = gr.g0; g < gr.n_groups; g += gr.step) {
            const int32_t r0 = g * SPMV_BLOCK;
            const int32_t nr = min(SPMV_BLOCK, n - r0);
            const GroupRow<T> row = spmv_group_row<T, -1>(ix, val, p, n, g, nr, w, xs, lds, gr);
            if ((int32_t)threadIdx.x < nr) {
                const int32_t i = r0 + threadIdx.x;
                q[i] = row.s;
                ppq += own_x<T, -1>(i, row, xs, p) * row.s;
            }
        }
        const T bpq = block_sum<T, SPMV_BLOCK>(ppq, red);
        if (threadIdx.x == 0) part[PART_A + xcd_block()] = bpq;
        if (!grid_barrier(bar, seq)) return;

        // alpha = rz_k / (p, q); r -= alpha q; partials of (r, M^-1 r), (r, r)
        const T pq = sum_partials_all<T, SPMV_BLOCK>(part + PART_A, G, red);
        if (!(pq > T(0)) || !isfinite(pq)) {
            if (lead) {
                st->pq = pq;
                st->iter = k;
                st->kk = -1;
                st->done = CG_BREAKDOWN;
            }
            return;
        }
        const T a = st->rz[k & 3] / pq;
        T prz = T(0), prr = T(0);
        for (int32_t i = i0; i < n; i += di) {
            const T ri = r[i] - a * q[i];
            r[i] = ri;
            prz += ri * (dinv[i] * ri);
            prr += ri * ri;
        }
        const T b1 = block_sum<T, SPMV_BLOCK>(prz, red);
        const T b2 = block_sum<T, SPMV_BLOCK>(prr, red);
        if (threadIdx.x == 0) {
            part[PART_RZ + blockIdx.x] = b1;
            part[PART_RR + blockIdx.x] = b2;
        }
        if (!grid_barrier(bar, seq)) return;

        // x += alpha p; stop tests; beta = rz_{k+1} / rz_k; p = M^-1 r + beta p
        const T rz = sum_partials_all<T, SPMV_BLOCK>(part + PART_RZ, G, red);
        const T rr = sum_partials_all<T, SPMV_BLOCK>(part + PART_RR, G, red);
        int32_t stop = CG_RUNNING;
        if (rr <= st->thresh) stop = CG_CONVERGED;
        else if (!(rz > T(0)) || !isfinite(rz)) stop = CG_BREAKDOWN;
        else if (rr <= st->pause_thresh) stop = CG_PAUSED;
        if (stop != CG_RUNNING) {
            for (int32_t i = i0; i < n; i += di) x[i] = x[i] + a * p[i];
            if (lead) {
                st->pq = pq;
                st->alpha = a;
                st->rr = rr;
                st->iter = k + 1;
                st->done = stop;
            }
            return;
        }
        const T beta = rz / st->rz[k & 3];
        for (int32_t i = i0; i < n; i += di) {
            const T pi = p[i];
            x[i] = x[i] + a * pi;
            p[i] = dinv[i] * r[i] + beta * pi;
        }
        if (lead) {
            st->rz[(k + 1) & 3] = rz;
            st->pq = pq;
            st->alpha = a;
            st->rr = rr;
            st->beta = beta;
            st->iter = k + 1;
        }
        if (!grid_barrier(bar, seq)) return;
    }
}

// ---------------------------------------------------------------------------
// The resident loop: the default on small systems whose rows hold at most
// RES_COLS entries (launch_cg_resident).
//
// A row belongs to one thread for the whole launch, with its entries, x, r,
// p and M^-1 in registers, and with p of the columns it couples to; every
// thread forms the new p of its columns itself (as the two-launch iteration
// does) from their z = M^-1 r.  So an iteration exchanges z and the three
// sums, and needs two exchanges where the loop above needs three barriers:
//   (p, q) partials;   alpha, r, z;   z and the (r, z), (r, r) partials;
//   stop tests, x, beta, p.
// An exchange is no barrier and has no fences.  What is exchanged is stored
// and loaded by agent-scope relaxed atomics, which pass the die's L2 by, so
// nothing is written back or invalidated; and every value is its own flag:
// its slot holds EMPTY (a NaN no value is stored as) until it is stored, and
// a reader loads until it is not.  So z needs no order with the partials, and
// a reader waits once for both.  z of columns in the block's own rows goes
// through LDS; a row is published only if it couples to another block's rows
// (the pattern is structurally symmetric, so only those have readers there).
// The slots rotate through RES_SETS sets; a thread empties its own slots of
// set k - 1 once its block has seen every (p, q) partial of iteration k (all
// blocks are then past iteration k - 1), and waits for those stores before
// the block's next (p, q) partial is published, so nobody can meet set k - 1
// again with old values in it.
//
// The partials are those of the launched kernels on systems of this size: one
// per group of SPMV_BLOCK consecutive rows for all three sums (vec_grid gives
// K2 one element per thread), summed in the same order, so every iterate is
// the three-launch form's bit for bit.  Waits are bounded (exchange.hpp).
//
// Bound by the two exchanges: a store and the load that meets it cross the
// die boundaries, about 1.5 us each way with the reductions.  Per iteration
// against two launches: FP64 6.6 / 12.8 us at 32768 rows, 8.4 / 14.4 at
// 130050, 11.3 / 19.9 at 262144; FP32 7.3 / 12.6, 9.0 / 14.2, 11.3 / 17.2.
// With r published in front of the partials, and read after them, the
// iteration at 32768 rows took 8.5 us.
// ---------------------------------------------------------------------------
constexpr int RES_COLS = 8;                    // entries per row at most
constexpr int RES_GROUPS = VEC_GRID_MAX;       // row groups at most

// every slot empty (all-ones words of either size), no abort
__global__ void clear_slots(uint32_t* slots, int32_t words, uint32_t* bar) {
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < words; i += gridDim.x * blockDim.x) slots[i] = ~0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) bar[0] = 0u;
}

// BT threads per block: BT / SPMV_BLOCK row groups.  slots: RES_SETS sets of
// 3 RES_GROUPS partials; zs: RES_SETS sets of n values of z.
template <typename T, int BT>
__global__ void __launch_bounds__(BT)
cg_resident(int32_t n, int32_t ng, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
            const T* __restrict__ val, const T* __restrict__ dinv, T* __restrict__ x, T* __restrict__ r,
            T* __restrict__ p, CgState<T>* st, int32_t k0, int32_t k_end, typename Word<T>::type* slots,
            typename Word<T>::type* zs, Wait wait) {
#pragma clang fp contract(off)
    typedef typename Word<T>::type W;
    constexpr W EMPTY = Word<T>::EMPTY;
    __shared__ T red1[BT / 64], red2[BT / 64];   // wave sums of this block's groups
    __shared__ T all[2][SPMV_BLOCK / 64];
    __shared__ T zl[BT];                         // z of this block's rows
    __shared__ int32_t bad;
    if (st->done != CG_RUNNING) return;
    const int32_t t = threadIdx.x, i = blockIdx.x * BT + t;
    const int32_t group = i / SPMV_BLOCK;
    const bool first = t % SPMV_BLOCK == 0 && group < ng;   // publishes the group's sums
    const int32_t k_stop = min(k_end, st->max_iter);
    const T thresh = st->thresh, pause_thresh = st->pause_thresh;
    T rz = st->rz[k0 & 3];
    int32_t len = 0, c[RES_COLS];
    T v[RES_COLS], pj[RES_COLS];
    T xi = T(0), ri = T(0), pi = T(0), di = T(0);
    bool remote = false;
    if (i < n) {
        const int32_t e0 = row_ptr[i];
        len = row_ptr[i + 1] - e0;
#pragma unroll
        for (int u = 0; u < RES_COLS; ++u) {
            c[u] = u < len ? col[e0 + u] : i;
            v[u] = u < len ? val[e0 + u] : T(0);
        }
#pragma unroll
        for (int u = 0; u < RES_COLS; ++u) pj[u] = p[c[u]];
        xi = x[i];
        ri = r[i];
        pi = p[i];
        di = dinv[i];
    } else {
#pragma unroll
        for (int u = 0; u < RES_COLS; ++u) {
            c[u] = i;
            v[u] = T(0);
            pj[u] = T(0);
        }
    }
    // columns of this block's own rows are read from zl, c = -1 - place; of the
    // others c is the byte offset
#pragma unroll
    for (int u = 0; u < RES_COLS; ++u) {
        const int32_t place = c[u] - (int32_t)blockIdx.x * BT;
        const bool own = place >= 0 && place < BT;
        remote |= !own;
        c[u] = own ? -1 - place : c[u] * (int32_t)sizeof(W);
    }
    if (t == 0) bad = 0;
    __syncthreads();
    int32_t k = k0, stop = CG_RUNNING;
    T pq = T(0), a = T(0), beta = T(0), rr = T(0);
    bool given_up = false;
    for (; k < k_stop; ++k) {
        W* const s_pq = slots + (k % RES_SETS) * 3 * RES_GROUPS;
        W* const s_rr = s_pq + RES_GROUPS;   // (r, z) and (r, r), a pair per group
        W* const z_k = zs + (int64_t)(k % RES_SETS) * n;
        // q = A p, partials of (p, q)
        T q = T(0);
#pragma unroll
        for (int u = 0; u < RES_COLS; ++u)
            if (u < len) q += v[u] * pj[u];
        T w1 = wave_sum(pi * q);
        if ((t & 63) == 0) red1[t >> 6] = w1;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the slots emptied last time are
        __syncthreads();
        if (first) agent_store(s_pq + group, Word<T>::of(sum_red(red1 + t / 64)));
        if (t < SPMV_BLOCK && !gather_slots<T, 1>(s_pq, ng, t, wait, all)) bad = 1;
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
        ri = ri - a * q;
        const T zi = di * ri;
        if (remote) agent_store(z_k + i, Word<T>::of(zi));
        zl[t] = zi;
        w1 = wave_sum(ri * zi);
        const T w2 = wave_sum(ri * ri);
        if ((t & 63) == 0) {
            red1[t >> 6] = w1;
            red2[t >> 6] = w2;
        }
        __syncthreads();
        if (first) {
            agent_store(s_rr + 2 * group, Word<T>::of(sum_red(red1 + t / 64)));
            agent_store(s_rr + 2 * group + 1, Word<T>::of(sum_red(red2 + t / 64)));
        }
        if (k > k0) {   // every block is past iteration k - 1
            if (remote) agent_store(zs + (int64_t)((k - 1) % RES_SETS) * n + i, EMPTY);
            if (first) {
                W* const old = slots + ((k - 1) % RES_SETS) * 3 * RES_GROUPS;
                agent_store(old + group, EMPTY);
                agent_store(old + RES_GROUPS + 2 * group, EMPTY);
                agent_store(old + RES_GROUPS + 2 * group + 1, EMPTY);
            }
        }
        W zj[RES_COLS];
        if (remote) {
#pragma unroll
            for (int u = 0; u < RES_COLS; ++u) zj[u] = c[u] >= 0 ? agent_load_at(z_k, (uint32_t)c[u]) : W(0);
        }
        if (t < SPMV_BLOCK && !gather_slots<T, 2>(s_rr, ng, t, wait, all)) bad = 1;
        if (remote) {
            for (uint32_t spins = 0;;) {
                bool empty = false;
#pragma unroll
                for (int u = 0; u < RES_COLS; ++u) empty |= zj[u] == EMPTY;
                if (!empty) break;
                if (wait_over(spins, wait)) {
                    bad = 1;
                    break;
                }
#pragma unroll
                for (int u = 0; u < RES_COLS; ++u)
                    if (zj[u] == EMPTY) zj[u] = agent_load_at(z_k, (uint32_t)c[u]);
            }
        }
        __syncthreads();
        if (bad) {
            given_up = true;
            break;
        }
        const T rzn = sum_red(all[0]);
        rr = sum_red(all[1]);
        // x += alpha p; stop tests; beta = rz_{k+1} / rz_k; p = z + beta p
        xi = xi + a * pi;
        if (rr <= thresh) stop = CG_CONVERGED;
        else if (!(rzn > T(0)) || !isfinite(rzn)) stop = CG_BREAKDOWN;
        else if (rr <= pause_thresh) stop = CG_PAUSED;
        if (stop != CG_RUNNING) {
            ++k;   // this iteration counts
            break;
        }
        beta = rzn / rz;
        rz = rzn;
        pi = zi + beta * pi;
#pragma unroll
        for (int u = 0; u < RES_COLS; ++u) {
            const T z = c[u] < 0 ? zl[-1 - c[u]] : Word<T>::value(zj[u]);
            pj[u] = z + beta * pj[u];
        }
    }
    if (given_up) {
        if (t == 0) atomicOr(wait.bar, 1u);
        return;
    }
    if (i < n) {
        x[i] = xi;
        r[i] = ri;
        p[i] = pi;
    }
    if (i == 0) {
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

// blocks of the cooperative launch for n rows: about two groups of rows per
// block, at most LOOP_GRID_MAX blocks (a barrier costs about one L2
// write-back and invalidate per block, so fewer, fuller blocks are cheaper
// up to the point where the SpMV phase lacks parallelism), a multiple of 8,
// at most what the device holds at once
constexpr int BAR_WORDS = FLAG0 + FLAG_STRIDE * SPMV_GRID_MAX;

template <typename T>
int loop_grid(int64_t n, int* out) {
    int dev = 0, cus = 0, per_cu = 0, coop = 0;
    RP_HIP_TRY(hipGetDevice(&dev));
    RP_HIP_TRY(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev));
    if (!coop) {
        *out = 0;
        return RP_OK;
    }
    RP_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    RP_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, cg_loop<T>, SPMV_BLOCK, 0));
    int64_t cap = std::min<int64_t>((int64_t)cus * per_cu, SPMV_GRID_MAX);
    cap -= cap % N_XCD;
    const int64_t groups = (n + SPMV_BLOCK - 1) / SPMV_BLOCK;
    int64_t g = std::min<int64_t>((groups + 1) / 2, LOOP_GRID_MAX);
    g = ((g + N_XCD - 1) / N_XCD) * N_XCD;
    *out = (int)std::max<int64_t>(std::min(g, cap), 0);
    return RP_OK;
}

}  // namespace

template <typename T>
int launch_cg_loop(rp_plan* p, int32_t n, const SpmvIdx& ix, const T* val, const T* dinv, T* x, T* r, T* pv, T* q,
                   CgState<T>* st, int32_t k0, int32_t k_end, hipStream_t s, bool* ran) {
    *ran = false;
    int grid = 0;
    RP_TRY(loop_grid<T>(n, &grid));
    if (grid < N_XCD) return RP_OK;
    if (!p->d_loop_bar) RP_HIP_TRY(hipMalloc(&p->d_loop_bar, BAR_WORDS * sizeof(uint32_t)));
    const LoopPlace place(p, grid);
    hipLaunchKernelGGL(clear_barrier, dim3(1), dim3(1024), 0, s, p->d_loop_bar, FLAG0 + FLAG_STRIDE * grid);
    RP_HIP_TRY(hipGetLastError());
    T* part = (T*)p->d_partials;
    uint32_t* bar = p->d_loop_bar;
    void* args[] = {&n, (void*)&ix, (void*)&val, (void*)&dinv, &x, &r, &pv, &q, &part, &st, &k0, &k_end, &bar};
    RP_HIP_TRY(hipLaunchCooperativeKernel((const void*)cg_loop<T>, dim3(grid), dim3(SPMV_BLOCK), args, 0, s));
    uint32_t abort_word = 0;
    RP_HIP_TRY(hipMemcpyAsync(&abort_word, p->d_loop_bar, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    RP_HIP_TRY(hipStreamSynchronize(s));
    if (abort_word) {
        set_error("the single-launch CG loop gave up waiting at a grid barrier");
        return RP_ERR_HIP;
    }
    *ran = true;
    return RP_OK;
}

namespace {

// The compute units of a device that one-launch loops hold.
//
// Every workgroup of a loop has to find its place while the others wait for its
// values, so loops on different streams must not take the units between them.
// (The runtime's cooperative launches keep apart by running one after the
// other, whatever they leave free.)  A loop therefore counts its workgroups in,
// a unit each, and is launched once all of them fit beside those of the loops
// that run.  Workgroups go to the dies in turn, so a die's share is counted up.
struct Units {
    std::mutex m;
    std::condition_variable freed;
    int held = 0;
    uint64_t next = 0, turn = 0;   // those who wait are served in the order they came
    int small = 0;                 // solves of small systems
};
constexpr int MAX_DEVICES = 64;
Units g_units[MAX_DEVICES];

int units(const rp_plan* p, int grid) { return std::min((grid + N_XCD - 1) / N_XCD * N_XCD, p->n_cus); }

}  // namespace

LoopPlace::LoopPlace(rp_plan* p, int grid) : device(p->device % MAX_DEVICES), need(units(p, grid)) {
    Units& u = g_units[device];
    std::unique_lock<std::mutex> lock(u.m);
    const uint64_t mine = u.next++;
    u.freed.wait(lock, [&] { return u.turn == mine && u.held + need <= p->n_cus; });
    ++u.turn;
    u.held += need;
    u.freed.notify_all();
}

LoopPlace::~LoopPlace() {
    Units& u = g_units[device];
    {
        std::lock_guard<std::mutex> lock(u.m);
        u.held -= need;
    }
    u.freed.notify_all();
}

// Small systems have the same iterates in launched kernels, which several
// streams overlap as finely as they come.  Loops are faster as long as the
// solves that run need the device no more than twice over; measured per solve
// with 1, 2, 4 and 8 threads, launches and loops, at 32^3 rows (64 units) 1.70 0.90
// 0.53 0.53 ms and 0.89 0.48 0.27 0.25; at 44^3 (168) 2.56 1.45 1.46 0.97 and 1.46
// 1.42 1.41 1.43; at 64^3 (256) 5.4 3.6 2.5 2.9 and 2.8 whatever the threads; mixed
// 64^3 5.3 3.3 2.2 2.2 and 3.3 3.1 3.1 3.1.
bool SmallSolve::loops_fit(rp_plan* p, int grid) {
    device = p->device % MAX_DEVICES;
    Units& u = g_units[device];
    std::lock_guard<std::mutex> lock(u.m);
    ++u.small;
    return u.small * units(p, grid) <= 2 * p->n_cus;
}

SmallSolve::~SmallSolve() {
    if (device < 0) return;
    std::lock_guard<std::mutex> lock(g_units[device].m);
    --g_units[device].small;
}

int launch_loop(rp_plan* p, const void* kernel, int grid, int block, void** args, const uint32_t* bar,
                hipStream_t s) {
    p->h_flags[LOOP_ABORT] = 1u;
    if (hipLaunchKernel(kernel, dim3(grid), dim3(block), args, 0, s) != hipSuccess) {
        (void)hipGetLastError();
        return RP_OK;
    }
    RP_HIP_TRY(hipMemcpyAsync(p->h_flags + LOOP_ABORT, bar, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    return RP_OK;
}

bool loop_gave_up(rp_plan* p) {
    if (p->h_flags[LOOP_ABORT] == 0u) {
        p->loop_given_up = 0;
        return false;
    }
    p->loop_rest = 1 << std::min(p->loop_given_up, 10);
    p->loop_given_up = std::min(p->loop_given_up + 1, 10);
    return true;
}

template <typename T>
const void* resident_kernel(int bt) {
    return bt == 512 ? (const void*)cg_resident<T, 512> : (const void*)cg_resident<T, 1024>;
}

// Threads per block of the resident loop, 0 where the plan or the device does
// not fit it (a row of more than RES_COLS entries; more rows than the device
// holds at a row per thread).  Measured per iteration, 512 against 1024
// threads: FP64 6.7 / 8.7 us at 32768 rows and 8.4 / 10.2 at 130050 (1024
// threads leave it 128 registers, and it spills), but only 1024 hold 262144
// rows (11.3); FP32 8.0 / 7.3 us and 9.8 / 9.2 (fewer blocks to wait for).
template <typename T>
int resident_block(rp_plan* p, int* out) {
    int& bt = p->resident_block[sizeof(T) == 4];
    if (bt < 0) {
        const int64_t n = p->n_rows;
        int fit = 0;
        if (p->max_row <= RES_COLS && n <= (int64_t)RES_GROUPS * SPMV_BLOCK)
            for (int t = sizeof(T) == 8 ? 512 : 1024; t <= 1024 && fit == 0; t *= 2) {
                int per_cu = 0;
                RP_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, resident_kernel<T>(t), t, 0));
                if (n <= (int64_t)p->n_cus * per_cu * t) fit = t;
            }
        bt = fit;
    }
    *out = bt;
    return RP_OK;
}

template int resident_block<double>(rp_plan*, int*);
template int resident_block<float>(rp_plan*, int*);

// words the loop exchanges its values through, of either precision
inline int64_t resident_slots(int64_t n) { return (int64_t)RES_SETS * (3 * RES_GROUPS + n); }

// whether there is memory for them
bool resident_room(rp_plan* p) {
    return got(p, &p->d_slots, resident_slots(p->n_rows) * sizeof(uint64_t)) &&
           got(p, &p->d_loop_bar, BAR_WORDS * sizeof(uint32_t));
}

// The iterations k0 .. min(k_end, budget) by the resident loop, enqueued, on a
// plan that fits it (resident_block > 0) and has room for it (resident_room).  See launch_loop.
template <typename T>
int launch_cg_resident(rp_plan* p, int32_t n, const int32_t* row_ptr, const int32_t* col, const T* val,
                       const T* dinv, T* x, T* r, T* pv, CgState<T>* st, int32_t k0, int32_t k_end, hipStream_t s) {
    const int bt = p->resident_block[sizeof(T) == 4];
    int32_t ng = (n + SPMV_BLOCK - 1) / SPMV_BLOCK;
    // slots of either precision: the sums, then z
    typedef typename Word<T>::type W;
    const int64_t len = resident_slots(n);
    W* slots = (W*)p->d_slots;
    W* zs = slots + RES_SETS * 3 * RES_GROUPS;
    uint32_t* bar = p->d_loop_bar;
    hipLaunchKernelGGL(clear_slots, dim3(256), dim3(256), 0, s, (uint32_t*)slots, (int32_t)(len * sizeof(W) / 4), bar);
    RP_HIP_TRY(hipGetLastError());
    Wait wait{bar, wait_spins(p)};
    void* args[] = {&n, &ng, (void*)&row_ptr, (void*)&col, (void*)&val, (void*)&dinv, &x, &r, &pv, &st, &k0, &k_end,
                    &slots, &zs, &wait};
    return launch_loop(p, resident_kernel<T>(bt), (n + bt - 1) / bt, bt, args, bar, s);
}

template int launch_cg_resident<double>(rp_plan*, int32_t, const int32_t*, const int32_t*, const double*,
                                        const double*, double*, double*, double*, CgState<double>*, int32_t, int32_t,
                                        hipStream_t);
template int launch_cg_resident<float>(rp_plan*, int32_t, const int32_t*, const int32_t*, const float*, const float*,
                                       float*, float*, float*, CgState<float>*, int32_t, int32_t, hipStream_t);
template int launch_cg_loop<double>(rp_plan*, int32_t, const SpmvIdx&, const double*, const double*, double*,
                                    double*, double*, double*, CgState<double>*, int32_t, int32_t, hipStream_t, bool*);
template int launch_cg_loop<float>(rp_plan*, int32_t, const SpmvIdx&, const float*, const float*, float*, float*,
                                   float*, float*, CgState<float>*, int32_t, int32_t, hipStream_t, bool*);

}  // namespace rp
