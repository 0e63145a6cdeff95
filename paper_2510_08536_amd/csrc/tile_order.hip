// A row order with locality for the tiled CG loop (cg_tile.hip), for plans
// whose own numbering has none: consecutive rows of it are compact pieces of
// the mesh, so that a tile's halo is about the surface of a blob instead of
// nearly every column of its rows.  Only the loop's private copies follow it.
//
//  1. Regions: rows at a fixed stride are seeds; each round, a row without a
//     region takes the lowest region among its neighbours' of the round before
//     (so the result does not depend on the order of execution).  Rows no seed
//     reaches go by index into regions of their own.
//  2. The pairs of regions with a coupling, collected in a hash table, and the
//     regions' sizes go to the host, which orders the regions: tile by tile it
//     adds the region with the most neighbours already in the tile and the
//     fewest not placed yet, and starts a tile next to what is placed, where
//     the fewest neighbours are left, so that no pockets remain.  (By the
//     neighbours in the tile alone the halos of 256 tiles of 128^3 rows were
//     2963 on average and 7634 at most; by both 2692 and 3703.)
//  3. Rows are placed region by region, ascending within a region.
#include <algorithm>
#include <queue>
#include <vector>

#include "rp_internal.hpp"

namespace rp {

namespace {

constexpr int OB = 256;
constexpr int64_t REGION_ROWS = 208;    // rows per seed: with 64 the halos are no shorter, the host's part 4 times as long
constexpr int64_t LEFT_ROWS = 1024;     // rows of a region of unreached rows
constexpr int REGION_MAX = 4096;        // rows of a region at most (sorted in LDS)
constexpr int ROUNDS = 64;              // growth rounds at most
constexpr int PROBES = 256;

int grid_of(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + OB - 1) / OB, 8192)); }

__global__ void __launch_bounds__(OB) order_seed(int32_t n, int32_t stride, int32_t* label) {
    for (int32_t i = blockIdx.x * OB + threadIdx.x; i < n; i += gridDim.x * OB)
        label[i] = i % stride == 0 ? i / stride : -1;
}

__global__ void __launch_bounds__(OB)
order_grow(int32_t n, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
           const int32_t* __restrict__ from, int32_t* __restrict__ to, uint32_t* grown) {
    bool any = false;
    for (int32_t i = blockIdx.x * OB + threadIdx.x; i < n; i += gridDim.x * OB) {
        int32_t l = from[i];
        if (l < 0) {
            uint32_t best = ~0u;   // unlabelled neighbours (-1) are the largest
            for (int32_t e = row_ptr[i]; e < row_ptr[i + 1]; ++e) best = min(best, (uint32_t)from[col[e]]);
            l = (int32_t)best;
            any |= l >= 0;
        }
        to[i] = l;
    }
    if (__any(any) && (threadIdx.x & 63) == 0) atomicOr(grown, 1u);
}

__global__ void order_clear(uint32_t* w, int64_t words, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * OB + threadIdx.x; i < words; i += (int64_t)gridDim.x * OB) w[i] = v;
}

// unreached rows; the regions' sizes
__global__ void __launch_bounds__(OB)
order_count(int32_t n, int32_t seeds, int32_t* __restrict__ label, uint32_t* __restrict__ size) {
    for (int32_t i = blockIdx.x * OB + threadIdx.x; i < n; i += gridDim.x * OB) {
        int32_t l = label[i];
        if (l < 0) {
            l = seeds + i / (int32_t)LEFT_ROWS;
            label[i] = l;
        }
        atomicAdd(size + l, 1u);
    }
}

// the pairs (a < b) of coupled regions into an open-addressed table of keys
__global__ void __launch_bounds__(OB)
order_pairs(int32_t n, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
            const int32_t* __restrict__ label, unsigned long long* __restrict__ table, uint32_t mask, uint32_t* full) {
    for (int32_t i = blockIdx.x * OB + threadIdx.x; i < n; i += gridDim.x * OB) {
        const int32_t a = label[i];
        for (int32_t e = row_ptr[i]; e < row_ptr[i + 1]; ++e) {
            const int32_t b = label[col[e]];
            if (b <= a) continue;
            const unsigned long long key = ((unsigned long long)(uint32_t)a << 32) | (uint32_t)b;
            uint32_t h = (uint32_t)a * 0x9E3779B1u ^ (uint32_t)b * 0x85EBCA6Bu;
            h ^= h >> 15;
            bool done = false;
            for (int q = 0; q < PROBES && !done; ++q, ++h) {
                unsigned long long* s = table + (h & mask);
                if (*(volatile unsigned long long*)s == key) done = true;
                else {
                    const unsigned long long old = atomicCAS(s, ~0ull, key);
                    done = old == ~0ull || old == key;
                }
            }
            if (!done) atomicOr(full, 1u);
        }
    }
}

__global__ void __launch_bounds__(OB)
order_place(int32_t n, const int32_t* __restrict__ label, const int32_t* __restrict__ start,
            uint32_t* __restrict__ used, int32_t* __restrict__ order) {
    for (int32_t i = blockIdx.x * OB + threadIdx.x; i < n; i += gridDim.x * OB) {
        const int32_t l = label[i];
        order[start[l] + (int32_t)atomicAdd(used + l, 1u)] = i;
    }
}

// each region's rows ascending (a block per region), and the inverse
__global__ void __launch_bounds__(OB)
order_sort(const int32_t* __restrict__ start, const uint32_t* __restrict__ size, int32_t* __restrict__ order,
           int32_t* __restrict__ inv) {
    __shared__ int32_t v[REGION_MAX];
    const int32_t s0 = start[blockIdx.x], m = (int32_t)size[blockIdx.x], t = threadIdx.x;
    int32_t P2 = 1;
    while (P2 < m) P2 *= 2;
    for (int32_t i = t; i < P2; i += OB) v[i] = i < m ? order[s0 + i] : INT32_MAX;
    __syncthreads();
    for (int32_t k = 2; k <= P2; k *= 2)
        for (int32_t j = k / 2; j > 0; j /= 2) {
            for (int32_t i = t; i < P2; i += OB) {
                const int32_t o = i ^ j;
                if (o > i && (v[i] > v[o]) == ((i & k) == 0)) {
                    const int32_t x = v[i];
                    v[i] = v[o];
                    v[o] = x;
                }
            }
            __syncthreads();
        }
    for (int32_t i = t; i < m; i += OB) {
        order[s0 + i] = v[i];
        inv[v[i]] = s0 + i;
    }
}

// the regions in the order they are placed: tiles of `cap` rows
std::vector<int32_t> order_regions(const std::vector<uint32_t>& size, const std::vector<unsigned long long>& pairs,
                                   int64_t cap) {
    const int32_t S = (int32_t)size.size();
    std::vector<int32_t> ptr(S + 1, 0), adj(2 * pairs.size());
    for (unsigned long long k : pairs) {
        ++ptr[(uint32_t)(k >> 32) + 1];
        ++ptr[(uint32_t)k + 1];
    }
    for (int32_t a = 0; a < S; ++a) ptr[a + 1] += ptr[a];
    std::vector<int32_t> at(ptr.begin(), ptr.end() - 1);
    for (unsigned long long k : pairs) {
        const int32_t a = (int32_t)(k >> 32), b = (int32_t)(uint32_t)k;
        adj[at[a]++] = b;
        adj[at[b]++] = a;
    }
    std::vector<int32_t> out, in_tile(S, 0), stamp(S, -1), score(S), open(S), edge;
    std::vector<uint8_t> placed(S, 0);
    out.reserve(S);
    for (int32_t a = 0; a < S; ++a) open[a] = ptr[a + 1] - ptr[a];
    int32_t tile = 0, next = 0;
    int64_t rows = 0;
    // candidates of the tile, best score first, then the lowest index; an entry
    // whose score has changed since is stale
    std::priority_queue<std::pair<int32_t, int32_t>> cand;
    auto enter = [&](int32_t a) {   // a's neighbours become candidates of the current tile
        for (int32_t e = ptr[a]; e < ptr[a + 1]; ++e) {
            const int32_t b = adj[e];
            if (placed[b]) continue;
            if (stamp[b] != tile) {
                stamp[b] = tile;
                in_tile[b] = 0;
            }
            score[b] = 2 * ++in_tile[b] - open[b];
            cand.emplace(score[b], -b);
        }
    };
    auto place = [&](int32_t a) {
        placed[a] = 1;
        out.push_back(a);
        for (int32_t e = ptr[a]; e < ptr[a + 1]; ++e) --open[adj[e]];
        enter(a);
        rows += size[a];
        if (rows < cap) return;
        // the tile is full: its open neighbours may start others; what it
        // spills is the next tile's
        while (!cand.empty()) {
            const int32_t b = -cand.top().second;
            cand.pop();
            if (!placed[b]) edge.push_back(b);
        }
        ++tile;
        rows %= cap;
        if (rows > 0) enter(a);
    };
    while ((int32_t)out.size() < S) {
        int32_t a = -1;
        while (!cand.empty() && a < 0) {
            const auto [g, nb] = cand.top();
            cand.pop();
            if (!placed[-nb] && stamp[-nb] == tile && score[-nb] == g) a = -nb;
        }
        if (a < 0) {   // next to what is placed, fewest neighbours left
            size_t keep = 0;
            for (int32_t b : edge)
                if (!placed[b]) {
                    edge[keep++] = b;
                    if (a < 0 || open[b] < open[a] || (open[b] == open[a] && b < a)) a = b;
                }
            edge.resize(keep);
        }
        if (a < 0) {
            while (placed[next]) ++next;
            a = next;
        }
        place(a);
    }
    return out;
}

struct Free {
    std::vector<void*> q;
    ~Free() {
        for (void* a : q)
            if (a) (void)hipFree(a);
    }
};

template <typename V>
bool temp(rp_plan* p, Free& f, V** q, int64_t count) {
    if (loop_malloc(p, (void**)q, sizeof(V) * (size_t)std::max<int64_t>(count, 1)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    f.q.push_back(*q);
    return true;
}

}  // namespace

// order[n] (row at each position) and inv[n], device arrays of the caller's,
// for tiles of `cap` rows; *ok = false where a region grew too large, or where
// there is no memory for it (*memory = false)
int tile_order(rp_plan* p, int64_t cap, int32_t* order, int32_t* inv, hipStream_t s, bool* ok, bool* memory) {
    *ok = false;
    const int32_t n = (int32_t)p->n_rows;
    const int32_t stride = (int32_t)REGION_ROWS;
    const int32_t seeds = (n + stride - 1) / stride;
    const int32_t S = seeds + (int32_t)((n + LEFT_ROWS - 1) / LEFT_ROWS);
    uint32_t slots = 1024;
    while (slots < 32u * (uint32_t)S && slots < (1u << 26)) slots *= 2;
    Free f;
    int32_t *la = nullptr, *lb = nullptr, *start = nullptr;
    uint32_t *size = nullptr, *used = nullptr, *flag = nullptr;
    unsigned long long* table = nullptr;
    if (!temp(p, f, &la, n) || !temp(p, f, &lb, n) || !temp(p, f, &start, S) || !temp(p, f, &size, 2 * (int64_t)S + 2) ||
        !temp(p, f, &table, slots)) {
        *memory = false;
        return RP_OK;
    }
    used = size + S;
    flag = used + S;   // grown, table full
    const dim3 g(grid_of(n)), b(OB);
    hipLaunchKernelGGL(order_clear, dim3(grid_of(2 * (int64_t)S + 2)), b, 0, s, size, 2 * (int64_t)S + 2, 0u);
    hipLaunchKernelGGL(order_clear, dim3(grid_of(2 * (int64_t)slots)), b, 0, s, (uint32_t*)table, 2 * (int64_t)slots, ~0u);
    hipLaunchKernelGGL(order_seed, g, b, 0, s, n, stride, la);
    for (int r = 0; r < ROUNDS; ++r) {
        hipLaunchKernelGGL(order_grow, g, b, 0, s, n, p->d_row_ptr, p->d_col, la, lb, flag);
        std::swap(la, lb);
        if (r % 8 != 7) continue;   // the host looks every eighth round
        uint32_t grown = 0;
        RP_HIP_TRY(hipMemcpyAsync(&grown, flag, sizeof(grown), hipMemcpyDeviceToHost, s));
        RP_HIP_TRY(hipStreamSynchronize(s));
        if (!grown) break;
        hipLaunchKernelGGL(order_clear, dim3(1), b, 0, s, flag, (int64_t)1, 0u);
    }
    hipLaunchKernelGGL(order_count, g, b, 0, s, n, seeds, la, size);
    hipLaunchKernelGGL(order_pairs, g, b, 0, s, n, p->d_row_ptr, p->d_col, la, table, slots - 1, flag + 1);
    RP_HIP_TRY(hipGetLastError());
    loop_host(p);
    std::vector<uint32_t> hs(2 * (size_t)S + 2);
    std::vector<unsigned long long> ht(slots);
    RP_HIP_TRY(hipMemcpyAsync(hs.data(), size, sizeof(uint32_t) * hs.size(), hipMemcpyDeviceToHost, s));
    RP_HIP_TRY(hipMemcpyAsync(ht.data(), table, sizeof(unsigned long long) * slots, hipMemcpyDeviceToHost, s));
    RP_HIP_TRY(hipStreamSynchronize(s));
    if (hs[2 * (size_t)S + 1]) return RP_OK;
    hs.resize(S);
    for (uint32_t v : hs)
        if (v > (uint32_t)REGION_MAX) return RP_OK;
    ht.erase(std::remove(ht.begin(), ht.end(), ~0ull), ht.end());
    std::sort(ht.begin(), ht.end());   // the table's order is that of arrival
    const std::vector<int32_t> seq = order_regions(hs, ht, cap);
    std::vector<int32_t> hstart(S);
    int32_t at = 0;
    for (int32_t a : seq) {
        hstart[a] = at;
        at += (int32_t)hs[a];
    }
    RP_HIP_TRY(hipMemcpyAsync(start, hstart.data(), sizeof(int32_t) * (size_t)S, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(order_place, g, b, 0, s, n, la, start, used, order);
    hipLaunchKernelGGL(order_sort, dim3(S), b, 0, s, start, size, order, inv);
    RP_HIP_TRY(hipGetLastError());
    RP_HIP_TRY(hipStreamSynchronize(s));   // the temporaries are released
    *ok = true;
    return RP_OK;
}

}  // namespace rp
