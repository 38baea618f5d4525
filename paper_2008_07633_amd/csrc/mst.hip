// Maximum-weight spanning forest on the GPU (the MST the paper uses in place
// of a low-stretch tree, Sec. 3.4).  Edges are totally ordered by (weight
// descending, edge id ascending), so the forest is unique and equals the one
// Kruskal's rule picks in that order.
//
// Boruvka rounds over a shrinking list of edges:
//   1. the list is compacted: endpoints become the roots of their components,
//      edges inside one component are dropped; the same pass finds every
//      component's best weight (an integer atomicMax of the weight's bits:
//      positive IEEE values order like them).  Once components are few, a
//      workgroup first collects its maxima in an LDS table, so that a
//      component most edges touch does not serialise their atomics;
//   2. an atomicMin of the edge id among the edges that reach the best weight;
//   3. each component hooks onto the component across its best edge; a pair
//      that chose the same edge is rooted at the smaller id (longer cycles
//      cannot occur under a total order);
//   4. pointer jumping flattens the hooks; the remaining roots are listed for
//      the next round.
// A list with several edges per node is taken in two parts: first the edges
// at or above a weight that about n edges reach (from a sample), a few rounds;
// then the others, of which most lie inside one component by then and are
// read once.  All edges of the first part precede the others in the order, so
// the forest is the same.
//
// List and root counts stay on the device; kernels run over them with a fixed
// grid and return at once when a list is empty.  The host reads the count
// after the first kRoundsBlind rounds of the second part and every
// kRoundsCheck rounds after that.  Only integer atomics are used, and every
// choice is by (weight, id), so the result does not depend on scheduling.
//
// Bound by random 8-byte reads and atomics, m at a time in the first version
// (every round over all edges, a host wait per round and per four pointer
// jumps): 4.9 ms for the 150^3 mesh (10.1M edges), now 1.5; about 12 ms for the
// 39.9M edges of the 4M-node Chung-Lu graph, now 3.4.
#include <algorithm>
#include <mutex>

#include "common.hpp"

namespace sfg {

namespace {

constexpr uint64_t kNoEdge = ~0ull;

template <typename TW>
__device__ __forceinline__ uint64_t wkey(TW w) {
    const double d = (double)w;
    uint64_t k;
    __builtin_memcpy(&k, &d, sizeof(k));
    return k;
}

// Live edges: roots of the two endpoints and the edge id.
struct EdgeList {
    int32_t *a, *b, *id;
};

// Device counters.
enum { kCntList0 = 0, kCntList1 = 1, kCntRoots0 = 2, kCntRoots1 = 3, kCntComps = 4, kCounters = 8 };

__global__ void k_mst_init(int64_t n, int32_t *par, uint64_t *best_w, uint64_t *best_e, int32_t *cnt) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < kCounters) cnt[p] = 0;
    if (p >= n) return;
    par[p] = (int32_t)p;
    best_w[p] = 0;
    best_e[p] = kNoEdge;
}

// Weight that about `want` of the m edges reach, from 1024 edges spread over
// the list (any value is right; it only splits the work).
template <typename TW>
__global__ __launch_bounds__(1024) void k_mst_pivot(int64_t m, const TW *__restrict__ w, int64_t want,
                                                    uint64_t *pivot) {
    __shared__ uint64_t s[1024];
    const int t = threadIdx.x;
    const int64_t lo = m * t / 1024, hi = m * (t + 1) / 1024;
    uint32_t h = (uint32_t)t * 0x9E3779B1u;
    h ^= h >> 15;
    const int64_t e = hi > lo ? lo + (int64_t)(h % (uint32_t)(hi - lo)) : lo;
    s[t] = e < m ? wkey(w[e]) : 0;
    __syncthreads();
    for (int kk = 2; kk <= 1024; kk <<= 1)
        for (int jj = kk >> 1; jj > 0; jj >>= 1) {
            const int o = t ^ jj;
            if (o > t) {
                const uint64_t x = s[t], y = s[o];
                if ((x < y) == ((t & kk) == 0)) {      // descending
                    s[t] = y;
                    s[o] = x;
                }
            }
            __syncthreads();
        }
    int64_t at = want * 1024 / m;
    if (at > 1023) at = 1023;
    if (t == 0) *pivot = s[at];
}

constexpr int kTabBits = 10, kTab = 1 << kTabBits;     // LDS table of component maxima
constexpr int kPerThread = 8;                          // edges of a chunk per thread
constexpr int kMstThreads = 512;
constexpr unsigned kMstGrid = 1024;                    // workgroups of a list kernel, each a stride of chunks

// Entries a thread takes of each chunk: fewer than kPerThread when the list
// is short, so that it spreads over the workgroups (eight dependent chains of
// a root or an edge in one thread kept a list of 20,000 entries at 30 us).
__device__ __forceinline__ int per_thread(int64_t m) {
    const int64_t per = (m + (int64_t)gridDim.x * kMstThreads - 1) / ((int64_t)gridDim.x * kMstThreads);
    return (int)(per < 1 ? 1 : (per > kPerThread ? kPerThread : per));
}

// read first: most edges lose, and skipping their atomics removes the
// contention (the maximum is still exact)
__device__ __forceinline__ void raise_global(uint64_t *best_w, int32_t c, uint64_t k) {
    if (k > best_w[c]) atomicMax((unsigned long long *)&best_w[c], (unsigned long long)k);
}

template <bool TABLE>
__device__ __forceinline__ void raise_best(uint64_t *best_w, int32_t *tc, unsigned long long *tb, int32_t c,
                                           uint64_t k) {
    if constexpr (TABLE) {
        const uint32_t h = ((uint32_t)c * 0x9E3779B1u) >> (32 - kTabBits);
        int32_t old = __hip_atomic_load(&tc[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (old == -1) old = atomicCAS(&tc[h], -1, c);
        if (old == -1 || old == c) {
            if (k > __hip_atomic_load(&tb[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
                atomicMax(&tb[h], (unsigned long long)k);
            return;
        }
    }
    raise_global(best_w, c, k);
}

// Workgroup-wide append: every thread has up to kPerThread entries with
// live[i]; returns the list position of its i-th one through pos[i].  One
// global atomic a call.
__device__ __forceinline__ void append_positions(const bool (&live)[kPerThread], int32_t (&pos)[kPerThread],
                                                 int32_t *counter, int32_t *sh /* 2 */) {
    const int lane = threadIdx.x & (kWave - 1);
    if (threadIdx.x == 0) sh[0] = 0;
    __syncthreads();
    int32_t mine = 0;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) mine += live[i] ? 1 : 0;
    int32_t incl = mine;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int32_t y = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += y;
    }
    int32_t base = 0;
    if (lane == kWave - 1 && incl > 0) base = atomicAdd(&sh[0], incl);
    base = __shfl(base, kWave - 1, kWave);
    __syncthreads();
    if (threadIdx.x == 0) sh[1] = sh[0] > 0 ? atomicAdd(counter, sh[0]) : 0;
    __syncthreads();
    int32_t at = sh[1] + base + incl - mine;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
        pos[i] = at;
        at += live[i] ? 1 : 0;
    }
}

// Compaction and best weights of one round.  SRC = 0: every allowed edge of
// the graph (components are single nodes); 1: those at or above the pivot
// (likewise); 2: those below it, appended to a list that holds the rest of
// the first part (par is flat); 3: the previous round's list, whose endpoints
// were roots before the last hooks.
template <typename TW, int SRC, bool TABLE>
__global__ __launch_bounds__(kMstThreads) void k_mst_list(int64_t m, const int32_t *__restrict__ u,
                                                          const int32_t *__restrict__ v, const TW *__restrict__ w,
                                                          const uint8_t *__restrict__ allowed,
                                                          const uint64_t *__restrict__ pivot,
                                                          const int32_t *__restrict__ par, EdgeList in,
                                                          const int32_t *__restrict__ in_cnt, EdgeList out,
                                                          int32_t *out_cnt, uint64_t *best_w) {
    __shared__ int32_t tc[TABLE ? kTab : 1];
    __shared__ unsigned long long tb[TABLE ? kTab : 1];
    __shared__ int32_t sh[2];
    if constexpr (SRC == 3) m = *in_cnt;
    const uint64_t piv = (SRC == 1 || SRC == 2) ? *pivot : 0;
    if constexpr (TABLE) {
        for (int i = threadIdx.x; i < kTab; i += kMstThreads) {
            tc[i] = -1;
            tb[i] = 0;
        }
        __syncthreads();
    }
    const int per = per_thread(m);
    const int64_t chunk = (int64_t)per * kMstThreads;
    for (int64_t c0 = blockIdx.x * chunk; c0 < m; c0 += gridDim.x * chunk) {
        int32_t a[kPerThread], b[kPerThread], id[kPerThread], pos[kPerThread];
        uint64_t k[kPerThread];
        bool live[kPerThread];
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            const int64_t e = c0 + (int64_t)i * kMstThreads + threadIdx.x;
            live[i] = i < per && e < m;
            a[i] = b[i] = id[i] = 0;
            k[i] = 0;
            if (!live[i]) continue;
            if constexpr (SRC == 3) {
                id[i] = in.id[e];
                a[i] = in.a[e];
                b[i] = in.b[e];
                k[i] = wkey(w[id[i]]);
            } else {
                id[i] = (int32_t)e;
                live[i] = !allowed || allowed[e] != 0;
                if (live[i]) {
                    k[i] = wkey(w[e]);
                    if constexpr (SRC == 1) live[i] = k[i] >= piv;
                    if constexpr (SRC == 2) live[i] = k[i] < piv;
                }
                if (live[i]) {
                    a[i] = u[e];
                    b[i] = v[e];
                }
            }
        }
        if constexpr (SRC >= 2) {
#pragma unroll
            for (int i = 0; i < kPerThread; ++i)
                if (live[i]) {
                    a[i] = par[a[i]];
                    b[i] = par[b[i]];
                }
        }
#pragma unroll
        for (int i = 0; i < kPerThread; ++i) {
            live[i] = live[i] && a[i] != b[i];
            if (live[i]) {
                raise_best<TABLE>(best_w, tc, tb, a[i], k[i]);
                raise_best<TABLE>(best_w, tc, tb, b[i], k[i]);
            }
        }
        append_positions(live, pos, out_cnt, sh);
#pragma unroll
        for (int i = 0; i < kPerThread; ++i)
            if (live[i]) {
                out.a[pos[i]] = a[i];
                out.b[pos[i]] = b[i];
                out.id[pos[i]] = id[i];
            }
        __syncthreads();
    }
    if constexpr (TABLE) {
        __syncthreads();
        for (int i = threadIdx.x; i < kTab; i += kMstThreads)
            if (tc[i] >= 0 && tb[i] > 0) raise_global(best_w, tc[i], tb[i]);
    }
}

// The edge of each component's best weight with the smallest id, packed with
// its place in the list.
template <typename TW>
__global__ __launch_bounds__(256) void k_mst_pick(const int32_t *__restrict__ cnt, EdgeList L,
                                                  const TW *__restrict__ w, const uint64_t *__restrict__ best_w,
                                                  uint64_t *best_e, int32_t *other_cnt) {
    const int32_t m = *cnt;
    if (blockIdx.x == 0 && threadIdx.x == 0) *other_cnt = 0;      // the list the next round fills
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < m; e += (int64_t)gridDim.x * 256) {
        const int32_t a = L.a[e], b = L.b[e], id = L.id[e];
        const uint64_t k = wkey(w[id]);
        const uint64_t me = ((uint64_t)(uint32_t)id << 32) | (uint64_t)e;
        if (k == best_w[a] && me < best_e[a]) atomicMin((unsigned long long *)&best_e[a], (unsigned long long)me);
        if (k == best_w[b] && me < best_e[b]) atomicMin((unsigned long long *)&best_e[b], (unsigned long long)me);
    }
}

// Roots (listed, or every node when roots == nullptr) hook across their best
// edge and mark it as a tree edge.
__global__ __launch_bounds__(256) void k_mst_hook(int64_t n, const int32_t *__restrict__ roots,
                                                  const int32_t *__restrict__ root_cnt, EdgeList L,
                                                  const uint64_t *__restrict__ best_e, int32_t *par, uint8_t *in_tree,
                                                  int32_t *next_cnt) {
    if (roots) n = *root_cnt;
    if (blockIdx.x == 0 && threadIdx.x == 0) *next_cnt = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int32_t c = roots ? roots[i] : (int32_t)i;
        const uint64_t e = best_e[c];
        if (e == kNoEdge) continue;
        const uint32_t at = (uint32_t)e;
        const int32_t a = L.a[at], b = L.b[at];
        const int32_t d = (a == c) ? b : a;
        in_tree[e >> 32] = 1;
        // a mutual pair (both chose e) is rooted at its smaller id
        par[c] = (best_e[d] == e && c < d) ? c : d;
    }
}

// Pointer jumping within the launch, at most kJumps jumps a root: the roots
// in flight shorten each other's chains, and whatever order their writes land
// in, par[c] stays an ancestor of c.  Other workgroups' writes may not be seen
// before the launch ends, so a chain surely gets kJumps times shorter only; the
// next kernel walks the rest.  On a path of 400,000 nodes with random ids and
// rising weights (one chain) a call takes 274 us, with 24 jumps 2,285; on
// meshes, power grids, k-NN and power-law graphs, whose chains are short, 0 to
// 64 jumps take the same time.
constexpr int kJumps = 64;

__global__ __launch_bounds__(256) void k_mst_jump(int64_t n, const int32_t *__restrict__ roots,
                                                  const int32_t *__restrict__ root_cnt, int32_t *par) {
    if (roots) n = *root_cnt;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int32_t c = roots ? roots[i] : (int32_t)i;
        int32_t p = __hip_atomic_load(&par[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        for (int j = 0; j < kJumps; ++j) {
            const int32_t g = __hip_atomic_load(&par[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (g == p) break;
            __hip_atomic_store(&par[c], g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            p = g;
        }
    }
}

// Every root of the round follows its (by now short) chain to the end; those
// that merged and are still roots are listed for the next round, and their
// best edges are cleared.
__global__ __launch_bounds__(kMstThreads) void k_mst_settle(int64_t n, const int32_t *__restrict__ roots,
                                                            const int32_t *__restrict__ root_cnt, int32_t *par,
                                                            uint64_t *best_w, uint64_t *best_e, int32_t *next,
                                                            int32_t *next_cnt) {
    __shared__ int32_t sh[2];
    if (roots) n = *root_cnt;
    const int per = per_thread(n);
    const int64_t chunk = (int64_t)per * kMstThreads;
    for (int64_t c0 = blockIdx.x * chunk; c0 < n; c0 += gridDim.x * chunk) {
        int32_t c[kPerThread], pos[kPerThread];
        bool live[kPerThread];
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            const int64_t i = c0 + (int64_t)j * kMstThreads + threadIdx.x;
            live[j] = false;
            c[j] = 0;
            if (j >= per || i >= n) continue;
            c[j] = roots ? roots[i] : (int32_t)i;
            int32_t p = __hip_atomic_load(&par[c[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (p == c[j]) {
                live[j] = best_e[c[j]] != kNoEdge;
                if (live[j]) {
                    best_w[c[j]] = 0;
                    best_e[c[j]] = kNoEdge;
                }
                continue;
            }
            for (;;) {
                const int32_t g = __hip_atomic_load(&par[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (g == p) break;
                p = g;
            }
            __hip_atomic_store(&par[c[j]], p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        append_positions(live, pos, next_cnt, sh);
#pragma unroll
        for (int j = 0; j < kPerThread; ++j)
            if (live[j]) next[pos[j]] = c[j];
        __syncthreads();
    }
}

// Between the parts: every node points at its root, every root is listed.
__global__ __launch_bounds__(kMstThreads) void k_mst_flatten(int64_t n, int32_t *par, int32_t *roots,
                                                             int32_t *root_cnt) {
    __shared__ int32_t sh[2];
    const int per = per_thread(n);
    const int64_t chunk = (int64_t)per * kMstThreads;
    for (int64_t c0 = blockIdx.x * chunk; c0 < n; c0 += gridDim.x * chunk) {
        int32_t c[kPerThread], pos[kPerThread];
        bool live[kPerThread];
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            const int64_t i = c0 + (int64_t)j * kMstThreads + threadIdx.x;
            live[j] = false;
            c[j] = (int32_t)i;
            if (j >= per || i >= n) continue;
            int32_t p = __hip_atomic_load(&par[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (p == c[j]) {
                live[j] = true;
                continue;
            }
            for (;;) {
                const int32_t g = __hip_atomic_load(&par[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (g == p) break;
                p = g;
            }
            __hip_atomic_store(&par[i], p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        append_positions(live, pos, root_cnt, sh);
#pragma unroll
        for (int j = 0; j < kPerThread; ++j)
            if (live[j]) roots[pos[j]] = c[j];
        __syncthreads();
    }
}

// Components of the forest so far.
__global__ __launch_bounds__(256) void k_mst_count(int64_t n, const int32_t *__restrict__ par, int32_t *cnt) {
    __shared__ int32_t part;
    if (threadIdx.x == 0) part = 0;
    __syncthreads();
    int32_t mine = 0;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += (int64_t)gridDim.x * 256)
        mine += par[p] == p ? 1 : 0;
    if (mine) atomicAdd(&part, mine);
    __syncthreads();
    if (threadIdx.x == 0 && part) atomicAdd(cnt, part);
}

// Edge lists with fewer edges per node than this are taken in one part.  In two
// parts and in one, FP64: a power grid of 1M nodes thinned to 1.43 edges a node
// 695 and 652 us, to 1.63 624 and 720; a 150^3 mesh thinned to 1.04 1,193 and
// 1,153, whole (2.98) 1,629 and 3,125.
constexpr double kSplitDensity = 1.6;
// Rounds on the first part (whatever is left joins the second).  With 3, 6 and
// 10: the 150^3 mesh 1,972, 1,623 and 1,603 us, the 4M-node Chung-Lu graph
// 5,303, 3,404 and 3,468; the 1M-node power grid 684, 734 and 789, the
// 400,000-point k-NN graph 774, 811 and 859.
constexpr int kRoundsFirst = 6;
// Rounds before the host first reads the list's length, and between its reads
// (1 to 8 and 1 to 6 differ by under 5% on these four graphs).
constexpr int kRoundsBlind = 4;
constexpr int kRoundsCheck = 3;

template <typename TW>
int64_t boruvka(int64_t n, int64_t m, const int32_t *u, const int32_t *v, const TW *w, const uint8_t *allowed,
                uint8_t *in_tree, DevArena &A, hipStream_t s) {
    int32_t *par = A.alloc<int32_t>(n + 1);
    uint64_t *best_w = A.alloc<uint64_t>(n + 1), *best_e = A.alloc<uint64_t>(n + 1);
    int32_t *roots[2] = {A.alloc<int32_t>(n + 1), A.alloc<int32_t>(n + 1)};
    int32_t *cnt = A.alloc<int32_t>(kCounters);
    uint64_t *pivot = A.alloc<uint64_t>(1);
    EdgeList L[2];
    for (EdgeList &l : L) {
        l.a = A.alloc<int32_t>(m + 1);
        l.b = A.alloc<int32_t>(m + 1);
        l.id = A.alloc<int32_t>(m + 1);
    }
    hipLaunchKernelGGL(k_mst_init, dim3(grid_for(n > kCounters ? n : kCounters, 256)), dim3(256), 0, s, n, par, best_w,
                       best_e, cnt);
    SFG_LAUNCH_CHECK();
    if (m > 0) fill_u8(in_tree, m, 0, s);
    const unsigned gl = (unsigned)std::min<int64_t>((m + kMstThreads - 1) / kMstThreads, kMstGrid);
    const unsigned gr = (unsigned)std::min<int64_t>((n + kMstThreads - 1) / kMstThreads, kMstGrid);
    const unsigned gm256 = std::min(grid_for(m, 256), 4u * kMstGrid), gn256 = std::min(grid_for(n, 256), 4u * kMstGrid);
    int cur = 0, rc = 0;          // the list and the root list in use
    const int32_t *rl = nullptr;  // nullptr: every node
    // one round after the compaction into L[cur]: pick, hook, flatten
    auto finish_round = [&] {
        hipLaunchKernelGGL(k_mst_pick<TW>, dim3(gm256), dim3(256), 0, s, cnt + cur, L[cur], w, best_w, best_e,
                           cnt + (1 - cur));
        SFG_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_mst_hook, dim3(gn256), dim3(256), 0, s, n, rl, cnt + kCntRoots0 + rc, L[cur], best_e, par,
                           in_tree, cnt + kCntRoots0 + (1 - rc));
        SFG_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_mst_jump, dim3(gn256), dim3(256), 0, s, n, rl, cnt + kCntRoots0 + rc, par);
        SFG_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_mst_settle, dim3(gr), dim3(kMstThreads), 0, s, n, rl, cnt + kCntRoots0 + rc, par, best_w,
                           best_e, roots[1 - rc], cnt + kCntRoots0 + (1 - rc));
        SFG_LAUNCH_CHECK();
        rc = 1 - rc;
        rl = roots[rc];
    };
    auto relist = [&](bool table) {
        if (table)
            hipLaunchKernelGGL((k_mst_list<TW, 3, true>), dim3(gl), dim3(kMstThreads), 0, s, m, u, v, w, allowed,
                               pivot, par, L[cur], cnt + cur, L[1 - cur], cnt + (1 - cur), best_w);
        else
            hipLaunchKernelGGL((k_mst_list<TW, 3, false>), dim3(gl), dim3(kMstThreads), 0, s, m, u, v, w, allowed,
                               pivot, par, L[cur], cnt + cur, L[1 - cur], cnt + (1 - cur), best_w);
        SFG_LAUNCH_CHECK();
        cur = 1 - cur;
    };
    if (m > 0) {
        int round = 0;
        if (!allowed && (double)m > kSplitDensity * (double)n) {
            hipLaunchKernelGGL(k_mst_pivot<TW>, dim3(1), dim3(1024), 0, s, m, w, n, pivot);
            SFG_LAUNCH_CHECK();
            hipLaunchKernelGGL((k_mst_list<TW, 1, false>), dim3(gl), dim3(kMstThreads), 0, s, m, u, v, w, allowed,
                               pivot, par, L[0], cnt, L[0], cnt, best_w);
            SFG_LAUNCH_CHECK();
            finish_round();
            for (round = 1; round < kRoundsFirst; ++round) {
                relist(round >= 2);
                finish_round();
            }
            // what the first part has left, then the second part's edges behind it
            relist(true);
            fill_i32(cnt + kCntRoots0 + (1 - rc), 1, 0, s);
            rc = 1 - rc;
            rl = roots[rc];
            hipLaunchKernelGGL(k_mst_flatten, dim3(gr), dim3(kMstThreads), 0, s, n, par, roots[rc],
                               cnt + kCntRoots0 + rc);
            SFG_LAUNCH_CHECK();
            hipLaunchKernelGGL((k_mst_list<TW, 2, true>), dim3(gl), dim3(kMstThreads), 0, s, m, u, v, w, allowed,
                               pivot, par, L[cur], cnt + cur, L[cur], cnt + cur, best_w);
            SFG_LAUNCH_CHECK();
        } else {
            hipLaunchKernelGGL((k_mst_list<TW, 0, false>), dim3(gl), dim3(kMstThreads), 0, s, m, u, v, w, allowed,
                               pivot, par, L[0], cnt, L[0], cnt, best_w);
            SFG_LAUNCH_CHECK();
        }
        finish_round();
        ++round;
        for (int blind = kRoundsBlind - 1;; blind = kRoundsCheck) {
            for (int j = 0; j < blind; ++j, ++round) {
                relist(round >= 2);
                finish_round();
            }
            // a round on an empty list hooks nothing, so the rounds after the last one change nothing
            relist(true);
            HostRead left(s);
            left.add(cnt + cur);
            left.wait();
            if (left.get<int32_t>(0) == 0) break;
            SFG_REQUIRE(round < 72, SFG_EHIP, "spanning_tree: too many rounds");
            finish_round();
            ++round;
        }
    }
    hipLaunchKernelGGL(k_mst_count, dim3(std::min(grid_for(n, 256), 512u)), dim3(256), 0, s, n, par, cnt + kCntComps);
    SFG_LAUNCH_CHECK();
    HostRead comps(s);
    comps.add(cnt + kCntComps);
    comps.wait();
    return comps.get<int32_t>(0);
}

// ------------------------------------------------------------------ small graphs: one workgroup
// All rounds in one launch: the edges stay in the threads' registers, the
// components in LDS.  The same choices, so the same forest.

constexpr int kSmallNodes = 8192, kSmallThreads = 1024;
constexpr int kSmallMaxItems = 32;
constexpr int64_t kSmallEdges = (int64_t)kSmallThreads * kSmallMaxItems;

template <typename TW, int ITEMS>
__global__ __launch_bounds__(kSmallThreads) void k_mst_small(int32_t n, int32_t m, const int32_t *__restrict__ u,
                                                             const int32_t *__restrict__ v, const TW *__restrict__ w,
                                                             const uint8_t *__restrict__ allowed, uint8_t *in_tree,
                                                             int32_t *comps) {
    extern __shared__ unsigned long long lds[];
    unsigned long long *bw = lds;                                     // [n] best weight
    int32_t *be = reinterpret_cast<int32_t *>(bw + n);                // [n] best edge
    int32_t *par = be + n;                                            // [n]
    __shared__ int32_t live_any, count;
    const int t = threadIdx.x;
    uint32_t ab[ITEMS];                // endpoints' components, 16 bits each
    unsigned long long k[ITEMS];
    uint32_t live = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int32_t e = i * kSmallThreads + t;
        ab[i] = 0;
        k[i] = 0;
        if (e < m) {
            in_tree[e] = 0;
            if (!allowed || allowed[e] != 0) {
                ab[i] = (uint32_t)u[e] | ((uint32_t)v[e] << 16);
                k[i] = wkey(w[e]);
                live |= 1u << i;
            }
        }
    }
    for (int32_t c = t; c < n; c += kSmallThreads) par[c] = c;
    if (t == 0) count = 0;
    // the component count at least halves while any edge is live: 13 rounds for 8192 nodes
    for (int round = 0; round < 16; ++round) {
        for (int32_t c = t; c < n; c += kSmallThreads) {
            bw[c] = 0;
            be[c] = 0x7fffffff;
        }
        if (t == 0) live_any = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (live >> i & 1u) {
                const int32_t a = par[ab[i] & 0xffffu], b = par[ab[i] >> 16];
                ab[i] = (uint32_t)a | ((uint32_t)b << 16);
                if (a == b) {
                    live &= ~(1u << i);
                } else {
                    if (k[i] > __hip_atomic_load(&bw[a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
                        atomicMax(&bw[a], k[i]);
                    if (k[i] > __hip_atomic_load(&bw[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
                        atomicMax(&bw[b], k[i]);
                }
            }
        if (live) live_any = 1;
        __syncthreads();
        if (!live_any) break;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (live >> i & 1u) {
                const int32_t a = ab[i] & 0xffffu, b = ab[i] >> 16, e = i * kSmallThreads + t;
                if (k[i] == bw[a]) atomicMin(&be[a], e);
                if (k[i] == bw[b]) atomicMin(&be[b], e);
            }
        __syncthreads();
        // hooks: the other end of a component's best edge, from its owner's registers
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (live >> i & 1u) {
                const int32_t a = ab[i] & 0xffffu, b = ab[i] >> 16, e = i * kSmallThreads + t;
                const bool ca = be[a] == e, cb = be[b] == e;
                if (ca || cb) in_tree[e] = 1;
                if (ca && cb) {
                    par[a > b ? a : b] = a > b ? b : a;
                } else if (ca) {
                    par[a] = b;
                } else if (cb) {
                    par[b] = a;
                }
            }
        __syncthreads();
        for (int jump = 0; jump < 13; ++jump) {      // 2^13 >= the longest chain
            bool moved = false;
            for (int32_t c = t; c < n; c += kSmallThreads) {
                const int32_t p = __hip_atomic_load(&par[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const int32_t g = __hip_atomic_load(&par[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (g != p) {
                    __hip_atomic_store(&par[c], g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    moved = true;
                }
            }
            if (!__syncthreads_or(moved)) break;
        }
    }
    __syncthreads();
    int32_t mine = 0;
    for (int32_t c = t; c < n; c += kSmallThreads) mine += par[c] == c ? 1 : 0;
    if (mine) atomicAdd(&count, mine);
    __syncthreads();
    if (t == 0) *comps = count;
}

template <typename TW, int ITEMS>
void launch_small(int64_t n, int64_t m, const int32_t *u, const int32_t *v, const TW *w, const uint8_t *allowed,
                  uint8_t *in_tree, int32_t *comps, hipStream_t s) {
    static std::once_flag once[kMaxDevices];
    int dev = 0;
    SFG_HIP(hipGetDevice(&dev));
    SFG_REQUIRE(dev >= 0 && dev < kMaxDevices, SFG_EUNSUPPORTED, "spanning_tree: device index over 63");
    const auto kernel = k_mst_small<TW, ITEMS>;
    std::call_once(once[dev], [&] {
        SFG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kSmallNodes * 16));
    });
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kSmallThreads), (size_t)n * 16, s, (int32_t)n, (int32_t)m, u, v, w,
                       allowed, in_tree, comps);
    SFG_LAUNCH_CHECK();
}

template <typename TW>
int64_t forest(int64_t n, int64_t m, const int32_t *u, const int32_t *v, const TW *w, const uint8_t *allowed,
               uint8_t *in_tree, DevArena &A, hipStream_t s) {
    if (n > kSmallNodes || m > kSmallEdges || m == 0) return boruvka<TW>(n, m, u, v, w, allowed, in_tree, A, s);
    int32_t *comps = A.alloc<int32_t>(1);
    if (m <= 8 * kSmallThreads) launch_small<TW, 8>(n, m, u, v, w, allowed, in_tree, comps, s);
    else launch_small<TW, kSmallMaxItems>(n, m, u, v, w, allowed, in_tree, comps, s);
    HostRead h(s);
    h.add(comps);
    h.wait();
    return h.get<int32_t>(0);
}

}  // namespace

int64_t spanning_tree_gpu(int64_t n, int64_t m, const int32_t *u, const int32_t *v, const void *w, sfg_dtype wt,
                          const uint8_t *allowed, uint8_t *in_tree, DevArena &A, hipStream_t s) {
    SFG_REQUIRE(wt == SFG_F64 || wt == SFG_F32, SFG_EINVAL, "spanning_tree: weights must be F64 or F32");
    const DevArena::Mark mark = A.mark();
    const int64_t comps = wt == SFG_F64 ? forest<double>(n, m, u, v, (const double *)w, allowed, in_tree, A, s)
                                        : forest<float>(n, m, u, v, (const float *)w, allowed, in_tree, A, s);
    A.release(mark);
    return comps;
}

}  // namespace sfg
