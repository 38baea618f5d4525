// Spanning-tree layout and exact tree-Laplacian solves.
//
// The condition-number estimate behind sigma-driven stopping (Eq. 2, and the
// sigma that Alg. 1 takes) needs solves with the sparsifier Laplacian L_P;
// they are done by conjugate gradients preconditioned with the spanning tree
// T inside P, and a tree Laplacian system is solved exactly in O(n) work.
//
// Layout (tree_order): root node 0; the Euler walk that crosses every tree
// edge once down and once up, taking at each node the neighbours in
// ascending id order starting after the one it came from.  On the device:
// tree CSR -> reverse arc by binary search -> successor of every arc -> list
// ranking (two levels of splitters, pointer jumping over the last) -> walk
// position of every arc -> down arcs scanned in walk order give the preorder.
// Per preorder position: node, parent position, subtree size, parent-edge
// weight and the walk steps that enter and leave it.
//
// Solve (tree_solve), x = L_T^+ b per column, no atomics, deterministic:
//   b is centred and gathered into preorder; the net demand below each edge
//   is a difference of two inclusive prefix sums (a subtree is a contiguous
//   preorder range); each edge's potential drop demand / w is written at its
//   down step and its negation at its up step of a walk-length array, whose
//   inclusive prefix sum at a node's down step is the node's potential
//   relative to the root (closed excursions cancel); the result is centred.
#include "common.hpp"

namespace sfg {

size_t csr_workspace_bytes(int64_t n, int64_t m);
void build_csr(int64_t n, int64_t m, const int32_t *u, const int32_t *v, const void *w, sfg_dtype wt,
               const uint8_t *mask, int32_t *rowptr, int32_t *col, void *val, int32_t *eid, void *deg, void *ws,
               size_t ws_bytes, hipStream_t s, int64_t included = 0);

namespace {

constexpr int kB = 256;
constexpr uint32_t kNil = 0xFFFFFFFFu;

// Grid-stride over a bounded grid, one atomic per workgroup: a single
// counter takes same-address atomics one at a time, so one per wave over
// millions of edges would cost milliseconds.
constexpr uint32_t kMaskBlocks = 1024;

__global__ void k_mask_eq(int64_t m, const uint8_t *__restrict__ keep, uint8_t want, uint8_t *__restrict__ out,
                          int32_t *__restrict__ count) {
    __shared__ int32_t part[kB / kWave];
    int32_t c = 0;
    for (int64_t e0 = (int64_t)blockIdx.x * blockDim.x; e0 < m; e0 += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = e0 + threadIdx.x;
        const bool in = e < m && keep[e] == want;
        if (e < m) out[e] = in ? 1 : 0;
        c += (int32_t)__popcll(__ballot(in));
    }
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t t = 0;
        for (int w = 0; w < kB / kWave; ++w) t += part[w];
        if (t) atomicAdd(count, t);
    }
}

// Successor of every arc a = (p -> q) in the walk: the arc after (q -> p) in
// row q, cyclically.  The arc entering the root last ends the list (kNil).
__device__ __forceinline__ void walk_arc(int32_t a, int32_t p, const int32_t *__restrict__ rowptr,
                                         const int32_t *__restrict__ col, int32_t *__restrict__ rev,
                                         int32_t *__restrict__ src, uint32_t *__restrict__ next) {
    const int32_t q = col[a];
    const int32_t q0 = rowptr[q], q1 = rowptr[q + 1];
    int32_t lo = q0, hi = q1;
    while (lo < hi) {   // p in row q (columns ascending)
        const int32_t mid = (lo + hi) >> 1;
        if (col[mid] < p) lo = mid + 1; else hi = mid;
    }
    // p is in row q for a symmetric CSR; the clamp only keeps a malformed
    // input's indexes inside row q
    const int32_t r = lo < q1 ? lo : q0;
    rev[a] = r;
    src[a] = p;
    int32_t nx = r + 1;
    if (nx == q1) nx = q0;
    next[a] = (q == 0 && nx == q0) ? kNil : (uint32_t)nx;
}

// A thread takes the arcs of a row of up to kArcRow.  Longer rows (the hubs of
// stars and power-law trees) are listed, a wavefront's arcs at a time, for the
// whole grid of the next launch, since each arc is a chain of dependent reads
// that one workgroup would take in turn.  Finding every arc's row by binary
// search over rowptr took 141 us for the 150^3 mesh's 6.7M arcs, this takes 71.
// With long rows left to the workgroup that holds their nodes, the layout of a
// spanning tree of the 500,000-node Chung-Lu graph (131 arcs on average in the
// first 256 rows) took 1,248 us; with the search 725, now 731.
constexpr int32_t kArcRow = 16;
constexpr int32_t kOwnPieces = 8;      // a row of more pieces is listed by its whole workgroup
constexpr uint32_t kLongArcBlocks = 512;

struct ArcPiece {
    int32_t row, first;
};

__global__ __launch_bounds__(kB) void k_walk_init(int64_t n, const int32_t *__restrict__ rowptr,
                                                  const int32_t *__restrict__ col, int32_t *__restrict__ rev,
                                                  int32_t *__restrict__ src, uint32_t *__restrict__ next,
                                                  ArcPiece *__restrict__ pieces, int32_t *__restrict__ count) {
    __shared__ int32_t row[kB], first[kB], num[kB], at[kB];
    __shared__ int32_t nrows, total, base;
    if (threadIdx.x == 0) nrows = total = 0;
    __syncthreads();
    const int64_t p = (int64_t)blockIdx.x * kB + threadIdx.x;
    int32_t j0 = 0, cnt = 0, to = 0;
    if (p < n) {
        j0 = rowptr[p];
        const int32_t len = rowptr[p + 1] - j0;
        if (len <= kArcRow) {
            for (int32_t i = 0; i < len; ++i) walk_arc(j0 + i, (int32_t)p, rowptr, col, rev, src, next);
        } else {
            cnt = (len - 1) / kWave + 1;
            to = atomicAdd(&total, cnt);
        }
    }
    __syncthreads();
    if (total == 0) return;
    if (threadIdx.x == 0) base = atomicAdd(count, total);
    __syncthreads();
    to += base;
    if (cnt <= kOwnPieces) {
        for (int32_t i = 0; i < cnt; ++i) pieces[to + i] = ArcPiece{(int32_t)p, j0 + i * kWave};
    } else {
        const int32_t s = atomicAdd(&nrows, 1);
        row[s] = (int32_t)p;
        first[s] = j0;
        num[s] = cnt;
        at[s] = to;
    }
    __syncthreads();
    const int32_t listed = nrows;
    for (int32_t s = 0; s < listed; ++s)
        for (int32_t i = threadIdx.x; i < num[s]; i += kB) pieces[at[s] + i] = ArcPiece{row[s], first[s] + i * kWave};
}

__global__ __launch_bounds__(kB) void k_walk_long(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                                                  int32_t *__restrict__ rev, int32_t *__restrict__ src,
                                                  uint32_t *__restrict__ next, const ArcPiece *__restrict__ pieces,
                                                  const int32_t *__restrict__ count) {
    const int32_t lane = threadIdx.x % kWave, cnt = *count;
    for (int64_t w = (int64_t)blockIdx.x * (kB / kWave) + threadIdx.x / kWave; w < cnt;
         w += (int64_t)gridDim.x * (kB / kWave)) {
        const ArcPiece t = pieces[w];
        if (lane < rowptr[t.row + 1] - t.first) walk_arc(t.first + lane, t.row, rowptr, col, rev, src, next);
    }
}

// ---- list ranking by splitters.  Of every kBucket consecutive elements one,
// at a hashed place, is a splitter (element 0, the list's head, is bucket
// 0's).  A thread per splitter walks to the next one: the walks' lengths make
// the next, shorter list.  Two levels leave 1/64 of the elements to pointer
// jumping; the distances then go back down by the same walks.  Every arc is
// visited twice per level instead of once per jumping round: 23 rounds took
// 1.40 ms for the 150^3 mesh's 6.7M arcs, all of this takes 0.36.
// A walk is a chain of dependent reads, 8 on average and about 8 ln(elements)
// at the longest; one that exceeds kMaxWalk (only a malformed list, or one
// made against the hash) raises `over`, and plain pointer jumping runs.
constexpr int kBucketLog = 3, kBucket = 1 << kBucketLog;
constexpr int kMaxWalk = 1024;
// Shorter lists: pointer jumping, 5 us a round.  Splitters and jumping take, in
// all of the layout, 316 and 269 us at 180,000 arcs (a grid), 325 and 313 at
// 320,000, 404 and 413 at 400,000 (a k-NN graph), 372 and 427 at 980,000.
constexpr int64_t kRankMin = int64_t(3) << 17;

__device__ __forceinline__ uint32_t splitter_at(uint32_t bucket) {   // place within the bucket
    uint32_t h = bucket * 0x9E3779B1u;
    h ^= h >> 15;
    h *= 0x85EBCA77u;
    h ^= h >> 13;
    return bucket == 0 ? 0u : h & (kBucket - 1);
}

// Splitter of bucket j of a list of len elements (the last bucket may be
// short: its splitter is then its first element).
__device__ __forceinline__ uint32_t splitter(uint32_t j, uint32_t len) {
    const uint32_t e = j * kBucket + splitter_at(j);
    return e < len ? e : j * kBucket;
}

__device__ __forceinline__ bool is_splitter(uint32_t e, uint32_t len) { return splitter(e >> kBucketLog, len) == e; }

// The shorter list: element j is splitter j; packed word: low 32 bits the
// next splitter's bucket (kNil at the end), high 32 bits the distance to it
// (to the last element at the end).  in: next words, or packed ones (LINKS).
template <bool LINKS>
__global__ __launch_bounds__(kB) void k_rank_up(uint32_t len, uint32_t buckets, const uint32_t *__restrict__ next,
                                                const uint64_t *__restrict__ link, uint64_t *__restrict__ out,
                                                int32_t *__restrict__ over) {
    const uint32_t j = blockIdx.x * kB + threadIdx.x;
    if (j >= buckets) return;
    uint32_t e = splitter(j, len), dist = 0;
    uint32_t to = kNil;
    int step = 0;
    for (; step < kMaxWalk; ++step) {
        if constexpr (LINKS) {
            const uint64_t x = link[e];
            dist += (uint32_t)(x >> 32);
            e = (uint32_t)x;
            if (e == kNil) break;
        } else {
            e = next[e];
            if (e == kNil) break;
            ++dist;
        }
        if (is_splitter(e, len)) {
            to = e >> kBucketLog;
            break;
        }
    }
    if (step == kMaxWalk) atomicOr(over, 1);
    out[j] = ((uint64_t)dist << 32) | to;
}

// Distances to the end from the splitters' (up: packed words whose high half
// is the distance) to every element of the list below.
template <bool LINKS>
__global__ __launch_bounds__(kB) void k_rank_down(uint32_t len, uint32_t buckets, const uint64_t *__restrict__ up,
                                                  const uint32_t *__restrict__ next, uint64_t *__restrict__ link,
                                                  uint32_t *__restrict__ dist_out) {
    const uint32_t j = blockIdx.x * kB + threadIdx.x;
    if (j >= buckets) return;
    uint32_t e = splitter(j, len), dist = (uint32_t)(up[j] >> 32);
    for (int step = 0; step < kMaxWalk; ++step) {
        if constexpr (LINKS) {
            const uint64_t x = link[e];
            link[e] = ((uint64_t)dist << 32) | (uint32_t)x;     // read by this walk alone
            dist -= (uint32_t)(x >> 32);
            e = (uint32_t)x;
        } else {
            dist_out[e] = dist;
            --dist;
            e = next[e];
        }
        if (e == kNil || is_splitter(e, len)) break;
    }
}

__global__ void k_rank_links(int64_t A, const uint32_t *__restrict__ next, uint64_t *__restrict__ link) {
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= A) return;
    const uint32_t nx = next[a];
    link[a] = nx == kNil ? (uint64_t)kNil : ((uint64_t)1 << 32) | nx;
}

__global__ void k_rank_dist(int64_t A, const uint64_t *__restrict__ link, uint32_t *__restrict__ dist) {
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a < A) dist[a] = (uint32_t)(link[a] >> 32);
}

// One round of pointer jumping over packed (next, distance) words.
__global__ void k_walk_jump(int64_t A, const uint64_t *__restrict__ in, uint64_t *__restrict__ out) {
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= A) return;
    const uint64_t x = in[a];
    const uint32_t nx = (uint32_t)x;
    if (nx == kNil) {
        out[a] = x;
        return;
    }
    const uint64_t y = in[nx];
    out[a] = (((x >> 32) + (y >> 32)) << 32) | (uint32_t)y;
}

// walk position of every arc, and a down flag at each walk position
__global__ void k_walk_pos(int64_t A, const uint32_t *__restrict__ dist, const int32_t *__restrict__ rev,
                           int32_t *__restrict__ pos, int32_t *__restrict__ down_at) {
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= A) return;
    const int32_t pa = (int32_t)(A - 1 - (int64_t)dist[a]);
    const int32_t pr = (int32_t)(A - 1 - (int64_t)dist[rev[a]]);
    pos[a] = pa;
    if (pa >= 0 && pa < A) down_at[pa] = pa < pr ? 1 : 0;
}

__global__ void k_tree_fill(int64_t A, const int32_t *__restrict__ pos, const int32_t *__restrict__ rev,
                            const int32_t *__restrict__ src, const int32_t *__restrict__ col,
                            const double *__restrict__ val, const int32_t *__restrict__ dbefore,
                            int32_t *__restrict__ pre_of, int32_t *__restrict__ order, int32_t *__restrict__ parnode,
                            int32_t *__restrict__ size, double *__restrict__ pw, int32_t *__restrict__ tdown,
                            int32_t *__restrict__ tup) {
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= A) return;
    const int32_t pa = pos[a], pr = pos[rev[a]];
    if (!(pa < pr)) return;   // up arc
    const int32_t q = col[a];
    const int32_t i = 1 + dbefore[pa];
    pre_of[q] = i;
    order[i] = q;
    parnode[i] = src[a];
    size[i] = (pr - pa + 1) >> 1;
    pw[i] = val[a];
    tdown[i] = pa;
    tup[i] = pr;
}

// A walk through all arcs has n - 1 down arcs, so every position 1..n-1 was
// written; if each holds another node than the root, whose position reads
// back as this one, the walk enters every node once: a spanning tree.
__global__ void k_tree_parent(int64_t n, const int32_t *__restrict__ order, const int32_t *__restrict__ pre_of,
                              const int32_t *__restrict__ parnode, int32_t *__restrict__ parent,
                              int32_t *__restrict__ bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || i == 0) return;
    const int32_t q = order[i];
    if (q <= 0 || q >= n || pre_of[q] != (int32_t)i) atomicOr(bad, 1);
    const int32_t pn = parnode[i];
    parent[i] = (pn >= 0 && pn < n) ? pre_of[pn] : -1;
}

__global__ void k_tree_root(int64_t n, int32_t *order, int32_t *parent, int32_t *size, double *pw, int32_t *tdown,
                            int32_t *tup, int32_t *pre_of) {
    order[0] = 0;
    parent[0] = -1;
    size[0] = (int32_t)n;
    pw[0] = 0.0;
    tdown[0] = -1;
    tup[0] = -1;
    pre_of[0] = 0;
}

// ------------------------------------------------------------------ FP64 block kernels (rows x k, row-major)
//
// A workgroup is kB threads laid out as G row lanes x k column lanes (G =
// kB / k); thread (g, c) owns column c of kRpt consecutive rows.

constexpr int kRpt = 16;

__device__ __forceinline__ int lanes_g(int k) { return kB / k; }

// Column sums, stage 1: per-workgroup partial sums over a strided set of rows.
__global__ __launch_bounds__(kB) void k_colsum(int64_t rows, int32_t k, const double *__restrict__ x,
                                               double *__restrict__ partial) {
    __shared__ double sh[kB];
    const int G = lanes_g(k);
    const int g = threadIdx.x / k, c = threadIdx.x % k;
    double acc = 0.0;
    if (g < G)
        for (int64_t r = (int64_t)blockIdx.x * G + g; r < rows; r += (int64_t)gridDim.x * G) acc += x[r * k + c];
    sh[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < k) {
        double t = 0.0;
        for (int gg = 0; gg < G; ++gg) t += sh[gg * k + threadIdx.x];
        partial[(int64_t)blockIdx.x * k + threadIdx.x] = t;
    }
}

// stage 2: out[c] = scale * sum of the partials, in workgroup order (sixteen
// loads in flight: 512 partials one after the other took 77 us, now 13)
__global__ void k_colsum_finish(int32_t nb, int32_t k, const double *__restrict__ partial, double scale,
                                double *__restrict__ out) {
    const int c = threadIdx.x;
    if (c >= k) return;
    double t = 0.0;
#pragma unroll 16
    for (int b = 0; b < nb; ++b) t += partial[(int64_t)b * k + c];
    out[c] = t * scale;
}

// per-column dot products, stage 1 (stage 2 is k_colsum_finish)
__global__ __launch_bounds__(kB) void k_coldot(int64_t rows, int32_t k, const double *__restrict__ x,
                                               const double *__restrict__ y, double *__restrict__ partial) {
    __shared__ double sh[kB];
    const int G = lanes_g(k);
    const int g = threadIdx.x / k, c = threadIdx.x % k;
    double acc = 0.0;
    if (g < G)
        for (int64_t r = (int64_t)blockIdx.x * G + g; r < rows; r += (int64_t)gridDim.x * G)
            acc += x[r * k + c] * y[r * k + c];
    sh[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < k) {
        double t = 0.0;
        for (int gg = 0; gg < G; ++gg) t += sh[gg * k + threadIdx.x];
        partial[(int64_t)blockIdx.x * k + threadIdx.x] = t;
    }
}

// k x k Gram block X^T Y, stage 1: thread t owns entries t, t + kB, ... of
// the k*k matrix over one of L = max(1, kB / k^2) row lanes
__global__ __launch_bounds__(kB) void k_gram(int64_t rows, int32_t k, const double *__restrict__ x,
                                             const double *__restrict__ y, double *__restrict__ partial) {
    __shared__ double sh[kB * 4];
    const int P = k * k;
    const int L = P >= kB ? 1 : kB / P;
    const int lane = P >= kB ? 0 : threadIdx.x / P;
    const int e0 = P >= kB ? threadIdx.x : threadIdx.x % P;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (lane < L)
        for (int64_t r = (int64_t)blockIdx.x * L + lane; r < rows; r += (int64_t)gridDim.x * L) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = e0 + q * kB;
                if (e < P && (q == 0 || P >= kB)) acc[q] += x[r * k + e / k] * y[r * k + e % k];
            }
        }
#pragma unroll
    for (int q = 0; q < 4; ++q) sh[q * kB + threadIdx.x] = acc[q];
    __syncthreads();
    for (int e = threadIdx.x; e < P; e += kB) {
        double t = 0.0;
        if (P >= kB) {
            t = sh[(e / kB) * kB + (e % kB)];
        } else {
            for (int l = 0; l < L; ++l) t += sh[l * P + e];
        }
        partial[(int64_t)blockIdx.x * P + e] = t;
    }
}

__global__ void k_gram_finish(int32_t nb, int32_t P, const double *__restrict__ partial, double *__restrict__ out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= P) return;
    double t = 0.0;
#pragma unroll 16
    for (int b = 0; b < nb; ++b) t += partial[(int64_t)b * P + e];
    out[e] = t;
}

// per-tile column totals of a rows x k block (tile = G * kRpt rows)
__global__ __launch_bounds__(kB) void k_scan_tiles(int64_t rows, int32_t k, const double *__restrict__ x,
                                                   double *__restrict__ tile_sum) {
    __shared__ double sh[kB];
    const int G = lanes_g(k);
    const int g = threadIdx.x / k, c = threadIdx.x % k;
    const int64_t base = (int64_t)blockIdx.x * G * kRpt + (int64_t)g * kRpt;
    double acc = 0.0;
    if (g < G)
        for (int r = 0; r < kRpt; ++r)
            if (base + r < rows) acc += x[(base + r) * k + c];
    sh[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < k) {
        double t = 0.0;
        for (int gg = 0; gg < G; ++gg) t += sh[gg * k + threadIdx.x];
        tile_sum[(int64_t)blockIdx.x * k + threadIdx.x] = t;
    }
}

// Exclusive scan of the tile totals in two levels.  k_scan_mid: a workgroup
// takes a group of G * kTpl tiles (lane (g, c): kTpl consecutive tiles of
// column c), replaces each tile total by its exclusive offset inside the
// group and writes the group total.  k_scan_top (one workgroup): exclusive
// offsets of the group totals, and the column totals after them.
constexpr int kTpl = 8;

__device__ __forceinline__ int64_t tiles_per_group(int k) { return (int64_t)lanes_g(k) * kTpl; }

__global__ __launch_bounds__(kB) void k_scan_mid(int64_t tiles, int32_t k, double *__restrict__ tile_sum,
                                                 double *__restrict__ group_sum) {
    __shared__ double sh[kB];
    const int G = lanes_g(k);
    const int g = threadIdx.x / k, c = threadIdx.x % k;
    const int64_t t0 = (int64_t)blockIdx.x * G * kTpl + (int64_t)g * kTpl;
    double v[kTpl];
    double acc = 0.0;
#pragma unroll
    for (int q = 0; q < kTpl; ++q) {
        v[q] = (g < G && t0 + q < tiles) ? tile_sum[(t0 + q) * k + c] : 0.0;
        acc += v[q];
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    if (g >= G) return;
    double off = 0.0;
    for (int gg = 0; gg < g; ++gg) off += sh[gg * k + c];
#pragma unroll
    for (int q = 0; q < kTpl; ++q) {
        if (t0 + q < tiles) tile_sum[(t0 + q) * k + c] = off;
        off += v[q];
    }
    if (g == G - 1) group_sum[(int64_t)blockIdx.x * k + c] = off;
}

__global__ __launch_bounds__(kB) void k_scan_top(int64_t groups, int32_t k, double *__restrict__ group_sum) {
    __shared__ double sh[kB];
    const int G = lanes_g(k);
    const int g = threadIdx.x / k, c = threadIdx.x % k;
    const int64_t chunk = (groups + G - 1) / G;
    const int64_t t0 = (int64_t)g * chunk, t1 = t0 + chunk < groups ? t0 + chunk : groups;
    double acc = 0.0;
    if (g < G)
        for (int64_t t = t0; t < t1; ++t) acc += group_sum[t * k + c];
    sh[threadIdx.x] = acc;
    __syncthreads();
    if (g >= G) return;
    double off = 0.0;
    for (int gg = 0; gg < g; ++gg) off += sh[gg * k + c];
    for (int64_t t = t0; t < t1; ++t) {
        const double x = group_sum[t * k + c];
        group_sum[t * k + c] = off;
        off += x;
    }
    if (g == 0) {   // column totals after the offsets
        double tot = 0.0;
        for (int gg = 0; gg < G; ++gg) tot += sh[gg * k + c];
        group_sum[groups * k + c] = tot;
    }
}

// inclusive prefix sums over rows: tile offset + lane offset + running sum
__global__ __launch_bounds__(kB) void k_scan_apply(int64_t rows, int32_t k, const double *__restrict__ x,
                                                   const double *__restrict__ tile_off,
                                                   const double *__restrict__ group_off, double *__restrict__ y) {
    __shared__ double sh[kB];
    const int G = lanes_g(k);
    const int g = threadIdx.x / k, c = threadIdx.x % k;
    const int64_t base = (int64_t)blockIdx.x * G * kRpt + (int64_t)g * kRpt;
    double v[kRpt];
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < kRpt; ++r) {
        v[r] = (g < G && base + r < rows) ? x[(base + r) * k + c] : 0.0;
        acc += v[r];
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    if (g >= G) return;
    double run = group_off[((int64_t)blockIdx.x / tiles_per_group(k)) * k + c] + tile_off[(int64_t)blockIdx.x * k + c];
    for (int gg = 0; gg < g; ++gg) run += sh[gg * k + c];
#pragma unroll
    for (int r = 0; r < kRpt; ++r) {
        run += v[r];
        if (base + r < rows) y[(base + r) * k + c] = run;
    }
}

// centred gather into preorder: bp[i] = b[order[i]] - mean
__global__ void k_gather_centre(int64_t n, int32_t k, const int32_t *__restrict__ order,
                                const double *__restrict__ b, const double *__restrict__ mean,
                                double *__restrict__ bp) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * k) return;
    const int64_t i = t / k;
    const int c = (int)(t - i * k);
    bp[t] = b[(int64_t)order[i] * k + c] - mean[c];
}

// potential drop of every parent edge, written at its down step and negated
// at its up step of the walk-length array
__global__ void k_edge_drop(int64_t n, int32_t k, const int32_t *__restrict__ size, const double *__restrict__ pw,
                            const int32_t *__restrict__ tdown, const int32_t *__restrict__ tup,
                            const double *__restrict__ S, double *__restrict__ walk) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * k || t < k) return;   // the root has no parent edge
    const int64_t i = t / k;
    const int c = (int)(t - i * k);
    const double hi = S[(i + size[i] - 1) * k + c];
    const double lo = S[(i - 1) * k + c];
    const double d = (hi - lo) / pw[i];
    walk[(int64_t)tdown[i] * k + c] = d;
    walk[(int64_t)tup[i] * k + c] = -d;
}

// potentials in preorder: xp[i] = prefix of the walk array at i's down step
__global__ void k_potential(int64_t n, int32_t k, const int32_t *__restrict__ tdown, const double *__restrict__ U,
                            double *__restrict__ xp) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * k) return;
    const int64_t i = t / k;
    const int c = (int)(t - i * k);
    xp[t] = i == 0 ? 0.0 : U[(int64_t)tdown[i] * k + c];
}

// centred scatter back to node order: x[order[i]] = xp[i] - mean
__global__ void k_scatter_centre(int64_t n, int32_t k, const int32_t *__restrict__ order,
                                 const double *__restrict__ xp, const double *__restrict__ mean,
                                 double *__restrict__ x) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * k) return;
    const int64_t i = t / k;
    const int c = (int)(t - i * k);
    x[(int64_t)order[i] * k + c] = xp[t] - mean[c];
}

// out[c] = sum of nb partials of column c: one workgroup of 1024 threads,
// lane (g, c) adds partials g, g + G, ... into four accumulators (loads in
// flight), then a fixed pairwise tree over the lanes
constexpr int kFinish = 1024;

__global__ __launch_bounds__(kFinish) void k_partials_finish(int32_t nb, int32_t k, const double *__restrict__ partial,
                                                             double *__restrict__ out) {
    __shared__ double sh[kFinish];
    const int G = kFinish / k;
    const int g = threadIdx.x / k, c = threadIdx.x % k;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    if (g < G) {
        int b = g;
        for (; b + 3 * G < nb; b += 4 * G) {
            a0 += partial[(int64_t)b * k + c];
            a1 += partial[(int64_t)(b + G) * k + c];
            a2 += partial[(int64_t)(b + 2 * G) * k + c];
            a3 += partial[(int64_t)(b + 3 * G) * k + c];
        }
        for (; b < nb; b += G) a0 += partial[(int64_t)b * k + c];
    }
    sh[threadIdx.x] = (a0 + a1) + (a2 + a3);
    __syncthreads();
    for (int st = 1; st < G; st <<= 1) {
        if (g < G && (g % (2 * st)) == 0 && g + st < G) sh[g * k + c] += sh[(g + st) * k + c];
        __syncthreads();
    }
    if ((int)threadIdx.x < k) out[threadIdx.x] = sh[threadIdx.x];
}

constexpr int kSumBlocks = 512;

int64_t scan_tiles(int64_t rows, int32_t k) {
    const int64_t tr = (int64_t)(kB / k) * kRpt;
    return (rows + tr - 1) / tr;
}

}  // namespace

// ------------------------------------------------------------------ block helpers shared by the estimate

size_t colsum_scratch_doubles(int32_t k) { return (size_t)kSumBlocks * k + 64; }

// out[c] = scale * sum_r x[r][c]; deterministic (fixed partition and order)
void block_colsum(int64_t rows, int32_t k, const double *x, double scale, double *out, double *scratch,
                  hipStream_t s) {
    int64_t nb = (rows * k + kB - 1) / kB;
    nb = nb < 1 ? 1 : (nb > kSumBlocks ? kSumBlocks : nb);
    hipLaunchKernelGGL(k_colsum, dim3((uint32_t)nb), dim3(kB), 0, s, rows, k, x, scratch);
    SFG_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_colsum_finish, dim3(1), dim3(64), 0, s, (int32_t)nb, k, scratch, scale, out);
    SFG_LAUNCH_CHECK();
}

// out[c] = sum_r x[r][c] * y[r][c]; deterministic
void block_dot(int64_t rows, int32_t k, const double *x, const double *y, double *out, double *scratch,
               hipStream_t s) {
    int64_t nb = (rows * k + kB - 1) / kB;
    nb = nb < 1 ? 1 : (nb > kSumBlocks ? kSumBlocks : nb);
    hipLaunchKernelGGL(k_coldot, dim3((uint32_t)nb), dim3(kB), 0, s, rows, k, x, y, scratch);
    SFG_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_colsum_finish, dim3(1), dim3(64), 0, s, (int32_t)nb, k, scratch, 1.0, out);
    SFG_LAUNCH_CHECK();
}

constexpr int kGramBlocks = 256;

size_t gram_scratch_doubles(int32_t k) { return (size_t)kGramBlocks * k * k + 64; }

// out (k x k, row-major) = X^T Y for rows x k blocks X, Y; k <= 32; deterministic
void block_gram(int64_t rows, int32_t k, const double *x, const double *y, double *out, double *scratch,
                hipStream_t s) {
    SFG_REQUIRE(k >= 1 && k <= 32, SFG_EINVAL, "gram: k must be in 1..32");
    const int P = k * k;
    const int L = P >= kB ? 1 : kB / P;
    int64_t nb = (rows + L - 1) / L;
    nb = nb < 1 ? 1 : (nb > kGramBlocks ? kGramBlocks : nb);
    hipLaunchKernelGGL(k_gram, dim3((uint32_t)nb), dim3(kB), 0, s, rows, k, x, y, scratch);
    SFG_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_gram_finish, dim3(grid_for(P, kB)), dim3(kB), 0, s, (int32_t)nb, P, scratch, out);
    SFG_LAUNCH_CHECK();
}

int64_t scan_groups(int64_t rows, int32_t k) {
    const int64_t tpg = (int64_t)(kB / k) * kTpl;
    return (scan_tiles(rows, k) + tpg - 1) / tpg;
}

// scratch: tile totals/offsets, then group totals/offsets and the column totals
size_t scan_scratch_doubles(int64_t rows, int32_t k) {
    return (size_t)(scan_tiles(rows, k) + scan_groups(rows, k) + 1) * k + 64;
}

// inclusive prefix sums down the rows of a rows x k block; y must not alias x
void block_scan(int64_t rows, int32_t k, const double *x, double *y, double *scratch, hipStream_t s) {
    if (rows <= 0) return;
    const int64_t tiles = scan_tiles(rows, k);
    hipLaunchKernelGGL(k_scan_tiles, dim3((uint32_t)tiles), dim3(kB), 0, s, rows, k, x, scratch);
    SFG_LAUNCH_CHECK();
    const int64_t groups = scan_groups(rows, k);
    double *gsum = scratch + (size_t)tiles * k;
    hipLaunchKernelGGL(k_scan_mid, dim3((uint32_t)groups), dim3(kB), 0, s, tiles, k, scratch, gsum);
    SFG_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kB), 0, s, groups, k, gsum);
    SFG_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_scan_apply, dim3((uint32_t)tiles), dim3(kB), 0, s, rows, k, x, scratch, gsum, y);
    SFG_LAUNCH_CHECK();
}

// Grid of a row-lane kernel over `rows` rows (at most kLaneBlocks workgroups).
constexpr int kLaneBlocks = 4096;

uint32_t lane_grid(int64_t rows, int32_t k) {
    const int64_t G = kB / k;
    int64_t nb = (rows + G - 1) / G;
    return (uint32_t)(nb < 1 ? 1 : (nb > kLaneBlocks ? kLaneBlocks : nb));
}

void finish_partials(int32_t nb, int32_t k, const double *partial, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_partials_finish, dim3(1), dim3(kFinish), 0, s, nb, k, partial, out);
    SFG_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ the preconditioner inside the conjugate gradients
//
// z = L_T^+ r up to a constant per column, for blocks in the tree's preorder
// (row i is node order[i]; constants are in the kernel of every Laplacian, so
// they change neither the iterates' residuals nor r . z for r orthogonal to
// the all-one vector).  Four launches after the kernel that updates r, which
// leaves r's tile sums: prefix sums S of r; the walk's potential drops, each
// step gathering its edge's two entries of S, with their tile sums; prefix
// sums along the walk, written at the steps that enter a node as z; r . z.
// All of them read a few MB, and an iteration is bound by the launches' own
// latency, so a launch's small sums are added up by the workgroups of the
// next one.  Conjugate gradients stopped at a loose tolerance carry the
// rounding of every sum into their result, so each sum that enters an iterate
// keeps the order that block_scan and k_partials_finish give it, whatever launch
// it is in; r . r, which only says when a column has converged, is added up
// tile by tile.
// On the 300 x 300 power grid (90,000 nodes, 8 columns) an iteration takes
// 73 us in seven launches; it took 98 us in sixteen.  (More launches: two for the
// offsets of each prefix sum over kDirectGroups groups of tiles, one for r . z
// beyond kDotPerLane, one for p . Ap beyond kPapRows, and the convergence test's
// where there is one.)

namespace {

constexpr int kT = 1024;               // threads of the kernels below: four per thread of block_scan's
constexpr int kTE = 4;                 // elements of a tile per thread
constexpr int kTileLds = kB * (kRpt + 1);

// e / k for e < 4352 and k <= 32 (error e / 2^18 < 1 / k): an integer division
// is some thirty instructions, and these kernels would need a dozen each.
struct ByK {
    int32_t k;
    uint32_t m;
    explicit ByK(int32_t k_) : k(k_), m((1u << 18) / (uint32_t)k_ + 1) {}
    __device__ __forceinline__ int div(int e) const { return (int)(((uint32_t)e * m) >> 18); }
    __device__ __forceinline__ int mod(int e) const { return e - div(e) * k; }
};

// A tile in LDS: element e = row * k + column, with a gap of k after every
// kRpt rows, so that the threads that add kRpt rows each hit different banks.
__device__ __forceinline__ int tile_lds(int e, const ByK &by) { return e + (by.div(e) / kRpt) * by.k; }

// Partial sums of k columns ([rows][k]) added in the order of
// k_partials_finish by a workgroup of kT threads; sh[c] = sum, c < k.
__device__ __forceinline__ void finish_rows(const double *__restrict__ partial, int32_t nb, const ByK &by, double *sh) {
    const int k = by.k, G = by.div(kFinish);
    const int g = by.div(threadIdx.x), c = by.mod(threadIdx.x);
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    if (g < G) {
        int b = g;
        for (; b + 3 * G < nb; b += 4 * G) {
            a0 += partial[(int64_t)b * k + c];
            a1 += partial[(int64_t)(b + G) * k + c];
            a2 += partial[(int64_t)(b + 2 * G) * k + c];
            a3 += partial[(int64_t)(b + 3 * G) * k + c];
        }
        for (; b < nb; b += G) a0 += partial[(int64_t)b * k + c];
    }
    sh[threadIdx.x] = (a0 + a1) + (a2 + a3);
    __syncthreads();
    for (int st = 1; st < G; st <<= 1) {
        if (g < G && (g & (2 * st - 1)) == 0 && g + st < G) sh[g * k + c] += sh[(g + st) * k + c];
        __syncthreads();
    }
}

// sh[0] + sh[k] + ... (rows terms), added in that order from 0 with eight
// reads in flight: one read after the other is 32 LDS latencies.
__device__ __forceinline__ double sum_lds(const double *sh, int rows, int k) {
    double t = 0.0;
#pragma unroll 8
    for (int i = 0; i < rows; ++i) t += sh[i * k];
    return t;
}

// Column sums of a tile in LDS in the order of k_scan_tiles; SQ: of the squares as well.
template <bool SQ>
__device__ __forceinline__ void tile_totals(const double *tile, const ByK &by, double *sh, double *__restrict__ out,
                                            double *__restrict__ out_sq) {
    const int k = by.k, G = by.div(kB);
    const int g = by.div(threadIdx.x), c = by.mod(threadIdx.x);
    const bool lane = threadIdx.x < kB && g < G;
    double acc = 0.0, sq = 0.0;
    if (lane)
        for (int r = 0; r < kRpt; ++r) {
            const double v = tile[(g * (kRpt + 1) + r) * k + c];
            acc += v;
            sq += v * v;
        }
    if (threadIdx.x < kB) {
        sh[threadIdx.x] = acc;
        sh[kB + threadIdx.x] = sq;
    }
    __syncthreads();
    const int h = threadIdx.x / 64, t = threadIdx.x % 64;
    if (h < (SQ ? 2 : 1) && t < k) {
        (h ? out_sq : out)[(int64_t)blockIdx.x * k + t] = sum_lds(sh + h * kB + t, G, k);
    }
}

// off[c] = the sum before this workgroup's tile.  Direct form: from the tile
// sums, at most four groups of tiles, one to a quarter of the workgroup, in
// the order of k_scan_mid and k_scan_top; tot[c] then gets the sum of all
// tiles up to this workgroup's group.  Else from those kernels' offsets.
__device__ __forceinline__ void tile_offset(int64_t tiles, const double *__restrict__ tile_sum,
                                            const double *__restrict__ group_off, const ByK &by, double *sh,
                                            double *off, double *tot) {
    const int k = by.k, G = by.div(kB);
    const int64_t b = blockIdx.x, tpg = (int64_t)G * kTpl;
    if (group_off) {
        const int64_t groups = (tiles + tpg - 1) / tpg;
        if ((int)threadIdx.x < k) {
            off[threadIdx.x] = group_off[(b / tpg) * k + threadIdx.x] + tile_sum[b * k + threadIdx.x];
            tot[threadIdx.x] = group_off[groups * k + threadIdx.x];
        }
        __syncthreads();
        return;
    }
    const int quarter = threadIdx.x / kB, lt = threadIdx.x % kB;
    const int g = by.div(lt), c = by.mod(lt);
    const int64_t t0 = ((int64_t)quarter * G + g) * kTpl;
    const int64_t mine = b / kTpl - (int64_t)quarter * G;          // lane of this tile, if in this quarter's group
    const int qb = (int)(b / tpg);
    double v[kTpl];
    double acc = 0.0;
#pragma unroll
    for (int q = 0; q < kTpl; ++q) {
        v[q] = (g < G && quarter <= qb && t0 + q < tiles) ? tile_sum[(t0 + q) * k + c] : 0.0;
        acc += v[q];
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    if (g == G - 1 || (g < G && g == mine)) {
        double run = sum_lds(sh + quarter * kB + c, g, k);
        double at = 0.0;
#pragma unroll
        for (int q = 0; q < kTpl; ++q) {
            if (q == (int)(b % kTpl)) at = run;
            run += v[q];
        }
        if (g == mine) off[c] = at;
        if (g == G - 1) tot[quarter * k + c] = run;
    }
    __syncthreads();
    if ((int)threadIdx.x < k) {
        double base = 0.0;
        for (int q = 0; q < qb; ++q) base += tot[q * k + threadIdx.x];
        off[threadIdx.x] = base + off[threadIdx.x];
        tot[threadIdx.x] = base + tot[qb * k + threadIdx.x];
    }
    __syncthreads();
}

// Inclusive prefix sums down a tile in LDS, in place, in the order of
// k_scan_apply; sh: kB doubles.
__device__ __forceinline__ void tile_prefix(double *tile, const ByK &by, const double *off, double *sh) {
    const int k = by.k, G = by.div(kB);
    const int g = by.div(threadIdx.x), c = by.mod(threadIdx.x);
    const bool lane = threadIdx.x < kB && g < G;
    double v[kRpt];
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < kRpt; ++r) {
        v[r] = lane ? tile[(g * (kRpt + 1) + r) * k + c] : 0.0;
        acc += v[r];
    }
    if (threadIdx.x < kB) sh[threadIdx.x] = acc;
    __syncthreads();
    if (lane) {
        double run = off[c];
        for (int gg = 0; gg < g; ++gg) run += sh[gg * k + c];
#pragma unroll
        for (int r = 0; r < kRpt; ++r) {
            run += v[r];
            tile[(g * (kRpt + 1) + r) * k + c] = run;
        }
    }
    __syncthreads();
}

__global__ void k_step_nodes(int64_t n, const int32_t *__restrict__ tdown, const int32_t *__restrict__ tup,
                             int32_t *__restrict__ step) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || i == 0) return;
    step[tdown[i]] = (int32_t)i;
    step[tup[i]] = ~(int32_t)i;
}

// The conjugate-gradient update x += alpha p, r -= alpha Ap (alpha_c = rz_c /
// pAp_c on active columns) with the tile sums of r and of r . r.  pap_rows:
// rows of partial sums of p . Ap, or 0: they are added up.  UPDATE = false:
// the tile sums of r alone.
template <bool UPDATE>
__global__ __launch_bounds__(kT) void k_cg_step(int64_t n, ByK by, uint32_t active,
                                                const uint32_t *__restrict__ dmask, const double *__restrict__ rz,
                                                const double *__restrict__ pap, int32_t pap_rows,
                                                const double *__restrict__ p, const double *__restrict__ ap,
                                                double *__restrict__ x, double *__restrict__ r,
                                                double *__restrict__ rr, double *__restrict__ tile_sum) {
    __shared__ double tile[kTileLds], sh[kT], alpha[32];
    const int k = by.k, E = by.div(kB) * kRpt * k;
    const int64_t t0 = (int64_t)blockIdx.x * E, nk = n * k;
    double rv[kTE], xv[kTE], pv[kTE], av[kTE];
#pragma unroll
    for (int q = 0; q < kTE; ++q) {
        const int e = (int)threadIdx.x + q * kT;
        const bool in = e < E && t0 + e < nk;
        rv[q] = in ? r[t0 + e] : 0.0;
        if constexpr (UPDATE) {
            xv[q] = in ? x[t0 + e] : 0.0;
            pv[q] = in ? p[t0 + e] : 0.0;
            av[q] = in ? ap[t0 + e] : 0.0;
        }
    }
    if constexpr (UPDATE) {
        if (pap_rows) {
            finish_rows(pap, pap_rows, by, sh);
        } else {
            if ((int)threadIdx.x < k) sh[threadIdx.x] = pap[threadIdx.x];
            __syncthreads();
        }
        if ((int)threadIdx.x < k) {
            const double d = sh[threadIdx.x];
            alpha[threadIdx.x] = d != 0.0 ? rz[threadIdx.x] / d : 0.0;
        }
        __syncthreads();
        const uint32_t act = dmask ? *dmask : active;
#pragma unroll
        for (int q = 0; q < kTE; ++q) {
            const int e = (int)threadIdx.x + q * kT;
            if (e >= E || t0 + e >= nk) continue;
            const int c = by.mod(e);
            if (!((act >> c) & 1u)) continue;
            const double a = alpha[c];
            xv[q] += a * pv[q];
            rv[q] -= a * av[q];
            x[t0 + e] = xv[q];
            r[t0 + e] = rv[q];
        }
    }
#pragma unroll
    for (int q = 0; q < kTE; ++q) {
        const int e = (int)threadIdx.x + q * kT;
        if (e < E) tile[tile_lds(e, by)] = rv[q];
    }
    __syncthreads();
    tile_totals<UPDATE>(tile, by, sh, tile_sum, rr);
}

// S = inclusive prefix sums of r down the rows; the last tile leaves the column totals.
__global__ __launch_bounds__(kT) void k_rows_prefix(int64_t n, ByK by, const double *__restrict__ r,
                                                    const double *__restrict__ tile_sum,
                                                    const double *__restrict__ group_off, double *__restrict__ S,
                                                    double *__restrict__ totals) {
    __shared__ double tile[kTileLds], sh[kT], off[32], tot[4 * 32];
    const int k = by.k, E = by.div(kB) * kRpt * k;
    const int64_t t0 = (int64_t)blockIdx.x * E, nk = n * k;
#pragma unroll
    for (int q = 0; q < kTE; ++q) {
        const int e = (int)threadIdx.x + q * kT;
        if (e < E) tile[tile_lds(e, by)] = t0 + e < nk ? r[t0 + e] : 0.0;
    }
    tile_offset(gridDim.x, tile_sum, group_off, by, sh, off, tot);
    if (blockIdx.x + 1 == gridDim.x && (int)threadIdx.x < k) totals[threadIdx.x] = tot[threadIdx.x];
    tile_prefix(tile, by, off, sh);
#pragma unroll
    for (int q = 0; q < kTE; ++q) {
        const int e = (int)threadIdx.x + q * kT;
        if (e < E && t0 + e < nk) S[t0 + e] = tile[tile_lds(e, by)];
    }
}

// The walk's potential drops: the step entering node i takes its parent edge's
// drop (net demand below the edge over its weight), the step leaving it the
// negative.  The demand's column mean comes off through the totals.
__global__ __launch_bounds__(kT) void k_walk_drops(int64_t n, int64_t A, ByK by, const int32_t *__restrict__ step,
                                                   const int32_t *__restrict__ size, const double *__restrict__ pw,
                                                   const double *__restrict__ S, const double *__restrict__ totals,
                                                   double *__restrict__ walk, double *__restrict__ tile_sum) {
    __shared__ double tile[kTileLds], sh[kT], mean[32];
    const int k = by.k, E = by.div(kB) * kRpt * k;
    if ((int)threadIdx.x < k) mean[threadIdx.x] = totals[threadIdx.x] / (double)n;
    const int64_t t0 = (int64_t)blockIdx.x * E, ak = A * k, row0 = (int64_t)blockIdx.x * by.div(kB) * kRpt;
    int32_t nd[kTE], sz[kTE];
    double w[kTE], lo[kTE], hi[kTE];
#pragma unroll
    for (int q = 0; q < kTE; ++q) {
        const int e = (int)threadIdx.x + q * kT;
        nd[q] = e < E && t0 + e < ak ? step[row0 + by.div(e)] : 1;      // node 1 exists wherever the walk has a step
    }
#pragma unroll
    for (int q = 0; q < kTE; ++q) {
        const int64_t i = nd[q] >= 0 ? nd[q] : ~nd[q];
        sz[q] = size[i];
        w[q] = pw[i];
    }
#pragma unroll
    for (int q = 0; q < kTE; ++q) {
        const int64_t i = nd[q] >= 0 ? nd[q] : ~nd[q];
        const int c = by.mod((int)threadIdx.x + q * kT);
        hi[q] = S[(i + sz[q] - 1) * k + c];
        lo[q] = S[(i - 1) * k + c];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kTE; ++q) {
        const int e = (int)threadIdx.x + q * kT;
        const double f = (hi[q] - lo[q]) - (double)sz[q] * mean[by.mod(e)];
        const double d = f / w[q];
        const bool in = e < E && t0 + e < ak;
        const double y = in ? (nd[q] >= 0 ? d : -d) : 0.0;
        if (in) walk[t0 + e] = y;
        if (e < E) tile[tile_lds(e, by)] = y;
    }
    __syncthreads();
    tile_totals<false>(tile, by, sh, tile_sum, nullptr);
}

// z at the nodes the walk enters: the prefix sum of the drops (the root's is 0).
__global__ __launch_bounds__(kT) void k_walk_prefix(int64_t A, ByK by, const double *__restrict__ walk,
                                                    const int32_t *__restrict__ step,
                                                    const double *__restrict__ tile_sum,
                                                    const double *__restrict__ group_off, double *__restrict__ z) {
    __shared__ double tile[kTileLds], sh[kT], off[32], tot[4 * 32];
    const int k = by.k, E = by.div(kB) * kRpt * k;
    const int64_t t0 = (int64_t)blockIdx.x * E, ak = A * k, row0 = (int64_t)blockIdx.x * by.div(kB) * kRpt;
    int32_t nd[kTE];
#pragma unroll
    for (int q = 0; q < kTE; ++q) {
        const int e = (int)threadIdx.x + q * kT;
        const bool in = e < E && t0 + e < ak;
        nd[q] = in ? step[row0 + by.div(e)] : -1;
        if (e < E) tile[tile_lds(e, by)] = in ? walk[t0 + e] : 0.0;
    }
    tile_offset(gridDim.x, tile_sum, group_off, by, sh, off, tot);
    tile_prefix(tile, by, off, sh);
#pragma unroll
    for (int q = 0; q < kTE; ++q) {
        const int e = (int)threadIdx.x + q * kT;
        if (nd[q] >= 0) z[(int64_t)nd[q] * k + by.mod(e)] = tile[tile_lds(e, by)];
    }
    if (blockIdx.x == 0 && (int)threadIdx.x < k) z[threadIdx.x] = 0.0;
}

// r . z over nb groups of rows (group b: rows b * G + g, then every nb * G
// further), as far as lane blockIdx.x of k_partials_finish adds them: groups
// blockIdx.x, + L, ... for L = kFinish / k lanes.  lane_sum: [lanes][k].
constexpr int kDotGroups = 24;         // groups in LDS at a time: 48 KB

__global__ __launch_bounds__(kT) void k_dot_lanes(int64_t n, ByK by, int32_t nb, const double *__restrict__ r,
                                                  const double *__restrict__ z, double *__restrict__ lane_sum) {
    __shared__ double prod[kDotGroups * kB], part[kDotGroups * 32];
    const int k = by.k, G = by.div(kB), L = by.div(kFinish);
    const int quarter = threadIdx.x / kB, lt = threadIdx.x % kB;
    const int32_t cnt = (nb - (int32_t)blockIdx.x + L - 1) / L;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int32_t i0 = 0; i0 < cnt; i0 += kDotGroups) {
        const int here = cnt - i0 < kDotGroups ? cnt - i0 : kDotGroups;
#pragma unroll
        for (int q = 0; q < kDotGroups / 4; ++q) {
            const int i = quarter + 4 * q;
            const int64_t b = blockIdx.x + (int64_t)(i0 + i) * L;
            double acc = 0.0;
            if (i < here && lt < G * k)
                for (int64_t t = b * G * k + lt; t < n * k; t += (int64_t)nb * G * k) acc += r[t] * z[t];
            prod[i * kB + lt] = acc;
        }
        __syncthreads();
        if ((int)threadIdx.x < here * k) {
            const int i = by.div(threadIdx.x), c = by.mod(threadIdx.x);
            part[threadIdx.x] = sum_lds(prod + i * kB + c, G, k);
        }
        __syncthreads();
        if ((int)threadIdx.x < k)
            for (int i = 0; i < here; ++i) {
                const int at = i0 + i, q = at < cnt / 4 * 4 ? at % 4 : 0;
                const double v = part[i * k + threadIdx.x];
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    if (w == q) a[w] += v;
            }
    }
    if ((int)threadIdx.x < k) lane_sum[(int64_t)blockIdx.x * k + threadIdx.x] = (a[0] + a[1]) + (a[2] + a[3]);
}

// r . z, per-workgroup partial sums (finished by k_partials_finish)
__global__ __launch_bounds__(kB) void k_dot_partials(int64_t n, ByK by, const double *__restrict__ r,
                                                     const double *__restrict__ z, double *__restrict__ partial) {
    __shared__ double sh[kB];
    const int k = by.k, G = by.div(kB);
    double acc = 0.0;
    if ((int)threadIdx.x < G * k)
        for (int64_t t = (int64_t)blockIdx.x * G * k + threadIdx.x; t < n * k; t += (int64_t)gridDim.x * G * k)
            acc += r[t] * z[t];
    sh[threadIdx.x] = acc;
    __syncthreads();
    if ((int)threadIdx.x < k) partial[(int64_t)blockIdx.x * k + threadIdx.x] = sum_lds(sh + threadIdx.x, G, k);
}

// k_dot_lanes has kFinish / k workgroups.  It saves a launch, and loses more
// than that where each has many elements: r . z over 380,000 rows of 8 takes
// 16 us (20 in two launches), over 552,000 of 32, on 32 workgroups, 292 (66).
constexpr int64_t kDotPerLane = 32768;

// Four groups of tiles are added up by the kernels that need the offsets (8
// columns: 524,000 rows, at most 64 KB read per workgroup); more get
// k_scan_mid and k_scan_top.
constexpr int64_t kDirectGroups = 4;

}  // namespace

static TreePrecond plan_tree_precond(Carver &c, int64_t n, int32_t k) {
    TreePrecond p;
    p.n = n;
    p.k = k;
    p.A = 2 * (n - 1);
    const int64_t A1 = p.A > 0 ? p.A : 1;
    p.rtiles = scan_tiles(n, k);
    p.wtiles = scan_tiles(A1, k);
    const bool by_lane = n * k <= kDotPerLane * (kFinish / k);
    p.lanes = by_lane ? kFinish / k : 1;
    p.step = c.take<int32_t>(A1);
    p.S = c.take<double>((size_t)n * k);
    p.walk = c.take<double>((size_t)A1 * k);
    p.rsum = c.take<double>((size_t)p.rtiles * k);
    p.wsum = c.take<double>((size_t)p.wtiles * k);
    p.rgroup = c.take<double>((size_t)(scan_groups(n, k) + 1) * k);
    p.wgroup = c.take<double>((size_t)(scan_groups(A1, k) + 1) * k);
    p.tot = c.take<double>(64);
    p.rz = c.take<double>((size_t)p.lanes * k);
    p.dot = by_lane ? nullptr : c.take<double>((size_t)lane_grid(n, k) * k);
    return p;
}

size_t tree_precond_bytes(int64_t n, int32_t k) {
    Carver c(nullptr);
    plan_tree_precond(c, n, k);
    return c.used + 256;
}

TreePrecond make_tree_precond(const sfg_tree *T, int32_t k, void *ws, hipStream_t s) {
    Carver c(ws);
    TreePrecond p = plan_tree_precond(c, T->n, k);
    hipLaunchKernelGGL(k_step_nodes, dim3(grid_for(T->n, kB)), dim3(kB), 0, s, T->n, T->tdown, T->tup, p.step);
    SFG_LAUNCH_CHECK();
    return p;
}

// rr: p.rtiles rows of partial sums.
void cg_step(const TreePrecond &p, uint32_t active, const uint32_t *dmask, const double *rz, const double *pap,
             int32_t pap_rows, const double *pd, const double *ap, double *x, double *r, double *rr, hipStream_t s) {
    hipLaunchKernelGGL(k_cg_step<true>, dim3((uint32_t)p.rtiles), dim3(kT), 0, s, p.n, ByK(p.k), active, dmask, rz, pap,
                       pap_rows, pd, ap, x, r, rr, p.rsum);
    SFG_LAUNCH_CHECK();
}

// The tile sums of r alone (before the first iteration).
void precond_row_sums(const TreePrecond &p, double *r, hipStream_t s) {
    hipLaunchKernelGGL(k_cg_step<false>, dim3((uint32_t)p.rtiles), dim3(kT), 0, s, p.n, ByK(p.k), 0u, nullptr, nullptr,
                       nullptr, 0, nullptr, nullptr, nullptr, r, nullptr, p.rsum);
    SFG_LAUNCH_CHECK();
}

// z, and r . z as p.lanes rows of lane sums in p.rz, from r and its tile sums.
void tree_precond(const sfg_tree *T, const TreePrecond &p, const double *r, double *z, hipStream_t s) {
    const int32_t k = p.k;
    const ByK by(k);
    auto offsets = [&](int64_t tiles, double *sum, double *group) -> const double * {
        const int64_t tpg = (int64_t)(kB / k) * kTpl, groups = (tiles + tpg - 1) / tpg;
        if (groups <= kDirectGroups) return nullptr;
        hipLaunchKernelGGL(k_scan_mid, dim3((uint32_t)groups), dim3(kB), 0, s, tiles, k, sum, group);
        SFG_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kB), 0, s, groups, k, group);
        SFG_LAUNCH_CHECK();
        return group;
    };
    const double *ro = offsets(p.rtiles, p.rsum, p.rgroup);
    hipLaunchKernelGGL(k_rows_prefix, dim3((uint32_t)p.rtiles), dim3(kT), 0, s, p.n, by, r, p.rsum, ro, p.S, p.tot);
    SFG_LAUNCH_CHECK();
    if (p.A > 0) {
        hipLaunchKernelGGL(k_walk_drops, dim3((uint32_t)p.wtiles), dim3(kT), 0, s, p.n, p.A, by, p.step, T->size,
                           T->pw, p.S, p.tot, p.walk, p.wsum);
        SFG_LAUNCH_CHECK();
    }
    const double *wo = offsets(p.wtiles, p.wsum, p.wgroup);
    hipLaunchKernelGGL(k_walk_prefix, dim3((uint32_t)p.wtiles), dim3(kT), 0, s, p.A, by, p.walk, p.step, p.wsum, wo, z);
    SFG_LAUNCH_CHECK();
    const int32_t nb = (int32_t)lane_grid(p.n, k);
    if (p.lanes > 1) {
        hipLaunchKernelGGL(k_dot_lanes, dim3((uint32_t)p.lanes), dim3(kT), 0, s, p.n, by, nb, r, z, p.rz);
        SFG_LAUNCH_CHECK();
    } else {
        hipLaunchKernelGGL(k_dot_partials, dim3((uint32_t)nb), dim3(kB), 0, s, p.n, by, r, z, p.dot);
        SFG_LAUNCH_CHECK();
        finish_partials(nb, k, p.dot, p.rz, s);
    }
}

// ------------------------------------------------------------------ tree layout

struct TreePlan {
    int32_t *rowptr, *col, *eid, *rev, *src, *pos, *down_at, *dbefore, *scan_scr, *pre_of, *parnode;
    // one range, cleared at the start: marked edges; pieces of long rows; bad (bad[1]: a walk of the list ranking was
    // over its bound)
    int32_t *count, *pieces, *bad;
    uint32_t *next, *dist;
    double *val, *deg;
    uint64_t *link0, *link1;
    uint8_t *mask;
    void *csr_ws;
    size_t csr_wsb;
};

static TreePlan plan_tree(Carver &c, int64_t n, int64_t m) {
    const int64_t A = 2 * (n - 1) > 0 ? 2 * (n - 1) : 0;
    TreePlan p;
    p.mask = c.take<uint8_t>(m + 1);
    p.count = c.take<int32_t>(4);
    p.pieces = p.count + 1;
    p.bad = p.count + 2;
    p.rowptr = c.take<int32_t>(n + 1);
    p.col = c.take<int32_t>(A + 1);
    p.eid = c.take<int32_t>(A + 1);
    p.val = c.take<double>(A + 1);
    p.deg = c.take<double>(n + 1);
    p.rev = c.take<int32_t>(A + 1);
    p.src = c.take<int32_t>(A + 1);
    p.pos = c.take<int32_t>(A + 1);
    p.down_at = c.take<int32_t>(A + 1);
    p.dbefore = c.take<int32_t>(A + 2);
    p.scan_scr = c.take<int32_t>(scan_scratch_ints(A + 1));
    p.link0 = c.take<uint64_t>(A + 1);
    p.link1 = c.take<uint64_t>(A + 1);
    p.pre_of = c.take<int32_t>(n + 1);
    p.parnode = c.take<int32_t>(n + 1);
    p.next = c.take<uint32_t>(A + 1);
    p.dist = c.take<uint32_t>(A + 1);
    p.csr_wsb = csr_workspace_bytes(n, m);
    p.csr_ws = c.take<char>(p.csr_wsb);
    return p;
}

size_t tree_order_workspace_bytes(int64_t n, int64_t m) {
    Carver c(nullptr);
    plan_tree(c, n < 1 ? 1 : n, m < 0 ? 0 : m);
    return c.used + 256;
}

// Preorder layout of the spanning tree formed by the edges with keep[e] == 1.
// Synchronises (edge count and the spanning check).
void tree_order(int64_t n, int64_t m, const int32_t *u, const int32_t *v, const void *w, sfg_dtype wt,
                const uint8_t *keep, int32_t *order, int32_t *parent, int32_t *size, double *pw, int32_t *tdown,
                int32_t *tup, void *ws, size_t ws_bytes, hipStream_t s) {
    SFG_REQUIRE(n >= 1 && m >= 0, SFG_EINVAL, "tree_order: need n >= 1 and m >= 0");
    SFG_REQUIRE(2 * m < (int64_t(1) << 31), SFG_EUNSUPPORTED, "tree_order: 2*m must be < 2^31");
    SFG_REQUIRE(wt == SFG_F64, SFG_EINVAL, "tree_order: weights must be F64");
    SFG_REQUIRE(ws_bytes >= tree_order_workspace_bytes(n, m), SFG_EWORKSPACE, "tree_order: workspace too small");
    SFG_REQUIRE(order && parent && size && pw && tdown && tup && (m == 0 || (u && v && w && keep)), SFG_EINVAL,
                "tree_order: null pointer");
    Carver c(ws);
    TreePlan p = plan_tree(c, n, m);
    const int64_t A = 2 * (n - 1);
    fill_i32(p.count, 4, 0, s);
    if (m > 0) {
        hipLaunchKernelGGL(k_mask_eq, dim3(std::min(grid_for(m, kB), kMaskBlocks)), dim3(kB), 0, s, m, keep,
                           (uint8_t)1, p.mask, p.count);
        SFG_LAUNCH_CHECK();
    }
    int32_t cnt = 0;
    SFG_HIP(hipMemcpyAsync(&cnt, p.count, 4, hipMemcpyDeviceToHost, s));
    SFG_HIP(hipStreamSynchronize(s));
    SFG_REQUIRE(cnt == n - 1, SFG_EINVAL,
                "tree_order: " + std::to_string(cnt) + " edges marked 1, a spanning tree has n - 1");
    hipLaunchKernelGGL(k_tree_root, dim3(1), dim3(1), 0, s, n, order, parent, size, pw, tdown, tup, p.pre_of);
    SFG_LAUNCH_CHECK();
    if (A == 0) return;
    // tree CSR with FP64 weights, columns ascending per row
    build_csr(n, m, u, v, w, SFG_F64, p.mask, p.rowptr, p.col, p.val, p.eid, p.deg, p.csr_ws, p.csr_wsb, s);
    const dim3 ga(grid_for(A, kB)), gn(grid_for(n, kB)), b(kB);
    // pieces of long rows: at most A / 64 + A / 17 of two words, in what later holds the walk positions
    ArcPiece *pieces = reinterpret_cast<ArcPiece *>(p.pos);
    hipLaunchKernelGGL(k_walk_init, gn, b, 0, s, n, p.rowptr, p.col, p.rev, p.src, p.next, pieces, p.pieces);
    SFG_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_walk_long, dim3(std::min(grid_for(A, kB * kArcRow), kLongArcBlocks)), b, 0, s, p.rowptr, p.col,
                       p.rev, p.src, p.next, pieces, p.pieces);
    SFG_LAUNCH_CHECK();
    // jumping over `len` packed words: the result is in a0
    uint64_t *a0 = p.link0, *a1 = p.link1;
    auto jump = [&](int64_t len) {
        for (int64_t span = 1; span < len; span <<= 1) {
            hipLaunchKernelGGL(k_walk_jump, dim3(grid_for(len, kB)), b, 0, s, len, a0, a1);
            SFG_LAUNCH_CHECK();
            std::swap(a0, a1);
        }
    };
    // the root's first arc (arc 0) must start a walk through all 2(n - 1) arcs
    auto check_walk = [&](int32_t &over) {
        uint64_t first = 0;
        SFG_HIP(hipMemcpyAsync(&first, a0, 8, hipMemcpyDeviceToHost, s));
        SFG_HIP(hipMemcpyAsync(&over, p.bad + 1, 4, hipMemcpyDeviceToHost, s));
        SFG_HIP(hipStreamSynchronize(s));
        if (!over && first != (((uint64_t)(A - 1) << 32) | kNil))
            fail(SFG_ENOTCONN, "tree_order: the edges marked 1 do not form a spanning tree");
    };
    int32_t over = A < kRankMin ? 1 : 0;
    if (!over) {
        const uint32_t len0 = (uint32_t)A, len1 = (len0 + kBucket - 1) / kBucket, len2 = (len1 + kBucket - 1) / kBucket;
        // the first level's words take link0's first len1 elements, the last level's the rest of link0 and link1
        uint64_t *l1 = p.link0;
        a0 = p.link0 + len1;
        hipLaunchKernelGGL(k_rank_up<false>, dim3(grid_for(len1, kB)), b, 0, s, len0, len1, p.next,
                           (const uint64_t *)nullptr, l1, p.bad + 1);
        SFG_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_rank_up<true>, dim3(grid_for(len2, kB)), b, 0, s, len1, len2, (const uint32_t *)nullptr,
                           l1, a0, p.bad + 1);
        SFG_LAUNCH_CHECK();
        jump(len2);
        check_walk(over);
        if (!over) {
            hipLaunchKernelGGL(k_rank_down<true>, dim3(grid_for(len2, kB)), b, 0, s, len1, len2, a0,
                               (const uint32_t *)nullptr, l1, (uint32_t *)nullptr);
            SFG_LAUNCH_CHECK();
            hipLaunchKernelGGL(k_rank_down<false>, dim3(grid_for(len1, kB)), b, 0, s, len0, len1, l1, p.next,
                               (uint64_t *)nullptr, p.dist);
            SFG_LAUNCH_CHECK();
        }
    }
    if (over) {
        a0 = p.link0;
        a1 = p.link1;
        fill_i32(p.bad, 2, 0, s);
        hipLaunchKernelGGL(k_rank_links, ga, b, 0, s, A, p.next, a0);
        SFG_LAUNCH_CHECK();
        jump(A);
        over = 0;
        check_walk(over);
        hipLaunchKernelGGL(k_rank_dist, ga, b, 0, s, A, a0, p.dist);
        SFG_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_walk_pos, ga, b, 0, s, A, p.dist, p.rev, p.pos, p.down_at);
    SFG_LAUNCH_CHECK();
    exclusive_scan_i32(p.down_at, p.dbefore, A, p.scan_scr, s);
    hipLaunchKernelGGL(k_tree_fill, ga, b, 0, s, A, p.pos, p.rev, p.src, p.col, p.val, p.dbefore, p.pre_of, order,
                       p.parnode, size, pw, tdown, tup);
    SFG_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_tree_parent, gn, b, 0, s, n, order, p.pre_of, p.parnode, parent, p.bad);
    SFG_LAUNCH_CHECK();
    int32_t bad = 0;
    SFG_HIP(hipMemcpyAsync(&bad, p.bad, 4, hipMemcpyDeviceToHost, s));
    SFG_HIP(hipStreamSynchronize(s));
    if (bad) fail(SFG_ENOTCONN, "tree_order: the edges marked 1 do not form a spanning tree");
}

// ------------------------------------------------------------------ tree solve

size_t tree_solve_workspace_bytes(int64_t n, int32_t k) {
    Carver c(nullptr);
    const int64_t A = 2 * (n - 1) > 0 ? 2 * (n - 1) : 1;
    c.take<double>((size_t)n * k);            // bp / xp
    c.take<double>((size_t)n * k);            // S
    c.take<double>((size_t)A * k);            // walk
    c.take<double>((size_t)A * k);            // U
    c.take<double>(128);                      // means
    c.take<double>(colsum_scratch_doubles(k));
    c.take<double>(scan_scratch_doubles(A > n ? A : n, k));
    return c.used + 256;
}

void tree_solve(const sfg_tree *T, int32_t k, const double *b, double *x, void *ws, size_t ws_bytes,
                hipStream_t s) {
    const int64_t n = T->n;
    SFG_REQUIRE(n >= 1 && k >= 1 && k <= 64, SFG_EINVAL, "tree_solve: need n >= 1 and 1 <= k <= 64");
    SFG_REQUIRE(ws_bytes >= tree_solve_workspace_bytes(n, k), SFG_EWORKSPACE, "tree_solve: workspace too small");
    SFG_REQUIRE(b && x && T->order && T->size && T->pw && T->tdown && T->tup, SFG_EINVAL, "tree_solve: null pointer");
    const int64_t A = 2 * (n - 1) > 0 ? 2 * (n - 1) : 1;
    Carver c(ws);
    double *bp = c.take<double>((size_t)n * k);
    double *S = c.take<double>((size_t)n * k);
    double *walk = c.take<double>((size_t)A * k);
    double *U = c.take<double>((size_t)A * k);
    double *mean = c.take<double>(128);
    double *csum = c.take<double>(colsum_scratch_doubles(k));
    double *sscr = c.take<double>(scan_scratch_doubles(A > n ? A : n, k));
    const dim3 gnk(grid_for(n * k, kB)), blk(kB);
    block_colsum(n, k, b, 1.0 / (double)n, mean, csum, s);
    hipLaunchKernelGGL(k_gather_centre, gnk, blk, 0, s, n, k, T->order, b, mean, bp);
    SFG_LAUNCH_CHECK();
    if (n > 1) {
        block_scan(n, k, bp, S, sscr, s);
        hipLaunchKernelGGL(k_edge_drop, gnk, blk, 0, s, n, k, T->size, T->pw, T->tdown, T->tup, S, walk);
        SFG_LAUNCH_CHECK();
        block_scan(A, k, walk, U, sscr, s);
    }
    hipLaunchKernelGGL(k_potential, gnk, blk, 0, s, n, k, T->tdown, U, bp);
    SFG_LAUNCH_CHECK();
    block_colsum(n, k, bp, 1.0 / (double)n, mean + 64, csum, s);
    hipLaunchKernelGGL(k_scatter_centre, gnk, blk, 0, s, n, k, T->order, bp, mean + 64, x);
    SFG_LAUNCH_CHECK();
}

}  // namespace sfg

extern "C" sfg_status sfg_tree_order(int64_t n, int64_t m, const int32_t *u, const int32_t *v, const void *w,
                                     sfg_dtype wt, const uint8_t *keep, int32_t *order, int32_t *parent,
                                     int32_t *size, double *pw, int32_t *tdown, int32_t *tup, void *ws,
                                     size_t ws_bytes, void *stream) {
    return sfg::guard([&] {
        sfg::tree_order(n, m, u, v, w, wt, keep, order, parent, size, pw, tdown, tup, ws, ws_bytes,
                        sfg::as_stream(stream));
    });
}

extern "C" sfg_status sfg_tree_solve(const sfg_tree *T, int32_t k, const double *b, double *x, void *ws,
                                     size_t ws_bytes, void *stream) {
    return sfg::guard([&] {
        SFG_REQUIRE(T, SFG_EINVAL, "tree_solve: null tree");
        sfg::tree_solve(T, k, b, x, ws, ws_bytes, sfg::as_stream(stream));
    });
}
