// Stable least-significant-digit radix sort of (unsigned key, int32 value)
// pairs, digits of up to 8 bits, only over the digit positions the caller
// names.
//
// Per pass: every 4096-key tile counts its digits in LDS; one exclusive scan
// over the digit-major [digit][tile] table gives each (digit, tile) its
// output base; the tile is then re-read and scattered.  A wavefront takes
// 1024 consecutive keys of the tile, 64 at a time, and keeps them in
// registers: a key's rank among the wavefront's equal digits is the
// wavefront's running count of the digit (LDS, private to the wavefront, so
// no barrier) plus its rank among the 64 from ballots.  Two barriers later
// the counts of all wavefronts give every key its place in the tile; keys and
// values go through LDS in that order, so that equal digits leave as one run
// of consecutive addresses.  Input order is kept among equal digits.  Integer
// counting only: the result is deterministic.
//
// Bound by HBM traffic (each pass reads and writes every pair once, plus the
// count's read).  Scattering each key straight from its thread, with three
// barriers per 256 keys, took 473 us a pass on average for the 27M to 39M
// inter-aggregate edges of the 4M-node Chung-Lu hierarchy (64-bit keys); this
// takes 237.
#include "common.hpp"

namespace sfg {

namespace {

constexpr int kRThreads = 256;
constexpr int kRItems = 16;                       // keys per thread
constexpr int kRTile = kRThreads * kRItems;
constexpr int kRWaves = kRThreads / kWave;
constexpr int kRSeg = kWave * kRItems;            // consecutive keys of one wavefront

// Where a pass reads its pairs: arrays, or the edges of a list keyed by their
// larger end (value = edge id), those outside the mask left out.
template <typename K>
struct PairSource {
    const K *keys;
    const int32_t *vals;
    __device__ __forceinline__ bool load(int64_t i, K &k) const {
        k = keys[i];
        return true;
    }
    __device__ __forceinline__ int32_t value(int64_t i) const { return vals[i]; }
};

struct EdgeSource {
    const int32_t *v;
    const uint8_t *mask;
    __device__ __forceinline__ bool load(int64_t i, uint32_t &k) const {
        k = (uint32_t)v[i];
        return !mask || mask[i] != 0;
    }
    __device__ __forceinline__ int32_t value(int64_t i) const { return (int32_t)i; }
};

// count: the number of input pairs when only the device knows it (at most n).
template <typename K, typename SRC>
__global__ __launch_bounds__(kRThreads) void k_radix_hist(SRC src, int64_t n, const int32_t *__restrict__ count,
                                                          int shift, uint32_t dmask, int32_t *hist, int32_t nb) {
    __shared__ int32_t h[256];
    const int t = threadIdx.x;
    h[t] = 0;
    __syncthreads();
    if (count) n = *count;
    const int64_t base = (int64_t)blockIdx.x * kRTile;
#pragma unroll 4
    for (int r = 0; r < kRItems; ++r) {
        const int64_t i = base + (int64_t)r * kRThreads + t;
        K k;
        if (i < n && src.load(i, k)) atomicAdd(&h[(uint32_t)(k >> shift) & dmask], 1);
    }
    __syncthreads();
    hist[(int64_t)t * nb + blockIdx.x] = h[t];
}

template <typename K, typename SRC>
__global__ __launch_bounds__(kRThreads) void k_radix_scatter(SRC src, K *kout, int32_t *vout, int64_t n,
                                                             const int32_t *__restrict__ count, int shift,
                                                             uint32_t dmask, const int32_t *__restrict__ offs,
                                                             int32_t nb) {
    __shared__ int32_t wc[kRWaves][256];          // a wavefront's count of each digit, then its first place
    __shared__ int32_t gofs[256];                 // output address of a digit's run less its place in the tile
    __shared__ int32_t wsum[kRWaves];
    __shared__ K buf[kRTile];
    const int t = threadIdx.x, lane = t & (kWave - 1), wid = t / kWave;
    if (count) n = *count;
    const int64_t tile = (int64_t)blockIdx.x * kRTile;
    if (tile >= n) return;
#pragma unroll
    for (int w = 0; w < kRWaves; ++w) wc[w][t] = 0;
    __syncthreads();
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t base = tile + (int64_t)wid * kRSeg + lane;
    K key[kRItems];
    int32_t val[kRItems];
    bool ok[kRItems];
#pragma unroll
    for (int r = 0; r < kRItems; ++r) {
        const int64_t i = base + r * kWave;
        key[r] = 0;
        val[r] = 0;
        ok[r] = false;
        if (i < n) {
            ok[r] = src.load(i, key[r]);
            val[r] = src.value(i);
        }
    }
    int32_t place[kRItems];
#pragma unroll
    for (int r = 0; r < kRItems; ++r) {
        const int d = ok[r] ? (int)((uint32_t)(key[r] >> shift) & dmask) : 256;   // left out: a group of its own
        uint64_t peers = ~0ull;
#pragma unroll
        for (int bit = 0; bit < 9; ++bit) {
            const bool on = (d >> bit) & 1;
            const uint64_t bal = __ballot(on);
            peers &= on ? bal : ~bal;
        }
        const int rank = __popcll(peers & lt);
        // the wavefront's count so far, read by all of the digit's lanes before its first lane moves it on
        int32_t before = 0;
        if (ok[r]) before = __hip_atomic_load(&wc[wid][d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_wave_barrier();
        if (ok[r] && rank == 0)
            __hip_atomic_store(&wc[wid][d], before + __popcll(peers), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_wave_barrier();
        place[r] = before + rank;
    }
    __syncthreads();
    // thread t: digit t's counts of the wavefronts, and its place in the tile
    int32_t c[kRWaves], tot = 0;
#pragma unroll
    for (int w = 0; w < kRWaves; ++w) {
        c[w] = tot;
        tot += wc[w][t];
    }
    int32_t incl = tot;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int32_t y = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += y;
    }
    if (lane == kWave - 1) wsum[wid] = incl;
    __syncthreads();
    int32_t first = incl - tot, taken = 0;
#pragma unroll
    for (int w = 0; w < kRWaves; ++w) {
        if (w < wid) first += wsum[w];
        taken += wsum[w];
    }
#pragma unroll
    for (int w = 0; w < kRWaves; ++w) wc[w][t] = first + c[w];
    gofs[t] = offs[(int64_t)t * nb + blockIdx.x] - first;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRItems; ++r)
        if (ok[r]) {
            place[r] += wc[wid][(uint32_t)(key[r] >> shift) & dmask];
            buf[place[r]] = key[r];
        }
    __syncthreads();
    int32_t out[kRItems];
#pragma unroll
    for (int r = 0; r < kRItems; ++r) {
        const int i = r * kRThreads + t;
        if (i < taken) {
            const K k = buf[i];
            out[r] = gofs[(uint32_t)(k >> shift) & dmask] + i;
            kout[out[r]] = k;
        }
    }
    __syncthreads();
    int32_t *vbuf = reinterpret_cast<int32_t *>(buf);
#pragma unroll
    for (int r = 0; r < kRItems; ++r)
        if (ok[r]) vbuf[place[r]] = val[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRItems; ++r) {
        const int i = r * kRThreads + t;
        if (i < taken) vout[out[r]] = vbuf[i];
    }
}

int64_t radix_tiles(int64_t n) { return (n + kRTile - 1) / kRTile; }

template <typename K, typename SRC>
void radix_pass(const SRC &src, K *kout, int32_t *vout, int64_t n, const int32_t *count, int shift, int bits,
                int32_t *hist, int32_t *offs, int32_t *scan, hipStream_t s) {
    const int64_t nb = radix_tiles(n);
    const uint32_t dmask = (1u << bits) - 1u;
    hipLaunchKernelGGL((k_radix_hist<K, SRC>), dim3((uint32_t)nb), dim3(kRThreads), 0, s, src, n, count, shift, dmask,
                       hist, (int32_t)nb);
    SFG_LAUNCH_CHECK();
    exclusive_scan_i32(hist, offs, 256 * nb, scan, s);
    hipLaunchKernelGGL((k_radix_scatter<K, SRC>), dim3((uint32_t)nb), dim3(kRThreads), 0, s, src, kout, vout, n,
                       count, shift, dmask, offs, (int32_t)nb);
    SFG_LAUNCH_CHECK();
}

}  // namespace

size_t radix_scratch_bytes(int64_t n) {
    const int64_t nb = radix_tiles(n);
    Carver c(nullptr);
    c.take<uint64_t>(n + 1);
    c.take<int32_t>(n + 1);
    c.take<int32_t>(256 * nb + 1);
    c.take<int32_t>(256 * nb + 1);
    c.take<int32_t>(scan_scratch_ints(256 * nb + 1));
    return c.used + 256;
}

// Sort in place (keys/vals hold the result).  `shifts` lists the digit
// positions (multiples of 8), least significant first.
void radix_sort_pairs(uint64_t *keys, int32_t *vals, int64_t n, const int *shifts, int nshift, void *scratch,
                      hipStream_t s) {
    if (n <= 1 || nshift == 0) return;
    const int64_t nb = radix_tiles(n);
    Carver c(scratch);
    uint64_t *ktmp = c.take<uint64_t>(n + 1);
    int32_t *vtmp = c.take<int32_t>(n + 1);
    int32_t *hist = c.take<int32_t>(256 * nb + 1);
    int32_t *offs = c.take<int32_t>(256 * nb + 1);
    int32_t *scr = c.take<int32_t>(scan_scratch_ints(256 * nb + 1));
    uint64_t *ka = keys, *kb = ktmp;
    int32_t *va = vals, *vb = vtmp;
    for (int p = 0; p < nshift; ++p) {
        radix_pass<uint64_t>(PairSource<uint64_t>{ka, va}, kb, vb, n, nullptr, shifts[p], 8, hist, offs, scr, s);
        std::swap(ka, kb);
        std::swap(va, vb);
    }
    if (ka != keys) {
        SFG_HIP(hipMemcpyAsync(keys, ka, n * sizeof(uint64_t), hipMemcpyDeviceToDevice, s));
        SFG_HIP(hipMemcpyAsync(vals, va, n * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
    }
}


struct EdgeSortPlan {
    int32_t *k[2], *v[2], *hist, *offs, *scan;
};

EdgeSortPlan plan_edge_sort(Carver &c, int64_t m) {
    const int64_t nb = radix_tiles(m);
    EdgeSortPlan p;
    for (int i = 0; i < 2; ++i) {
        p.k[i] = c.take<int32_t>(m + 1);
        p.v[i] = c.take<int32_t>(m + 1);
    }
    p.hist = c.take<int32_t>(256 * nb + 1);
    p.offs = c.take<int32_t>(256 * nb + 1);
    p.scan = c.take<int32_t>(scan_scratch_ints(256 * nb + 1));
    return p;
}

size_t edge_sort_bytes(int64_t m) {
    Carver c(nullptr);
    plan_edge_sort(c, m);
    return c.used + 256;
}

// v of the edges in [0, n), m >= 1; mask nullptr = every edge.  Enqueues only.
EdgeSort sort_edges_by_v(int64_t n, int64_t m, const int32_t *v, const uint8_t *mask, void *scratch,
                         hipStream_t s) {
    Carver c(scratch);
    const EdgeSortPlan p = plan_edge_sort(c, m);
    int bits = 1;
    while (bits < 31 && (int64_t(1) << bits) < n) ++bits;
    const int passes = (bits + 7) / 8, width = (bits + passes - 1) / passes;
    const int32_t *count = p.offs + 256 * radix_tiles(m);      // every pass's scan leaves the same total there
    int at = 0;
    for (int q = 0; q < passes; ++q) {
        const int shift = q * width;
        if (q == 0)
            radix_pass<uint32_t>(EdgeSource{v, mask}, (uint32_t *)p.k[0], p.v[0], m, nullptr, shift, width, p.hist,
                                 p.offs, p.scan, s);
        else
            radix_pass<uint32_t>(PairSource<uint32_t>{(const uint32_t *)p.k[at], p.v[at]}, (uint32_t *)p.k[1 - at],
                                 p.v[1 - at], m, count, shift, width, p.hist, p.offs, p.scan, s);
        if (q > 0) at = 1 - at;
    }
    return EdgeSort{p.k[at], p.v[at], count, p.k[1 - at], p.v[1 - at]};
}

}  // namespace sfg
