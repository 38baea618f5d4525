// Internal helpers of libsfg (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <hip/hip_bf16.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "sfg.h"

namespace sfg {

// ---------------------------------------------------------------- errors

struct Error {
    sfg_status st;
    std::string msg;
};

void set_last_error(const std::string &msg);
void clear_last_error();

[[noreturn]] inline void fail(sfg_status st, const std::string &msg) { throw Error{st, msg}; }

#define SFG_HIP(call)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (call);                                                              \
        if (e_ != hipSuccess)                                                                \
            ::sfg::fail(SFG_EHIP, std::string(#call) + ": " + hipGetErrorString(e_) + " at " + \
                                      __FILE__ + ":" + std::to_string(__LINE__));            \
    } while (0)

#define SFG_LAUNCH_CHECK() SFG_HIP(hipGetLastError())

#define SFG_REQUIRE(cond, st, msg)               \
    do {                                         \
        if (!(cond)) ::sfg::fail((st), (msg));   \
    } while (0)

// Wrap an entry point body: maps internal errors to status codes.
template <typename F>
inline sfg_status guard(F &&f) {
    try {
        f();
        clear_last_error();
        return SFG_OK;
    } catch (const Error &e) {
        set_last_error(e.msg);
        return e.st;
    } catch (const std::exception &e) {
        set_last_error(std::string("internal error: ") + e.what());
        return SFG_EHIP;
    } catch (...) {
        set_last_error("internal error");
        return SFG_EHIP;
    }
}

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

// ---------------------------------------------------------------- workspace carving

// Bump allocator over a caller workspace.  With base == nullptr it only
// measures, so the same plan function gives sfg_workspace_bytes().
struct Carver {
    char *base;
    size_t used = 0;
    explicit Carver(void *b) : base(static_cast<char *>(b)) {}
    template <typename T>
    T *take(size_t count) {
        used = (used + 255) & ~size_t(255);
        T *p = base ? reinterpret_cast<T *>(base + used) : nullptr;
        used += count * sizeof(T);
        return p;
    }
};

inline size_t dtype_size(sfg_dtype t) {
    switch (t) {
        case SFG_F64: return 8;
        case SFG_F32: return 4;
        case SFG_F16: return 2;
        case SFG_BF16: return 2;
    }
    return 0;
}

inline bool valid_dtype(int t) { return t >= SFG_F64 && t <= SFG_BF16; }

// ---------------------------------------------------------------- device helpers

constexpr int kWave = 64;
constexpr int kNumXcd = 8;
constexpr int kMaxDevices = 64;

// Size of the per-device scratch array of sfg_select_topk_noalloc.
constexpr size_t kSelectNoallocBytes = size_t(128) << 20;

// Workgroups are dealt round-robin to the 8 XCDs; remap so that each XCD
// walks one contiguous range of logical blocks (neighbouring rows share that
// XCD's L2).  Bijective for any grid size.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t nb) {
    uint32_t q = nb / kNumXcd, r = nb % kNumXcd;
    uint32_t x = b % kNumXcd, i = b / kNumXcd;
    return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// The same in chunks dealt round-robin: XCD x takes chunks x, x + 8, ... of
// kXcdChunk consecutive logical blocks.  Every XCD then gets a sample of the
// whole index range.  What is left of the last whole round of chunks, all of a
// small graph among it, is one contiguous range per XCD.
constexpr uint32_t kXcdChunk = 64;

__device__ __forceinline__ uint32_t xcd_remap_chunked(uint32_t b, uint32_t nb) {
    constexpr uint32_t round = kNumXcd * kXcdChunk;
    const uint32_t whole = nb / round * round;      // a multiple of 8: b and b - whole are on one XCD
    if (b >= whole) return whole + xcd_remap(b - whole, nb - whole);
    const uint32_t x = b % kNumXcd, i = b / kNumXcd;
    return ((i / kXcdChunk) * kNumXcd + x) * kXcdChunk + i % kXcdChunk;
}

// How a kernel over the rows of a graph deals its workgroups to the XCDs: one
// contiguous range of rows each keeps neighbouring rows in one L2 (meshes,
// trees, preorders), but where one range would hold over 1.5 times its share of
// the entries (a power-law graph numbered by degree: 3.8 to 5 times) its XCD
// would be the last by far, and chunks are dealt.  Graphs averaging under 8
// entries per row have no such rows to speak of and are not asked.  (A sweep
// reads one word that the kernel of the column means left: nine loads in front
// of every workgroup cost 2 to 5% where the block stays in the caches.)
// Measured, FP32, 16 vectors: the 4M-node Chung-Lu graph, contiguous 3,486 us a
// sweep, chunks 1,417; relabelled in a tree's preorder (1.01 times the share)
// 1,739 and 1,744; 27-point meshes in their own order of 64,000 nodes 15.5 and
// 16.9 (FP64 20.6 and 23.2), of 2.1M nodes 351 and 329.  A row of a million
// entries among 25 million makes 1.28 of its range, and hub rows have
// workgroups of their own, hence no less than 1.5.
__device__ __forceinline__ bool xcd_uneven(const int32_t *__restrict__ rowptr, int64_t n) {
    uint32_t most = 0;
#pragma unroll
    for (int x = 0; x < kNumXcd; ++x) {
        const uint32_t part = (uint32_t)(rowptr[n * (x + 1) / kNumXcd] - rowptr[n * x / kNumXcd]);
        most = part > most ? part : most;
    }
    return 2ull * kNumXcd * most > 3ull * (uint32_t)(rowptr[n] - rowptr[0]);
}

// Between a wavefront's writes to LDS and its other lanes' reads of them (and
// before the next writes there).  Its LDS accesses run in program order; the
// fences keep the compiler from moving them, which wave_barrier alone, no
// access to memory, does not.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Quotients with one denominator, bit for bit as the operator gives them: the
// compiler's own steps for a division (a reciprocal refined by Newton's method,
// the product, the remainder's correction) with the reciprocal taken once.  Its
// scaling of extreme operands does nothing while the operands' exponents differ
// by less than 96 (FP64: 768) and neither the quotient nor the remainder is
// near the smallest numbers; the callers keep them well inside.
__device__ __forceinline__ float refined_rcp(float d) {
    const float y = __builtin_amdgcn_rcpf(d);
    return __builtin_fmaf(__builtin_fmaf(-d, y, 1.f), y, y);
}
__device__ __forceinline__ float quotient(float a, float d, float y) {
    float q = a * y;
    q = __builtin_fmaf(__builtin_fmaf(-d, q, a), y, q);
    return __builtin_fmaf(__builtin_fmaf(-d, q, a), y, q);
}
__device__ __forceinline__ double refined_rcp(double d) {
    double y = __builtin_amdgcn_rcp(d);
    y = __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
    return __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
}
__device__ __forceinline__ double quotient(double a, double d, double y) {
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-d, q, a), y, q);
}

// Whether quotient() may take a[0..V) / d: no zero, infinity or NaN, exponents
// within 40 (300) of 1's.  On the exponent fields, which NaN and infinity have
// the largest of and zero the smallest.
template <int V>
__device__ __forceinline__ bool mid_range(const float (&a)[V], float d) {
    uint32_t lo = 0x7f800000u, hi = 0;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const uint32_t e = __float_as_uint(a[i]) & 0x7f800000u;
        lo = e < lo ? e : lo;
        hi = e > hi ? e : hi;
    }
    constexpr uint32_t kLo = (127u - 40u) << 23, kHi = (127u + 40u) << 23;
    const uint32_t ed = __float_as_uint(d);
    return lo > kLo && hi < kHi && ed > kLo && ed < kHi;
}
template <int V>
__device__ __forceinline__ bool mid_range(const double (&a)[V], double d) {
    uint32_t lo = 0x7ff00000u, hi = 0;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const uint32_t e = (uint32_t)__double2hiint(a[i]) & 0x7ff00000u;
        lo = e < lo ? e : lo;
        hi = e > hi ? e : hi;
    }
    constexpr uint32_t kLo = (1023u - 300u) << 20, kHi = (1023u + 300u) << 20;
    const uint32_t ed = (uint32_t)__double2hiint(d);
    return lo > kLo && hi < kHi && ed > kLo && ed < kHi;
}

// out[i] = a[i] / d
template <int V, typename T>
__device__ __forceinline__ void divide_row(const T (&a)[V], T d, T (&out)[V]) {
    if (mid_range<V>(a, d)) {
        const T y = refined_rcp(d);
#pragma unroll
        for (int i = 0; i < V; ++i) out[i] = quotient(a[i], d, y);
    } else {
#pragma unroll
        for (int i = 0; i < V; ++i) out[i] = a[i] / d;
    }
}

template <typename T> struct DT;
template <> struct DT<double> { static constexpr sfg_dtype id = SFG_F64; };
template <> struct DT<float> { static constexpr sfg_dtype id = SFG_F32; };
template <> struct DT<__half> { static constexpr sfg_dtype id = SFG_F16; };
template <> struct DT<__hip_bfloat16> { static constexpr sfg_dtype id = SFG_BF16; };

// value conversions (round to nearest even on narrowing)
template <typename TO, typename FROM> __device__ __forceinline__ TO cvt(FROM x);
template <> __device__ __forceinline__ double cvt<double, double>(double x) { return x; }
template <> __device__ __forceinline__ double cvt<double, float>(float x) { return (double)x; }
template <> __device__ __forceinline__ float cvt<float, float>(float x) { return x; }
template <> __device__ __forceinline__ float cvt<float, double>(double x) { return (float)x; }
template <> __device__ __forceinline__ float cvt<float, __half>(__half x) { return __half2float(x); }
template <> __device__ __forceinline__ float cvt<float, __hip_bfloat16>(__hip_bfloat16 x) {
    return __bfloat162float(x);
}
template <> __device__ __forceinline__ __half cvt<__half, float>(float x) { return __float2half(x); }
template <> __device__ __forceinline__ __hip_bfloat16 cvt<__hip_bfloat16, float>(float x) {
    return __float2bfloat16(x);
}
// FP64 to FP16 / BF16 with one rounding.  Rounding to float first and then to
// the 16-bit type rounds twice and can land one unit off (a double just above
// a 16-bit midpoint can round to that midpoint in float, then tie to even).
// Rounding to float toward zero and setting the last bit when anything was
// dropped ("round to odd") keeps the information the second rounding needs:
// with at least two extra significand bits in the intermediate format (float
// has 13 more than FP16 and 16 more than BF16, also in their subnormal ranges)
// the round to nearest even that follows gives the correctly rounded result
// (Boldo and Melquiond, "Emulation of FMA and correctly rounded sums: proved
// algorithms using rounding to odd", IEEE Trans. Computers 57(4), 2008).
__device__ __forceinline__ float round_to_odd_float(double x) {
    float f = (float)x;
    // rounded away from zero (also to infinity on overflow): one step back toward zero, which for a
    // sign-magnitude encoding is the bit pattern minus one
    if (__builtin_fabs((double)f) > __builtin_fabs(x)) f = __uint_as_float(__float_as_uint(f) - 1u);
    if ((double)f != x && f == f) f = __uint_as_float(__float_as_uint(f) | 1u);
    return f;
}
template <> __device__ __forceinline__ __half cvt<__half, double>(double x) {
    return __float2half(round_to_odd_float(x));
}
template <> __device__ __forceinline__ __hip_bfloat16 cvt<__hip_bfloat16, double>(double x) {
    return __float2bfloat16(round_to_odd_float(x));
}
template <> __device__ __forceinline__ double cvt<double, __half>(__half x) { return (double)__half2float(x); }
template <> __device__ __forceinline__ double cvt<double, __hip_bfloat16>(__hip_bfloat16 x) {
    return (double)__bfloat162float(x);
}

// ---------------------------------------------------------------- shared device routines

// Exclusive prefix sum of int32 counts; out may alias nothing.  n elements in,
// n+1 written (out[n] = total).  Scratch: scan_scratch_ints(n) ints.
size_t scan_scratch_ints(int64_t n);
void exclusive_scan_i32(const int32_t *in, int32_t *out, int64_t n, int32_t *scratch, hipStream_t s);

// Fill with a value (kernel, not a memset node, so it is safe under capture).
void fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s);
void fill_u8(uint8_t *p, int64_t n, uint8_t v, hipStream_t s);

// Scalars read back to pinned host memory.  add() enqueues a copy of one value
// of at most 8 bytes; wait() blocks until every copy added so far is done
// (an event, not the stream: work enqueued after the last add() keeps the GPU
// busy meanwhile), then get() gives the values.  The buffer and its event come
// from a per-device pool of at most kPoolMax free ones and go back when the
// object dies (after its copies have landed).
class HostRead {
  public:
    explicit HostRead(hipStream_t s);
    ~HostRead();
    HostRead(const HostRead &) = delete;
    HostRead &operator=(const HostRead &) = delete;
    template <typename T>
    int add(const T *device) {
        static_assert(sizeof(T) <= 8, "one scalar");
        return add_bytes(device, sizeof(T));
    }
    void wait();
    template <typename T>
    T get(int slot) const {
        T v;
        std::memcpy(&v, static_cast<const char *>(it_.host) + 8 * slot, sizeof(T));
        return v;
    }
    struct Item {
        void *host = nullptr;
        hipEvent_t ev = nullptr;
    };

  private:
    int add_bytes(const void *device, size_t bytes);
    Item it_;
    hipStream_t s_;
    int dev_ = 0, used_ = 0;
    bool pending_ = false;
};

// The included edges of a list, sorted by (larger end, edge id).
struct EdgeSort {
    int32_t *v, *e;              // [m + 1] larger end and id, in order
    const int32_t *count;        // device: how many
    int32_t *spare0, *spare1;    // [m + 1] buffers the result does not occupy
};

// Node numbering for the sweeps of a sparsify call or of one hierarchy level
// (the rules are with score_level and level_node_order).
struct NodeOrder {
    int64_t launches = 0;       // planned column-part sweep launches (set by the caller)
    bool decided = false;
    bool use = false;
    int32_t *order = nullptr;   // [n] node at new position i
    int32_t *inv = nullptr;     // [n] new position of node j
    int32_t *u = nullptr;       // [m] endpoints in the new numbering
    int32_t *v = nullptr;
};

// Device buffers owned by one allocating call (sfg_sparsify, ...), carved
// from chunks of at least 256 MB.  A call that ends with finish() (its stream
// drained) hands its chunks to a per-device cache (up to 16 GiB) that later
// calls reuse; otherwise (an error path, work possibly in flight) they are
// freed stream-ordered.  release(mark()) gives back everything taken since
// the mark, for later requests of the same call: its users' work must be on
// the arena's stream (or joined to it), so that the next user runs after them.
// SFG_FAIL_ALLOC_AFTER=n makes the (n+1)-th buffer request fail, to test the
// error path.
struct DevArena {
    struct Chunk {
        void *p;
        size_t size;
    };
    hipStream_t s;
    struct Mark {
        size_t chunks, used;
    };
    std::vector<Chunk> chunks;
    std::vector<Chunk> spare;   // released chunks of this call
    size_t used = 0;            // bytes carved from the last of `chunks`
    int dev = 0;
    bool synced = false;
    long fail_after = -1;
    long count = 0;
    explicit DevArena(hipStream_t st);
    ~DevArena();
    DevArena(const DevArena &) = delete;
    DevArena &operator=(const DevArena &) = delete;
    void *raw(size_t bytes);
    Mark mark() const { return {chunks.size(), used}; }
    void release(const Mark &m);
    void finish();   // wait for the stream; the chunks may then be cached
    template <typename T>
    T *alloc(size_t n) {
        return static_cast<T *>(raw(n * sizeof(T)));
    }
};

// Buffers of the tree preconditioner inside the conjugate gradients (blocks
// in the tree's preorder; tree.hip, kappa.hip).
struct TreePrecond {
    int64_t n = 0, A = 0;              // nodes, walk steps
    int32_t k = 0, lanes = 0;          // columns; rows of rz
    int64_t rtiles = 0, wtiles = 0;    // tiles of block_scan over the rows, over the walk
    int32_t *step = nullptr;           // [A] i at the step entering node i, ~i at the step leaving it
    double *S = nullptr, *walk = nullptr;                                            // [n][k], [A][k]
    double *rsum = nullptr, *wsum = nullptr, *rgroup = nullptr, *wgroup = nullptr;   // tile sums, group sums
    double *tot = nullptr;             // [k] column totals of r
    double *rz = nullptr;              // [lanes][k] lane sums of r . z (one lane: their sum, from partials in dot)
    double *dot = nullptr;
};

// Graphs averaging 8 or more entries per row (see xcd_uneven).
inline bool dense_rows(const sfg_csr *H) { return H->nnz >= 8 * H->n; }

inline uint32_t grid_for(int64_t items, int block) {
    int64_t g = (items + block - 1) / block;
    return (uint32_t)(g < 1 ? 1 : g);
}

}  // namespace sfg
