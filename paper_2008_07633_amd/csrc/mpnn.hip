// Learned edge-criticality surrogate: a two-layer message-passing network
// over G with an edge head, trained on the scores the plain method produces.
// (Not part of the paper; it prunes candidates before exact scoring.)
//
//   A1 = D^-1 A X            X: 8 standardised node features
//   H1 = relu([X | A1 | 1] W1)       W1: (2*8+1) x 32
//   A2 = D^-1 A H1
//   H2 = relu([H1 | A2 | 1] W2)      W2: (2*32+1) x 32
//   z_e = [|H2_p - H2_q| | H2_p * H2_q | f_e | 1]   (69)
//   yhat_e = [relu(z_e W3) | 1] . w4      W3: 69 x 32, w4: 33
// Parameters are one FP32 vector [W1 | W2 | W3 | w4] (4865 values); each
// block stacks the self weights, the neighbour weights and the bias, so a
// weight gradient is one product U^T dP of the layer's input [x | a | 1].
//
// Kernels: FP32 aggregations reuse the smoothing sweep (omega = 1).
// Inference (BF16 activations) runs the layers, each with its aggregation, and
// the edge head on the matrix cores: a wavefront takes 16 nodes or edges,
// builds their x, a or z rows as BF16 MFMA operands, multiplies by the BF16
// weights into FP32 accumulators, and applies the ReLU (and the head's last
// dot product) in FP32.  Training
// (and FP32 inference) runs on the matrix cores too, in FP32
// (v_mfma_f32_32x32x2_f32).  One kernel takes the edge head forward and
// backward, 32 edges per wavefront: predictions, loss, the gradients sent to
// both ends' nodes and the head's weight gradients, which stay in accumulators
// over all of a wavefront's tiles.  Per-edge gradients reach the nodes through
// an incidence CSR in ascending edge order; weight gradients are added over
// fixed partitions in a fixed order: no FP atomics, so training is
// deterministic.  One loss and gradient on a 40^3 mesh (64,000 nodes, 123,201
// edges) took 1.21 ms on the vector units, with every layer's inputs written
// out for its weight gradient, and takes 0.19.
#include <algorithm>
#include <cmath>
#include <vector>

#include <type_traits>

#include "common.hpp"

namespace sfg {

void spmm_rownorm_f32(const sfg_csr *H, int32_t k, const float *x, float *y, hipStream_t s);
size_t csr_workspace_bytes(int64_t n, int64_t m);
void build_csr(int64_t n, int64_t m, const int32_t *u, const int32_t *v, const void *w, sfg_dtype wt,
               const uint8_t *mask, int32_t *rowptr, int32_t *col, void *val, int32_t *eid, void *deg, void *ws,
               size_t ws_bytes, hipStream_t s, int64_t included = 0);

namespace {

constexpr int kF = 8;                 // node features
constexpr int kH = 32;                // hidden width
constexpr int kE = 4;                 // edge features
constexpr int kZ = 2 * kH + kE;       // edge-head input
constexpr int kU1 = 2 * kF + 1;       // rows of W1
constexpr int kU2 = 2 * kH + 1;       // rows of W2
constexpr int kZ1 = kZ + 1;           // rows of W3
constexpr int kOffW1 = 0;
constexpr int kOffW2 = kOffW1 + kU1 * kH;
constexpr int kOffW3 = kOffW2 + kU2 * kH;
constexpr int kOffW4 = kOffW3 + kZ1 * kH;
constexpr int kParams = kOffW4 + kH + 1;
static_assert(kParams == 4865, "parameter count");
constexpr float kTiny = 1e-30f;

// ------------------------------------------------------------------ features

// |x_p - x_q|^2 over the kc cheap vectors, added in column order (KC > 0: kc =
// KC, a multiple of 4, loaded as 16-byte vectors)
template <int KC>
__device__ __forceinline__ float dist2(const float *__restrict__ xc, int32_t kc, const float *xp, int64_t q) {
    float d2 = 0.f;
    if constexpr (KC > 0) {
#pragma unroll
        for (int c4 = 0; c4 < KC / 4; ++c4) {
            const float4 b = *reinterpret_cast<const float4 *>(xc + q * KC + 4 * c4);
            const float bq[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float d = xp[4 * c4 + c] - bq[c];
                d2 = __builtin_fmaf(d, d, d2);
            }
        }
    } else {
        const float *xq = xc + q * kc;
        for (int c = 0; c < kc; ++c) {
            const float d = xp[c] - xq[c];
            d2 = __builtin_fmaf(d, d, d2);
        }
    }
    return d2;
}

// sum_j w_j |x_p - x_col[j]|^2 over a row, in entry order, two entries in flight
template <int KC>
__device__ __forceinline__ float row_energy(const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                                            const float *__restrict__ val, const float *__restrict__ xc, int32_t kc,
                                            const float *xp, int64_t p) {
    float e = 0.f;
    const int32_t j0 = rp[p], j1 = rp[p + 1];
    int32_t j = j0;
    for (; j + 2 <= j1; j += 2) {
        const int64_t q0 = col[j], q1 = col[j + 1];
        const float w0 = val[j], w1 = val[j + 1];
        const float d0 = dist2<KC>(xc, kc, xp, q0), d1 = dist2<KC>(xc, kc, xp, q1);
        e = __builtin_fmaf(w0, d0, e);
        e = __builtin_fmaf(w1, d1, e);
    }
    if (j < j1) e = __builtin_fmaf(val[j], dist2<KC>(xc, kc, xp, col[j]), e);
    return e;
}

template <int KC>
__global__ void k_node_feat(int64_t n, const int32_t *__restrict__ grp, const int32_t *__restrict__ gcol,
                            const float *__restrict__ gval, const float *__restrict__ gdeg,
                            const int32_t *__restrict__ trp, const int32_t *__restrict__ tcol,
                            const float *__restrict__ tval, const float *__restrict__ tdeg,
                            const float *__restrict__ xc, int32_t kc, const float *__restrict__ norm, float *nf) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    float xp[KC > 0 ? KC : 64];
    if constexpr (KC > 0) {
#pragma unroll
        for (int c4 = 0; c4 < KC / 4; ++c4) {
            const float4 a = *reinterpret_cast<const float4 *>(xc + p * KC + 4 * c4);
            xp[4 * c4] = a.x;
            xp[4 * c4 + 1] = a.y;
            xp[4 * c4 + 2] = a.z;
            xp[4 * c4 + 3] = a.w;
        }
    } else {
        for (int c = 0; c < kc; ++c) xp[c] = xc[p * kc + c];
    }
    float amp = 0.f;
    for (int c = 0; c < (KC > 0 ? KC : kc); ++c) amp = __builtin_fmaf(xp[c], xp[c], amp);
    const float eg = row_energy<KC>(grp, gcol, gval, xc, kc, xp, p);
    const float et = row_energy<KC>(trp, tcol, tval, xc, kc, xp, p);
    float f[kF];
    f[0] = 1.f;
    f[1] = logf(gdeg[p]);
    f[2] = logf(tdeg[p]);
    f[3] = logf((float)(grp[p + 1] - grp[p]));
    f[4] = logf((float)(trp[p + 1] - trp[p]));
    f[5] = logf(amp + kTiny);
    f[6] = logf(eg / gdeg[p] + kTiny);
    f[7] = logf(et / tdeg[p] + kTiny);
    float o[kF];
#pragma unroll
    for (int i = 0; i < kF; ++i) o[i] = (norm && i > 0) ? (f[i] - norm[i]) * norm[kF + i] : f[i];
    if constexpr (KC > 0) {
        *reinterpret_cast<float4 *>(nf + p * kF) = make_float4(o[0], o[1], o[2], o[3]);
        *reinterpret_cast<float4 *>(nf + p * kF + 4) = make_float4(o[4], o[5], o[6], o[7]);
    } else {
#pragma unroll
        for (int i = 0; i < kF; ++i) nf[p * kF + i] = o[i];
    }
}

template <int KC>
__global__ void k_edge_feat(int64_t ne, const int32_t *__restrict__ cand, const int32_t *__restrict__ u,
                            const int32_t *__restrict__ v, const float *__restrict__ w, const float *__restrict__ xc,
                            int32_t kc, const float *__restrict__ tdeg, const float *__restrict__ norm, float *ef) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ne) return;
    const int32_t e = cand ? cand[i] : (int32_t)i;
    const int32_t p = u[e], q = v[e];
    float xp[KC > 0 ? KC : 64];
    if constexpr (KC > 0) {
#pragma unroll
        for (int c4 = 0; c4 < KC / 4; ++c4) {
            const float4 a = *reinterpret_cast<const float4 *>(xc + (int64_t)p * KC + 4 * c4);
            xp[4 * c4] = a.x;
            xp[4 * c4 + 1] = a.y;
            xp[4 * c4 + 2] = a.z;
            xp[4 * c4 + 3] = a.w;
        }
    } else {
        for (int c = 0; c < kc; ++c) xp[c] = xc[(int64_t)p * kc + c];
    }
    const float d2 = dist2<KC>(xc, kc, xp, q);
    const float lp = logf(tdeg[p]), lq = logf(tdeg[q]);
    float f[kE] = {logf(w[e]), logf(w[e] * d2 + kTiny), fminf(lp, lq), fmaxf(lp, lq)};
#pragma unroll
    for (int j = 0; j < kE; ++j) {
        float x = f[j];
        if (norm) x = (x - norm[2 * kF + j]) * norm[2 * kF + kE + j];
        ef[i * kE + j] = x;
    }
}

// ------------------------------------------------------------------ inference on the matrix cores
//
// A wavefront takes 16 nodes or edges; lane l works for item l % 16 as its
// quarter q = l / 16.  Products are formed transposed (hidden x item), so that
// a lane ends up with runs of four hidden values of its own item:
//   v_mfma_f32_16x16x32_bf16: A (16 x 32): row l % 16, columns 8 q + 0..7
//                             B (32 x 16): column l % 16, rows 8 q + 0..7
//   v_mfma_f32_16x16x16_bf16: the same with 4 q + 0..3
//   D (16 x 16): column l % 16, rows 4 q + 0..3
// with the weights as A (two blocks of 16 hidden values), which a wavefront
// keeps in registers over all its tiles, and the items' values as B.  The
// layers' products run in the order of the inputs with the bias last: what
// they leave is rounded to BF16, and a sum in another order rounds some of it
// to the other side.
//
// The aggregation is part of the layer: the four lanes of a node gather the
// eight columns of its neighbours' rows that their quarter of B needs, where a
// sweep of its own wrote the aggregate and the layer read it back.  The layers
// are bound by memory and as much by the vector units (conversions, addresses,
// the aggregate's divisions), all three by latency until a wavefront loaded
// its next tiles ahead.  On the 128^3 mesh (2.1 million nodes, 12.5 million
// entries, 4.2 million edges; floors at the rate of a large copy): layer 1 90
// (sweep) + 48 -> 76 us (58), layer 2 150 + 116 -> 118 us (71), head 182 ->
// 90 us (51).

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bfx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bfx8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// two values rounded to BF16, the first in the low half
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    const bfx2 r = __builtin_convertvector((f32x2){a, b}, bfx2);
    uint32_t o;
    __builtin_memcpy(&o, &r, sizeof(o));
    return o;
}

__device__ __forceinline__ bfx8 operand8(const uint32_t (&w)[4]) {
    bfx8 r;
    __builtin_memcpy(&r, w, sizeof(r));
    return r;
}

__device__ __forceinline__ bf16x4 operand4(uint32_t a, uint32_t b) {
    const uint32_t w[2] = {a, b};
    bf16x4 r;
    __builtin_memcpy(&r, w, sizeof(r));
    return r;
}

// eight BF16 values of a row (16 bytes) to FP32
__device__ __forceinline__ void unpack8(const uint4 &r, float (&f)[8]) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(w[i] << 16);
        f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}

// Rows 4 q .. 4 q + 3 from r0 of a (rows x 32) FP32 weight block, hidden value
// 16 b + l % 16, as two words of an A operand
__device__ __forceinline__ void weights4(const float *__restrict__ W, int r0, int q, int b, int c, uint32_t *w) {
    const float *at = W + (r0 + 4 * q) * kH + 16 * b + c;
    w[0] = pack2(at[0], at[kH]);
    w[1] = pack2(at[2 * kH], at[3 * kH]);
}

// [b][r] = v[16 b + 4 q + r]: a lane's hidden values
__device__ __forceinline__ void hidden8(const float *__restrict__ v, int q, f32x4 (&o)[2]) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[b][r] = v[16 * b + 4 * q + r];
}

// h[node] = relu(acc): hidden value 16 b + 4 q + r lies at 8 q + 4 b + r of its
// row, so that a lane stores, and gathers, 16 bytes.
__device__ __forceinline__ void store_relu(const f32x4 (&acc)[2], int q, __hip_bfloat16 *__restrict__ hrow) {
    uint4 o;
    o.x = pack2(fmaxf(acc[0][0], 0.f), fmaxf(acc[0][1], 0.f));
    o.y = pack2(fmaxf(acc[0][2], 0.f), fmaxf(acc[0][3], 0.f));
    o.z = pack2(fmaxf(acc[1][0], 0.f), fmaxf(acc[1][1], 0.f));
    o.w = pack2(fmaxf(acc[1][2], 0.f), fmaxf(acc[1][3], 0.f));
    *reinterpret_cast<uint4 *>(hrow + 8 * q) = o;
}

// The bias as one more row of the product, after the others: the first of
// quarter 0's four, whose item value is 1
__device__ __forceinline__ bf16x4 bias_row(float v, int q) { return operand4(q == 0 ? pack2(v, 0.f) : 0u, 0u); }

// Wavefronts per SIMD, and so workgroups per CU, that the kernels below are
// compiled for; the grid is that many workgroups on every CU and no more, so
// that the weights are loaded once, all workgroups run from start to end and
// neighbouring tiles stay close in time (the head with 5 workgroups per CU
// took 96 us, with 6 89; with 5.5, its last ones alone at the end, 147).  One
// wavefront more than here spills.
constexpr int kLayerWaves(int U) { return U <= 4 ? 5 : (U <= 6 ? 4 : 3); }
constexpr int kHeadWaves = 6;

inline uint32_t tile_grid(uint32_t nvb, int waves) { return std::min(nvb, 256u * (uint32_t)waves); }

// One row of the graph on its way through a wavefront's tiles: its extent is
// loaded two tiles ahead, its first U entries one tile ahead, so that only the
// gathered rows themselves are waited for.
template <int U>
struct RowAhead {
    int32_t j0, j1, c[U];
    float w[U], d;

    __device__ __forceinline__ void extent(int64_t p, const int32_t *__restrict__ rowptr) {
        j0 = rowptr[p];
        j1 = rowptr[p + 1];
    }
    // A short row's U entries run into the next rows' (valid, and masked where
    // they are used); only the graph's last rows are clamped.
    __device__ __forceinline__ void entries(int64_t p, int32_t nnz, const int32_t *__restrict__ col,
                                            const float *__restrict__ val, const float *__restrict__ deg) {
        d = deg[p];
        if (nnz - j0 >= U) {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                c[i] = col[j0 + i];
                w[i] = val[j0 + i];
            }
        } else {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                c[i] = i < nnz - j0 ? col[j0 + i] : (int32_t)p;
                w[i] = i < nnz - j0 ? val[j0 + i] : 0.f;
            }
        }
    }

    // every lane's row has at least U entries: no masks
    __device__ __forceinline__ bool full() const { return __all(j1 - j0 >= U); }
};

// acc[i] += w x[i] over entries U, U + 1, ... of a row of len entries (counted
// from its first: at 2^31 - 2 entries the last rows' indices step over 2^31), B
// in flight.  AHEAD: the next B columns and weights are loaded before the
// gathered rows are added; a hub row is one chain, and its loads would be two
// waits a step.  (Layer 2 where it has the registers: inference on the
// 50,000-node Chung-Lu graph takes 500 us, 558 without.  In layer 1, where a
// wavefront holds 64 rows of two loads an entry, it took 310 us for 290 on
// 20,000 nodes, and so did more entries in flight.)  RAW: what load() returns
// of a row, taken apart by add().
template <int U, int B, bool AHEAD, typename RAW, typename LOAD, typename ADD>
__device__ __forceinline__ void gather_rest(int32_t len, const int32_t *__restrict__ col,
                                            const float *__restrict__ val, LOAD load, ADD add) {
    if (len <= U) return;
    int32_t cj[B];
    float wj[B];
    auto entries = [&](int32_t j) {
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int32_t jj = j + i < len ? j + i : len - 1;
            cj[i] = col[jj];
            wj[i] = val[jj];
        }
    };
    if constexpr (AHEAD) entries(U);
    for (int32_t j = U; j < len; j += B) {
        RAW x[B];
        float w[B];
        if constexpr (!AHEAD) entries(j);
#pragma unroll
        for (int i = 0; i < B; ++i) {
            load(cj[i], x[i]);
            w[i] = wj[i];
        }
        if constexpr (AHEAD)
            if (j + B < len) entries(j + B);
#pragma unroll
        for (int i = 0; i < B; ++i)
            if (j + i < len) add(w[i], x[i]);
    }
}

struct Row8 {
    float v[8];
};

// a[i] = acc[i] / d + 0 self[i]: the sweep's form with omega = 1, bit for bit,
// with one reciprocal for all eight columns in divide_row's range.  After a
// ReLU many sums are zero (+0), whose quotient by these steps is +0 as well.
__device__ __forceinline__ void row_mean(const float (&acc)[8], const float (&self)[8], float d, float (&a)[8]) {
    uint32_t lo = 0x7f800000u, hi = 0;      // NaN and infinity are the largest
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const uint32_t b = __float_as_uint(acc[t]), mag = b & 0x7fffffffu;
        hi = mag > hi ? mag : hi;
        const uint32_t low = b == 0 ? 0x7f800000u : mag;
        lo = low < lo ? low : lo;
    }
    if (__all(lo > __float_as_uint(0x1p-40f) && hi < __float_as_uint(0x1p40f) && d > 0x1p-40f && d < 0x1p40f)) {
        const float y = refined_rcp(d);
#pragma unroll
        for (int t = 0; t < 8; ++t) a[t] = quotient(acc[t], d, y) + 0.f * self[t];
    } else {
#pragma unroll
        for (int t = 0; t < 8; ++t) a[t] = acc[t] / d + 0.f * self[t];
    }
}

// h1 = relu([x | D^-1 A x | 1] W1).  A wavefront takes 64 nodes, one per lane
// (a row of x is 32 bytes), and turns their [x | a] rows through LDS into the
// operands of four tiles.
template <int U>
__global__ __launch_bounds__(256, kLayerWaves(U)) void k_layer1_mfma(int64_t n, uint32_t nvb, bool dense,
                                                     const int32_t *__restrict__ rowptr,
                                                     const int32_t *__restrict__ col, const float *__restrict__ val,
                                                     const float *__restrict__ deg, const float *__restrict__ x,
                                                     const float *__restrict__ W, __hip_bfloat16 *__restrict__ h) {
    static_assert(kF == 8, "[x | a] is one product of 16");
    __shared__ uint32_t turn[4][64][10];      // 40-byte rows: 8-byte aligned, spread over the banks
    const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15, wv = threadIdx.x >> 6;
    bf16x4 wa[2], wb[2];
    const bf16x4 one = bias_row(1.f, q);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        uint32_t w[2];
        weights4(W, 0, q, b, c, w);
        wa[b] = operand4(w[0], w[1]);
        wb[b] = bias_row(W[2 * kF * kH + 16 * b + c], q);
    }
    auto load = [&](int64_t row, float (&o)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = x[row * kF + i];
    };
    const bool uneven = dense && xcd_uneven(rowptr, n);
    auto first = [&](uint32_t vb) {
        return ((int64_t)(uneven ? xcd_remap_chunked(vb, nvb) : xcd_remap(vb, nvb)) * 4 + wv) * 64;
    };
    auto row_of = [&](uint32_t vb) {
        const int64_t p = (vb < nvb ? first(vb) : 0) + lane;
        return p < n ? p : n - 1;
    };
    RowAhead<U> cur, nxt;
    int64_t p = row_of(blockIdx.x), pn = row_of(blockIdx.x + gridDim.x);
    const int32_t nnz = rowptr[n];
    cur.extent(p, rowptr);
    nxt.extent(pn, rowptr);
    cur.entries(p, nnz, col, val, deg);
    for (uint32_t vb = blockIdx.x; vb < nvb; vb += gridDim.x) {
        float self[8], xv[U][8], acc[8];
        load(p, self);
#pragma unroll
        for (int i = 0; i < U; ++i) load(cur.c[i], xv[i]);
        nxt.entries(pn, nnz, col, val, deg);
        RowAhead<U> after;
        const int64_t pa = row_of(vb + 2 * gridDim.x);
        after.extent(pa, rowptr);
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = 0.f;
        auto add = [&](int i) {
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[t] = __builtin_fmaf(cur.w[i], xv[i][t], acc[t]);
        };
        if (cur.full()) {
#pragma unroll
            for (int i = 0; i < U; ++i) add(i);
        } else {
#pragma unroll
            for (int i = 0; i < U; ++i)
                if (i < cur.j1 - cur.j0) add(i);
        }
        gather_rest<U, U, false, Row8>(
            cur.j1 - cur.j0, col + cur.j0, val + cur.j0, [&](int64_t row, Row8 &o) { load(row, o.v); },
            [&](float w, const Row8 &row) {
#pragma unroll
                for (int t = 0; t < 8; ++t) acc[t] = __builtin_fmaf(w, row.v[t], acc[t]);
            });
        float a[8];
        row_mean(acc, self, cur.d, a);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            turn[wv][lane][t] = pack2(self[2 * t], self[2 * t + 1]);
            turn[wv][lane][4 + t] = pack2(a[2 * t], a[2 * t + 1]);
        }
        wave_lds_sync();
        const int64_t base = first(vb);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int64_t node = base + 16 * g + c;
            const uint32_t *t = turn[wv][16 * g + c];
            const bf16x4 bv = operand4(t[2 * q], t[2 * q + 1]);
            f32x4 out[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                out[b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wa[b], bv, f32x4{}, 0, 0, 0);
                out[b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wb[b], one, out[b], 0, 0, 0);
            }
            if (node < n) store_relu(out, q, h + node * kH);
        }
        wave_lds_sync();
        cur = nxt;
        nxt = after;
        p = pn;
        pn = pa;
    }
}

// h2 = relu([h1 | D^-1 A h1 | 1] W2): lane quarter q holds columns 4q .. 4q + 3
// and 16 + 4q .. 16 + 4q + 3.
template <int U>
__global__ __launch_bounds__(256, kLayerWaves(U)) void k_layer2_mfma(int64_t n, uint32_t nvb, bool dense,
                                                     const int32_t *__restrict__ rowptr,
                                                     const int32_t *__restrict__ col, const float *__restrict__ val,
                                                     const float *__restrict__ deg,
                                                     const __hip_bfloat16 *__restrict__ h1,
                                                     const float *__restrict__ W, __hip_bfloat16 *__restrict__ h2) {
    static_assert(kH == 32, "eight columns per lane");
    const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15, wv = threadIdx.x >> 6;
    bf16x4 wa[4][2], wb[2];      // rows 16 t .. 16 t + 15 of W2: two of h1, two of the aggregate
    const bf16x4 one = bias_row(1.f, q);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint32_t w[2];
            weights4(W, 16 * t, q, b, c, w);
            wa[t][b] = operand4(w[0], w[1]);
        }
        wb[b] = bias_row(W[2 * kH * kH + 16 * b + c], q);
    }
    auto raw = [&](int64_t row) { return *reinterpret_cast<const uint4 *>(h1 + row * kH + 8 * q); };
    const bool uneven = dense && xcd_uneven(rowptr, n);
    auto first = [&](uint32_t vb) {
        return ((int64_t)(uneven ? xcd_remap_chunked(vb, nvb) : xcd_remap(vb, nvb)) * 4 + wv) * 16;
    };
    auto row_of = [&](uint32_t vb) {
        const int64_t p = (vb < nvb ? first(vb) : 0) + c;
        return p < n ? p : n - 1;
    };
    RowAhead<U> cur, nxt;
    int64_t p = row_of(blockIdx.x), pn = row_of(blockIdx.x + gridDim.x);
    const int32_t nnz = rowptr[n];
    cur.extent(p, rowptr);
    nxt.extent(pn, rowptr);
    cur.entries(p, nnz, col, val, deg);
    for (uint32_t vb = blockIdx.x; vb < nvb; vb += gridDim.x) {
        uint4 xr[U];
        const uint4 own = raw(p);
#pragma unroll
        for (int i = 0; i < U; ++i) xr[i] = raw(cur.c[i]);
        nxt.entries(pn, nnz, col, val, deg);
        RowAhead<U> after;
        const int64_t pa = row_of(vb + 2 * gridDim.x);
        after.extent(pa, rowptr);
        float self[8], acc[8], a[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = 0.f;
        auto add = [&](int i) {
            float xv[8];
            unpack8(xr[i], xv);
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[t] = __builtin_fmaf(cur.w[i], xv[t], acc[t]);
        };
        if (cur.full()) {
#pragma unroll
            for (int i = 0; i < U; ++i) add(i);
        } else {
#pragma unroll
            for (int i = 0; i < U; ++i)
                if (i < cur.j1 - cur.j0) add(i);
        }
        gather_rest<U, U, (U > 4), uint4>(
            cur.j1 - cur.j0, col + cur.j0, val + cur.j0, [&](int64_t row, uint4 &o) { o = raw(row); },
            [&](float w, const uint4 &row) {
                float xv[8];
                unpack8(row, xv);
#pragma unroll
                for (int t = 0; t < 8; ++t) acc[t] = __builtin_fmaf(w, xv[t], acc[t]);
            });
        unpack8(own, self);
        row_mean(acc, self, cur.d, a);
        const bf16x4 item[4] = {operand4(own.x, own.y), operand4(own.z, own.w),
                                operand4(pack2(a[0], a[1]), pack2(a[2], a[3])),
                                operand4(pack2(a[4], a[5]), pack2(a[6], a[7]))};
        f32x4 out[2] = {};
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                out[b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wa[t][b], item[t], out[b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < 2; ++b) out[b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wb[b], one, out[b], 0, 0, 0);
        const int64_t node = first(vb) + c;
        if (node < n) store_relu(out, q, h2 + node * kH);
        cur = nxt;
        nxt = after;
        p = pn;
        pn = pa;
    }
}

// yhat_e = relu(z_e W3) . w4[0:32] + w4[32]; lane quarter q holds eight columns
// of |hp - hq| and of hp * hq (as k_layer2_mfma left them) and edge feature q.
// Candidates are loaded two tiles ahead, their ends one tile ahead.  All of an
// accumulator's products have one shape: the compiler (ROCm 7.2) puts a
// 16x16x16 right behind the 16x16x32 that writes its accumulator, without the
// wait states the longer product needs, and with the edge features' product as
// a 16x16x16 the sums lacked the products of hp * hq.
__global__ __launch_bounds__(256, kHeadWaves) void k_head_mfma(int64_t ne, uint32_t nvb,
                                                   const int32_t *__restrict__ cand,
                                                   const int32_t *__restrict__ u, const int32_t *__restrict__ v,
                                                   const __hip_bfloat16 *__restrict__ h,
                                                   const float *__restrict__ ef, const float *__restrict__ W3,
                                                   const float *__restrict__ w4, float *__restrict__ pred) {
    static_assert(kH == 32 && kE == 4, "head layout");
    const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15, wv = threadIdx.x >> 6;
    bfx8 wd[2], wp[2], we[2];
    f32x4 bias[2], last[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        uint32_t w[4];
        weights4(W3, 0, q, b, c, w);
        weights4(W3, 16, q, b, c, w + 2);
        wd[b] = operand8(w);
        weights4(W3, kH, q, b, c, w);
        weights4(W3, kH + 16, q, b, c, w + 2);
        wp[b] = operand8(w);
        const uint32_t f[4] = {pack2(W3[(2 * kH + q) * kH + 16 * b + c], 0.f), 0u, 0u, 0u};
        we[b] = operand8(f);
    }
    hidden8(W3 + kZ * kH, q, bias);
    hidden8(w4, q, last);
    const float w0 = w4[kH];
    auto item = [&](uint32_t vb) {
        const int64_t i = (vb < nvb ? ((int64_t)xcd_remap(vb, nvb) * 4 + wv) * 16 : 0) + c;
        return i < ne ? i : ne - 1;
    };
    auto edge = [&](int64_t i) { return cand ? cand[i] : (int32_t)i; };
    int64_t in = item(blockIdx.x + gridDim.x);
    int32_t e = edge(item(blockIdx.x)), en = edge(in);
    int32_t pu = u[e], pv = v[e];
    float f = ef[item(blockIdx.x) * kE + q];
    for (uint32_t vb = blockIdx.x; vb < nvb; vb += gridDim.x) {
        const uint4 rp = *reinterpret_cast<const uint4 *>(h + (int64_t)pu * kH + 8 * q);
        const uint4 rq = *reinterpret_cast<const uint4 *>(h + (int64_t)pv * kH + 8 * q);
        const int32_t nu = u[en], nv = v[en];
        const float nf = ef[in * kE + q];
        in = item(vb + 2 * gridDim.x);
        en = edge(in);
        float hp[8], hq[8];
        unpack8(rp, hp);
        unpack8(rq, hq);
        uint32_t dw[4], pw[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            dw[t] = pack2(hp[2 * t] - hq[2 * t], hp[2 * t + 1] - hq[2 * t + 1]) & 0x7fff7fffu;
            pw[t] = pack2(hp[2 * t] * hq[2 * t], hp[2 * t + 1] * hq[2 * t + 1]);
        }
        const uint32_t ew[4] = {pack2(f, 0.f), 0u, 0u, 0u};
        const bfx8 bd = operand8(dw), bp = operand8(pw), be = operand8(ew);
        float o = 0.f;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wd[b], bd, bias[b], 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wp[b], bp, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(we[b], be, acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) o = __builtin_fmaf(fmaxf(acc[r], 0.f), last[b][r], o);
        }
        o += __shfl_xor(o, 16);
        o += __shfl_xor(o, 32);
        const int64_t i = ((int64_t)xcd_remap(vb, nvb) * 4 + wv) * 16 + c;
        if (i < ne && q == 0) pred[i] = o + w0;
        pu = nu;
        pv = nv;
        f = nf;
    }
}

// ------------------------------------------------------------------ FP32 on the matrix cores
//
// v_mfma_f32_32x32x2_f32 (one 32 x 32 x 2 block per wavefront), lane l, half
// h = l / 32:
//   A (32 x 2):  row l % 32, column h
//   B (2 x 32):  column l % 32, row h
//   D (32 x 32): as above: column l % 32, rows tile_row(r, h), r = 0..15
// The order of the k index is free, so a step may take any two of the k
// values, one per half, as long as A and B agree: rows of a 32-wide operand
// are loaded as 16-byte pieces (half h of piece t holds k = 8t + 4h + 0..3),
// and a sum over the rows of a D tile takes its registers as they are.
// (Bound by the matrix cores' 64 cycles a step: 116 steps per 32 edges in the
// head, about 12 us for 123,201 edges on 1024 SIMDs.)

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // rows need not be 16-byte aligned

__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ int tile_row(int r, int half) { return 8 * (r / 4) + 4 * half + (r % 4); }

// h = relu([x | a | 1] W), 32 nodes per wavefront.
template <int FIN>
__global__ __launch_bounds__(256) void k_dense_f32(int64_t n, const float *__restrict__ x, const float *__restrict__ a,
                                                   const float *__restrict__ W, float *__restrict__ h) {
    constexpr int NX = FIN / 8;
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    float wx[NX][4], wa[NX][4];
#pragma unroll
    for (int t = 0; t < NX; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            wx[t][q] = W[(8 * t + 4 * half + q) * kH + col];
            wa[t][q] = W[(FIN + 8 * t + 4 * half + q) * kH + col];
        }
    const float bias = W[2 * FIN * kH + col];
    const int64_t base = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 32;
    if (base >= n) return;
    const int64_t row = base + col < n ? base + col : n - 1;      // past the end: computed, not stored
    f32x4u vx[NX], va[NX];
#pragma unroll
    for (int t = 0; t < NX; ++t) {
        vx[t] = *reinterpret_cast<const f32x4u *>(x + row * FIN + 8 * t + 4 * half);
        va[t] = *reinterpret_cast<const f32x4u *>(a + row * FIN + 8 * t + 4 * half);
    }
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = bias;
#pragma unroll
    for (int t = 0; t < NX; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = mfma32(vx[t][q], wx[t][q], acc);
#pragma unroll
    for (int t = 0; t < NX; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = mfma32(va[t][q], wa[t][q], acc);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t node = base + tile_row(r, half);
        if (node < n) h[node * kH + col] = fmaxf(acc[r], 0.f);
    }
}

// Sum of the workgroup's four wavefronts' tiles (NT accumulator tiles each,
// rows of the gradient in order) into partial[block][row * 32 + column], the
// wavefronts added in order.
template <int NT>
__device__ __forceinline__ void store_tiles(const f32x16 (&acc)[NT], int rows, float *sh /* 4 x 1056 */,
                                            float *__restrict__ partial) {
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31, wv = threadIdx.x >> 6;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) sh[wv * 1056 + tile_row(r, half) * 33 + col] = acc[t][r];
        __syncthreads();
        for (int e = threadIdx.x; e < 1024; e += 256) {
            const int i = e >> 5, j = e & 31;
            if (32 * t + i < rows) {
                const float *q = sh + i * 33 + j;
                partial[(32 * t + i) * kH + j] = ((q[0] + q[1056]) + q[2112]) + q[3168];
            }
        }
    }
}

// One number per lane, summed over the workgroup (lanes 0..31 of a wavefront
// hold 32 columns; both halves are added): partial[0..31].
__device__ __forceinline__ void store_cols(float v, float *sh /* 4 x 32 */, float *__restrict__ partial) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    v += __shfl_xor(v, 32, 64);
    __syncthreads();
    if (lane < 32) sh[wv * 32 + lane] = v;
    __syncthreads();
    if (threadIdx.x < 32)
        partial[threadIdx.x] = ((sh[threadIdx.x] + sh[32 + threadIdx.x]) + sh[64 + threadIdx.x]) + sh[96 + threadIdx.x];
}

constexpr int kTrainBlocks = 256;     // workgroups of the kernels that leave weight-gradient partials
constexpr int kNent3 = kZ1 * kH;      // W3 entries of a head partial, then w4's 33, then the loss
constexpr int kHeadPart = kNent3 + kH + 1 + 1;

// Edge head, 32 edges per wavefront: yhat_e = relu(z_e W3) . w4[0:32] + w4[32].
// TRAIN: a wavefront takes every 4 gridDim-th tile; besides the predictions it
// forms the output errors d_e = scale (yhat_e - y_e), the squared errors, the
// gradients at both ends' H2 rows (dhp, dhq per edge) and the head's weight
// gradients, its share of which goes to part[block][kHeadPart].
template <bool TRAIN>
__global__ __launch_bounds__(256) void k_head_f32(int64_t ne, const int32_t *__restrict__ cand,
                                                  const int32_t *__restrict__ u, const int32_t *__restrict__ v,
                                                  const float *__restrict__ h, const float *__restrict__ ef,
                                                  const float *__restrict__ W3, const float *__restrict__ w4,
                                                  float *__restrict__ pred, const float *__restrict__ target,
                                                  float scale, float *__restrict__ dhp, float *__restrict__ dhq,
                                                  float *__restrict__ part) {
    static_assert(kH == 32 && kE == 4, "head layout");
    __shared__ float s_d[4][32 * 33];                       // a wavefront's 32 x 32 tile, transposed through here
    __shared__ float s_p[TRAIN ? 4 : 1][TRAIN ? 32 * 33 : 1], s_q[TRAIN ? 4 : 1][TRAIN ? 32 * 33 : 1];
    __shared__ float s_e[TRAIN ? 4 : 1][TRAIN ? 32 * 8 : 1], s_err[TRAIN ? 4 : 1][TRAIN ? 32 : 1];
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31, wv = threadIdx.x >> 6;
    float w0[4][4], w1[4][4], we[4], wt0[TRAIN ? 4 : 1][4], wt1[TRAIN ? 4 : 1][4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 8 * t + 4 * half + q;
            w0[t][q] = W3[k * kH + col];
            w1[t][q] = W3[(kH + k) * kH + col];
            if constexpr (TRAIN) {
                wt0[t][q] = W3[col * kH + k];
                wt1[t][q] = W3[(kH + col) * kH + k];
            }
        }
    // the last four k of a half: the edge features, or the bias
#pragma unroll
    for (int q = 0; q < 4; ++q) we[q] = half == 0 ? W3[(2 * kH + q) * kH + col] : (q == 0 ? W3[kZ * kH + col] : 0.f);
    const float w4c = w4[col], w4b = w4[kH];
    f32x16 gw[TRAIN ? 3 : 1] = {};
    float g4 = 0.f, g4b = 0.f, loss = 0.f;
    const int64_t tiles = (ne + 31) / 32;
    for (int64_t tile = (int64_t)blockIdx.x * 4 + wv; tile < tiles; tile += (int64_t)gridDim.x * 4) {
        const int64_t base = tile * 32;
        const bool valid = base + col < ne;
        const int64_t i = valid ? base + col : ne - 1;
        const int32_t e = cand ? cand[i] : (int32_t)i;
        const float *hp = h + (int64_t)u[e] * kH + 4 * half, *hq = h + (int64_t)v[e] * kH + 4 * half;
        f32x4u a[4], b[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            a[t] = *reinterpret_cast<const f32x4u *>(hp + 8 * t);
            b[t] = *reinterpret_cast<const f32x4u *>(hq + 8 * t);
        }
        const f32x4u f = *reinterpret_cast<const f32x4u *>(ef + i * kE);
        float y = 0.f;
        if constexpr (TRAIN) y = target[i];
        f32x16 acc = {};
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc = mfma32(fabsf(a[t][q] - b[t][q]), w0[t][q], acc);
                acc = mfma32(a[t][q] * b[t][q], w1[t][q], acc);
            }
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = mfma32(half == 0 ? f[q] : (q == 0 ? 1.f : 0.f), we[q], acc);
        // the last layer: each lane scales its column, then two lanes add a row
        float *sd = s_d[wv];
#pragma unroll
        for (int r = 0; r < 16; ++r) sd[tile_row(r, half) * 33 + col] = fmaxf(acc[r], 0.f) * w4c;
        wave_lds_sync();
        float o = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) o += sd[col * 33 + 16 * half + j];
        o += __shfl_xor(o, 32, 64);
        o += w4b;
        if (half == 0 && valid) pred[i] = o;
        if constexpr (TRAIN) {
            float *sp = s_p[wv], *sq = s_q[wv], *se = s_e[wv], *sx = s_err[wv];
            const float err = valid ? o - y : 0.f;
            const float d = err * scale;
            if (half == 0) {
                loss = __builtin_fmaf(err, err, loss);
                g4b += d;
                sx[col] = d;
#pragma unroll
                for (int q = 0; q < 4; ++q) se[col * 8 + q] = f[q];
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    sp[col * 33 + 8 * t + 4 * half + q] = a[t][q];
                    sq[col * 33 + 8 * t + 4 * half + q] = b[t][q];
                }
            wave_lds_sync();
            // dG in the D layout (d is 0 on edges past the end), the w4 gradient, and W3's: z^T dG
            float dg[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = tile_row(r, half);
                const float dr = sx[row];
                g4 = __builtin_fmaf(fmaxf(acc[r], 0.f), dr, g4);
                dg[r] = acc[r] > 0.f ? dr * w4c : 0.f;
                const float pa = sp[row * 33 + col], pb = sq[row * 33 + col];
                const float ze = col < kE ? se[row * 8 + (col & 3)] : (col == kE ? 1.f : 0.f);
                gw[0] = mfma32(fabsf(pa - pb), dg[r], gw[0]);
                gw[1] = mfma32(pa * pb, dg[r], gw[1]);
                gw[2] = mfma32(ze, dg[r], gw[2]);
            }
            // dz = dG W3^T needs dG with a row per lane
#pragma unroll
            for (int r = 0; r < 16; ++r) sd[tile_row(r, half) * 33 + col] = dg[r];
            wave_lds_sync();
            f32x16 dz0 = {}, dz1 = {};
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float x = sd[col * 33 + 8 * t + 4 * half + q];
                    dz0 = mfma32(x, wt0[t][q], dz0);
                    dz1 = mfma32(x, wt1[t][q], dz1);
                }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = tile_row(r, half);
                const float pa = sp[row * 33 + col], pb = sq[row * 33 + col];
                const float sg = pa > pb ? 1.f : (pa < pb ? -1.f : 0.f);
                if (base + row < ne) {
                    dhp[(base + row) * kH + col] = dz0[r] * sg + dz1[r] * pb;
                    dhq[(base + row) * kH + col] = -dz0[r] * sg + dz1[r] * pa;
                }
            }
            wave_lds_sync();      // the next tile writes over this one's LDS
        }
    }
    if constexpr (TRAIN) {
        float *out = part + (int64_t)blockIdx.x * kHeadPart;
        store_tiles<3>(gw, kZ1, &s_d[0][0], out);
        store_cols(g4, &s_err[0][0], out + kNent3);
        // w4's bias and the loss: sums over the first half's 32 lanes, then the wavefronts
        for (int st = 16; st > 0; st >>= 1) {
            g4b += __shfl_xor(g4b, st, 64);
            loss += __shfl_xor(loss, st, 64);
        }
        __syncthreads();
        if (lane == 0) {
            s_err[0][wv] = g4b;
            s_err[0][4 + wv] = loss;
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            const float *q = s_err[0] + 4 * threadIdx.x;
            out[kNent3 + kH + threadIdx.x] = ((q[0] + q[1]) + q[2]) + q[3];
        }
    }
}

// dH2 at each node from its incident candidate edges, in ascending edge
// order, masked by the layer's ReLU (h > 0 exactly where its input was).
__global__ void k_gather_dh(int64_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                            const int32_t *__restrict__ eid, const float *__restrict__ dhp,
                            const float *__restrict__ dhq, const float *__restrict__ h, float *dpre) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;     // eight lanes a node, four columns each
    const int64_t p = t >> 3;
    const int c = (int)(t & 7) * 4;
    if (p >= n) return;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int32_t j = rp[p]; j < rp[p + 1]; ++j) {
        const int64_t i = eid[j];
        const float4 g = *reinterpret_cast<const float4 *>((col[j] > p ? dhp : dhq) + i * kH + c);
        acc[0] += g.x;
        acc[1] += g.y;
        acc[2] += g.z;
        acc[3] += g.w;
    }
    const float4 hv = *reinterpret_cast<const float4 *>(h + p * kH + c);
    *reinterpret_cast<float4 *>(dpre + p * kH + c) =
        make_float4(hv.x > 0.f ? acc[0] : 0.f, hv.y > 0.f ? acc[1] : 0.f, hv.z > 0.f ? acc[2] : 0.f,
                    hv.w > 0.f ? acc[3] : 0.f);
}

// Weight gradients of a dense layer, [x | a | 1]^T dP, as partials per
// workgroup (a wavefront takes every 4 gridDim-th tile of 32 nodes; rows of
// the tile two at a time are the k steps).  dP is dpre (layer 2, which also
// forms its input gradients t1 = dP Ws^T and t2 = (dP Wn^T) / D), or, in layer
// 1, t1 + c2 where the layer's output h is positive.
template <int FIN, bool INPUTS>
__global__ __launch_bounds__(256) void k_dense_grad(int64_t n, const float *__restrict__ x,
                                                    const float *__restrict__ a, const float *__restrict__ dpre,
                                                    const float *__restrict__ c2, const float *__restrict__ h,
                                                    const float *__restrict__ W, const float *__restrict__ deg,
                                                    float *__restrict__ t1, float *__restrict__ t2,
                                                    float *__restrict__ part) {
    constexpr int kRows = 2 * FIN + 1, NT = FIN == kH ? 2 : 1;
    static_assert(FIN == kH || 2 * FIN + 1 <= 32, "tiles of the weight gradient");
    __shared__ float sh[4 * 1056];
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31, wv = threadIdx.x >> 6;
    float ws[INPUTS ? 4 : 1][4], wn[INPUTS ? 4 : 1][4];
    if constexpr (INPUTS) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ws[t][q] = W[col * kH + 8 * t + 4 * half + q];
                wn[t][q] = W[(FIN + col) * kH + 8 * t + 4 * half + q];
            }
    }
    f32x16 gw[NT] = {};
    float gb = 0.f;
    const int64_t tiles = (n + 31) / 32;
    for (int64_t tile = (int64_t)blockIdx.x * 4 + wv; tile < tiles; tile += (int64_t)gridDim.x * 4) {
        const int64_t base = tile * 32;
        float dp[16], zx[16], za[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t node = base + 2 * r + half;
            const bool in = node < n;
            const int64_t at = (in ? node : n - 1) * kH + col;
            if constexpr (INPUTS)
                dp[r] = dpre[at];
            else
                dp[r] = h[at] > 0.f ? dpre[at] + c2[at] : 0.f;
            if (!in) dp[r] = 0.f;
            const int64_t row = (in ? node : n - 1) * FIN;
            if constexpr (FIN == kH) {
                zx[r] = x[row + col];
                za[r] = a[row + col];
            } else {
                zx[r] = col < FIN ? x[row + col] : (col < 2 * FIN ? a[row + col - FIN] : (col == 2 * FIN ? 1.f : 0.f));
                za[r] = 0.f;
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            gw[0] = mfma32(zx[r], dp[r], gw[0]);
            if constexpr (FIN == kH) {
                gw[NT - 1] = mfma32(za[r], dp[r], gw[NT - 1]);
                gb += dp[r];
            }
        }
        if constexpr (INPUTS) {
            const int64_t node = base + col < n ? base + col : n - 1;
            f32x4u d[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) d[t] = *reinterpret_cast<const f32x4u *>(dpre + node * kH + 8 * t + 4 * half);
            f32x16 o1 = {}, o2 = {};
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    o1 = mfma32(d[t][q], ws[t][q], o1);
                    o2 = mfma32(d[t][q], wn[t][q], o2);
                }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t p = base + tile_row(r, half);
                if (p < n) {
                    t1[p * kH + col] = o1[r];
                    t2[p * kH + col] = o2[r] * (1.f / deg[p]);
                }
            }
        }
    }
    float *out = part + (int64_t)blockIdx.x * kRows * kH;
    store_tiles<NT>(gw, FIN == kH ? 2 * FIN : kRows, sh, out);
    if constexpr (FIN == kH) store_cols(gb, sh, out + 2 * FIN * kH);
}

// The whole gradient and the loss from the partials: 8 lanes an entry, each
// adding every eighth partial, then pairs, fours and eights.
__global__ __launch_bounds__(256) void k_grad_finish(int nb1, int nb2, int nb3, const float *__restrict__ p1,
                                                     const float *__restrict__ p2, const float *__restrict__ p3,
                                                     float inv_ne, float *__restrict__ grad, float *__restrict__ loss) {
    // lanes of an entry are 32 apart, so that a load covers 32 consecutive entries
    __shared__ float sh[8][32];
    const int e = blockIdx.x * 32 + (threadIdx.x & 31), g = threadIdx.x >> 5;
    const float *p = nullptr;
    int nb = 0, stride = 0;
    if (e < kOffW2) {
        p = p1 + e;
        nb = nb1;
        stride = kU1 * kH;
    } else if (e < kOffW3) {
        p = p2 + (e - kOffW2);
        nb = nb2;
        stride = kU2 * kH;
    } else if (e < kParams + 1) {
        p = p3 + (e - kOffW3);
        nb = nb3;
        stride = kHeadPart;
    }
    float s0 = 0.f, s1 = 0.f;
    int b = g;
    for (; b + 8 < nb; b += 16) {
        s0 += p[(int64_t)b * stride];
        s1 += p[(int64_t)(b + 8) * stride];
    }
    if (b < nb) s0 += p[(int64_t)b * stride];
    sh[g][threadIdx.x & 31] = s0 + s1;
    __syncthreads();
    if (g == 0 && e < kParams + 1) {
        const int l = threadIdx.x;
        const float t =
            ((sh[0][l] + sh[1][l]) + (sh[2][l] + sh[3][l])) + ((sh[4][l] + sh[5][l]) + (sh[6][l] + sh[7][l]));
        if (e < kParams) grad[e] = t;
        else *loss = t * inv_ne;
    }
}

__global__ void k_gather_uv(int64_t ne, const int32_t *__restrict__ cand, const int32_t *__restrict__ u,
                            const int32_t *__restrict__ v, int32_t *cu, int32_t *cv, float *ones) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ne) return;
    const int32_t e = cand ? cand[i] : (int32_t)i;
    cu[i] = u[e];
    cv[i] = v[e];
    ones[i] = 1.f;
}

__global__ void k_fill_f32(int64_t n, float val, float *p) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = val;
}

__global__ void k_adam(int64_t n, float *theta, const float *__restrict__ g, float *m, float *v, float lr, float b1,
                       float b2, float c1, float c2, float eps) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / c1, vh = vi / c2;
    theta[i] = theta[i] - lr * mh / (sqrtf(vh) + eps);
}

// ------------------------------------------------------------------ plans

struct FwdPlan {
    void *a, *h1, *h2;
};

FwdPlan plan_fwd(Carver &c, int64_t n, sfg_dtype act) {
    FwdPlan p;
    const size_t s = dtype_size(act);
    p.a = act == SFG_F32 ? c.take<char>((size_t)n * kH * s) : nullptr;   // the BF16 layers aggregate in registers
    p.h1 = c.take<char>((size_t)n * kH * s);
    p.h2 = c.take<char>((size_t)n * kH * s);
    return p;
}

struct TrainPlan {
    float *a1, *h1, *a2, *h2, *dhp, *dhq, *dpre2, *t1, *t2, *c2, *ones_n, *ones_e, *part1, *part2, *part3, *incval,
        *incdeg;
    int32_t *cu, *cv, *irp, *icol, *ieid;
    void *csr_ws;
};

// Workgroups of a partial-sum kernel over tiles of 32 rows, four tiles each.
int train_blocks(int64_t rows) {
    const int64_t b = (rows + 127) / 128;
    return (int)(b > kTrainBlocks ? kTrainBlocks : b);
}

TrainPlan plan_train(Carver &c, int64_t n, int64_t ne) {
    TrainPlan p;
    p.a1 = c.take<float>(n * kF);
    p.h1 = c.take<float>(n * kH);
    p.a2 = c.take<float>(n * kH);
    p.h2 = c.take<float>(n * kH);
    p.dhp = c.take<float>((ne + 1) * kH);
    p.dhq = c.take<float>((ne + 1) * kH);
    p.dpre2 = c.take<float>(n * kH);
    p.t1 = c.take<float>(n * kH);
    p.t2 = c.take<float>(n * kH);
    p.c2 = c.take<float>(n * kH);
    p.ones_n = c.take<float>(n);
    p.ones_e = c.take<float>(ne + 1);
    p.part1 = c.take<float>((size_t)kTrainBlocks * kU1 * kH);
    p.part2 = c.take<float>((size_t)kTrainBlocks * kU2 * kH);
    p.part3 = c.take<float>((size_t)kTrainBlocks * kHeadPart);
    p.incval = c.take<float>(2 * ne + 1);
    p.incdeg = c.take<float>(n);
    p.cu = c.take<int32_t>(ne + 1);
    p.cv = c.take<int32_t>(ne + 1);
    p.irp = c.take<int32_t>(n + 1);
    p.icol = c.take<int32_t>(2 * ne + 1);
    p.ieid = c.take<int32_t>(2 * ne + 1);
    p.csr_ws = c.take<char>(csr_workspace_bytes(n, ne));
    return p;
}

void check_graph(const sfg_csr *G) {
    SFG_REQUIRE(G && G->rowptr && G->col && G->val && G->deg && G->n >= 1, SFG_EINVAL, "mpnn: graph CSR required");
    SFG_REQUIRE(G->vt == SFG_F32, SFG_EUNSUPPORTED, "mpnn: the graph CSR must be F32");
}

}  // namespace

size_t mpnn_forward_workspace_bytes(int64_t n, sfg_dtype act) {
    Carver c(nullptr);
    plan_fwd(c, n, act);
    return c.used + 256;
}

size_t mpnn_train_workspace_bytes(int64_t n, int64_t ne) {
    Carver c(nullptr);
    plan_train(c, n, ne);
    return c.used + 256;
}

}  // namespace sfg

extern "C" int64_t sfg_mpnn_param_count(void) { return sfg::kParams; }

extern "C" sfg_status sfg_mpnn_features(const sfg_csr *G, const sfg_csr *T, const float *xc, int32_t kc, int64_t ne,
                                        const int32_t *cand, const int32_t *u, const int32_t *v, const float *w,
                                        const float *norm, float *node_feat, float *edge_feat, void *stream) {
    return sfg::guard([&] {
        using namespace sfg;
        hipStream_t s = as_stream(stream);
        check_graph(G);
        check_graph(T);
        SFG_REQUIRE(T->n == G->n, SFG_EINVAL, "mpnn_features: G and T must have the same nodes");
        SFG_REQUIRE(xc && kc >= 1 && kc <= 64 && node_feat, SFG_EINVAL, "mpnn_features: bad block");
        SFG_REQUIRE(ne >= 0 && (ne == 0 || (u && v && w && edge_feat)), SFG_EINVAL, "mpnn_features: null pointer");
        const int64_t n = G->n;
        // 4- and 16-vector cheap embeddings with 16-byte aligned rows take vector loads
        const bool aligned = (uintptr_t)xc % 16 == 0 && (uintptr_t)node_feat % 16 == 0;
        const int kv = aligned && (kc == 4 || kc == 16) ? kc : 0;
        auto node = [&](auto kt) {
            constexpr int KC = decltype(kt)::value;
            hipLaunchKernelGGL(k_node_feat<KC>, dim3(grid_for(n, 256)), dim3(256), 0, s, n, G->rowptr, G->col,
                               (const float *)G->val, (const float *)G->deg, T->rowptr, T->col,
                               (const float *)T->val, (const float *)T->deg, xc, kc, norm, node_feat);
            SFG_LAUNCH_CHECK();
            if (ne > 0) {
                hipLaunchKernelGGL(k_edge_feat<KC>, dim3(grid_for(ne, 256)), dim3(256), 0, s, ne, cand, u, v, w, xc,
                                   kc, (const float *)T->deg, norm, edge_feat);
                SFG_LAUNCH_CHECK();
            }
        };
        if (kv == 4)
            node(std::integral_constant<int, 4>());
        else if (kv == 16)
            node(std::integral_constant<int, 16>());
        else
            node(std::integral_constant<int, 0>());
    });
}

extern "C" sfg_status sfg_mpnn_forward(const sfg_csr *G, const float *params, const float *node_feat, int64_t ne,
                                       const int32_t *cand, const int32_t *u, const int32_t *v,
                                       const float *edge_feat, sfg_dtype act, float *pred, void *ws, size_t ws_bytes,
                                       void *stream) {
    return sfg::guard([&] {
        using namespace sfg;
        hipStream_t s = as_stream(stream);
        check_graph(G);
        SFG_REQUIRE(params && node_feat, SFG_EINVAL, "mpnn_forward: null pointer");
        SFG_REQUIRE(act == SFG_F32 || act == SFG_BF16, SFG_EUNSUPPORTED, "mpnn_forward: activations F32 or BF16");
        SFG_REQUIRE(ws_bytes >= mpnn_forward_workspace_bytes(G->n, act), SFG_EWORKSPACE,
                    "mpnn_forward: workspace too small");
        const int64_t n = G->n;
        Carver c(ws);
        FwdPlan p = plan_fwd(c, n, act);
        const dim3 b(256);
        if (act == SFG_F32) {
            float *a = (float *)p.a, *h1 = (float *)p.h1, *h2 = (float *)p.h2;
            spmm_rownorm_f32(G, kF, node_feat, a, s);
            hipLaunchKernelGGL(k_dense_f32<kF>, dim3(grid_for(n, 128)), b, 0, s, n, node_feat, a, params + kOffW1, h1);
            SFG_LAUNCH_CHECK();
            spmm_rownorm_f32(G, kH, h1, a, s);
            hipLaunchKernelGGL(k_dense_f32<kH>, dim3(grid_for(n, 128)), b, 0, s, n, h1, a, params + kOffW2, h2);
            SFG_LAUNCH_CHECK();
        } else {
            __hip_bfloat16 *h1 = (__hip_bfloat16 *)p.h1, *h2 = (__hip_bfloat16 *)p.h2;
            // the first U entries of a row are in flight together: the average row of a lattice (6), 4 below, 8 above
            const bool dense = dense_rows(G);
            auto layers = [&](auto ut) {
                constexpr int U = decltype(ut)::value;
                const uint32_t nb1 = grid_for(n, 256), nb2 = grid_for(n, 64);
                hipLaunchKernelGGL(k_layer1_mfma<U>, dim3(tile_grid(nb1, kLayerWaves(U))), b, 0, s, n, nb1, dense,
                                   G->rowptr, G->col, (const float *)G->val, (const float *)G->deg, node_feat,
                                   params + kOffW1, h1);
                SFG_LAUNCH_CHECK();
                hipLaunchKernelGGL(k_layer2_mfma<U>, dim3(tile_grid(nb2, kLayerWaves(U))), b, 0, s, n, nb2, dense,
                                   G->rowptr, G->col, (const float *)G->val, (const float *)G->deg, h1,
                                   params + kOffW2, h2);
                SFG_LAUNCH_CHECK();
            };
            if (G->nnz <= 4 * n)
                layers(std::integral_constant<int, 4>());
            else if (G->nnz <= 6 * n)
                layers(std::integral_constant<int, 6>());
            else
                layers(std::integral_constant<int, 8>());
        }
        if (ne == 0) return;
        SFG_REQUIRE(u && v && edge_feat && pred, SFG_EINVAL, "mpnn_forward: null pointer");
        if (act == SFG_F32) {
            hipLaunchKernelGGL(k_head_f32<false>, dim3(grid_for(ne, 128)), b, 0, s, ne, cand, u, v,
                               (const float *)p.h2, edge_feat, params + kOffW3, params + kOffW4, pred, nullptr, 0.f,
                               nullptr, nullptr, nullptr);
        } else {
            const uint32_t nvb = grid_for(ne, 64);
            hipLaunchKernelGGL(k_head_mfma, dim3(tile_grid(nvb, kHeadWaves)), b, 0, s, ne, nvb, cand, u, v,
                               (const __hip_bfloat16 *)p.h2, edge_feat, params + kOffW3, params + kOffW4, pred);
        }
        SFG_LAUNCH_CHECK();
    });
}

extern "C" sfg_status sfg_mpnn_loss_grad(const sfg_csr *G, const float *params, const float *node_feat, int64_t ne,
                                         const int32_t *cand, const int32_t *u, const int32_t *v,
                                         const float *edge_feat, const float *target, float *pred, float *loss,
                                         float *grad, void *ws, size_t ws_bytes, void *stream) {
    return sfg::guard([&] {
        using namespace sfg;
        hipStream_t s = as_stream(stream);
        check_graph(G);
        SFG_REQUIRE(ne >= 1, SFG_EINVAL, "mpnn_loss_grad: need at least one edge");
        SFG_REQUIRE(params && node_feat && u && v && edge_feat && target && pred && loss && grad, SFG_EINVAL,
                    "mpnn_loss_grad: null pointer");
        const int64_t n = G->n;
        SFG_REQUIRE(ws_bytes >= mpnn_train_workspace_bytes(n, ne), SFG_EWORKSPACE,
                    "mpnn_loss_grad: workspace too small");
        Carver c(ws);
        TrainPlan p = plan_train(c, n, ne);
        const dim3 gn(grid_for(n, 256)), ge(grid_for(ne, 256)), b(256);
        // ---- forward
        spmm_rownorm_f32(G, kF, node_feat, p.a1, s);
        hipLaunchKernelGGL(k_dense_f32<kF>, dim3(grid_for(n, 128)), b, 0, s, n, node_feat, p.a1, params + kOffW1, p.h1);
        SFG_LAUNCH_CHECK();
        spmm_rownorm_f32(G, kH, p.h1, p.a2, s);
        hipLaunchKernelGGL(k_dense_f32<kH>, dim3(grid_for(n, 128)), b, 0, s, n, p.h1, p.a2, params + kOffW2, p.h2);
        SFG_LAUNCH_CHECK();
        // ---- edge head, forward and backward
        const int nbe = train_blocks(ne), nbn = train_blocks(n);
        hipLaunchKernelGGL(k_head_f32<true>, dim3(nbe), b, 0, s, ne, cand, u, v, p.h2, edge_feat, params + kOffW3,
                           params + kOffW4, pred, target, 2.f / (float)ne, p.dhp, p.dhq, p.part3);
        SFG_LAUNCH_CHECK();
        // edge gradients to nodes through the incidence CSR of the candidate edges
        hipLaunchKernelGGL(k_gather_uv, ge, b, 0, s, ne, cand, u, v, p.cu, p.cv, p.ones_e);
        SFG_LAUNCH_CHECK();
        build_csr(n, ne, p.cu, p.cv, p.ones_e, SFG_F32, nullptr, p.irp, p.icol, p.incval, p.ieid, p.incdeg, p.csr_ws,
                  csr_workspace_bytes(n, ne), s);
        hipLaunchKernelGGL(k_gather_dh, dim3(grid_for(n * 8, 256)), b, 0, s, n, p.irp, p.icol, p.ieid, p.dhp, p.dhq,
                           p.h2, p.dpre2);
        SFG_LAUNCH_CHECK();
        // ---- layer 2
        hipLaunchKernelGGL((k_dense_grad<kH, true>), dim3(nbn), b, 0, s, n, p.h1, p.a2, p.dpre2, nullptr, nullptr,
                           params + kOffW2, (const float *)G->deg, p.t1, p.t2, p.part2);
        SFG_LAUNCH_CHECK();
        // A (dP Wn^T / D): the sweep with unit degrees is the plain product
        hipLaunchKernelGGL(k_fill_f32, gn, b, 0, s, n, 1.f, p.ones_n);
        SFG_LAUNCH_CHECK();
        sfg_csr Gu = *G;
        Gu.deg = p.ones_n;
        spmm_rownorm_f32(&Gu, kH, p.t2, p.c2, s);
        // ---- layer 1, and the sums over the partials
        hipLaunchKernelGGL((k_dense_grad<kF, false>), dim3(nbn), b, 0, s, n, node_feat, p.a1, p.t1, p.c2, p.h1,
                           params + kOffW1, nullptr, nullptr, nullptr, p.part1);
        SFG_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_grad_finish, dim3(grid_for(kParams + 1, 32)), b, 0, s, nbn, nbn, nbe, p.part1, p.part2,
                           p.part3, 1.f / (float)ne, grad, loss);
        SFG_LAUNCH_CHECK();
    });
}

extern "C" sfg_status sfg_mpnn_adam(float *params, const float *grad, float *m, float *v, int64_t n, int64_t step,
                                    double lr, double beta1, double beta2, double eps, void *stream) {
    return sfg::guard([&] {
        using namespace sfg;
        SFG_REQUIRE(params && grad && m && v && n >= 1 && step >= 1, SFG_EINVAL, "mpnn_adam: bad arguments");
        const float c1 = (float)(1.0 - std::pow(beta1, (double)step));
        const float c2 = (float)(1.0 - std::pow(beta2, (double)step));
        hipLaunchKernelGGL(k_adam, dim3(grid_for(n, 256)), dim3(256), 0, as_stream(stream), n, params, grad, m, v,
                           (float)lr, (float)beta1, (float)beta2, c1, c2, (float)eps);
        SFG_LAUNCH_CHECK();
    });
}
