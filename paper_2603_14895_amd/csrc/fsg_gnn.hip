// fsg_gnn.hip -- learned surrogate of the Monte Carlo SIR spread: a
// mean-aggregation message-passing network (the message / aggregate / update
// structure of Eq. ms, Eq. agg, Eq. updata, here with learned functions),
// BF16 weights and activations with FP32 accumulation on MFMA, trained on the
// simulator's own Monte Carlo output by hand-written forward and backward
// kernels and Adam.
//
// Network (per node v, per seed set s; R = n_sets * n rows):
//   x_v  = [seed_v, 20 beta, log1p(indeg_v) / 8, 1,
//           20 beta log1p(indeg_v) / 8, log1p(k_s) / 8, log1p(D_s) / 16, 0 ... 0]
//                                                                   (16 wide)
//   with k_s the number of seeds of the set and D_s the sum of their
//   in-degrees (query-wide terms: a node further than three hops from every
//   seed sees the seed set only through them)
//   h1_v = ReLU(W1 [x_v | mean_{u in N-(v)} x_u] + b1)            (32 -> 64)
//   h2_v = ReLU(W2 [h1_v | mean h1_u] + b2)                        (128 -> 64)
//   h3_v = ReLU(W3 [h2_v | mean h2_u] + b3)                        (128 -> 64)
//   p_v  = sigmoid(wo . h3_v + bo)
// Loss: mean binary cross-entropy against per-node infection frequencies.
// A mean over an empty neighbourhood is 0.  Every stored BF16 value of the
// forward pass is its defining expression rounded once (to nearest even,
// through FP32): the means exactly so (FP64 sums), the layer outputs up to
// the FP32 rounding of the MFMA sums.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/fsg.h"
#include "fsg_internal.hpp"

namespace fsg {
namespace gnn {

constexpr int kF0 = 16;   // input features (padded)
constexpr int kHid = 64;  // hidden width
constexpr int kK1 = 2 * kF0, kK2 = 2 * kHid;
// flat FP32 parameter layout
constexpr int kW1 = 0, kB1 = kW1 + kK1 * kHid, kW2 = kB1 + kHid, kB2 = kW2 + kK2 * kHid,
              kW3 = kB2 + kHid, kB3 = kW3 + kK2 * kHid, kWo = kB3 + kHid, kBo = kWo + kHid,
              kP = kBo + 1;
// BF16 copies of W1, W2, W3 ([K][64] row-major each)
constexpr int kWb1 = 0, kWb2 = kWb1 + kK1 * kHid, kWb3 = kWb2 + kK2 * kHid,
              kWbN = kWb3 + kK2 * kHid;
constexpr int kHeadBlocks = 512;  // most blocks of the head's partial sums (deterministic sums)
constexpr int kDwBlocks = 512;    // most blocks of a weight-gradient product
constexpr int kMaxMembers = 64;   // ensemble members one spread estimate may combine
constexpr int kSlices = 4;        // members a spread estimate runs side by side

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__host__ __device__ inline uint16_t to_bf16(float f)
{
    union {
        float f;
        uint32_t u;
    } x;
    x.f = f;
    if ((x.u & 0x7F800000u) == 0x7F800000u) return (uint16_t)((x.u >> 16) | ((x.u & 0xFFFF) ? 0x40 : 0));
    x.u += 0x7FFFu + ((x.u >> 16) & 1u);  // round to nearest even
    return (uint16_t)(x.u >> 16);
}

__host__ __device__ inline float from_bf16(uint16_t h)
{
    union {
        uint32_t u;
        float f;
    } x;
    x.u = (uint32_t)h << 16;
    return x.f;
}

// ------------------------------------------------------------- kernels ----

// Value of lane J of the caller's 16-lane row (DPP row broadcast); every lane
// of the row must be active.
template <int J>
__device__ __forceinline__ uint32_t row_bcast(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x150 + J, 0xF, 0xF, false);
}

// Query-wide terms of every seed set: block b of a set adds up the seeds and
// their in-degrees in its share of the nodes into part[set][b] (kStatParts
// pairs; the set's first reader adds them).  Integer sums, so the result does
// not depend on the order of the additions.
constexpr int kStatParts = 32;

__global__ void __launch_bounds__(256) k_query_stats(const uint8_t *mask, const int32_t *ptr,
                                                     int32_t n, unsigned long long *part)
{
    const int s = blockIdx.x / kStatParts, b = blockIdx.x - s * kStatParts;
    const uint8_t *m = mask + (int64_t)s * n;
    unsigned long long k = 0, d = 0;
    for (int v = b * 256 + (int)threadIdx.x; v < n; v += kStatParts * 256)
        if (m[v]) {
            ++k;
            d += (unsigned long long)(ptr[v + 1] - ptr[v]);
        }
    for (int off = 32; off >= 1; off >>= 1) {
        k += __shfl_xor(k, off, 64);
        d += __shfl_xor(d, off, 64);
    }
    __shared__ unsigned long long sk[4], sd[4];
    if ((threadIdx.x & 63) == 0) {
        sk[threadIdx.x >> 6] = k;
        sd[threadIdx.x >> 6] = d;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = sk[0] + sk[1] + sk[2] + sk[3];
        part[2 * blockIdx.x + 1] = sd[0] + sd[1] + sd[2] + sd[3];
    }
}

// Input features.  Of the seven features of a row three depend on the node:
// x0 (seed), x2 (log degree) and x4 (its product with the rate); they go
// packed, 8 bytes a row, to Q, which the first aggregation gathers.  The
// others are the same for every node of a set (x1, x3, x5, x6) or zero: they
// go to C[set] as one 16-feature row with zeros at x0, x2, x4.  inv, if not
// null, gets 1 / indeg of every node (backward).  Grid: (blocks over nodes,
// n_sets).
__global__ void __launch_bounds__(256) k_input(uint2 *Q, uint16_t *C, const uint8_t *mask,
                                               const float *beta, const int32_t *ptr,
                                               const unsigned long long *part, int32_t n, float *inv)
{
    const int s = blockIdx.y;
    const double xb = 20.0 * (double)beta[s];
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        unsigned long long k = 0, d = 0;
        if (threadIdx.x < kStatParts) {
            k = part[2 * (s * kStatParts + threadIdx.x)];
            d = part[2 * (s * kStatParts + threadIdx.x) + 1];
        }
        for (int off = 32; off >= 1; off >>= 1) {
            k += __shfl_xor(k, off, 64);
            d += __shfl_xor(d, off, 64);
        }
        if (threadIdx.x < kF0) {
            float x = 0.f;
            if (threadIdx.x == 1) x = (float)xb;
            if (threadIdx.x == 3) x = 1.f;
            if (threadIdx.x == 5) x = (float)(log1p((double)k) * 0.125);
            if (threadIdx.x == 6) x = (float)(log1p((double)d) * 0.0625);
            C[s * kF0 + threadIdx.x] = to_bf16(x);
        }
    }
    for (int v = blockIdx.x * 256 + (int)threadIdx.x; v < n; v += (int)gridDim.x * 256) {
        const int64_t r = (int64_t)s * n + v;
        const int d = ptr[v + 1] - ptr[v];
        const double xd = log1p((double)d) * 0.125;
        const uint32_t x0 = to_bf16(mask[r] ? 1.f : 0.f), x2 = to_bf16((float)xd),
                       x4 = to_bf16((float)(xb * xd));
        Q[r] = make_uint2(x0 | (x2 << 16), x4);
        if (inv != nullptr && s == 0) inv[v] = d > 0 ? 1.f / (float)d : 0.f;
    }
}

// Adds the four BF16 values packed in q to four FP64 sums (exactly: a BF16
// value widens to FP64 without rounding).
__device__ __forceinline__ void add_bf16x4(double &a0, double &a1, double &a2, double &a3,
                                           uint2 q)
{
    a0 += (double)from_bf16((uint16_t)q.x);
    a1 += (double)from_bf16((uint16_t)(q.x >> 16));
    a2 += (double)from_bf16((uint16_t)q.y);
    a3 += (double)from_bf16((uint16_t)(q.y >> 16));
}

// BF16 of sum / deg: FP64 quotient, rounded to FP32, then to BF16 (nearest
// even at both steps); 0 for an empty neighbourhood.
__device__ __forceinline__ uint16_t mean_bf16(double sum, int deg)
{
    return deg > 0 ? to_bf16((float)(sum / (double)deg)) : (uint16_t)0;
}

// Mean aggregation over in-neighbours (pull CSR), BF16 result.  The BF16
// neighbour values are added in FP64, which holds such a sum exactly (8-bit
// significands: exact while the values span fewer than about 2^40 and the row
// has fewer than 2^5 ... 2^31 entries), and divided by the degree in FP64; the
// quotient goes to FP32 and then to BF16, both rounding to nearest even.  The
// stored mean is therefore the exact mean rounded as the definition rounds it,
// whatever the order of the additions.  (An FP32 sum scaled by a rounded
// 1/deg lands on the other side of a BF16 tie now and then; those one-unit
// flips then reach every later layer.)
//
// Rows above kWideRow arcs take a block each, the first blocks of the grid
// (largest first), so they run alongside the others.  The others are taken by
// decreasing degree (`order`, built with the graph): rows that share a wave
// then have about the same number of arcs (in node order of a Chung-Lu graph
// half the gather slots of a wave were padding: 258 us a layer for 8 sets of
// 1e5 nodes, 244 like this).
constexpr int kAggThreads = 512;
constexpr int kAggWaves = kAggThreads / 64;

// First layer: X1[r] = [x (16) | mean x (16)] from the packed features.  The
// mean of a feature that is the same for all nodes of a set is that feature
// (deg c / deg is exact), so only three are summed.  Four lanes a row split
// its arcs; an 8-byte gather an arc where the full feature row is 32 bytes
// (8 sets of 1e5 nodes: 93 us instead of 200 with the input's rows written and
// gathered whole).
__device__ __forceinline__ void input_row_out(uint16_t *X1, const uint16_t *C, const uint2 *Q,
                                              int64_t r, int s, int deg, double a0, double a2,
                                              double a4, int part)
{
    // lanes `part` of four: 16 bytes each of the 64-byte row
    const uint16_t *c = C + (int64_t)s * kF0 + (part & 1) * 8;
    uint4 o = *reinterpret_cast<const uint4 *>(c);  // x_{8p} .. x_{8p+7}; zeros at 0, 2, 4
    if (part == 0) {
        const uint2 q = Q[r];
        o.x |= q.x & 0xFFFFu;
        o.y |= q.x >> 16;
        o.z |= q.y & 0xFFFFu;
    } else if (part >= 2) {
        if (deg == 0) o = make_uint4(0u, 0u, 0u, 0u);
        if (part == 2) {
            o.x |= mean_bf16(a0, deg);
            o.y |= mean_bf16(a2, deg);
            o.z |= mean_bf16(a4, deg);
        }
    }
    *reinterpret_cast<uint4 *>(X1 + r * kK1 + 8 * part) = o;
}

__global__ void __launch_bounds__(kAggThreads) k_mean_input(uint16_t *X1, const uint2 *Q,
                                                            const uint16_t *C, const int32_t *ptr,
                                                            const int32_t *src, int32_t n,
                                                            int32_t n_sets, const int32_t *wide,
                                                            int32_t n_wide, const int32_t *order)
{
    __shared__ double s_part[kAggWaves][3];
    const int nwb = n_wide * n_sets;
    const int lane = threadIdx.x & 63;
    if ((int)blockIdx.x < nwb) {
        const int s = (int)blockIdx.x / n_wide;
        const int v = wide[(int)blockIdx.x - s * n_wide];
        const int e0 = ptr[v], deg = ptr[v + 1] - e0;
        const uint2 *q = Q + (int64_t)s * n;
        double a0 = 0.0, a2 = 0.0, a4 = 0.0, un = 0.0;
        for (uint32_t k = threadIdx.x; k < (uint32_t)deg; k += kAggThreads)
            add_bf16x4(a0, a2, a4, un, q[src[e0 + (int)k]]);
        for (int off = 32; off >= 1; off >>= 1) {
            a0 += __shfl_xor(a0, off, 64);
            a2 += __shfl_xor(a2, off, 64);
            a4 += __shfl_xor(a4, off, 64);
        }
        if (lane == 0) {
            s_part[threadIdx.x >> 6][0] = a0;
            s_part[threadIdx.x >> 6][1] = a2;
            s_part[threadIdx.x >> 6][2] = a4;
        }
        __syncthreads();
        if (threadIdx.x < 4) {
            a0 = a2 = a4 = 0.0;
            for (int w = 0; w < kAggWaves; ++w) {
                a0 += s_part[w][0];
                a2 += s_part[w][1];
                a4 += s_part[w][2];
            }
            input_row_out(X1, C, Q, (int64_t)s * n + v, s, deg, a0, a2, a4, threadIdx.x);
        }
        return;
    }
    const int32_t nl = n - n_wide;
    const int64_t R = (int64_t)nl * n_sets;
    const int64_t t0 = (int64_t)((int)blockIdx.x - nwb) * kAggThreads + threadIdx.x;
    const int64_t rows = (int64_t)((int)gridDim.x - nwb) * (kAggThreads / 4);
    const int part = (int)(t0 & 3);
    for (int64_t i = t0 >> 2; i < R; i += rows) {
        const int s = (int)(i / nl);
        const int v = order[i - (int64_t)s * nl];
        const int64_t r = (int64_t)s * n + v;
        const int e0 = ptr[v], e1 = ptr[v + 1], deg = e1 - e0;
        const uint2 *q = Q + (int64_t)s * n;
        double a0 = 0.0, a2 = 0.0, a4 = 0.0, un = 0.0;
        for (int e = e0 + part; e < e1; e += 32) {  // eight gathers in flight
            uint2 x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = q[src[min(e + 4 * j, e1 - 1)]];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                add_bf16x4(a0, a2, a4, un, e + 4 * j < e1 ? x[j] : make_uint2(0u, 0u));
        }
        for (int off = 1; off < 4; off <<= 1) {  // a row's four lanes are here together
            a0 += __shfl_xor(a0, off, 64);
            a2 += __shfl_xor(a2, off, 64);
            a4 += __shfl_xor(a4, off, 64);
        }
        input_row_out(X1, C, Q, r, s, deg, a0, a2, a4, part);
    }
}

// Calls f(slot, q, w) for the arcs [e0, e1) of the row that the caller's 16
// lanes own, q the lane's four BF16 features (8 bytes) of the arc's source row
// and w its weight (or 1): the 16 lanes load 16 consecutive sources with one
// load and receive each by DPP row broadcast, and 8 gathers are in flight (16
// for the weighted sums, whose kernel has half the waves to cover them: 405 to
// 390 us; the mean is faster with 8, 244 us against 252).
// Slots past the row's end carry q = 0.  All lanes of the wave call this
// together (the rows of its four groups differ).
template <bool WEIGHTED, typename F>
__device__ __forceinline__ void gather_rows(const uint16_t *base, int ld, const int32_t *src,
                                            const float *wt, int e0, int e1, F f)
{
    const int li = threadIdx.x & 15;
    const int d = e1 - e0;
    int dmax = 0;
#pragma unroll
    for (int l = 0; l < 64; l += 16) dmax = max(dmax, __builtin_amdgcn_readlane(d, l));
    auto src_at = [&](int b) -> uint32_t { return b + li < d ? (uint32_t)src[e0 + b + li] : 0u; };
    uint32_t cur = src_at(0);
    for (int b = 0; b < dmax; b += 16) {
        uint32_t w = 0;
        if (WEIGHTED) w = __builtin_bit_cast(uint32_t, wt[cur]);
        const uint32_t nxt = b + 16 < dmax ? src_at(b + 16) : 0u;
        auto take = [&](auto... js) {
            uint2 q[sizeof...(js)];
            int i = 0;
            ((q[i++] = *reinterpret_cast<const uint2 *>(
                  base + (uint64_t)row_bcast<decltype(js)::value>(cur) * (uint32_t)ld)),
             ...);
            i = 0;
            ((f(b + decltype(js)::value < d ? q[i] : make_uint2(0u, 0u),
                WEIGHTED ? __builtin_bit_cast(float, row_bcast<decltype(js)::value>(w)) : 1.f),
              ++i),
             ...);
        };
        if (WEIGHTED && dmax - b > 8) {
            take(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{},
                 std::integral_constant<int, 2>{}, std::integral_constant<int, 3>{},
                 std::integral_constant<int, 4>{}, std::integral_constant<int, 5>{},
                 std::integral_constant<int, 6>{}, std::integral_constant<int, 7>{},
                 std::integral_constant<int, 8>{}, std::integral_constant<int, 9>{},
                 std::integral_constant<int, 10>{}, std::integral_constant<int, 11>{},
                 std::integral_constant<int, 12>{}, std::integral_constant<int, 13>{},
                 std::integral_constant<int, 14>{}, std::integral_constant<int, 15>{});
        } else {
            take(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{},
                 std::integral_constant<int, 2>{}, std::integral_constant<int, 3>{},
                 std::integral_constant<int, 4>{}, std::integral_constant<int, 5>{},
                 std::integral_constant<int, 6>{}, std::integral_constant<int, 7>{});
            if (dmax - b > 8)
                take(std::integral_constant<int, 8>{}, std::integral_constant<int, 9>{},
                     std::integral_constant<int, 10>{}, std::integral_constant<int, 11>{},
                     std::integral_constant<int, 12>{}, std::integral_constant<int, 13>{},
                     std::integral_constant<int, 14>{}, std::integral_constant<int, 15>{});
        }
        cur = nxt;
    }
}

// Hidden layers: X[r][64 .. 127] = mean of X[s*n + u][0 .. 63].  A wave takes
// four rows, 16 lanes each (four features a lane, 128 bytes a gathered row),
// so a row's sums stay in its lanes and the divisions of four rows are shared
// by one wave.  Bound by the gathers (2 GB a layer for 8 sets of 1e5 nodes, 2e6
// arcs, mostly from the Infinity Cache) and the widening to FP64: 244 us a
// layer; with a wave a row, its lanes over neighbours and a butterfly at the
// end, 490.
__global__ void __launch_bounds__(kAggThreads) k_mean(uint16_t *X, const int32_t *ptr,
                                                      const int32_t *src, int32_t n, int32_t n_sets,
                                                      const int32_t *wide, int32_t n_wide,
                                                      const int32_t *order)
{
    __shared__ double s_part[4 * kAggWaves][kHid];
    const int nwb = n_wide * n_sets;
    const int gi = threadIdx.x >> 4, li = threadIdx.x & 15;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    auto add = [&](uint2 q, float) { add_bf16x4(a0, a1, a2, a3, q); };
    if ((int)blockIdx.x < nwb) {
        const int s = (int)blockIdx.x / n_wide;
        const int v = wide[(int)blockIdx.x - s * n_wide];
        const int e0 = ptr[v], deg = ptr[v + 1] - e0;
        const int per = ((deg + 4 * kAggWaves - 1) / (4 * kAggWaves) + 15) & ~15;
        int lo, hi;
        share_of(deg, per, gi, lo, hi);
        gather_rows<false>(X + (int64_t)s * n * kK2 + 4 * li, kK2, src, nullptr, e0 + lo, e0 + hi, add);
        s_part[gi][4 * li] = a0;
        s_part[gi][4 * li + 1] = a1;
        s_part[gi][4 * li + 2] = a2;
        s_part[gi][4 * li + 3] = a3;
        __syncthreads();
        if ((int)threadIdx.x < kHid) {
            double acc = 0.0;
            for (int g = 0; g < 4 * kAggWaves; ++g) acc += s_part[g][threadIdx.x];
            X[((int64_t)s * n + v) * kK2 + kHid + threadIdx.x] = mean_bf16(acc, deg);
        }
        return;
    }
    const int32_t nl = n - n_wide;
    const int64_t R = (int64_t)nl * n_sets;
    const int64_t step = (int64_t)((int)gridDim.x - nwb) * (kAggThreads / 16);
    // every lane of a wave stays in the loop while its first row exists
    const int64_t first = ((int64_t)((int)blockIdx.x - nwb) * kAggThreads + (threadIdx.x & ~63)) >> 4;
    for (int64_t i0 = first; i0 < R; i0 += step) {
        const int64_t i = i0 + (gi & 3);
        int64_t sb = 0, r = 0;
        int e0 = 0, e1 = 0;
        const bool mine = i < R;
        if (mine) {
            const int s = (int)(i / nl);
            const int v = order[i - (int64_t)s * nl];
            sb = (int64_t)s * n;
            r = sb + v;
            e0 = ptr[v];
            e1 = ptr[v + 1];
        }
        a0 = a1 = a2 = a3 = 0.0;
        gather_rows<false>(X + sb * kK2 + 4 * li, kK2, src, nullptr, e0, e1, add);
        if (mine) {
            const int deg = e1 - e0;
            uint2 o;
            o.x = (uint32_t)mean_bf16(a0, deg) | ((uint32_t)mean_bf16(a1, deg) << 16);
            o.y = (uint32_t)mean_bf16(a2, deg) | ((uint32_t)mean_bf16(a3, deg) << 16);
            *reinterpret_cast<uint2 *>(X + r * kK2 + kHid + 4 * li) = o;
        }
    }
}

// ---- products on MFMA -------------------------------------------------------
// All run with the output's columns as the instruction's rows and the data
// rows as its columns, so a lane ends with four consecutive columns of one
// data row in each 16 x 16 tile and stores 8 bytes at a time.

__device__ __forceinline__ bf16x4 as_bf16x4(uint2 q) { return __builtin_bit_cast(bf16x4, q); }

// Weights of one slice (a network of an ensemble, or the one trained).
struct Weights {
    const uint16_t *w;  // BF16 [K][64]
    const float *b;     // [64]
    const float *wo;    // [64], head only
    const float *bo;
};
struct SliceWeights {
    Weights s[kSlices];
};

// The head's outputs: probabilities of the rows, and when training (y not
// null) dZ of the last layer and per-block partial sums of the gradients of wo
// and bo and of the loss ([64], [1], [1] per block).
struct HeadArgs {
    float *prob;
    const float *y;
    uint16_t *dZ;
    float *part;  // [blocks][66]
    float rows;
};

// out = ReLU(A . W + bias) in BF16, 16 rows a wave and pass, the weights in
// registers; grid (blocks, slices), slice y works on its `rows` rows with its
// own weights.  A slice stride of 0 for A shares the input.  With HEAD the
// rows stay in registers: p = sigmoid(wo . h + bo) and, when training, dz =
// (p - y) / R, dZ = BF16(dz wo [h > 0]) and the sums of dz h, dz and the
// cross-entropy (stable form from the logit) -- the last layer's activations
// and their gradients in 32 bits never reach memory.  Out may be A's own rows
// (a wave reads its rows before it writes them).
// Bound by reading A (205 MB for 8e5 rows): 80 us; 104 with 2-byte LDS reads
// of the weights per product; the separate head took
// 498 (a row a wave), inside the last layer 105 for both.
template <int K, bool HEAD>
__global__ void __launch_bounds__(256) k_layer(const uint16_t *A, int64_t a_stride, SliceWeights sw,
                                               uint16_t *out, int64_t out_stride, int64_t rows,
                                               HeadArgs h)
{
    const Weights w = sw.s[blockIdx.y];
    A += a_stride * (int64_t)blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    // the weights reach their lanes through LDS (16-byte loads, then two bytes
    // at a time once a block)
    __shared__ __align__(16) uint16_t s_w[K * kHid];
    for (int i = threadIdx.x; i < K * kHid / 8; i += 256)
        *reinterpret_cast<uint4 *>(&s_w[8 * i]) = *reinterpret_cast<const uint4 *>(w.w + 8 * i);
    __syncthreads();
    bf16x4 wf[K / 16][4];
#pragma unroll
    for (int k = 0; k < K / 16; ++k)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) wf[k][t][j] = (short)s_w[(16 * k + 4 * lk + j) * kHid + 16 * t + li];
    float bias[4][4], wo[4][4], gw[4][4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            bias[t][i] = w.b[16 * t + 4 * lk + i];
            if (HEAD) {
                wo[t][i] = w.wo[16 * t + 4 * lk + i];
                gw[t][i] = 0.f;
            }
        }
    const float bo = HEAD ? w.bo[0] : 0.f;
    float gb = 0.f, ls = 0.f;
    const int64_t step = (int64_t)gridDim.x * 64;
    const int64_t first = ((int64_t)blockIdx.x * 4 + wave) * 16;
    for (int64_t r0 = first; r0 < rows; r0 += step) {
        const int64_t r = r0 + li;
        const bool in = r < rows;
        const uint16_t *pa = A + min(r, rows - 1) * K + 4 * lk;
        uint2 af[K / 16];
#pragma unroll
        for (int k = 0; k < K / 16; ++k) af[k] = *reinterpret_cast<const uint2 *>(pa + 16 * k);
        f32x4 acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < K / 16; ++k)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wf[k][t], as_bf16x4(af[k]), acc[t], 0, 0, 0);
        uint16_t hv[4][4];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float v = acc[t][i] + bias[t][i];
                hv[t][i] = to_bf16(v > 0.f ? v : 0.f);
            }
        if (!HEAD) {
            if (in) {
                uint16_t *po = out + out_stride * (int64_t)blockIdx.y + r * kK2 + 4 * lk;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    *reinterpret_cast<uint2 *>(po + 16 * t) =
                        make_uint2((uint32_t)hv[t][0] | ((uint32_t)hv[t][1] << 16),
                                   (uint32_t)hv[t][2] | ((uint32_t)hv[t][3] << 16));
            }
            continue;
        }
        // logit: column c's product plus that of c ^ 32, c ^ 16, ... c ^ 1 in
        // turn (t, then lanes, then i hold the bits of c)
        float p0[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) x[t] = from_bf16(hv[t][i]) * wo[t][i];
            p0[i] = (x[0] + x[2]) + (x[1] + x[3]);
            p0[i] += __shfl_xor(p0[i], 32, 64);
            p0[i] += __shfl_xor(p0[i], 16, 64);
        }
        const float z = ((p0[0] + p0[2]) + (p0[1] + p0[3])) + bo;
        const float p = 1.f / (1.f + expf(-z));
        if (in && lk == 0) h.prob[(int64_t)blockIdx.y * rows + r] = p;
        if (h.y == nullptr || !in) continue;
        const float t = h.y[r];
        const float dz = (p - t) / h.rows;
        uint16_t *po = h.dZ + r * kHid + 4 * lk;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t g[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float x = from_bf16(hv[q][i]);
                gw[q][i] += dz * x;
                g[i] = to_bf16(x > 0.f ? dz * wo[q][i] : 0.f);
            }
            *reinterpret_cast<uint2 *>(po + 16 * q) = make_uint2(g[0] | (g[1] << 16), g[2] | (g[3] << 16));
        }
        if (lk == 0) {
            gb += dz;
            ls += fmaxf(z, 0.f) - z * t + log1pf(expf(-fabsf(z)));
        }
    }
    if (!HEAD || h.y == nullptr) return;
    __shared__ float s_g[4][kHid];
    __shared__ float s_b[4][2];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x = gw[t][i];
            for (int off = 1; off < 16; off <<= 1) x += __shfl_xor(x, off, 64);
            if (li == 0) s_g[wave][16 * t + 4 * lk + i] = x;
        }
    for (int off = 1; off < 64; off <<= 1) {
        gb += __shfl_xor(gb, off, 64);
        ls += __shfl_xor(ls, off, 64);
    }
    if (lane == 0) {
        s_b[wave][0] = gb;
        s_b[wave][1] = ls;
    }
    __syncthreads();
    float *pp = h.part + (int64_t)blockIdx.x * 66;
    if (threadIdx.x < kHid)
        pp[threadIdx.x] = s_g[0][threadIdx.x] + s_g[1][threadIdx.x] + s_g[2][threadIdx.x] + s_g[3][threadIdx.x];
    else if (threadIdx.x < kHid + 2) {
        const int i = threadIdx.x - kHid;
        pp[threadIdx.x] = s_b[0][i] + s_b[1][i] + s_b[2][i] + s_b[3][i];
    }
}

// Backward through one layer and the transposed mean in one kernel:
//   dH[u] = dZ[u] . Wa^T + G[u] . Wb^T,  G[u] = sum_{v : u in N-(v)} dZ[v] / indeg(v),
//   dZprev[u] = BF16(dH[u] [h_u > 0]),
// Wa and Wb the upper and lower halves of W, G pulled over the out-arcs of u
// (the in-CSR of the reversed graph) and h the layer's input.  Aggregating dZ
// (128 bytes a row) before the product instead of dZ . Wb^T (256 bytes, 32 bits)
// after it halves the gathered bytes and leaves no gradient in 32 bits in
// memory; G is summed in FP32 and multiplied in FP32 (v_mfma_f32_16x16x4_f32),
// so nothing is rounded to 16 bits that was not before.  A wave takes 16 rows:
// its four 16-lane groups pull four rows at a time into its own LDS tile, then
// it multiplies.  Rows above kWideRow out-arcs take a block each, first in the
// grid.  Bound by the gathers (2 GB a layer for 8 sets of 1e5 nodes): 390 us a
// layer, where the product, the two gathers of its FP32 rows and the masking
// pass took 1170.
constexpr int kBwdThreads = 256;
constexpr int kGPitch = kHid + 4;  // floats of a G row in LDS
constexpr int kWPitch = kHid + 4;  // values of a weight row in LDS

__global__ void __launch_bounds__(kBwdThreads) k_layer_bwd(const uint16_t *dZ, const uint16_t *W,
                                                           const uint16_t *H, uint16_t *out,
                                                           const float *inv, const int32_t *rptr,
                                                           const int32_t *rdst, int32_t n,
                                                           int32_t n_sets, const int32_t *wide,
                                                           int32_t n_wide, const int32_t *order)
{
    __shared__ __align__(16) uint16_t s_w[kK2 * kWPitch];
    __shared__ __align__(16) float s_g[kBwdThreads / 64][16][kGPitch];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const int nwb = n_wide * n_sets;
    float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
    auto add = [&](uint2 q, float w) {
        g.x += from_bf16((uint16_t)q.x) * w;
        g.y += from_bf16((uint16_t)(q.x >> 16)) * w;
        g.z += from_bf16((uint16_t)q.y) * w;
        g.w += from_bf16((uint16_t)(q.y >> 16)) * w;
    };
    if ((int)blockIdx.x < nwb) {
        const int s = (int)blockIdx.x / n_wide;
        const int u = wide[(int)blockIdx.x - s * n_wide];
        const int64_t r = (int64_t)s * n + u;
        const int e0 = rptr[u], deg = rptr[u + 1] - e0;
        const int groups = kBwdThreads / 16, gi = threadIdx.x >> 4;
        const int per = ((deg + groups - 1) / groups + 15) & ~15;
        int lo, hi;
        share_of(deg, per, gi, lo, hi);
        gather_rows<true>(dZ + (int64_t)s * n * kHid + 4 * li, kHid, rdst, inv, e0 + lo, e0 + hi, add);
        *reinterpret_cast<float4 *>(&s_g[wave][lk][4 * li]) = g;
        __syncthreads();
        if (threadIdx.x < kHid) {
            float x = 0.f;
            for (int w = 0; w < kBwdThreads / 64; ++w)
                for (int k = 0; k < 4; ++k) x += s_g[w][k][threadIdx.x];
            s_g[0][8][threadIdx.x] = x;
            s_g[0][9][threadIdx.x] = from_bf16(dZ[r * kHid + threadIdx.x]);
        }
        __syncthreads();
        if (threadIdx.x < kHid) {
            const uint16_t *wa = W + threadIdx.x * kHid, *wb = W + (kHid + threadIdx.x) * kHid;
            float x = 0.f, y = 0.f;
            for (int c = 0; c < kHid; ++c) {
                x += s_g[0][9][c] * from_bf16(wa[c]);
                y += s_g[0][8][c] * from_bf16(wb[c]);
            }
            out[r * kHid + threadIdx.x] =
                to_bf16(from_bf16(H[r * kK2 + threadIdx.x]) > 0.f ? x + y : 0.f);
        }
        return;
    }
    // weights in LDS (in registers they leave room for two waves a SIMD,
    // too few to cover the gathers: 547 us a layer, 390 like this)
    for (int i = threadIdx.x; i < kK2 * kHid / 4; i += kBwdThreads)
        *reinterpret_cast<uint2 *>(&s_w[(i >> 4) * kWPitch + 4 * (i & 15)]) =
            *reinterpret_cast<const uint2 *>(W + 4 * i);
    __syncthreads();
    const int32_t nl = n - n_wide;
    const int64_t R = (int64_t)nl * n_sets;
    const int64_t step = (int64_t)((int)gridDim.x - nwb) * (kBwdThreads / 4);
    for (int64_t i0 = ((int64_t)((int)blockIdx.x - nwb) * (kBwdThreads / 64) + wave) * 16; i0 < R; i0 += step) {
        // row li of the tile (the same in the four lane groups)
        const int64_t i = i0 + li;
        const bool mine = i < R;
        const int64_t ic = mine ? i : R - 1;
        const int s = (int)(ic / nl);
        const int u = order[ic - (int64_t)s * nl];
        const int64_t r = (int64_t)s * n + u;
        const int p0 = rptr[u], p1 = mine ? rptr[u + 1] : p0;
#pragma unroll 1
        for (int k = 0; k < 4; ++k) {
            const int from = (lane & 48) | (4 * k + lk);  // this group's row of the pass
            const int e0 = __shfl(p0, from, 64), e1 = __shfl(p1, from, 64);
            const int sk = __shfl(s, from, 64);
            g = make_float4(0.f, 0.f, 0.f, 0.f);
            gather_rows<true>(dZ + (int64_t)sk * n * kHid + 4 * li, kHid, rdst, inv, e0, e1, add);
            *reinterpret_cast<float4 *>(&s_g[wave][4 * k + lk][4 * li]) = g;
        }
        // the tile is the wave's own: its LDS accesses stay in order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint2 zf[4], hf[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            zf[q] = *reinterpret_cast<const uint2 *>(dZ + r * kHid + 16 * q + 4 * lk);
            hf[q] = *reinterpret_cast<const uint2 *>(H + r * kK2 + 16 * q + 4 * lk);
        }
        f32x4 acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 gv = *reinterpret_cast<const float4 *>(&s_g[wave][li][16 * q + 4 * lk]);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const uint16_t *wr = &s_w[(16 * t + li) * kWPitch + 16 * q + 4 * lk];
                const uint2 wa = *reinterpret_cast<const uint2 *>(wr);
                const uint2 b = *reinterpret_cast<const uint2 *>(wr + kHid * kWPitch);
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_bf16x4(wa), as_bf16x4(zf[q]), acc[t],
                                                                  0, 0, 0);
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(from_bf16((uint16_t)b.x), gv.x, acc[t], 0, 0, 0);
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(from_bf16((uint16_t)(b.x >> 16)), gv.y, acc[t], 0, 0, 0);
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(from_bf16((uint16_t)b.y), gv.z, acc[t], 0, 0, 0);
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(from_bf16((uint16_t)(b.y >> 16)), gv.w, acc[t], 0, 0, 0);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (mine) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint32_t o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t hb = i < 2 ? hf[t].x : hf[t].y;
                    const float hx = from_bf16((uint16_t)(hb >> (16 * (i & 1))));
                    o[i] = to_bf16(hx > 0.f ? acc[t][i] : 0.f);
                }
                *reinterpret_cast<uint2 *>(out + r * kHid + 16 * t + 4 * lk) =
                    make_uint2(o[0] | (o[1] << 16), o[2] | (o[3] << 16));
            }
        }
    }
}

// Weight and bias gradients of one layer: part[b][k][c] = sum over the block's
// rows of X[row][k] dZ[row][c] on MFMA (32x32x16, the rows are the
// contraction), then the column sums of dZ.  Chunks of 64 rows: a thread loads
// 16 bytes of two neighbouring rows and writes them to LDS transposed, two
// rows of one column to a word, so an operand (8 rows of one column) is one
// 16-byte LDS read; the next chunk's loads are in flight meanwhile.  K = 128:
// wave w owns features 32 w .. 32 w + 31; K = 32: wave w owns 16 rows of each
// chunk and writes a partial of its own.  Bound by reading X and dZ once (307 MB
// for 8e5 rows): 64 us; with 2-byte LDS staging and reads 346.
constexpr int kDwPitch = 36;  // words of an LDS column (32 row pairs)
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 mbf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <int K>
constexpr int dw_part_len() { return K * kHid; }

template <int K>
__global__ void __launch_bounds__(256) k_layer_dw(const uint16_t *X, const uint16_t *dZ, float *part,
                                                  float *part_b, int64_t R)
{
    __shared__ __align__(16) uint32_t sX[K * kDwPitch];
    __shared__ __align__(16) uint32_t sZ[kHid * kDwPitch];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int kXT = K / 64 > 0 ? K / 64 : 1;  // tasks (row pair, 8 columns) a thread: X
    // task i of thread t: columns 8 q .. 8 q + 7 of row pair p
    auto xq = [&](int i) { return K == 128 ? ((int)threadIdx.x & 3) + 4 * (((int)threadIdx.x >> 7) + 2 * i)
                                           : (int)threadIdx.x & 3; };
    const int p = ((int)threadIdx.x >> 2) & 31;
    const int zq = ((int)threadIdx.x & 3) + 4 * ((int)threadIdx.x >> 7);
    const bool has_x = K == 128 || threadIdx.x < 128;
    uint4 x0[kXT], x1[kXT], z0, z1;
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
    auto load = [&](int64_t c0) {
        const int64_t ra = c0 + 2 * p, rb = ra + 1;
#pragma unroll
        for (int i = 0; i < kXT; ++i) {
            x0[i] = has_x && ra < R ? *reinterpret_cast<const uint4 *>(X + ra * K + 8 * xq(i)) : zero;
            x1[i] = has_x && rb < R ? *reinterpret_cast<const uint4 *>(X + rb * K + 8 * xq(i)) : zero;
        }
        z0 = ra < R ? *reinterpret_cast<const uint4 *>(dZ + ra * kHid + 8 * zq) : zero;
        z1 = rb < R ? *reinterpret_cast<const uint4 *>(dZ + rb * kHid + 8 * zq) : zero;
    };
    auto put = [&](uint32_t *dst, int q, const uint4 &a, const uint4 &b) {
        const uint32_t av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            dst[(8 * q + 2 * i) * kDwPitch + p] = (av[i] & 0xFFFFu) | (bv[i] << 16);
            dst[(8 * q + 2 * i + 1) * kDwPitch + p] = (av[i] >> 16) | (bv[i] & 0xFFFF0000u);
        }
    };
    float gb[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) gb[i] = 0.f;
    f32x16 acc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
    const int64_t stride = (int64_t)gridDim.x * 64;
    int64_t c0 = (int64_t)blockIdx.x * 64;
    load(c0);
    for (; c0 < R; c0 += stride) {
        __syncthreads();
        if (has_x) {
#pragma unroll
            for (int i = 0; i < kXT; ++i) put(sX, xq(i), x0[i], x1[i]);
        }
        put(sZ, zq, z0, z1);
        const uint32_t zv[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            gb[2 * (i & 3)] += from_bf16((uint16_t)zv[i]);
            gb[2 * (i & 3) + 1] += from_bf16((uint16_t)(zv[i] >> 16));
        }
        __syncthreads();
        load(c0 + stride);  // (past the end: zeros)
        const int m = lane & 31, kh = lane >> 5;
        auto step = [&](int ks, int f0) {  // 16 rows: pairs 8 ks + 4 kh .. + 3
            const uint4 a = *reinterpret_cast<const uint4 *>(&sX[(f0 + m) * kDwPitch + 8 * ks + 4 * kh]);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint4 b = *reinterpret_cast<const uint4 *>(&sZ[(32 * t + m) * kDwPitch + 8 * ks + 4 * kh]);
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(mbf16x8, a),
                                                                 __builtin_bit_cast(mbf16x8, b), acc[t], 0, 0, 0);
            }
        };
        if (K == 128) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) step(ks, 32 * wave);
        } else {
            step(wave, 0);
        }
    }
    float *pb = part + ((int64_t)blockIdx.x * (K == 128 ? 1 : 4) + (K == 128 ? 0 : wave)) * dw_part_len<K>();
    const int f0 = K == 128 ? 32 * wave : 0;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i)
            pb[(f0 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3)) * kHid + 32 * t + (lane & 31)] = acc[t][i];
    // column sums of dZ: the 32 threads of a column group in order
    __syncthreads();
    float *sB = reinterpret_cast<float *>(sZ);  // [8 groups][32][8]
#pragma unroll
    for (int i = 0; i < 8; ++i) sB[(zq * 32 + p) * 8 + i] = gb[i];
    __syncthreads();
    if (threadIdx.x < kHid) {
        float x = 0.f;
        for (int k = 0; k < 32; ++k) x += sB[((threadIdx.x >> 3) * 32 + k) * 8 + (threadIdx.x & 7)];
        part_b[(int64_t)blockIdx.x * kHid + threadIdx.x] = x;
    }
}

// Sums of partials, several arrays a launch: out[i] = scale * sum_b part[b * pitch + i],
// i < len.  A block takes 32 outputs, its 32 groups of 32 lanes every 32nd
// partial each (four loads in flight), and the groups' sums are added in order: the same sum every
// time, without one lane walking hundreds of partials (120 us a launch, nine
// launches a training step; now under 20 us for all).
struct Sum {
    const float *part;
    float *out;
    int32_t nb, pitch, len, blocks;  // blocks = ceil(len / 32)
    float scale;
};
constexpr int kMaxSums = 9;
struct Sums {
    Sum s[kMaxSums];
};

constexpr int kSumGroups = 32;

__global__ void __launch_bounds__(32 * kSumGroups) k_sums(Sums all)
{
    int b = (int)blockIdx.x, k = 0;
    while (b >= all.s[k].blocks) b -= all.s[k++].blocks;
    const Sum s = all.s[k];
    __shared__ float s_x[kSumGroups][32];
    const int i = b * 32 + ((int)threadIdx.x & 31), g = (int)threadIdx.x >> 5;
    float x[4] = {0.f, 0.f, 0.f, 0.f};
    if (i < s.len) {
        const float *p = s.part + i;
        int q = g;
        for (; q + 3 * kSumGroups < s.nb; q += 4 * kSumGroups)
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] += p[(int64_t)(q + j * kSumGroups) * s.pitch];
        for (; q < s.nb; q += kSumGroups) x[0] += p[(int64_t)q * s.pitch];
    }
    s_x[g][threadIdx.x & 31] = (x[0] + x[1]) + (x[2] + x[3]);
    __syncthreads();
    if (g == 0 && i < s.len) {
        float t = 0.f;
        for (int q = 0; q < kSumGroups; ++q) t += s_x[q][threadIdx.x];
        s.out[i] = t * s.scale;
    }
}

// Adam (Kingma and Ba, ICLR 2015, Algorithm 1) on the FP32 master
// parameters, every operation rounded to FP32 (no contraction; division and
// square root correctly rounded):
//   m = b1 m + (1 - b1) g,  v = b2 v + (1 - b2) g^2,
//   p = p - lr (m / c1) / (sqrt(v / c2) + eps),  c1 = 1 - b1^t, c2 = 1 - b2^t,
// then the BF16 copies of W1..W3.
__global__ void k_adam(float *p, const float *g, float *m, float *v, int n, float lr, float b1,
                       float b2, float eps, float c1, float c2, uint16_t *wb)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * (gi * gi);
        m[i] = mi;
        v[i] = vi;
        const float upd = (mi / c1) / (sqrtf(vi / c2) + eps);
        const float pi = p[i] - lr * upd;
        p[i] = pi;
        if (i < kB1) wb[kWb1 + i] = to_bf16(pi);
        else if (i >= kW2 && i < kB2) wb[kWb2 + (i - kW2)] = to_bf16(pi);
        else if (i >= kW3 && i < kB3) wb[kWb3 + (i - kW3)] = to_bf16(pi);
    }
}

__global__ void k_params_to_bf16(const float *p, uint16_t *wb)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kWbN; i += gridDim.x * blockDim.x) {
        float x;
        if (i < kWb2) x = p[kW1 + i];
        else if (i < kWb3) x = p[kW2 + (i - kWb2)];
        else x = p[kW3 + (i - kWb3)];
        wb[i] = to_bf16(x);
    }
}

// Per-set sums of the node probabilities (the predicted spread) in a fixed
// order: block b of set s
// sums rows [b c, (b+1) c) of the set (c = ceil(n / kSumParts)) into
// part[s][b]; k_set_final then adds the kSumParts partials of each set.
constexpr int kSumParts = 128;

__global__ void __launch_bounds__(256) k_set_part(const float *prob, int32_t n, float *part)
{
    __shared__ float s[256];
    const int set = blockIdx.x / kSumParts, b = blockIdx.x - set * kSumParts;
    const int c = (n + kSumParts - 1) / kSumParts;
    const int lo = min(n, b * c), hi = min(n, lo + c);
    float acc = 0.f;
    for (int v = lo + (int)threadIdx.x; v < hi; v += blockDim.x) acc += prob[(int64_t)set * n + v];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

__global__ void __launch_bounds__(kSumParts) k_set_final(const float *part, float *out)
{
    __shared__ float s[kSumParts];
    s[threadIdx.x] = part[blockIdx.x * kSumParts + threadIdx.x];
    __syncthreads();
    for (int off = kSumParts / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = s[0];
}

__global__ void k_mask_clear(uint8_t *mask, int32_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        mask[i] = 0;
}

__global__ void k_mask_set(uint8_t *mask, const int32_t *seeds, int64_t ns)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ns;
         i += (int64_t)gridDim.x * blockDim.x)
        mask[seeds[i]] = 1;
}

}  // namespace gnn
}  // namespace fsg

using namespace fsg;
using namespace fsg::gnn;

// ------------------------------------------------------------------ host ----

struct fsg_gnn {
    int32_t hidden = kHid, layers = 3;
    uint64_t seed = 0;
    std::vector<float> init;
    bool bound = false;
    char *state = nullptr;  // device: params, m, v, grads (FP32 [P] each), BF16 weights
    int64_t step = 0;
    float last_loss = 0.f;
    float *p() const { return (float *)state; }
    float *m() const { return (float *)state + kP; }
    float *v() const { return (float *)state + 2 * kP; }
    float *g() const { return (float *)state + 3 * kP; }
    uint16_t *wb() const { return (uint16_t *)((float *)state + 4 * kP); }
};

namespace {

size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

#define GNN_TRY(expr)                                                                 \
    do {                                                                              \
        if (fsg::inject_device_fault())                                                       \
            return set_error(FSG_EDEVICE, (std::string(#expr) + ": injected fault").c_str()); \
        hipError_t e_ = (expr);                                                       \
        if (e_ != hipSuccess)                                                         \
            return set_error(FSG_EDEVICE, (std::string(#expr) + ": " + hipGetErrorString(e_)).c_str()); \
    } while (0)

unsigned grid_of(int64_t work, int block, int cap = 65536)
{
    int64_t g = (work + block - 1) / block;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(g, cap));
}

// Blocks (partials) of the weight-gradient products and of the head.
int dw_blocks(int64_t R) { return (int)std::max<int64_t>(1, std::min<int64_t>(kDwBlocks, R / 256)); }
int head_blocks(int64_t R) { return (int)std::max<int64_t>(1, std::min<int64_t>(kHeadBlocks, (R + 63) / 64)); }

// Workspace of one pass over R = n_sets n rows: training (and the forward
// pass), or a spread estimate, which runs kSlices members side by side on one
// set and updates their layers in place.
struct GnnWs {
    size_t Q, C, X1, X2, X3, prob, dZ, dZ2, inv, part1, part2, part3, pb1, pb2, pb3, phead, beta,
        stat, sums, setp, mask, seeds, total;
};

GnnWs gnn_layout(int64_t n, int32_t n_sets)
{
    GnnWs w;
    const size_t R = (size_t)n * (size_t)n_sets;
    const size_t nb = (size_t)dw_blocks((int64_t)R), hb = (size_t)head_blocks((int64_t)R);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = al256(off + std::max<size_t>(bytes, 4));
        return o;
    };
    w.Q = take(R * 8);
    w.C = take((size_t)n_sets * kF0 * 2);
    w.X1 = take(R * kK1 * 2);
    w.beta = take((size_t)n_sets * 4);
    w.stat = take((size_t)n_sets * kStatParts * 16);
    w.sums = take((size_t)std::max<int32_t>(n_sets, kMaxMembers) * 4);
    w.mask = take((size_t)n);
    w.seeds = take((size_t)n * 4);
    w.setp = take((size_t)kSlices * kSumParts * 4);
    w.prob = take((n_sets == 1 ? (size_t)kSlices : (size_t)1) * R * 4);
    w.X2 = take(R * kK2 * 2);
    const size_t slices = w.X2 + (size_t)kSlices * R * kK2 * 2;  // a spread estimate's X2, end
    w.X3 = take(R * kK2 * 2);
    w.dZ = take(R * kHid * 2);
    w.dZ2 = take(R * kHid * 2);
    w.inv = take((size_t)n * 4);
    w.part1 = take(nb * 4 * dw_part_len<kK1>() * 4);
    w.part2 = take(nb * dw_part_len<kK2>() * 4);
    w.part3 = take(nb * dw_part_len<kK2>() * 4);
    w.pb1 = take(nb * kHid * 4);
    w.pb2 = take(nb * kHid * 4);
    w.pb3 = take(nb * kHid * 4);
    w.phead = take(hb * 66 * 4);
    if (n_sets == 1) off = std::max(off, al256(slices));
    w.total = off;
    return w;
}

uint64_t splitmix(uint64_t &x)
{
    uint64_t z = (x += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

struct GraphView {
    int64_t n = 0, nnz = 0, dmax = 0, n_wide = 0, wide_arcs = 0;
    const int32_t *ptr = nullptr, *src = nullptr, *wide = nullptr, *order = nullptr;
};

int view_of(const fsg_graph *g, GraphView *v, const char *what)
{
    if (!graph_view(g, &v->n, &v->nnz, &v->dmax, &v->ptr, &v->src, &v->wide, &v->n_wide, &v->order,
                    &v->wide_arcs))
        return set_error(FSG_EINVAL, (std::string(what) + " is NULL or not bound").c_str());
    return FSG_OK;
}

// Blocks of an aggregation: one a wide row, then the others, `per` rows a block.
unsigned agg_grid(const GraphView &G, int64_t n_sets, int per)
{
    return (unsigned)(G.n_wide * n_sets) + grid_of((G.n - G.n_wide) * n_sets, per);
}

Weights layer_weights(const fsg_gnn *g, int layer)
{
    const int wb[3] = {kWb1, kWb2, kWb3}, b[3] = {kB1, kB2, kB3};
    return Weights{g->wb() + wb[layer], g->p() + b[layer], g->p() + kWo, g->p() + kBo};
}

// Persistent blocks of a product over `rows` rows of each of `slices` slices:
// 64 rows a pass, three blocks a compute unit (what the weights in registers
// leave room for), so that a block's weights serve as many rows as possible.
unsigned layer_grid(int64_t rows, int slices) { return grid_of(rows, 64, std::max(1, 768 / slices)); }

// Query-wide terms, features and the first layer's input rows of n_sets sets.
int input_enqueue(const GraphView &G, int32_t n_sets, const uint8_t *mask, char *base, const GnnWs &w,
                  bool want_inv, hipStream_t st)
{
    unsigned long long *part = (unsigned long long *)(base + w.stat);
    uint2 *Q = (uint2 *)(base + w.Q);
    uint16_t *C = (uint16_t *)(base + w.C);
    for (int64_t s0 = 0; s0 < n_sets; s0 += 65535) {  // grid y, and a launch's 2^32 threads
        const int32_t c = (int32_t)std::min<int64_t>(65535, n_sets - s0);
        hipLaunchKernelGGL(k_query_stats, dim3((unsigned)(c * kStatParts)), dim3(256), 0, st,
                           mask + s0 * G.n, G.ptr, (int32_t)G.n, part + s0 * kStatParts * 2);
        GNN_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_input, dim3(grid_of(G.n, 256), (unsigned)c), dim3(256), 0, st,
                           Q + s0 * G.n, C + s0 * kF0, mask + s0 * G.n,
                           (const float *)(base + w.beta) + s0, G.ptr,
                           (const unsigned long long *)part + s0 * kStatParts * 2, (int32_t)G.n,
                           want_inv && s0 == 0 ? (float *)(base + w.inv) : nullptr);
        GNN_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(k_mean_input, dim3(agg_grid(G, n_sets, kAggThreads / 4)),
                       dim3(kAggThreads), 0, st, (uint16_t *)(base + w.X1), (const uint2 *)Q,
                       (const uint16_t *)C, G.ptr, G.src, (int32_t)G.n, n_sets, G.wide,
                       (int32_t)G.n_wide, G.order);
    GNN_TRY(hipGetLastError());
    return FSG_OK;
}

int mean_enqueue(uint16_t *X, const GraphView &G, int32_t n_sets, hipStream_t st)
{
    hipLaunchKernelGGL(k_mean, dim3(agg_grid(G, n_sets, kAggThreads / 16)),
                       dim3(kAggThreads), 0, st, X, G.ptr, G.src, (int32_t)G.n, n_sets, G.wide,
                       (int32_t)G.n_wide, G.order);
    GNN_TRY(hipGetLastError());
    return FSG_OK;
}

// The three layers and the head over `slices` slices of `rows` rows each, the
// first layer's input shared by the slices (in_stride 0) or one per slice.
// sets: seed sets the aggregations run over (slices times the sets of a
// slice).  X3 may be X2: then the second layer is written over the first.
int layers_enqueue(const SliceWeights (&sw)[3], int slices, int64_t rows, int64_t in_stride,
                   const GraphView &G, int32_t sets, char *base, const GnnWs &w, uint16_t *X2,
                   uint16_t *X3, const HeadArgs &head, unsigned head_grid, hipStream_t st)
{
    const uint16_t *X1 = (const uint16_t *)(base + w.X1);
    const dim3 grid(layer_grid(rows, slices), (unsigned)slices), hgrid(head_grid, (unsigned)slices);
    const HeadArgs none{};
    hipLaunchKernelGGL((k_layer<kK1, false>), grid, dim3(256), 0, st, X1, in_stride, sw[0], X2,
                       rows * kK2, rows, none);
    GNN_TRY(hipGetLastError());
    int rc = mean_enqueue(X2, G, sets, st);
    if (rc) return rc;
    hipLaunchKernelGGL((k_layer<kK2, false>), grid, dim3(256), 0, st, (const uint16_t *)X2, rows * kK2,
                       sw[1], X3, rows * kK2, rows, none);
    GNN_TRY(hipGetLastError());
    rc = mean_enqueue(X3, G, sets, st);
    if (rc) return rc;
    hipLaunchKernelGGL((k_layer<kK2, true>), hgrid, dim3(256), 0, st, (const uint16_t *)X3, rows * kK2,
                       sw[2], (uint16_t *)nullptr, (int64_t)0, rows, head);
    GNN_TRY(hipGetLastError());
    return FSG_OK;
}

// Forward pass of one network over n_sets sets; probabilities to prob.  With
// targets also dZ of the last layer and the head's partial sums.
int forward_all(const fsg_gnn *gn, const GraphView &G, int32_t n_sets, const uint8_t *mask,
                float *prob, const float *y, char *base, const GnnWs &w, hipStream_t st)
{
    const int64_t R = G.n * n_sets;
    int rc = input_enqueue(G, n_sets, mask, base, w, y != nullptr, st);
    if (rc) return rc;
    SliceWeights sw[3];
    for (int l = 0; l < 3; ++l) sw[l].s[0] = layer_weights(gn, l);
    HeadArgs h{};
    h.prob = prob;
    h.y = y;
    h.dZ = (uint16_t *)(base + w.dZ);
    h.part = (float *)(base + w.phead);
    h.rows = (float)R;
    return layers_enqueue(sw, 1, R, 0, G, n_sets, base, w, (uint16_t *)(base + w.X2),
                          (uint16_t *)(base + w.X3), h,
                          y ? (unsigned)head_blocks(R) : layer_grid(R, 1), st);
}

// Weight-gradient partials of one layer (K columns of Xin).
template <int K>
int dw_enqueue(const uint16_t *Xin, const uint16_t *dZ, float *part, float *part_b, int64_t R,
               hipStream_t st)
{
    hipLaunchKernelGGL((k_layer_dw<K>), dim3((unsigned)dw_blocks(R)), dim3(256), 0, st, Xin, dZ, part,
                       part_b, R);
    GNN_TRY(hipGetLastError());
    return FSG_OK;
}

// dZ of the layer below from dZ of this one (BF16 weights w, input rows H).
int bwd_enqueue(const GraphView &Gr, int32_t n_sets, const uint16_t *dZ, const uint16_t *w,
                const uint16_t *H, uint16_t *out, const float *inv, hipStream_t st)
{
    const unsigned g = (unsigned)(Gr.n_wide * n_sets) + grid_of((Gr.n - Gr.n_wide) * n_sets, 64, 2048);
    hipLaunchKernelGGL(k_layer_bwd, dim3(g), dim3(kBwdThreads), 0, st, dZ, w, H, out, inv, Gr.ptr,
                       Gr.src, (int32_t)Gr.n, n_sets, Gr.wide, (int32_t)Gr.n_wide, Gr.order);
    GNN_TRY(hipGetLastError());
    return FSG_OK;
}

int check_ws(void *ws, size_t bytes, size_t need)
{
    if (!ws || bytes < need) return set_error(FSG_EWORKSPACE, "gnn workspace too small");
    if (((uintptr_t)ws & 255) != 0) return set_error(FSG_EWORKSPACE, "workspace not 256-byte aligned");
    return FSG_OK;
}

// One Adam step (step count t = ++g->step) with gradient grads (device [kP]).
int adam_enqueue(fsg_gnn *g, const float *grads, float lr, hipStream_t st)
{
    g->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    // 1 - beta^t: beta^t rounded once to FP32 (powf is correctly rounded)
    const float c1 = 1.f - powf(b1, (float)g->step), c2 = 1.f - powf(b2, (float)g->step);
    hipLaunchKernelGGL(k_adam, dim3(grid_of(kP, 256)), dim3(256), 0, st, g->p(), grads, g->m(),
                       g->v(), (int)kP, lr, b1, b2, 1e-8f, c1, c2, g->wb());
    GNN_TRY(hipGetLastError());
    return FSG_OK;
}

int upload_betas(const float *beta, int32_t n_sets, char *base, const GnnWs &w, hipStream_t st)
{
    for (int32_t i = 0; i < n_sets; ++i)
        if (!(beta[i] >= 0.f && beta[i] <= 1.f)) return set_error(FSG_EINVAL, "beta outside [0, 1]");
    GNN_TRY(hipMemcpyAsync(base + w.beta, beta, (size_t)n_sets * 4, hipMemcpyHostToDevice, st));
    return FSG_OK;
}

}  // namespace

extern "C" {

int fsg_gnn_create(int32_t hidden, int32_t layers, uint64_t init_seed, fsg_gnn **out)
{
    try {
        if (!out) return set_error(FSG_EINVAL, "out is NULL");
        *out = nullptr;
        if (hidden != kHid || layers != 3)
            return set_error(FSG_EUNSUPPORTED, "this build has hidden = 64 and 3 layers");
        fsg::inject_alloc_fault();
        fsg_gnn *g = new fsg_gnn;
        g->seed = init_seed;
        g->init.assign(kP, 0.f);
        uint64_t x = init_seed;
        auto fill = [&](int off, int fan_in, int count) {  // uniform(-a, a), a = sqrt(6 / (fan_in + 64))
            const float a = sqrtf(6.f / (float)(fan_in + kHid));
            for (int i = 0; i < count; ++i) {
                const double u = (double)(splitmix(x) >> 11) * (1.0 / 9007199254740992.0);
                g->init[(size_t)(off + i)] = (float)((2.0 * u - 1.0) * a);
            }
        };
        fill(kW1, kK1, kK1 * kHid);
        fill(kW2, kK2, kK2 * kHid);
        fill(kW3, kK2, kK2 * kHid);
        fill(kWo, kHid, kHid);
        *out = g;
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return set_error(FSG_ENOMEM, "host allocation failed");
    }
}

int fsg_gnn_destroy(fsg_gnn *g)
{
    delete g;
    return FSG_OK;
}

int fsg_gnn_param_count(const fsg_gnn *g, int64_t *count)
{
    if (!g || !count) return set_error(FSG_EINVAL, "NULL argument");
    *count = kP;
    return FSG_OK;
}

int fsg_gnn_state_size(const fsg_gnn *g, size_t *bytes)
{
    if (!g || !bytes) return set_error(FSG_EINVAL, "NULL argument");
    *bytes = al256((size_t)4 * kP * 4 + (size_t)kWbN * 2);
    return FSG_OK;
}

int fsg_gnn_bind(fsg_gnn *g, void *dev_state, size_t bytes, void *stream)
{
    if (!g) return set_error(FSG_EINVAL, "gnn is NULL");
    size_t need = 0;
    fsg_gnn_state_size(g, &need);
    int rc = check_ws(dev_state, bytes, need);
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    g->state = (char *)dev_state;
    GNN_TRY(hipMemcpyAsync(g->p(), g->init.data(), (size_t)kP * 4, hipMemcpyHostToDevice, st));
    GNN_TRY(hipMemsetAsync(g->m(), 0, (size_t)3 * kP * 4, st));
    hipLaunchKernelGGL(k_params_to_bf16, dim3(grid_of(kWbN, 256)), dim3(256), 0, st,
                       (const float *)g->p(), g->wb());
    GNN_TRY(hipGetLastError());
    GNN_TRY(hipStreamSynchronize(st));
    g->bound = true;
    g->step = 0;
    return FSG_OK;
}

int fsg_gnn_workspace_size(const fsg_gnn *g, const fsg_graph *graph, int32_t n_sets, size_t *bytes)
{
    if (!g || !bytes) return set_error(FSG_EINVAL, "NULL argument");
    GraphView G;
    int rc = view_of(graph, &G, "graph");
    if (rc) return rc;
    if (n_sets < 1) return set_error(FSG_EINVAL, "n_sets must be >= 1");
    if ((int64_t)n_sets * G.n > ((int64_t)1 << 31)) return set_error(FSG_EUNSUPPORTED, "n_sets * n above 2^31");
    *bytes = gnn_layout(G.n, n_sets).total;
    return FSG_OK;
}

}  // extern "C"

namespace fsg {
namespace gnn {
// Forward pass into dev_prob, enqueued on the stream without waiting.
int forward_enqueue(fsg_gnn *g, const fsg_graph *graph, int32_t n_sets, const uint8_t *dev_mask,
                    const float *beta, float *dev_prob, void *ws, size_t ws_bytes, void *stream)
{
    if (!g || !g->bound) return set_error(FSG_EINVAL, "gnn is NULL or not bound");
    GraphView G;
    int rc = view_of(graph, &G, "graph");
    if (rc) return rc;
    if (n_sets < 1 || !dev_mask || !beta || !dev_prob) return set_error(FSG_EINVAL, "bad arguments");
    const GnnWs w = gnn_layout(G.n, n_sets);
    rc = check_ws(ws, ws_bytes, w.total);
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    char *base = (char *)ws;
    rc = upload_betas(beta, n_sets, base, w, st);
    if (rc) return rc;
    return forward_all(g, G, n_sets, dev_mask, dev_prob, nullptr, base, w, st);
}
}  // namespace gnn
}  // namespace fsg

extern "C" {

int fsg_gnn_forward(fsg_gnn *g, const fsg_graph *graph, int32_t n_sets, const uint8_t *dev_mask,
                    const float *beta, float *dev_prob, void *ws, size_t ws_bytes, void *stream)
{
    const int rc = fsg::gnn::forward_enqueue(g, graph, n_sets, dev_mask, beta, dev_prob, ws,
                                             ws_bytes, stream);
    if (rc) return rc;
    GNN_TRY(hipStreamSynchronize((hipStream_t)stream));
    return FSG_OK;
}

int fsg_gnn_train_step(fsg_gnn *g, const fsg_graph *graph, const fsg_graph *reverse,
                       int32_t n_sets, const uint8_t *dev_mask, const float *beta,
                       const float *dev_target, float lr, int32_t apply_update, float *loss,
                       void *ws, size_t ws_bytes, void *stream)
{
    if (!g || !g->bound) return set_error(FSG_EINVAL, "gnn is NULL or not bound");
    GraphView G, Gr;
    int rc = view_of(graph, &G, "graph");
    if (rc) return rc;
    rc = view_of(reverse, &Gr, "reverse graph");
    if (rc) return rc;
    if (Gr.n != G.n || Gr.nnz != G.nnz) return set_error(FSG_EINVAL, "reverse graph does not match");
    if (n_sets < 1 || !dev_mask || !beta || !dev_target) return set_error(FSG_EINVAL, "bad arguments");
    if (!(lr >= 0.f)) return set_error(FSG_EINVAL, "lr must be >= 0");
    const GnnWs w = gnn_layout(G.n, n_sets);
    rc = check_ws(ws, ws_bytes, w.total);
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    char *base = (char *)ws;
    rc = upload_betas(beta, n_sets, base, w, st);
    if (rc) return rc;
    rc = forward_all(g, G, n_sets, dev_mask, (float *)(base + w.prob), dev_target, base, w, st);
    if (rc) return rc;
    const int64_t R = G.n * n_sets;
    float *grads = g->g();
    const uint16_t *X1 = (const uint16_t *)(base + w.X1), *X2 = (const uint16_t *)(base + w.X2),
                   *X3 = (const uint16_t *)(base + w.X3);
    uint16_t *dZ = (uint16_t *)(base + w.dZ), *dZ2 = (uint16_t *)(base + w.dZ2);
    const float *inv = (const float *)(base + w.inv);
    float *p1 = (float *)(base + w.part1), *p2 = (float *)(base + w.part2),
          *p3 = (float *)(base + w.part3), *b1 = (float *)(base + w.pb1),
          *b2 = (float *)(base + w.pb2), *b3 = (float *)(base + w.pb3),
          *ph = (float *)(base + w.phead);
    // layer 3: input X3 = [h2 | mean h2]; layer 2: X2; layer 1: X1, no
    // gradient to the inputs
    rc = dw_enqueue<kK2>(X3, dZ, p3, b3, R, st);
    if (rc) return rc;
    rc = bwd_enqueue(Gr, n_sets, dZ, g->wb() + kWb3, X3, dZ2, inv, st);
    if (rc) return rc;
    rc = dw_enqueue<kK2>(X2, dZ2, p2, b2, R, st);
    if (rc) return rc;
    rc = bwd_enqueue(Gr, n_sets, dZ2, g->wb() + kWb2, X2, dZ, inv, st);
    if (rc) return rc;
    rc = dw_enqueue<kK1>(X1, dZ, p1, b1, R, st);
    if (rc) return rc;
    float *dloss = (float *)(base + w.sums);
    const int nb = dw_blocks(R), hb = head_blocks(R);
    const int l1 = dw_part_len<kK1>(), l2 = dw_part_len<kK2>();
    const Sums sums = {{{p3, grads + kW3, nb, l2, l2, 0, 1.f},
                        {p2, grads + kW2, nb, l2, l2, 0, 1.f},
                        {p1, grads + kW1, 4 * nb, l1, l1, 0, 1.f},
                        {b3, grads + kB3, nb, kHid, kHid, 0, 1.f},
                        {b2, grads + kB2, nb, kHid, kHid, 0, 1.f},
                        {b1, grads + kB1, nb, kHid, kHid, 0, 1.f},
                        {ph, grads + kWo, hb, 66, kHid, 0, 1.f},
                        {ph + kHid, grads + kBo, hb, 66, 1, 0, 1.f},
                        {ph + kHid + 1, dloss, hb, 66, 1, 0, 1.f / (float)R}}};
    Sums launch = sums;
    int blocks = 0;
    for (Sum &x : launch.s) {
        x.blocks = (x.len + 31) / 32;
        blocks += x.blocks;
    }
    hipLaunchKernelGGL(k_sums, dim3((unsigned)blocks), dim3(32 * kSumGroups), 0, st, launch);
    GNN_TRY(hipGetLastError());
    if (apply_update) {
        rc = adam_enqueue(g, grads, lr, st);
        if (rc) return rc;
    }
    float hl = 0.f;
    GNN_TRY(hipMemcpyAsync(&hl, dloss, 4, hipMemcpyDeviceToHost, st));
    GNN_TRY(hipStreamSynchronize(st));
    g->last_loss = hl;
    if (loss) *loss = hl;
    return FSG_OK;
}

int fsg_gnn_get_params(const fsg_gnn *g, float *out, int64_t n, void *stream)
{
    if (!g || !g->bound || !out || n != kP) return set_error(FSG_EINVAL, "bad arguments");
    hipStream_t st = (hipStream_t)stream;
    GNN_TRY(hipMemcpyAsync(out, g->p(), (size_t)kP * 4, hipMemcpyDeviceToHost, st));
    GNN_TRY(hipStreamSynchronize(st));
    return FSG_OK;
}

int fsg_gnn_set_params(fsg_gnn *g, const float *in, int64_t n, void *stream)
{
    if (!g || !g->bound || !in || n != kP) return set_error(FSG_EINVAL, "bad arguments");
    hipStream_t st = (hipStream_t)stream;
    GNN_TRY(hipMemcpyAsync(g->p(), in, (size_t)kP * 4, hipMemcpyHostToDevice, st));
    GNN_TRY(hipMemsetAsync(g->m(), 0, (size_t)2 * kP * 4, st));
    hipLaunchKernelGGL(k_params_to_bf16, dim3(grid_of(kWbN, 256)), dim3(256), 0, st,
                       (const float *)g->p(), g->wb());
    GNN_TRY(hipGetLastError());
    GNN_TRY(hipStreamSynchronize(st));
    g->step = 0;
    return FSG_OK;
}

int fsg_gnn_get_grads(const fsg_gnn *g, float *out, int64_t n, void *stream)
{
    if (!g || !g->bound || !out || n != kP) return set_error(FSG_EINVAL, "bad arguments");
    hipStream_t st = (hipStream_t)stream;
    GNN_TRY(hipMemcpyAsync(out, g->g(), (size_t)kP * 4, hipMemcpyDeviceToHost, st));
    GNN_TRY(hipStreamSynchronize(st));
    return FSG_OK;
}

int fsg_gnn_apply_update(fsg_gnn *g, const float *dev_grad, float lr, void *stream)
{
    if (!g || !g->bound) return set_error(FSG_EINVAL, "gnn is NULL or not bound");
    if (!(lr >= 0.f) || !(lr < INFINITY)) return set_error(FSG_EINVAL, "lr must be finite and >= 0");
    hipStream_t st = (hipStream_t)stream;
    const int rc = adam_enqueue(g, dev_grad ? dev_grad : (const float *)g->g(), lr, st);
    if (rc) return rc;
    GNN_TRY(hipStreamSynchronize(st));
    return FSG_OK;
}

int fsg_gnn_get_state(const fsg_gnn *g, float *m, float *v, uint16_t *wb, int64_t *step,
                      int64_t n, void *stream)
{
    if (!g || !g->bound || n != kP) return set_error(FSG_EINVAL, "bad arguments");
    hipStream_t st = (hipStream_t)stream;
    if (m) GNN_TRY(hipMemcpyAsync(m, g->m(), (size_t)kP * 4, hipMemcpyDeviceToHost, st));
    if (v) GNN_TRY(hipMemcpyAsync(v, g->v(), (size_t)kP * 4, hipMemcpyDeviceToHost, st));
    if (wb) GNN_TRY(hipMemcpyAsync(wb, g->wb(), (size_t)kWbN * 2, hipMemcpyDeviceToHost, st));
    GNN_TRY(hipStreamSynchronize(st));
    if (step) *step = g->step;
    return FSG_OK;
}

int fsg_estimate_spread(fsg_gnn *const *members, int32_t n_members, const fsg_graph *graph,
                        const int32_t *seeds, int64_t n_seeds, double beta, double gamma,
                        int64_t max_steps, const fsg_spread_gate *gate, int64_t B_fallback,
                        uint64_t rng_key, void *ws, size_t ws_bytes, void *sim_ws,
                        size_t sim_ws_bytes, uint32_t *dev_counts, double *spread,
                        double *uncertainty, int32_t *used_fallback, void *stream)
{
    if (!members || n_members < 1 || n_members > kMaxMembers || !gate || !spread ||
        !uncertainty || !used_fallback)
        return set_error(FSG_EINVAL, "bad arguments (1 <= n_members <= 64, gate not NULL)");
    GraphView G;
    int rc = view_of(graph, &G, "graph");
    if (rc) return rc;
    if (n_seeds < 0 || (n_seeds > 0 && !seeds)) return set_error(FSG_EINVAL, "bad seed array");
    for (int64_t i = 0; i < n_seeds; ++i)
        if (seeds[i] < 0 || seeds[i] >= G.n) return set_error(FSG_EINVAL, "seed out of range");
    std::vector<int32_t> distinct(seeds, seeds + n_seeds);
    std::sort(distinct.begin(), distinct.end());
    const int64_t k = std::unique(distinct.begin(), distinct.end()) - distinct.begin();
    *used_fallback = 0;
    *uncertainty = 0.0;
    if (k == 0) {  // nothing is ever infected
        *spread = 0.0;
        return FSG_OK;
    }
    const GnnWs w = gnn_layout(G.n, 1);
    rc = check_ws(ws, ws_bytes, w.total);
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    char *base = (char *)ws;
    uint8_t *mask = (uint8_t *)(base + w.mask);
    int32_t *dseeds = (int32_t *)(base + w.seeds);
    hipLaunchKernelGGL(k_mask_clear, dim3(grid_of(G.n, 256)), dim3(256), 0, st, mask, (int32_t)G.n);
    GNN_TRY(hipGetLastError());
    // each seed once: the array on the device has room for n
    GNN_TRY(hipMemcpyAsync(dseeds, distinct.data(), (size_t)k * 4, hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_mask_set, dim3(grid_of(k, 256)), dim3(256), 0, st, mask,
                       (const int32_t *)dseeds, k);
    GNN_TRY(hipGetLastError());
    // every member's spread into the device sums, then one copy.  The
    // features and the first aggregation are the members' in common; then
    // kSlices members at a time run as slices of one launch per layer (four
    // members of 1e5 nodes: 14 launches instead of 44).
    float *sums = (float *)(base + w.sums);
    const float fb = (float)beta;
    for (int32_t m = 0; m < n_members; ++m)
        if (!members[m] || !members[m]->bound) return set_error(FSG_EINVAL, "gnn is NULL or not bound");
    rc = upload_betas(&fb, 1, base, w, st);
    if (rc) return rc;
    rc = input_enqueue(G, 1, mask, base, w, false, st);
    if (rc) return rc;
    uint16_t *X2 = (uint16_t *)(base + w.X2);
    float *part = (float *)(base + w.setp);
    for (int32_t m0 = 0; m0 < n_members; m0 += kSlices) {
        const int c = std::min<int>(kSlices, n_members - m0);
        SliceWeights sw[3];
        for (int l = 0; l < 3; ++l)
            for (int i = 0; i < c; ++i) sw[l].s[i] = layer_weights(members[m0 + i], l);
        HeadArgs h{};
        h.prob = (float *)(base + w.prob);
        rc = layers_enqueue(sw, c, G.n, 0, G, c, base, w, X2, X2, h, layer_grid(G.n, c), st);
        if (rc) return rc;
        hipLaunchKernelGGL(k_set_part, dim3((unsigned)(c * kSumParts)), dim3(256), 0, st,
                           (const float *)(base + w.prob), (int32_t)G.n, part);
        GNN_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_set_final, dim3((unsigned)c), dim3(kSumParts), 0, st,
                           (const float *)part, sums + m0);
        GNN_TRY(hipGetLastError());
    }
    float hs[kMaxMembers];
    GNN_TRY(hipMemcpyAsync(hs, sums, (size_t)n_members * 4, hipMemcpyDeviceToHost, st));
    GNN_TRY(hipStreamSynchronize(st));
    std::vector<double> sp(hs, hs + n_members);
    double mean = 0, var = 0;
    for (double x : sp) mean += x;
    mean /= n_members;
    for (double x : sp) var += (x - mean) * (x - mean);
    var = n_members > 1 ? var / (n_members - 1) : 0.0;
    const double unc = mean > 0 ? sqrt(var) / mean : 1e30;
    *uncertainty = unc;
    *spread = mean;
    if (gate->calibrated) {
        const double x = 20.0 * beta, kd = (double)k, lk = log(kd);
        const double f[FSG_CALIB_TERMS] = {1.0, x, x * x, x * x * x, 1.0 / kd, x / kd,
                                           1.0 / (kd * kd), lk, x * lk};
        double z = 0.0;
        for (int i = 0; i < FSG_CALIB_TERMS; ++i) z += gate->calib[i] * f[i];
        *spread = mean * exp(z);
    }
    if (unc > gate->tau || k < gate->min_seeds) {
        if (B_fallback < 1 || !dev_counts) return set_error(FSG_EINVAL, "fallback needs B_fallback and counts");
        fsg_params prm;
        memset(&prm, 0, sizeof(prm));
        prm.model = FSG_SIR;
        prm.beta = beta;
        prm.gamma = gamma;
        prm.max_steps = max_steps;
        fsg_run_info info;
        rc = fsg_simulate(graph, &prm, seeds, n_seeds, B_fallback, 0, rng_key, nullptr, sim_ws,
                          sim_ws_bytes, nullptr, dev_counts, &info, stream);
        if (rc) return rc;
        std::vector<uint32_t> cnt((size_t)G.n);
        GNN_TRY(hipMemcpyAsync(cnt.data(), dev_counts, (size_t)G.n * 4, hipMemcpyDeviceToHost, st));
        GNN_TRY(hipStreamSynchronize(st));
        double tot = 0;
        for (uint32_t c : cnt) tot += c;
        *spread = tot / (double)B_fallback;
        *used_fallback = 1;
    }
    return FSG_OK;
}

}  // extern "C"
