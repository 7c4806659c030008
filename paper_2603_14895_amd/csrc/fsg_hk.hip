// fsg_hk.hip -- batched Hegselmann-Krause opinion dynamics as synchronous
// pull message passing (Appendix A.2, "Micro-accelerated implementation of
// HK model"): every arc j -> i carries the pair (h_j, 1) when
// |h_i - h_j| < eps and (0, 0) otherwise; node i sums the pairs and takes
// the quotient, keeping h_i when no pair is non-zero.  B independent
// replicates (initial opinion vectors) run side by side.
//
// State: FP32 opinions [n][B] (replicate fastest), double-buffered between
// the caller's array and the workspace.  No randomness.
//
// Arithmetic contract: per (node, replicate) the filtered opinions are
// summed in IEEE single precision in CSR order of the in-arcs, one rounding
// per addition, then divided once (round to nearest even) by the count.
// The kernels keep that order exactly, so the result is the same bits as a
// plain sequential loop, and so are all later eps decisions.
//
// Kernel (one launch per step):
//   * rows with more than kWideRow in-arcs ("hubs", largest first) get
//     the first blocks of the grid: one block per (hub, 16 to 64
//     replicates); its four waves gather and filter tiles of arcs into LDS
//     two tiles ahead (source indices one tile further), and wave 0 adds each
//     replicate's column in arc order;
//   * every other row, by decreasing degree: one lane per (row, 4
//     replicates) or (row, replicate), looping over the row's in-arcs with the
//     next source indices in flight.
// A step that changes no opinion leaves its ring flag clear; the next step's
// kernel then returns at once, so several steps can be queued between host
// polls.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "../../include/fsg.h"
#include "fsg_internal.hpp"

namespace fsg {
namespace hk {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;

struct Args {
    const int32_t *ptr;   // [n+1]
    const int32_t *src;   // [nnz]
    const int32_t *wide;  // [n_wide] hub rows, largest first
    const int32_t *order; // [n - n_wide] the other rows, by decreasing in-degree
    int32_t n;
    int32_t n_wide;
    int32_t chunks;       // column chunks of a hub row
    int32_t hub_blocks;   // n_wide * chunks
    int64_t B;
    uint32_t per_row;     // lanes of a light row: ceil(B / vec)
    uint32_t lanes;       // (n - n_wide) * per_row
    float eps;
    float mu, omm;        // weighted HK: fraction moved towards the mean, and 1 - mu
    const float *x;       // opinions after the previous step
    float *y;             // opinions after this step
    uint32_t *flags;      // ring: 1 iff the step changed an opinion
    int32_t slot;         // this step's ring index
    int32_t prev;         // previous step's ring index, -1: none
};

__device__ __forceinline__ void mark_changed(const Args &a, bool ch)
{
    if (__ballot(ch) != 0ull && (threadIdx.x & 63) == 0) a.flags[a.slot] = 1u;
}

// One eps-filtered message: h_j when the two opinions differ by less than eps,
// else 0, and the count.  Adding +0.0 instead of skipping is the same bits: the
// sum starts at +0.0 and round-to-nearest never yields -0.0 from it.
__device__ __forceinline__ float filtered(float hv, float hj, float eps, int &mv)
{
    const bool in = fabsf(hv - hj) < eps;
    mv += in ? 1 : 0;
    return in ? hj : 0.0f;
}

__device__ __forceinline__ void take(float hv, float hj, float eps, float &mc, int &mv)
{
    mc += filtered(hv, hj, eps, mv);
}

__device__ __forceinline__ float settle(const Args &a, float hv, float mc, int mv)
{
    if (mv == 0) return hv;
    const float m = __fdiv_rn(mc, (float)mv);
    // weighted HK: (1 - mu) h + mu m, two rounded products and a rounded sum
    // (no contraction); mu = 1 is plain HK
    return a.mu == 1.0f ? m : __fadd_rn(__fmul_rn(a.omm, hv), __fmul_rn(a.mu, m));
}

// ---- hub rows ---------------------------------------------------------------
//
// A hub row's sums are one chain of additions per replicate, in arc order, so
// a block takes C replicates of a hub and keeps the chain fed: its four waves
// gather tiles of arcs two tiles ahead, filter them by eps and count (which
// needs no order) as they put them to LDS, a column a replicate, and wave 0
// adds, one addition an arc and a 16-byte LDS read every four.  A tile is
// 4 P 64 / C arcs: with fewer replicates a block the tiles are longer and cover
// the gathers' latency, which bounds the step where the hub's chain does; with
// more, a gather reads whole cache lines and fewer blocks repeat the
// filtering, which counts once the graph's gathers take longer than the chain;
// and P = 8 leaves room for six waves a SIMD instead of four.  20 steps, by n B:
//   20,000 x 50   C = 64 1.81 ms, 32 1.03, 16 0.79  (2.61 with filtering, counting
//                 and adding by wave 0)
//   100,000 x 150 C = 64 4.33 ms, 32 3.06, 16 3.37
//   200,000 x 256 C = 64 11.5 ms, 32 12.8, 16 13.1; C = 64 with P = 8 12.0
//   1,000,000 x 256, 10 steps: C = 64 33.1 ms, with P = 8 30.8
template <int C, int P>
struct Hub {
    static constexpr int kArcsPerLoad = 64 / C;          // arcs of one gather instruction
    static constexpr int kPerWave = P;                   // gather instructions a wave and tile
    static constexpr int kTile = kWaves * kPerWave * kArcsPerLoad;  // arcs of a tile
    static constexpr int kPitch = kTile + 4;             // floats of a replicate's column in LDS
};

template <int P>
struct HubTile {
    int32_t s[P];
    float g[P];
};

// Read-only view of the source indices in the constant address space: with
// C = 64 a load's arc is the same for the whole wave, so the indices come in
// through scalar loads and the gathers that use them wait on the scalar
// counter only, never on older gathers still in flight.
typedef const __attribute__((address_space(4))) int32_t csrc_t;

// Sources of tile t (clamped to the last tile; arcs past the row end repeat
// its last arc), this wave's share.
template <int C, int P>
__device__ __forceinline__ void hub_src(const int32_t *src, int e0, int e1, int nt, int w, int t,
                                        int32_t (&s)[P])
{
    constexpr int A = Hub<C, P>::kArcsPerLoad;
    // (below 2^31 with every clamp: arcs are at most 2^31 - 256 and a tile's
    // last share begins at most 240 past the row's end)
    const int base = e0 + min(t, nt - 1) * Hub<C, P>::kTile + w * (P * A);
    if (C == 64) {
        csrc_t *cs = (csrc_t *)src;
#pragma unroll
        for (int i = 0; i < P; ++i) s[i] = cs[min(base + i, e1 - 1)];
    } else {
        const int a = (threadIdx.x & 63) / C;
#pragma unroll
        for (int i = 0; i < P; ++i) s[i] = src[min(base + a * P + i, e1 - 1)];
    }
}

// C = 64: one buffer resource per source row (its B opinions; base and range
// in scalar registers) and one fixed 32-bit lane offset: the gathers need no
// per-load address registers, and lanes past column B read 0 through the
// range check instead of touching memory.
constexpr int kRsrcWord3 = 0x00020000;  // raw 32-bit buffer access (gfx9 family)

template <int C, int P>
__device__ __forceinline__ void hub_gather(const Args &a, int64_t col, uint32_t voff,
                                           const int32_t (&s)[P], float (&g)[P])
{
    const uint32_t row_bytes = (uint32_t)a.B * 4u;
#pragma unroll
    for (int i = 0; i < P; ++i) {
        if (C == 64) {
            __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(a.x + (int64_t)s[i] * a.B), (short)0, (int)row_bytes, kRsrcWord3);
            g[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, 0, 0));
        } else {
            g[i] = a.x[(int64_t)s[i] * a.B + col];
        }
    }
}

// Tiles t = 0 .. nt-1.  Per half-iteration k: sources of tile k+3, gathers of
// tile k+2, the sum of tile k from LDS by wave 0, then the gathers of tile
// k+1, issued one half earlier, go filtered to the other LDS buffer.  Loads
// past the last tile re-read it, so the loop body has no conditional loads.
template <int C, int P>
__device__ void hub_row(const Args &a, float *lds)
{
    typedef Hub<C, P> H;
    const int hb = blockIdx.x;
    const int32_t v = a.wide[hb / a.chunks];
    const int64_t c0 = (int64_t)(hb % a.chunks) * C;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cl = lane & (C - 1);
    const bool live = c0 + cl < a.B;
    const int64_t col = live ? c0 + cl : a.B - 1;
    const uint32_t voff = (uint32_t)(c0 + cl) * 4u;  // past the row for idle lanes: reads 0
    const int e0 = a.ptr[v], e1 = a.ptr[v + 1];
    const int nt = (e1 - e0 + H::kTile - 1) / H::kTile;
    const float hv = a.x[(int64_t)v * a.B + col];
    float *buf0 = lds, *buf1 = lds + H::kPitch * C;
    float mc = 0.0f;
    int mv = 0;
    // a tile's gathers, filtered, to LDS: a column a replicate in arc order, the
    // P consecutive arcs of a lane four at a time (arcs past the row end: 0)
    auto put = [&](float *buf, int t, const float (&g)[H::kPerWave]) {
        const int left = e1 - e0 - t * H::kTile;  // arcs from the tile's first
        const int k0 = (w * H::kArcsPerLoad + lane / C) * H::kPerWave;
        float f[H::kPerWave];
#pragma unroll
        for (int i = 0; i < H::kPerWave; ++i) {
            f[i] = 0.0f;
            if (k0 + i < left) f[i] = filtered(hv, g[i], a.eps, mv);
        }
#pragma unroll
        for (int i = 0; i < H::kPerWave; i += 4)
            *reinterpret_cast<float4 *>(buf + cl * H::kPitch + k0 + i) =
                make_float4(f[i], f[i + 1], f[i + 2], f[i + 3]);
    };
    auto sum = [&](const float *buf) {
        const float *p = buf + cl * H::kPitch;
#pragma unroll 1
        for (int i = 0; i < H::kTile; i += 32) {
            float4 x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = *reinterpret_cast<const float4 *>(p + i + 4 * j);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                mc += x[j].x;
                mc += x[j].y;
                mc += x[j].z;
                mc += x[j].w;
            }
        }
    };
    HubTile<P> A, Bt;  // tiles with even / odd index
    hub_src<C, P>(a.src, e0, e1, nt, w, 0, A.s);
    hub_src<C, P>(a.src, e0, e1, nt, w, 1, Bt.s);
    hub_gather<C, P>(a, col, voff, A.s, A.g);
    hub_src<C, P>(a.src, e0, e1, nt, w, 2, A.s);
    hub_gather<C, P>(a, col, voff, Bt.s, Bt.g);
    put(buf0, 0, A.g);
    __syncthreads();
    // at even k: buf0 = tile k, Bt.g = tile k+1 in flight, A.s = sources of tile k+2
    for (int k = 0; k < nt; k += 2) {
        hub_src<C, P>(a.src, e0, e1, nt, w, k + 3, Bt.s);
        hub_gather<C, P>(a, col, voff, A.s, A.g);
        if (w == 0) sum(buf0);
        put(buf1, k + 1, Bt.g);
        __syncthreads();
        if (k + 1 >= nt) break;
        hub_src<C, P>(a.src, e0, e1, nt, w, k + 4, A.s);
        hub_gather<C, P>(a, col, voff, Bt.s, Bt.g);
        if (w == 0) sum(buf1);
        put(buf0, k + 2, A.g);
        __syncthreads();
    }
    // the counts of the waves and of the lanes that share a replicate
    int *cnt = reinterpret_cast<int *>(lds);
    __syncthreads();
    cnt[w * 64 + lane] = mv;
    __syncthreads();
    if (w == 0) {
        mv = 0;
        for (int i = cl; i < kBlock; i += C) mv += cnt[i];
        const float nv = settle(a, hv, mc, mv);
        if (live && lane < C) a.y[(int64_t)v * a.B + col] = nv;
        mark_changed(a, live && nv != hv);
    }
}

// ---- light rows -------------------------------------------------------------

// VEC replicates of a row a lane: 4 with 16-byte loads (B >= 4; where B is no
// multiple of 4 the loads are 4-byte aligned and the row's last lane takes its
// last four replicates, some of them again: the same values), else 1.  The
// rows go by decreasing degree, so rows that share a wave have about as many
// arcs and the longest begin first.  U gathers are in flight, the next
// sources with them.
template <int VEC>
struct __attribute__((aligned(4))) Pack {
    float f[VEC];
};

template <int VEC, bool ALIGNED>
__device__ __forceinline__ Pack<VEC> load_pack(const float *p)
{
    if constexpr (VEC == 4 && ALIGNED) {
        const float4 x = *reinterpret_cast<const float4 *>(p);
        return Pack<4>{{x.x, x.y, x.z, x.w}};
    } else {
        return *reinterpret_cast<const Pack<VEC> *>(p);
    }
}

template <int VEC, bool ALIGNED, int U>
__device__ void light_row(const Args &a, uint32_t idx)
{
    bool ch = false;
    if (idx < a.lanes) {
        const uint32_t i = idx / a.per_row;
        const int64_t v = a.order[i];
        const int64_t c = min((int64_t)(idx - i * a.per_row) * VEC, a.B - VEC);
        const int e0 = a.ptr[v], e1 = a.ptr[v + 1];
        const float *X = a.x + c;
        const Pack<VEC> hv = load_pack<VEC, ALIGNED>(X + v * a.B);
        float mc[VEC];
        int mv[VEC];
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            mc[k] = 0.0f;
            mv[k] = 0;
        }
        if (e0 < e1) {
            // indices past the row end repeat its last arc (loaded, never taken)
            const int last = e1 - 1;
            int32_t s[U];
#pragma unroll
            for (int j = 0; j < U; ++j) s[j] = a.src[min(e0 + j, last)];
            for (int e = e0; e < e1; e += U) {
                Pack<VEC> g[U];
#pragma unroll
                for (int j = 0; j < U; ++j) g[j] = load_pack<VEC, ALIGNED>(X + (int64_t)s[j] * a.B);
                // the next batch's sources go out while the gathers are in flight
#pragma unroll
                for (int j = 0; j < U; ++j) s[j] = a.src[min(e + U + j, last)];
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    if (e + j < e1) {
#pragma unroll
                        for (int k = 0; k < VEC; ++k) take(hv.f[k], g[j].f[k], a.eps, mc[k], mv[k]);
                    }
                }
            }
        }
        Pack<VEC> out;
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            out.f[k] = settle(a, hv.f[k], mc[k], mv[k]);
            ch |= out.f[k] != hv.f[k];
        }
        float *Y = a.y + v * a.B + c;
        if constexpr (VEC == 4 && ALIGNED)
            *reinterpret_cast<float4 *>(Y) = make_float4(out.f[0], out.f[1], out.f[2], out.f[3]);
        else
            *reinterpret_cast<Pack<VEC> *>(Y) = out;
    }
    mark_changed(a, ch);
}

template <int VEC, bool ALIGNED, int C, int P>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(P == 8 ? 6 : 4)))
void k_hk_step(Args a)
{
    __shared__ __align__(16) float lds[2 * Hub<C, P>::kPitch * C];
    if (a.prev >= 0 && a.flags[a.prev] == 0u) return;  // converged: nothing moves
    if ((int)blockIdx.x < a.hub_blocks) {
        hub_row<C, P>(a, lds);
        return;
    }
    light_row<VEC, ALIGNED, VEC == 4 ? 4 : 8>(a, (uint32_t)(blockIdx.x - a.hub_blocks) * kBlock + threadIdx.x);
}

// Per replicate: nodes with opinion above `act`, added to counts (zeroed).
// Lanes go over replicates (several rows a wave where B <= 32), the waves of a
// block meet in LDS and each block adds once per replicate (an atomic a thread
// before: 2e4 nodes at B = 50 took 169 us, now 9).
__global__ void __launch_bounds__(256) k_hk_count(const float *h, int64_t n, int64_t B, int64_t y0,
                                                  float act, uint32_t *counts)
{
    const int lane = threadIdx.x & 63;
    const int R = B <= 32 ? 64 / (int)B : 1;  // rows a wave and pass
    const int slot = B <= 32 ? lane / (int)B : 0;
    const int64_t col = B <= 32 ? lane - slot * (int)B : (y0 + (int64_t)blockIdx.y) * 64 + lane;
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), nwave = (int64_t)gridDim.x * 4;
    uint32_t c = 0;
    if (slot < R && col < B) {
        int64_t v = wave * R + slot;
        for (; v + 3 * nwave * R < n; v += 4 * nwave * R) {  // four loads in flight
            const float x0 = h[v * B + col], x1 = h[(v + nwave * R) * B + col],
                        x2 = h[(v + 2 * nwave * R) * B + col], x3 = h[(v + 3 * nwave * R) * B + col];
            c += (x0 > act ? 1u : 0u) + (x1 > act ? 1u : 0u) + (x2 > act ? 1u : 0u) + (x3 > act ? 1u : 0u);
        }
        for (; v < n; v += nwave * R) c += h[v * B + col] > act ? 1u : 0u;
    }
    __shared__ uint32_t s_c[256];
    s_c[threadIdx.x] = c;
    __syncthreads();
    if (threadIdx.x < 64 && slot == 0 && col < B) {
        uint32_t t = 0;
        for (int w = 0; w < 4; ++w)
            for (int k = 0; k < R; ++k) t += s_c[w * 64 + k * (int)(B <= 32 ? B : 0) + lane];
        if (t) atomicAdd(&counts[col], t);
    }
}

__global__ void k_fill_u32(uint32_t *p, int64_t count)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0u;
}

size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

struct View {
    int64_t n = 0, nnz = 0, dmax = 0, n_wide = 0, wide_arcs = 0;
    const int32_t *ptr = nullptr, *src = nullptr, *wide = nullptr, *order = nullptr;
};

int view_of(const fsg_graph *g, View *v)
{
    if (!graph_view(g, &v->n, &v->nnz, &v->dmax, &v->ptr, &v->src, &v->wide, &v->n_wide, &v->order,
                    &v->wide_arcs))
        return set_error(FSG_EINVAL, "graph is NULL or not bound");
    return FSG_OK;
}

#define HK_TRY(expr)                                                                          \
    do {                                                                                      \
        if (fsg::inject_device_fault())                                                        \
            return set_error(FSG_EDEVICE, (std::string(#expr) + ": injected fault").c_str());  \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess)                                                                 \
            return set_error(FSG_EDEVICE, (std::string(#expr) + ": " + hipGetErrorString(e_)).c_str()); \
    } while (0)

constexpr int kMaxSync = 256;

int sync_of(const fsg_schedule *s)
{
    int v = s && s->steps_per_sync > 0 ? s->steps_per_sync : 16;
    return std::min(v, kMaxSync);
}

// Replicates of a hub a block takes where the state is small (see Hub).  With
// 16 the longest hub's chain runs faster, with 32 fewer blocks repeat the
// gathers and the filtering: a step takes the longer of the two, at 13 and 17 ns
// an arc of the longest row and 27 and 30 ps an arc and block of all hubs
// (measured).  A power law's chain decides for 16 (2e4 nodes of mean degree 100,
// B = 64, 10 steps: 1.06 ms, 1.33 with 32), a graph that is all hubs for 32 (4000
// rows of 600 arcs, B = 64: 1.75 ms with 16, 1.29 with 32; 16,000 of 300: 5.26
// and 2.97).
int small_hub_cols(const View &G, int64_t B)
{
    auto ns = [&](int64_t cols, double chain, double work) {
        return std::max(chain * (double)G.dmax,
                        work * (double)G.wide_arcs * (double)((B + cols - 1) / cols));
    };
    return ns(16, 13.0, 0.027) <= ns(32, 17.0, 0.030) ? 16 : 32;
}

size_t ws_bytes_for(int64_t n, int64_t B, int sync)
{
    return al256((size_t)n * (size_t)B * 4) + al256((size_t)(sync + 1) * 4);
}

}  // namespace hk
}  // namespace fsg

using namespace fsg;
using namespace fsg::hk;

extern "C" {

int fsg_hk_workspace_size(const fsg_graph *g, int64_t B, const fsg_schedule *sched, size_t *bytes)
{
    View G;
    int rc = view_of(g, &G);
    if (rc) return rc;
    if (!bytes) return set_error(FSG_EINVAL, "bytes is NULL");
    if (B < 1) return set_error(FSG_EINVAL, "B must be >= 1");
    *bytes = ws_bytes_for(G.n, B, sync_of(sched));
    return FSG_OK;
}

int fsg_hk(const fsg_graph *g, float eps, int64_t max_steps, int64_t B, float *dev_h,
           const fsg_schedule *sched, void *dev_ws, size_t ws_bytes, float act,
           uint32_t *dev_counts, fsg_run_info *info, void *stream)
{
    return fsg_whk(g, eps, 1.0f, max_steps, B, dev_h, sched, dev_ws, ws_bytes, act, dev_counts,
                   info, stream);
}

int fsg_whk(const fsg_graph *g, float eps, float mu, int64_t max_steps, int64_t B, float *dev_h,
            const fsg_schedule *sched, void *dev_ws, size_t ws_bytes, float act,
            uint32_t *dev_counts, fsg_run_info *info, void *stream)
{
    View G;
    int rc = view_of(g, &G);
    if (rc) return rc;
    if (!dev_h) return set_error(FSG_EINVAL, "dev_h is NULL");
    if (B < 1) return set_error(FSG_EINVAL, "B must be >= 1");
    if (max_steps < 0) return set_error(FSG_EINVAL, "max_steps must be >= 0");
    if (!(eps >= 0.0f) || isinf(eps)) return set_error(FSG_EINVAL, "eps must be finite and >= 0");
    if (!(mu >= 0.0f && mu <= 1.0f)) return set_error(FSG_EINVAL, "mu must be in [0, 1]");
    if (isnan(act)) return set_error(FSG_EINVAL, "act is NaN");
    const int vec = (B % 4 == 0) ? 4 : 1;
    if (G.n * (B / vec) >= ((int64_t)1 << 31) - kBlock || B >= ((int64_t)1 << 28))
        return set_error(FSG_EUNSUPPORTED, "n * B too large");
    if (G.n_wide * ((B + 63) / 64) >= ((int64_t)1 << 30))
        return set_error(FSG_EUNSUPPORTED, "too many hub blocks");
    // Replicates of a hub a block takes (measured lines: see Hub), and of a light
    // row a lane: four share the index loads and the address, one gives a small
    // state four times the waves (5,000 x 301: 0.85 ms with one, 1.2 with four;
    // 50,000 x 64: 1.67 and 1.59).
    const int64_t size = G.n * B;
    const int lane_vec = B >= 4 && size >= ((int64_t)1 << 22) ? 4 : 1;
    const int hub_cols = lane_vec == 1 || size < 6000000 ? small_hub_cols(G, B)
                                                         : (size < ((int64_t)1 << 25) ? 32 : 64);
    const int chunks = (int)((B + hub_cols - 1) / hub_cols);
    const int sync = sync_of(sched);
    const size_t need = ws_bytes_for(G.n, B, sync);
    if (!dev_ws || ws_bytes < need) return set_error(FSG_EWORKSPACE, "HK workspace too small");
    if (((uintptr_t)dev_ws & 255) != 0 || ((uintptr_t)dev_h & 15) != 0)
        return set_error(FSG_EWORKSPACE, "workspace not 256-byte aligned or dev_h not 16-byte aligned");
    const bool timed = sched && sched->time_kernels;
    hipStream_t st = (hipStream_t)stream;

    float *buf[2] = {dev_h, (float *)dev_ws};
    uint32_t *flags = (uint32_t *)((char *)dev_ws + al256((size_t)G.n * (size_t)B * 4));
    const int ring = sync + 1;
    Args a;
    memset(&a, 0, sizeof(a));
    a.ptr = G.ptr;
    a.src = G.src;
    a.wide = G.wide;
    a.n = (int32_t)G.n;
    a.n_wide = (int32_t)G.n_wide;
    a.chunks = chunks;
    a.hub_blocks = (int32_t)(G.n_wide * chunks);
    a.order = G.order;
    a.B = B;
    a.per_row = (uint32_t)((B + lane_vec - 1) / lane_vec);
    a.lanes = (uint32_t)((G.n - G.n_wide) * (int64_t)a.per_row);
    a.eps = eps;
    a.mu = mu;
    a.omm = 1.0f - mu;
    a.flags = flags;
    const int64_t grid = std::max<int64_t>(1, a.hub_blocks + ((int64_t)a.lanes + kBlock - 1) / kBlock);
    auto launch = [&]() {
        const dim3 g((unsigned)grid), b(kBlock);
        const bool al = B % 4 == 0;
        if (lane_vec == 1 && hub_cols == 16)
            hipLaunchKernelGGL((k_hk_step<1, false, 16, 16>), g, b, 0, st, a);
        else if (lane_vec == 1)
            hipLaunchKernelGGL((k_hk_step<1, false, 32, 16>), g, b, 0, st, a);
        else if (hub_cols == 16 && al)
            hipLaunchKernelGGL((k_hk_step<4, true, 16, 16>), g, b, 0, st, a);
        else if (hub_cols == 16)
            hipLaunchKernelGGL((k_hk_step<4, false, 16, 16>), g, b, 0, st, a);
        else if (hub_cols == 32 && al)
            hipLaunchKernelGGL((k_hk_step<4, true, 32, 16>), g, b, 0, st, a);
        else if (hub_cols == 32)
            hipLaunchKernelGGL((k_hk_step<4, false, 32, 16>), g, b, 0, st, a);
        else if (size < ((int64_t)1 << 27) && al)
            hipLaunchKernelGGL((k_hk_step<4, true, 64, 16>), g, b, 0, st, a);
        else if (size < ((int64_t)1 << 27))
            hipLaunchKernelGGL((k_hk_step<4, false, 64, 16>), g, b, 0, st, a);
        else if (al)
            hipLaunchKernelGGL((k_hk_step<4, true, 64, 8>), g, b, 0, st, a);
        else
            hipLaunchKernelGGL((k_hk_step<4, false, 64, 8>), g, b, 0, st, a);
    };

    std::vector<hipEvent_t> ev;
    struct Ev {
        std::vector<hipEvent_t> &e;
        ~Ev()
        {
            for (auto x : e)
                if (x) (void)hipEventDestroy(x);
        }
    } ev_guard{ev};
    if (timed) {
        ev.assign(2 * (size_t)sync, nullptr);
        for (auto &x : ev) HK_TRY(hipEventCreate(&x));
    }
    std::vector<uint32_t> hflags((size_t)ring);
    double kernel_ms = 0.0;
    int64_t launches = 0, t = 0;
    bool converged = false;
    while (!converged && t < max_steps) {
        const int64_t c = std::min<int64_t>(sync, max_steps - t);
        HK_TRY(launch_ring_clear(flags, ring, (int32_t)(t % ring), st));
        for (int64_t i = 1; i <= c; ++i) {
            const int64_t step = t + i;
            a.x = buf[(step - 1) & 1];
            a.y = buf[step & 1];
            a.slot = (int32_t)(step % ring);
            a.prev = step > 1 ? (int32_t)((step - 1) % ring) : -1;
            if (timed) HK_TRY(hipEventRecord(ev[2 * (i - 1)], st));
            launch();
            HK_TRY(hipGetLastError());
            if (timed) HK_TRY(hipEventRecord(ev[2 * (i - 1) + 1], st));
        }
        HK_TRY(hipMemcpyAsync(hflags.data(), flags, (size_t)ring * 4, hipMemcpyDeviceToHost, st));
        HK_TRY(hipStreamSynchronize(st));
        int64_t done = t + c;
        for (int64_t i = 1; i <= c; ++i)
            if (hflags[(size_t)((t + i) % ring)] == 0u) {
                done = t + i;
                converged = true;
                break;
            }
        if (timed)
            for (int64_t i = 1; i <= done - t; ++i) {
                float ms = 0.f;
                HK_TRY(hipEventElapsedTime(&ms, ev[2 * (i - 1)], ev[2 * (i - 1) + 1]));
                kernel_ms += ms;
                ++launches;
            }
        t = done;
    }
    if (t & 1)
        HK_TRY(hipMemcpyAsync(dev_h, buf[1], (size_t)G.n * (size_t)B * 4, hipMemcpyDeviceToDevice, st));
    if (dev_counts) {
        hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, st, dev_counts, B);
        HK_TRY(hipGetLastError());
        // 64 replicates a block column, 16 rows a wave or more
        const int64_t cols = B <= 32 ? 1 : (B + 63) / 64;
        const int64_t rows = std::max<int64_t>(1, std::min<int64_t>(G.n / 64 + 1, std::max<int64_t>(1, 1024 / cols)));
        for (int64_t y0 = 0; y0 < cols; y0 += 65535) {  // grid y
            const int64_t cy = std::min<int64_t>(65535, cols - y0);
            hipLaunchKernelGGL(k_hk_count, dim3((unsigned)rows, (unsigned)cy), dim3(256), 0, st,
                               (const float *)dev_h, G.n, B, y0, act, dev_counts);
            HK_TRY(hipGetLastError());
        }
    }
    HK_TRY(hipStreamSynchronize(st));
    if (info) {
        info->steps_run = t;
        info->absorbed = converged ? 1 : 0;
        info->tail_steps = 0;
        info->step_kernel_ms = kernel_ms;
        info->step_launches = launches;
        info->setup_ms = 0.0;
        info->finalize_ms = 0.0;
        info->philox_calls = 0;
    }
    return FSG_OK;
}

}  // extern "C"
