// fsg_kernels.hip -- the synchronous pull step of batched Monte Carlo
// propagation for gfx950 (FS_GPlib, arxiv 2603.14895, Sec. 3.1: message
// Eq. ms, aggregation Eq. agg, update Eq. updata; batched over replicates as
// Eq. batch).
//
// Work decomposition.  A row v of the pull CSR lists the sources of the arcs
// into v.  Rows are grouped into contiguous tiles of roughly equal in-edge
// load (the target-node partition of Sec. 3.2 applied per workgroup).  Inside
// a wave, G * S lanes own one row: G lanes over the row's replicate words
// (64 replicates per uint64 word, so the G lanes of a neighbour gather read
// 8*G contiguous bytes) and S lanes over its in-edge list.  Per-lane partial
// results are merged with order-free operations (OR for cascades, integer
// addition of bit-sliced counters for counts), so every schedule gives the
// same bits.  Rows with more than `heavy` in-edges are cut into segments whose
// partial results go to a workspace; the wave that finishes a row's last
// segment merges them.
//
// No MFMA here: the step is a sparse gather plus integer/ALU work.
#include "fsg_device.hpp"
#include "fsg_internal.hpp"

#include <algorithm>

namespace fsg {

// Infection thresholds staged in LDS by the step kernel (k = 0 .. kTinfLds-1):
// counts of 16 and more look here, smaller ones in the code table.  A block
// stages them before its first row, so more cost every block what few counts
// use (SIR, 1e6 nodes: 2048 thresholds 84.8 ms a run, 256 81.9, 32 81.8).
constexpr int kTinfLds = 32;

// Threshold of k infected neighbours: LDS copy when staged, global otherwise.
__device__ __forceinline__ uint32_t tinf_at(const StepArgs &a, const uint32_t *tl, int tl_n,
                                            uint32_t k)
{
    if (k > (uint32_t)a.khat) k = (uint32_t)a.khat;
    return (int)k < tl_n ? tl[k] : a.tinf[k];
}

// ---------------------------------------------------------------- IC ----
// Message of arc e = (u -> v) in replicate r: u newly active at t-1 and the
// arc's one trial fires (the trial does not depend on t, and an arc is
// consulted only once per replicate since u is newly active only once).
// Aggregation: OR over arcs.  Update: 0 -> 1 on any message, 1 -> 2.
__device__ __forceinline__ void ic_edge(const StepArgs &a, int e, uint64_t f, uint64_t gbase,
                                        uint32_t tv, uint64_t &acc)
{
    if (!f) return;
    const uint32_t te = a.edge_t ? a.edge_t[e] : tv;
    if (te == 0u) return;
    if (te == kAlways) {
        acc |= f;
        return;
    }
    while (f) {
        const int b = __builtin_ctzll(f);
        const int gs = b - (int)((gbase + (uint64_t)b) & 3u);  // block's first bit
        const uint64_t gm = block_bits(gbase, b);
        const uint64_t bits = f & gm;
        f &= ~gm;
        const uint32_t blk = (uint32_t)((gbase + (uint64_t)b) >> 2);
        const U4 o = philox10((uint32_t)e, blk, 0u, kDomIcEdge << 24, a.key0, a.key1);
        const uint32_t ou[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int bb = gs + j;
            if (bb < 0 || bb > 63) continue;
            if (((bits >> bb) & 1ull) && ou[j] < te) acc |= 1ull << bb;
        }
    }
}

// x or y by a lane's own choice, in registers (as values: an array indexed by
// the lane would be laid out in memory).
__device__ __forceinline__ uint64_t pick2(bool second, uint64_t x, uint64_t y)
{
    const uint32_t m = second ? 0xFFFFFFFFu : 0u;
    const uint32_t lo = ((uint32_t)x & ~m) | ((uint32_t)y & m);
    const uint32_t hi = ((uint32_t)(x >> 32) & ~m) | ((uint32_t)(y >> 32) & m);
    return (uint64_t)hi << 32 | lo;
}

// The trials of eight arcs e, e + S, ... whose sources' words are x0 .. x7 (masked
// by the caller): each lane walks the blocks of four replicates of all words in one
// loop, where a loop per arc took as long as the lane with the most of that
// arc (IC, 3e5 nodes, 1000 replicates: 12.9 -> 9.6 ms).
__device__ __forceinline__ void ic_trials(const StepArgs &a, int e, int S, uint64_t x0, uint64_t x1,
                                          uint64_t x2, uint64_t x3, uint64_t x4, uint64_t x5,
                                          uint64_t x6, uint64_t x7, uint64_t gbase, uint32_t tv,
                                          uint64_t &acc)
{
    if ((a.goff & 3u) != 0u) {  // blocks of four are not nibbles of the word
        ic_edge(a, e, x0 & ~acc, gbase, tv, acc);
        ic_edge(a, e + S, x1 & ~acc, gbase, tv, acc);
        ic_edge(a, e + 2 * S, x2 & ~acc, gbase, tv, acc);
        ic_edge(a, e + 3 * S, x3 & ~acc, gbase, tv, acc);
        ic_edge(a, e + 4 * S, x4 & ~acc, gbase, tv, acc);
        ic_edge(a, e + 5 * S, x5 & ~acc, gbase, tv, acc);
        ic_edge(a, e + 6 * S, x6 & ~acc, gbase, tv, acc);
        ic_edge(a, e + 7 * S, x7 & ~acc, gbase, tv, acc);
        return;
    }
    // bit k: the word of arc k not yet begun
    uint32_t left = (x0 ? 1u : 0u) | (x1 ? 2u : 0u) | (x2 ? 4u : 0u) | (x3 ? 8u : 0u) |
                    (x4 ? 16u : 0u) | (x5 ? 32u : 0u) | (x6 ? 64u : 0u) | (x7 ? 128u : 0u);
    const uint32_t blk0 = (uint32_t)(gbase >> 2);
    uint64_t need = 0;
    uint32_t te = tv, arc = 0;
    while (left != 0u || need != 0ull) {
        if (need == 0ull) {
            const int k = __builtin_ctz(left);
            left &= left - 1u;
            need = pick2((k & 4) != 0, pick2((k & 2) != 0, pick2((k & 1) != 0, x0, x1), pick2((k & 1) != 0, x2, x3)),
                         pick2((k & 2) != 0, pick2((k & 1) != 0, x4, x5), pick2((k & 1) != 0, x6, x7))) & ~acc;
            arc = (uint32_t)(e + k * S);
            if (a.edge_t) te = a.edge_t[arc];
            if (te == kAlways) acc |= need;
            if (te == 0u || te == kAlways) need = 0ull;
        }
        if (need != 0ull) {
            const int gs = __builtin_ctzll(need) & ~3;
            const uint32_t bits = (uint32_t)(need >> gs) & 0xFu;
            need &= ~(0xFull << gs);
            const U4 o = philox10(arc, blk0 + ((uint32_t)gs >> 2), 0u, kDomIcEdge << 24, a.key0, a.key1);
            uint32_t f = o.w < te ? 1u : 0u;
            f = f + f + (o.z < te ? 1u : 0u);
            f = f + f + (o.y < te ? 1u : 0u);
            f = f + f + (o.x < te ? 1u : 0u);
            acc |= (uint64_t)(f & bits) << gs;
        }
    }
}

// Trials of a lane's share of the arcs [e0, e1) into v for the replicates
// `cand` of word w: with whole 16-lane rows (S = 1, G >= 16, 32-bit offsets)
// the lane's group takes all of [e0, e1), else arcs e0 + s, e0 + s + S, ...
__device__ __forceinline__ void ic_arcs(const StepArgs &a, int G, int S, bool valid, int e0, int e1,
                                        int s, int w, uint64_t cand, uint32_t tv, uint64_t &acc)
{
    const int64_t W = a.W;
    const uint64_t gbase = a.goff + 64ull * (uint64_t)w;
    if (S == 1 && G >= 16 && a.fast32) {
        // 16 arcs of the row per pass: lane lr of each 16-lane DPP row loads
        // source e0 + base + lr, the row's lanes receive them by row
        // broadcast and gather their word of each; arcs past the row's end
        // read the all-zero row n, so they never reach a trial
        const int lr = (int)(threadIdx.x & 15u);
        int dmax = 0;
        const int d = valid ? e1 - e0 : 0;
        for (int l = 0; l < 64; l += G) dmax = max(dmax, __builtin_amdgcn_readlane(d, l));
        if (dmax > 0 && __ballot(cand != 0ull) != 0ull) {
            const uint32_t W8 = (uint32_t)a.W * 8u, w8 = (uint32_t)w * 8u, zero = (uint32_t)a.n;
            const char *prev = reinterpret_cast<const char *>(a.prev);
            auto src_at = [&](int base) -> uint32_t {
                const int e = e0 + base + lr;
                return e < e1 ? (uint32_t)ld32_off32(a.src, (uint32_t)e) : zero;
            };
            auto word = [&](uint32_t u) -> uint64_t {
                return *reinterpret_cast<const uint64_t *>(prev + __umul24(cand ? u : zero, W8) + w8);
            };
            uint32_t cur = src_at(0);
            for (int base = 0; base < dmax; base += 16) {
                const uint32_t nxt = base + 16 < dmax ? src_at(base + 16) : zero;
                {
                    const uint64_t x0 = word(row_bcast<0>(cur)), x1 = word(row_bcast<1>(cur)),
                                   x2 = word(row_bcast<2>(cur)), x3 = word(row_bcast<3>(cur)),
                                   x4 = word(row_bcast<4>(cur)), x5 = word(row_bcast<5>(cur)),
                                   x6 = word(row_bcast<6>(cur)), x7 = word(row_bcast<7>(cur));
                    const uint64_t m = cand & ~acc;
                    ic_trials(a, e0 + base, 1, x0 & m, x1 & m, x2 & m, x3 & m, x4 & m, x5 & m, x6 & m,
                              x7 & m, gbase, tv, acc);
                }
                if (dmax - base > 8) {
                    const uint64_t x0 = word(row_bcast<8>(cur)), x1 = word(row_bcast<9>(cur)),
                                   x2 = word(row_bcast<10>(cur)), x3 = word(row_bcast<11>(cur)),
                                   x4 = word(row_bcast<12>(cur)), x5 = word(row_bcast<13>(cur)),
                                   x6 = word(row_bcast<14>(cur)), x7 = word(row_bcast<15>(cur));
                    const uint64_t m = cand & ~acc;
                    ic_trials(a, e0 + base + 8, 1, x0 & m, x1 & m, x2 & m, x3 & m, x4 & m, x5 & m, x6 & m,
                              x7 & m, gbase, tv, acc);
                }
                cur = nxt;
            }
        }
    } else if (cand && a.fast32) {
        // four gathers in flight, the next four sources with them; slots
        // past the end read the all-zero row n
        const uint32_t Wu = (uint32_t)a.W, ww = (uint32_t)w, zero = (uint32_t)a.n;
        auto src_at = [&](int e) -> uint32_t {
            return e < e1 ? (uint32_t)ld32_off32(a.src, (uint32_t)e) : zero;
        };
        int e = e0 + s;
        uint32_t u0 = src_at(e), u1 = src_at(e + S), u2 = src_at(e + 2 * S), u3 = src_at(e + 3 * S);
        for (; e < e1; e += 4 * S) {
            const uint64_t f0 = ld64_off32(a.prev, __umul24(u0, Wu) + ww);
            const uint64_t f1 = ld64_off32(a.prev, __umul24(u1, Wu) + ww);
            const uint64_t f2 = ld64_off32(a.prev, __umul24(u2, Wu) + ww);
            const uint64_t f3 = ld64_off32(a.prev, __umul24(u3, Wu) + ww);
            const int en = e + 4 * S;
            u0 = src_at(en);
            u1 = src_at(en + S);
            u2 = src_at(en + 2 * S);
            u3 = src_at(en + 3 * S);
            const uint64_t m = cand & ~acc;
            ic_trials(a, e, S, f0 & m, f1 & m, f2 & m, f3 & m, 0ull, 0ull, 0ull, 0ull, gbase, tv, acc);
        }
    } else if (cand) {
        walk_arcs(
            (uint32_t)e0 + (uint32_t)s, (uint32_t)e1, (uint32_t)S,
            [&](uint32_t e) {  // four independent gathers in flight per lane
                const int u0 = a.src[e], u1 = a.src[e + S], u2 = a.src[e + 2 * S],
                          u3 = a.src[e + 3 * S];
                const uint64_t f0 = a.prev[(int64_t)u0 * W + w], f1 = a.prev[(int64_t)u1 * W + w],
                               f2 = a.prev[(int64_t)u2 * W + w], f3 = a.prev[(int64_t)u3 * W + w];
                const uint64_t m = cand & ~acc;
                ic_trials(a, (int)e, S, f0 & m, f1 & m, f2 & m, f3 & m, 0ull, 0ull, 0ull, 0ull, gbase,
                          tv, acc);
            },
            [&](uint32_t e) {
                ic_edge(a, (int)e, a.prev[(int64_t)a.src[e] * W + w] & cand & ~acc, gbase, tv, acc);
            });
    }
}

__device__ __forceinline__ void ic_row_word(const StepArgs &a, int G, int S, bool valid, int v,
                                            int w, int e0, int e1, uint32_t tv, int s, uint64_t lm,
                                            bool &any)
{
    const int64_t idx = (int64_t)v * a.W + w;
    const uint64_t A = valid ? a.aux[idx] : ~0ull;
    const uint64_t cand = valid ? (~A & tail_mask(w, a.B) & lm) : 0ull;
    uint64_t acc = 0;
    ic_arcs(a, G, S, valid, e0, e1, s, w, cand, tv, acc);
    acc = or_reduce_lanes(acc, G, S);
    if (!valid || s != 0) return;
    a.next[idx] = acc;
    a.aux[idx] = A | acc;
    any |= acc != 0;
}

// Bit-sliced count of the in-neighbours whose word has the replicate's bit
// set: four independent gathers in flight per lane, folded in with carry-save
// adders.  Counts are kept for every replicate of the word; callers use them
// only under their own state mask.  The fast path addresses sources and
// planes with 32-bit offsets from uniform bases and 24-bit index products.
template <int L>
__device__ __forceinline__ void count_edges(const StepArgs &a, int e, int e1, int S, int w,
                                            uint64_t (&c)[L])
{
    if (a.fast32) {
        // the next four sources are loaded while the gathers of these four
        // are in flight; slots past the end read the all-zero row n, so the
        // last pass takes one round trip as well
        const uint32_t W = (uint32_t)a.W, ww = (uint32_t)w, zero = (uint32_t)a.n;
        auto src_at = [&](int i) -> uint32_t {
            return i < e1 ? (uint32_t)ld32_off32(a.src, (uint32_t)i) : zero;
        };
        uint32_t u0 = src_at(e), u1 = src_at(e + S), u2 = src_at(e + 2 * S), u3 = src_at(e + 3 * S);
        for (; e < e1; e += 4 * S) {
            const uint64_t x0 = ld64_off32(a.prev, __umul24(u0, W) + ww);
            const uint64_t x1 = ld64_off32(a.prev, __umul24(u1, W) + ww);
            const uint64_t x2 = ld64_off32(a.prev, __umul24(u2, W) + ww);
            const uint64_t x3 = ld64_off32(a.prev, __umul24(u3, W) + ww);
            const int en = e + 4 * S;
            u0 = src_at(en);
            u1 = src_at(en + S);
            u2 = src_at(en + 2 * S);
            u3 = src_at(en + 3 * S);
            bs_add4<L>(c, x0, x1, x2, x3);
        }
        return;
    }
    const int64_t W = a.W;
    walk_arcs(
        (uint32_t)e, (uint32_t)e1, (uint32_t)S,
        [&](uint32_t i) {
            const int u0 = a.src[i], u1 = a.src[i + S], u2 = a.src[i + 2 * S], u3 = a.src[i + 3 * S];
            bs_add4<L>(c, a.prev[(int64_t)u0 * W + w], a.prev[(int64_t)u1 * W + w],
                       a.prev[(int64_t)u2 * W + w], a.prev[(int64_t)u3 * W + w]);
        },
        [&](uint32_t i) { bs_add1<L>(c, a.prev[(int64_t)a.src[i] * W + w]); });
}

// The same count when a row owns whole 16-lane rows of the wave (G >= 16,
// S = 1) and 32-bit offsets apply: the 16 lanes load 16 consecutive sources
// of their row with one vector load (the next chunk's load issued before the
// current chunk's gathers), and each source reaches every lane of the row by a
// DPP row broadcast; the gathers then go out eight at a time without waiting
// on index loads.  Positions past the row's end carry source n, whose plane
// row is all zero, as does every position of a lane whose word needs no
// count.  All 64 lanes of the wave must call this together.
template <int L>
__device__ __forceinline__ void count_edges_bcast(const StepArgs &a, int G, bool valid, int e0,
                                                  int e1, int w, bool need, uint64_t (&c)[L])
{
    const int lr = (int)(threadIdx.x & 15u);
    int dmax = 0;  // longest valid row of the wave (word 0 of a row is valid iff the row is)
    const int d = valid ? e1 - e0 : 0;
    for (int l = 0; l < 64; l += G) dmax = max(dmax, __builtin_amdgcn_readlane(d, l));
    if (dmax == 0 || __ballot(need) == 0ull) return;
    const uint32_t W8 = (uint32_t)a.W * 8u, w8 = (uint32_t)w * 8u, zero = (uint32_t)a.n;
    const char *prev = reinterpret_cast<const char *>(a.prev);
    auto src_at = [&](int base) -> uint32_t {
        const int e = e0 + base + lr;
        return e < e1 ? (uint32_t)ld32_off32(a.src, (uint32_t)e) : zero;
    };
    auto word = [&](uint32_t u) -> uint64_t {
        return *reinterpret_cast<const uint64_t *>(prev + __umul24(need ? u : zero, W8) + w8);
    };
    uint32_t cur = src_at(0);
    for (int base = 0; base < dmax; base += 16) {
        const uint32_t nxt = base + 16 < dmax ? src_at(base + 16) : zero;
        {
            const uint64_t x0 = word(row_bcast<0>(cur)), x1 = word(row_bcast<1>(cur)),
                           x2 = word(row_bcast<2>(cur)), x3 = word(row_bcast<3>(cur)),
                           x4 = word(row_bcast<4>(cur)), x5 = word(row_bcast<5>(cur)),
                           x6 = word(row_bcast<6>(cur)), x7 = word(row_bcast<7>(cur));
            bs_add4<L>(c, x0, x1, x2, x3);
            bs_add4<L>(c, x4, x5, x6, x7);
        }
        if (dmax - base > 8) {
            const uint64_t x0 = word(row_bcast<8>(cur)), x1 = word(row_bcast<9>(cur)),
                           x2 = word(row_bcast<10>(cur)), x3 = word(row_bcast<11>(cur)),
                           x4 = word(row_bcast<12>(cur)), x5 = word(row_bcast<13>(cur)),
                           x6 = word(row_bcast<14>(cur)), x7 = word(row_bcast<15>(cur));
            bs_add4<L>(c, x0, x1, x2, x3);
            bs_add4<L>(c, x4, x5, x6, x7);
        }
        cur = nxt;
    }
}

// ------------------------------------------------------ SI / SIS / SIR ----
// Appendix A.1: the log-survival messages of the k infected in-neighbours sum
// to k log(1-beta), so a susceptible node is infected with probability
// 1 - (1-beta)^k; the k-indexed thresholds come from the host.  One draw per
// (node, replicate, step) decides whichever transition the node's state
// allows (infection if S, recovery if I).
// Draw classes of the aligned decision path: a 5-bit code per replicate from
// five bit planes, code = k for k = 1 .. 15 infected in-neighbours, 16 for
// sixteen or more (threshold from the exact count), 17 = infected with a
// recovery draw, 18 = latent (SEIR / SEIS) with an E -> I draw.  The table
// maps a code to its threshold (0 for codes that never fire here); its last
// entry is not a threshold but the mask of the codes 1 .. 15 whose threshold
// always fires (those replicates take no draw).
constexpr int kCodeTable = 32;
constexpr int kCodeAlwaysMask = kCodeTable - 1;

__device__ __forceinline__ uint32_t code_threshold(const StepArgs &a, int code)
{
    if (code >= 1 && code <= 15) return a.tinf[code < a.khat ? code : a.khat];
    if (code == 17) return a.trec;
    if (code == 18) return a.talpha;
    return 0u;
}

// The code table into LDS, by the first wave of a block (a lane an entry, the
// mask from their ballot: one thread reading all fifteen thresholds held every
// block, SIR at 2e4 nodes 5.03 -> 4.85 ms a run of 169 steps).
__device__ __forceinline__ void stage_codes(const StepArgs &a, uint32_t *s_code)
{
    if (threadIdx.x >= kCodeTable) return;
    const uint32_t t = code_threshold(a, threadIdx.x);
    const uint64_t always = __ballot(threadIdx.x >= 1 && threadIdx.x <= 15 && t == kAlways);
    s_code[threadIdx.x] = threadIdx.x == kCodeAlwaysMask ? (uint32_t)always : t;
}

// Bit plane K of a bit-sliced counter (zero past its last plane).
template <int K, int L>
__device__ __forceinline__ uint64_t plane(const uint64_t (&c)[L])
{
    if constexpr (K < L) return c[K];
    else return 0ull;
}

// Spread the four bits of a nibble to bit 0 of the four bytes of a word.
__device__ __forceinline__ uint32_t spread4(uint32_t n, uint32_t mul, uint32_t mask)
{
    return __umul24(n, mul) & mask;
}

// SWIR (states S, W weakened, I, R; a reading of the model the paper only
// names): with k infected in-neighbours a susceptible replicate becomes I if
// its draw fires against thr(1-(1-kappa)^k), else W if it fires against
// thr(1-(1-kappa-mu)^k); a weakened one becomes I against thr(1-(1-nu)^k);
// an infected one is removed after one step.  One draw per (node, replicate,
// step), taken only where k >= 1; counts are exact per replicate here (the
// model is off the hot path).  `wk` is the weakened plane.
__device__ __forceinline__ uint32_t swir_table(const uint32_t *t, int32_t khat, uint32_t k)
{
    return t[k > (uint32_t)khat ? (uint32_t)khat : k];
}

template <int LC>
__device__ __forceinline__ void swir_decide(const StepArgs &a, int G, int S, bool valid, int v,
                                            int w, int64_t idx, uint64_t h, uint64_t r, uint64_t wk,
                                            uint64_t sus, const uint64_t (&c)[LC], int s,
                                            uint64_t share, bool &any)
{
    const uint64_t gbase = a.goff + 64ull * (uint64_t)w;
    uint64_t need = (sus | wk) & bs_nonzero<LC>(c) & share;
    uint64_t toI = 0, toW = 0;
    while (need) {
        const int b = __builtin_ctzll(need);
        const int gs = b - (int)((gbase + (uint64_t)b) & 3u);  // first bit of the block
        const uint32_t blk = (uint32_t)((gbase + (uint64_t)b) >> 2);
        const uint32_t nn = nibble_at(need, gs);
        need &= ~nibble_to_word(0xFu, gs);
        const U4 o = philox10((uint32_t)v, blk, a.step, kDomNodeStep << 24, a.key0, a.key1);
        const uint32_t ou[4] = {o.x, o.y, o.z, o.w};
        const uint32_t ns = nibble_at(sus, gs);
        uint32_t fi = 0, fw = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!((nn >> j) & 1u)) continue;
            const uint32_t k = bs_get<LC>(c, gs + j);
            if ((ns >> j) & 1u) {
                if (fires(ou[j], swir_table(a.tinf, a.khat, k)))
                    fi |= 1u << j;
                else if (fires(ou[j], swir_table(a.tsiw, a.khat_siw, k)))
                    fw |= 1u << j;
            } else if (fires(ou[j], swir_table(a.twi, a.khat_wi, k))) {
                fi |= 1u << j;
            }
        }
        toI |= nibble_to_word(fi, gs);
        toW |= nibble_to_word(fw, gs);
    }
    toI = or_reduce_lanes(toI, G, S);
    toW = or_reduce_lanes(toW, G, S);
    if (!valid || s != 0) return;
    a.next[idx] = toI;               // infected for one step
    a.lat[idx] = (wk & ~toI) | toW;
    a.aux[idx] = r | h;              // removed after it
    any |= toI != 0;
}

template <int LC>
__device__ __forceinline__ void epi_decide(const StepArgs &a, int G, int S, bool valid, int v,
                                           int w, int64_t idx, uint64_t h, uint64_t r, uint64_t e,
                                           uint64_t sus, const uint64_t (&c)[LC], int s,
                                           uint64_t share, const uint32_t *tl, int tl_n,
                                           const uint32_t *tcode, bool &any)
{
    if (a.model == kSWIR) {
        swir_decide<LC>(a, G, S, valid, v, w, idx, h, r, e, sus, c, s, share, any);
        return;
    }
    const uint64_t gbase = a.goff + 64ull * (uint64_t)w;
    const bool draw_rec = a.trec != 0u && a.trec != kAlways;
    const bool draw_lat = a.talpha != 0u && a.talpha != kAlways;
    const uint32_t trec = a.trec, tlat = a.talpha;
    uint64_t inf = 0, rec = 0, act = 0;  // S -> I or E, I -> R or S, E -> I
    uint32_t ncalls = 0;                 // generator calls of this lane
    if (tcode != nullptr && (a.goff & 3u) == 0u) {
        // generator blocks are nibbles of the word: one draw per block with
        // any replicate that needs one, the class of each replicate read from
        // five bit planes, its threshold from the code table
        uint64_t rest = 0;  // sixteen or more
#pragma unroll
        for (int l = 4; l < LC; ++l) rest |= c[l];
        const uint64_t c0 = plane<0>(c), c1 = plane<1>(c), c2 = plane<2>(c), c3 = plane<3>(c);
        const uint64_t ninf = sus & share & (c0 | c1 | c2 | c3 | rest);  // k >= 1
        uint64_t always = 0;  // classes whose threshold always fires
        const uint32_t acodes = tcode[kCodeAlwaysMask];
        if (acodes) {
            for (int k = 1; k <= 15; ++k)
                if ((acodes >> k) & 1u)
                    always |= ~rest & ((k & 1) ? c0 : ~c0) & ((k & 2) ? c1 : ~c1) &
                              ((k & 4) ? c2 : ~c2) & ((k & 8) ? c3 : ~c3);
            always &= ninf;
        }
        const uint64_t ndraw = ninf & ~always;
        const uint64_t nrec = draw_rec ? (h & share) : 0ull;
        const uint64_t nlat = draw_lat ? (e & share) : 0ull;
        const uint64_t low = ndraw & ~rest;
        const uint64_t P0 = (low & c0) | nrec, P1 = (low & c1) | nlat, P2 = low & c2,
                       P3 = low & c3, P4 = (ndraw & rest) | nrec | nlat;
        uint64_t need = ndraw | nrec | nlat;
        uint64_t fire = 0;
        const uint32_t blk0 = (uint32_t)(gbase >> 2);
        while (need) {
            const int b = __builtin_ctzll(need);
            const int gs = b & ~3;
            need &= ~(0xFull << gs);
            const bool hi = gs >= 32;
            const uint32_t sh = (uint32_t)gs & 31u;
            auto nib = [&](uint64_t P) -> uint32_t {
                return ((hi ? (uint32_t)(P >> 32) : (uint32_t)P) >> sh) & 0xFu;
            };
            const uint32_t n0 = nib(P0), n1 = nib(P1), n2 = nib(P2), n3 = nib(P3), n4 = nib(P4);
            // byte j of T = 4 * code of replicate j (a byte offset into the table)
            const uint32_t T = spread4(n0, 0x810204u, 0x04040404u) |
                               (spread4(n1, 0x204081u, 0x01010101u) << 3) |
                               (spread4(n2, 0x204081u, 0x01010101u) << 4) |
                               (spread4(n3, 0x204081u, 0x01010101u) << 5) |
                               (spread4(n4, 0x204081u, 0x01010101u) << 6);
            const char *tb = reinterpret_cast<const char *>(tcode);
            const uint32_t q0 = *reinterpret_cast<const uint32_t *>(tb + (T & 0xFFu));
            const uint32_t q1 = *reinterpret_cast<const uint32_t *>(tb + ((T >> 8) & 0xFFu));
            const uint32_t q2 = *reinterpret_cast<const uint32_t *>(tb + ((T >> 16) & 0xFFu));
            const uint32_t q3 = *reinterpret_cast<const uint32_t *>(tb + (T >> 24));
            const U4 o = philox10((uint32_t)v, blk0 + ((uint32_t)gs >> 2), a.step,
                                  kDomNodeStep << 24, a.key0, a.key1);
            ++ncalls;
            uint32_t f = (o.w < q3) ? 1u : 0u;
            f = f + f + ((o.z < q2) ? 1u : 0u);
            f = f + f + ((o.y < q1) ? 1u : 0u);
            f = f + f + ((o.x < q0) ? 1u : 0u);
            const uint32_t nb = n4 & ~n0 & ~n1;  // code 16: sixteen or more infected neighbours
            if (nb) {
                const uint32_t ou[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((nb >> j) & 1u)
                        f |= (fires(ou[j], tinf_at(a, tl, tl_n, bs_get<LC>(c, gs + j))) ? 1u : 0u)
                             << j;
            }
            fire |= (uint64_t)f << gs;
        }
        inf = (fire & ~h & ~e) | always;
        rec = fire & h;
        act = fire & e;
    } else {
        uint64_t need = sus & bs_nonzero<LC>(c);
        if (draw_rec) need |= h;
        if (draw_lat) need |= e;
        need &= share;
        const SmallCounts sm = bs_small<LC>(c);
        const uint64_t big = sus & ~(sm.m1 | sm.m2 | sm.m3) & bs_nonzero<LC>(c);  // k >= 4
        const uint32_t t1 = tinf_at(a, tl, tl_n, 1u), t2 = tinf_at(a, tl, tl_n, 2u),
                       t3 = tinf_at(a, tl, tl_n, 3u);
        while (need) {
            const int b = __builtin_ctzll(need);
            const int gs = b - (int)((gbase + (uint64_t)b) & 3u);  // first bit of the block
            const uint32_t blk = (uint32_t)((gbase + (uint64_t)b) >> 2);
            const uint32_t nn = nibble_at(need, gs);
            need &= ~nibble_to_word(0xFu, gs);
            const U4 o = philox10((uint32_t)v, blk, a.step, kDomNodeStep << 24, a.key0, a.key1);
            ++ncalls;
            const uint32_t ou[4] = {o.x, o.y, o.z, o.w};
            const uint32_t nh = nibble_at(h, gs), ne = nibble_at(e, gs), n1 = nibble_at(sm.m1, gs),
                           n2 = nibble_at(sm.m2, gs), n3 = nibble_at(sm.m3, gs),
                           nb = nibble_at(big, gs);
            uint32_t tb[4] = {0u, 0u, 0u, 0u};
            if (nb) {  // a replicate of this block has four or more infected neighbours
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((nb >> j) & 1u) tb[j] = tinf_at(a, tl, tl_n, bs_get<LC>(c, gs + j));
            }
            uint32_t fi = 0, fr = 0, fe = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool isI = (nh >> j) & 1u, isE = (ne >> j) & 1u;
                uint32_t t = ((n1 >> j) & 1u) ? t1
                                              : (((n2 >> j) & 1u) ? t2 : (((n3 >> j) & 1u) ? t3 : tb[j]));
                t = isI ? trec : (isE ? tlat : t);
                const uint32_t f = (((nn >> j) & 1u) && fires(ou[j], t)) ? 1u : 0u;
                fi |= ((isI || isE) ? 0u : f) << j;
                fr |= (isI ? f : 0u) << j;
                fe |= (isE ? f : 0u) << j;
            }
            inf |= nibble_to_word(fi, gs);
            rec |= nibble_to_word(fr, gs);
            act |= nibble_to_word(fe, gs);
        }
    }
    if (a.draws) {  // counting runs only (all 64 lanes are here together)
        for (int off = 32; off >= 1; off >>= 1) ncalls += (uint32_t)__shfl_xor((int)ncalls, off, 64);
        if ((threadIdx.x & 63) == 0 && ncalls) atomicAdd(a.draws, (unsigned long long)ncalls);
    }
    inf = or_reduce_lanes(inf, G, S);
    rec = or_reduce_lanes(rec, G, S);
    act = or_reduce_lanes(act, G, S);
    if (a.trec == kAlways) rec = h;
    if (a.talpha == kAlways) act = e;
    if (!valid || s != 0) return;
    if (a.lat) {  // SEIR / SEIS: infection leads to E, E -> I
        const uint64_t nh = (h & ~rec) | act;
        const uint64_t ne = (e & ~act) | inf;
        a.next[idx] = nh;
        a.lat[idx] = ne;
        if (a.model == kSEIR) a.aux[idx] = r | rec;
        any |= (nh | ne) != 0;
        return;
    }
    const uint64_t nh = (h & ~rec) | inf;
    const uint64_t nr = (a.model == kSIS) ? r : (r | rec);
    a.next[idx] = nh;
    a.aux[idx] = nr;
    any |= nh != 0;
}

// Tail mode: node v has an infected replicate after step t (bitmap t % 4).
__device__ __forceinline__ void mark_infected(const StepArgs &a, int v)
{
    atomicOr(&a.ibm[(size_t)(a.step & 3u) * (size_t)a.ibm_words + (size_t)(v >> 5)], 1u << (v & 31));
}

template <int L>
__device__ __forceinline__ void epi_row_word(const StepArgs &a, int G, int S, bool valid, int v,
                                             int w, int e0, int e1, int s, uint64_t share,
                                             const uint32_t *tl, int tl_n, const uint32_t *tcode,
                                             uint64_t lm, bool &any)
{
    const int64_t idx = (int64_t)v * a.W + w;
    const uint64_t h = valid ? a.prev[idx] : 0ull;
    const uint64_t r = valid ? a.aux[idx] : 0ull;
    const uint64_t e = (valid && a.lat) ? a.lat[idx] : 0ull;
    const uint64_t sus = valid ? (~(h | r | e) & tail_mask(w, a.B) & lm) : 0ull;
    // replicates whose decision needs the count (SWIR: weakened ones too)
    const uint64_t counted = a.model == kSWIR ? (sus | (e & lm)) : sus;
    uint64_t c[L];
#pragma unroll
    for (int l = 0; l < L; ++l) c[l] = 0;
    if (S == 1 && G >= 16 && a.fast32)
        count_edges_bcast<L>(a, G, valid, e0, e1, w, counted != 0ull, c);
    else if (counted)
        count_edges<L>(a, e0 + s, e1, S, w, c);
    bs_reduce_lanes<L>(c, G, S);
    epi_decide<L>(a, G, S, valid, v, w, idx, h, r, e, sus, c, s, share, tl, tl_n, tcode, any);
}

// ---------------------------------------------------------------- LT ----
// In-weights 1/indeg and threshold U/2^32 drawn once per (node, replicate):
// v activates once c active in-neighbours satisfy c >= ceil(U indeg / 2^32)
// (and c >= 1).
constexpr int kPlaneBlocks = 4;

template <int LC>
__device__ __forceinline__ void lt_decide(const StepArgs &a, int G, int S, bool valid, int v,
                                          int w, int64_t idx, uint64_t act, uint64_t inact,
                                          uint32_t indeg, const uint64_t (&c)[LC], int s,
                                          uint64_t share, bool use_need, bool &any)
{
    const uint64_t gbase = a.goff + 64ull * (uint64_t)w;
    uint64_t nw = 0;
    const int P = indeg ? 32 - __builtin_clz(indeg) : 0;  // planes of the stored thresholds
    uint64_t nz = 0;
#pragma unroll
    for (int l = 0; l < LC; ++l) nz |= c[l];
    const uint64_t cand = inact & share & nz;
    // Stored thresholds cost bitlen(indeg) word loads, a fresh draw one
    // Philox call per 4-replicate block with a candidate: the wave reads the
    // planes when some lane has more than kPlaneBlocks such blocks.
    bool planes = false;
    if (use_need && a.need != nullptr) {
        uint64_t blk = cand | (cand >> 1) | (cand >> 2) | (cand >> 3);
        blk &= 0x1111111111111111ull;
        planes = __ballot(__popcll(blk) > kPlaneBlocks) != 0ull;
    }
    if (planes && P <= LC) {
        // v activates in replicate r iff c_r >= need_r, i.e. iff c - need
        // does not borrow (the chain runs plane by plane over the word)
        if (cand) {
            const uint64_t *np = a.need + (int64_t)v * a.Lp * a.W + w;
            uint64_t borrow = 0;
#pragma unroll
            for (int l = 0; l < LC; ++l) {
                const uint64_t nl = l < P ? np[(int64_t)l * a.W] : 0ull;
                borrow = maj3(~c[l], nl, borrow);
            }
            nw = cand & ~borrow;
        }
    } else if ((a.goff & 3u) == 0u) {
        // aligned generator blocks, branch-free per block: c = c0 + 2 c1
        // when no higher plane is set; v activates iff c 2^32 >= U indeg,
        // i.e. iff c > hi or (c == hi and lo == 0) for U indeg = hi 2^32 + lo.
        // Replicates whose every in-neighbour is active (c == indeg) always
        // activate and need no draw.
        uint64_t rest = 0;
#pragma unroll
        for (int l = 2; l < LC; ++l) rest |= c[l];
        const uint64_t c0 = c[0], c1 = LC > 1 ? c[LC > 1 ? 1 : 0] : 0ull;
        const uint64_t cand = inact & share & (c0 | c1 | rest);
        uint64_t full = cand;  // c == indeg, plane by plane
#pragma unroll
        for (int l = 0; l < LC; ++l) full &= ((indeg >> l) & 1u) ? c[l] : ~c[l];
        if (((uint64_t)indeg >> LC) != 0ull) full = 0;  // c < 2^LC <= indeg
        uint64_t need = cand & ~full;
        uint64_t fire = 0;
        const uint32_t blk0 = (uint32_t)(gbase >> 2);
        while (need) {
            const int b = __builtin_ctzll(need);
            const int gs = b & ~3;
            const bool hi32 = gs >= 32;
            const uint32_t sh = (uint32_t)gs & 31u;
            const uint32_t nn = ((hi32 ? (uint32_t)(need >> 32) : (uint32_t)need) >> sh) & 0xFu;
            need &= ~(0xFull << gs);
            const uint32_t n0 = ((hi32 ? (uint32_t)(c0 >> 32) : (uint32_t)c0) >> sh) & 0xFu;
            const uint32_t n1 = ((hi32 ? (uint32_t)(c1 >> 32) : (uint32_t)c1) >> sh) & 0xFu;
            const uint32_t nr = ((hi32 ? (uint32_t)(rest >> 32) : (uint32_t)rest) >> sh) & 0xFu;
            const U4 o = philox10((uint32_t)v, blk0 + ((uint32_t)gs >> 2), 0u, kDomLtThresh << 24,
                                  a.key0, a.key1);
            const uint32_t ou[4] = {o.x, o.y, o.z, o.w};
            uint32_t f = 0;
#pragma unroll
            for (int j = 3; j >= 0; --j) {
                uint32_t k = ((n0 >> j) & 1u) + 2u * ((n1 >> j) & 1u);
                if ((nr >> j) & 1u) k = bs_get<LC>(c, gs + j);  // four or more active
                const uint64_t prod = (uint64_t)ou[j] * (uint64_t)indeg;
                const uint32_t ph = (uint32_t)(prod >> 32), pl = (uint32_t)prod;
                f = f + f + ((k > ph || (k == ph && pl == 0u)) ? 1u : 0u);
            }
            fire |= (uint64_t)(f & nn) << gs;
        }
        nw = fire | full;
    } else {
    uint64_t cand = inact & bs_nonzero<LC>(c) & share;
    const SmallCounts sm = bs_small<LC>(c);
    while (cand) {
        const int b = __builtin_ctzll(cand);
        const int gs = b - (int)((gbase + (uint64_t)b) & 3u);
        const uint32_t blk = (uint32_t)((gbase + (uint64_t)b) >> 2);
        const uint32_t nc = nibble_at(cand, gs);
        cand &= ~nibble_to_word(0xFu, gs);
        const U4 o = philox10((uint32_t)v, blk, 0u, kDomLtThresh << 24, a.key0, a.key1);
        const uint32_t ou[4] = {o.x, o.y, o.z, o.w};
        const uint32_t n1 = nibble_at(sm.m1, gs), n2 = nibble_at(sm.m2, gs),
                       n3 = nibble_at(sm.m3, gs);
        uint32_t fa = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!((nc >> j) & 1u)) continue;
            uint32_t k = ((n1 >> j) & 1u) ? 1u : (((n2 >> j) & 1u) ? 2u : (((n3 >> j) & 1u) ? 3u : 0u));
            if (k == 0u) k = bs_get<LC>(c, gs + j);  // four or more active neighbours
            // c >= 1 here, so max(1, need) = need
            const uint64_t need = ((uint64_t)ou[j] * (uint64_t)indeg + 0xFFFFFFFFull) >> 32;
            if ((uint64_t)k >= need) fa |= 1u << j;
        }
        nw |= nibble_to_word(fa, gs);
    }
    }
    nw = or_reduce_lanes(nw, G, S);
    if (!valid || s != 0) return;
    a.next[idx] = act | nw;
    if (nw != 0ull && a.stamp != nullptr)
        a.stamp[(size_t)(a.step & 1u) * (size_t)a.n + (size_t)v] = a.step;
    any |= nw != 0;
}

template <int L>
__device__ __forceinline__ void lt_row_word(const StepArgs &a, int G, int S, bool valid, int v,
                                            int w, int e0, int e1, uint32_t indeg, int s,
                                            uint64_t share, uint64_t lm, bool &any)
{
    const int64_t idx = (int64_t)v * a.W + w;
    const uint64_t act = valid ? a.prev[idx] : 0ull;
    const uint64_t inact = valid ? (~act & tail_mask(w, a.B) & lm) : 0ull;
    uint64_t c[L];
#pragma unroll
    for (int l = 0; l < L; ++l) c[l] = 0;
    if (S == 1 && G >= 16 && a.fast32)
        count_edges_bcast<L>(a, G, valid, e0, e1, w, inact != 0ull, c);
    else if (inact)
        count_edges<L>(a, e0 + s, e1, S, w, c);
    bs_reduce_lanes<L>(c, G, S);
    lt_decide<L>(a, G, S, valid, v, w, idx, act, inact, indeg, c, s, share, true, any);
}

__device__ __forceinline__ uint32_t wc_threshold(uint32_t indeg)
{
    // weighted cascade p = 1/indeg: floor(2^32 / indeg), 1 -> always
    return indeg <= 1u ? kAlways : (uint32_t)(0x100000000ull / (uint64_t)indeg);
}

template <int KIND, int L>
__device__ __forceinline__ void row_word(const StepArgs &a, int G, int S, bool valid, int v, int w,
                                         int e0, int e1, uint32_t indeg, int s,
                                         uint64_t share_fixed, const uint32_t *tl, int tl_n,
                                         const uint32_t *tcode, uint64_t lm, bool &any)
{
    // draws of lane s: generator blocks congruent to s mod S; for S <= 16 the
    // pattern repeats every word, otherwise it depends on the word
    const uint64_t share =
        S <= 16 ? share_fixed : share_bits(a.goff + 64ull * (uint64_t)w, s, S);
    if (KIND == kKindIC) {
        uint32_t tv = a.ic_t;
        if (a.ic_prob == kIcWeightedCascade) tv = wc_threshold(indeg);
        ic_row_word(a, G, S, valid, v, w, e0, e1, tv, s, lm, any);
    } else if (KIND == kKindEpidemic) {
        epi_row_word<L>(a, G, S, valid, v, w, e0, e1, s, share, tl, tl_n, tcode, lm, any);
    } else {
        lt_row_word<L>(a, G, S, valid, v, w, e0, e1, indeg, s, share, lm, any);
    }
}

// Words a wave works on at step t = a.step.  A word whose flag is clear
// after step t-1 cannot change at step t (no frontier, no infectious or
// latent replicate, or no activation under fixed thresholds).  If its flag
// after step t-2 is clear too, the state buffer step t writes already holds
// the word's state (state t-2 = t-1 = t) and the word is left out; otherwise
// it takes a pass with its candidates masked off, which copies it forward.
// `any` lists the words worked on, `live` those with candidates; with word
// flags, pass k gives lane gw the (k G + gw)-th word of `any`.
struct WordMap {
    uint64_t any, live;
    int passes, count;
    bool compact;
};

// All 64 lanes of the wave call this together.
__device__ __forceinline__ WordMap word_map(const StepArgs &a, int G)
{
    WordMap m;
    m.compact = a.wflags != nullptr;
    if (!m.compact) {
        m.any = m.live = ~0ull;
        m.count = a.W;
    } else {
        const uint32_t t = a.step, wr = (uint32_t)a.wring;
        const uint32_t *f1 = a.wflags + (size_t)((t - 1u) % wr) * (size_t)a.W;
        const uint32_t *f2 = a.wflags + (size_t)((t + wr - 2u) % wr) * (size_t)a.W;
        const int lane = (int)(threadIdx.x & 63u);
        uint32_t x1 = 0u, x2 = 0u;
        if (lane < a.W) {
            x1 = f1[lane];
            x2 = f2[lane];
        }
        m.live = __ballot(x1 != 0u);
        m.any = __ballot((x1 | x2) != 0u);
        m.count = __popcll(m.any);
    }
    m.passes = (m.count + G - 1) / G;
    return m;
}

// Position of the j-th (from 0) set bit of m; j < popcount(m).
__device__ __forceinline__ int nth_set_bit(uint64_t m, int j)
{
    int pos = 0;
    int c = __popc((uint32_t)m);
    if (j >= c) {
        j -= c;
        m >>= 32;
        pos = 32;
    }
    uint32_t x = (uint32_t)m;
    c = __popc(x & 0xFFFFu);
    if (j >= c) { j -= c; x >>= 16; pos += 16; }
    c = __popc(x & 0xFFu);
    if (j >= c) { j -= c; x >>= 8; pos += 8; }
    c = __popc(x & 0xFu);
    if (j >= c) { j -= c; x >>= 4; pos += 4; }
    c = __popc(x & 0x3u);
    if (j >= c) { j -= c; x >>= 2; pos += 2; }
    if (j >= (int)(x & 1u)) pos += 1;
    return pos;
}

// Word of lane gw in pass k, whether it exists, and its candidate mask.
__device__ __forceinline__ int word_of(const WordMap &m, int k, int G, int gw, bool &ok,
                                       uint64_t &lm)
{
    const int j = k * G + gw;
    ok = j < m.count;
    if (!m.compact) {
        lm = ~0ull;
        return ok ? j : 0;
    }
    const int w = ok ? nth_set_bit(m.any, j) : 0;
    lm = ((m.live >> w) & 1ull) ? ~0ull : 0ull;
    return w;
}

// Records the word flags of step a.step: lanes of one pass that share gw
// share the word, so the ballot is folded onto its low G bits and lane gw
// stores for its word.  All 64 lanes of the wave call this together.
__device__ __forceinline__ void note_words(const StepArgs &a, int G, int w, bool ok, bool anyw)
{
    if (a.wflags == nullptr) return;
    uint64_t m = __ballot(anyw);
    if (m == 0ull) return;
    for (int sh = 32; sh >= G; sh >>= 1) m |= m >> sh;
    const int lane = (int)(threadIdx.x & 63u);
    if (lane < G && ((m >> lane) & 1ull) && ok)
        a.wflags[(size_t)(a.step % (uint32_t)a.wring) * (size_t)a.W + (size_t)w] = 1u;
}

// Waves of a block that share one segment, and the words of LDS through
// which they merge it: the counts (IC: the fired replicates) of waves 1 .. 3,
// L planes of up to 64 words each.
constexpr int kSegWaves = 4;
template <int KIND, int L>
constexpr int seg_lds_words()
{
    return (kSegWaves - 1) * 64 * (KIND == kKindIC ? 1 : L);
}

// Lanes over the segments of a merged row, beside G over its words (at most
// 16, the widest split the draw-sharing masks cover).
__device__ __forceinline__ int merge_lanes(const StepArgs &a)
{
    const int lanes = 64 >> a.lgG;
    return lanes < 16 ? lanes : 16;
}

// Merge of the segment partials of heavy row j, then the same update as a
// light row: G lanes over words times S2 lanes over the row's segments, whose
// counts are summed across lanes in LC planes.  A wave has 64 / (G S2) such
// lane groups; j and `act` (whether the group has a row) are the group's.
template <int KIND, int LP, int LC>
__device__ __forceinline__ void combine_row(const StepArgs &a, int j, bool act, const WordMap &wm,
                                            const uint32_t *tl, int tl_n, const uint32_t *tcode,
                                            bool &any)
{
    const int lane = threadIdx.x & 63;
    const int G = a.G;
    const int S2 = merge_lanes(a);
    const int ss = (lane >> a.lgG) % S2;
    const int gw = lane & (G - 1);
    const int v = a.heavy_rows[j];
    const int sg0 = a.heavy_seg[j], sg1 = a.heavy_seg[j + 1];
    const uint64_t share = share_bits(a.goff, ss, S2);
    for (int k = 0; k < wm.passes; ++k) {
        bool ok;
        uint64_t lm;
        const int ww = word_of(wm, k, G, gw, ok, lm);
        const bool valid = act && ok;
        const int64_t idx = (int64_t)v * a.W + ww;
        bool anyw = false;
        if (KIND == kKindIC) {
            uint64_t acc = 0;
            if (valid && lm)
                for (int sg = sg0 + ss; sg < sg1; sg += S2) acc |= a.partial[(int64_t)sg * a.W + ww];
            acc = or_reduce_lanes(acc, G, S2);
            if (valid && ss == 0) {
                const uint64_t A = a.aux[idx];
                acc &= ~A;
                a.next[idx] = acc;
                a.aux[idx] = A | acc;
                anyw = acc != 0;
            }
            if (a.ibm != nullptr && anyw) mark_infected(a, v);  // tail mode
        } else {
            uint64_t c[LC];
#pragma unroll
            for (int l = 0; l < LC; ++l) c[l] = 0;
            if (valid && lm) {
                for (int sg = sg0 + ss; sg < sg1; sg += S2) {
                    uint64_t d[LC];
#pragma unroll
                    for (int l = 0; l < LC; ++l)
                        d[l] = (l < LP) ? a.partial[((int64_t)sg * LP + l) * a.W + ww] : 0ull;
                    bs_add<LC>(c, d);
                }
            }
            bs_reduce_lanes<LC>(c, G, S2);
            if (KIND == kKindEpidemic) {
                const uint64_t h = valid ? a.prev[idx] : 0ull;
                const uint64_t r = valid ? a.aux[idx] : 0ull;
                const uint64_t e = (valid && a.lat) ? a.lat[idx] : 0ull;
                const uint64_t sus = valid ? (~(h | r | e) & tail_mask(ww, a.B) & lm) : 0ull;
                const uint64_t counted = a.model == kSWIR ? (sus | (e & lm)) : sus;
#pragma unroll
                for (int l = 0; l < LC; ++l) c[l] &= counted;
                epi_decide<LC>(a, G, S2, valid, v, ww, idx, h, r, e, sus, c, ss, share, tl, tl_n,
                               tcode, anyw);
                if (a.ibm != nullptr && anyw) mark_infected(a, v);  // tail mode
            } else {
                const uint64_t act_w = valid ? a.prev[idx] : 0ull;
                const uint64_t inact = valid ? (~act_w & tail_mask(ww, a.B) & lm) : 0ull;
#pragma unroll
                for (int l = 0; l < LC; ++l) c[l] &= inact;
                const uint32_t indeg = (uint32_t)(a.ptr[v + 1] - a.ptr[v]);
                lt_decide<LC>(a, G, S2, valid, v, ww, idx, act_w, inact, indeg, c, ss, share, false,
                              anyw);
                if (a.ibm != nullptr && anyw) mark_infected(a, v);  // tail mode
            }
        }
        note_words(a, G, ww, ok, anyw);
        any |= anyw;
    }
}

__device__ __forceinline__ bool bit_of(const uint32_t *bm, int v)
{
    return ((bm[v >> 5] >> (v & 31)) & 1u) != 0u;
}

// Tail mode without the out-adjacency: whether node v or a source of its arcs
// e0 .. e1 that lane i of k tests has its bit in the bitmap of step t-1.
__device__ __forceinline__ bool tail_fresh(const StepArgs &a, int v, int e0, int e1, int i, int k)
{
    const uint32_t *inf1 = a.ibm + (size_t)((a.step - 1u) & 3u) * a.ibm_words;
    return bit_of(inf1, v) ||
           any_arcs((uint32_t)e0 + (uint32_t)i, (uint32_t)e1, (uint32_t)k,
                    [&](uint32_t p, uint32_t q, uint32_t r, uint32_t t) {
                        const int u0 = a.src[p], u1 = a.src[q], u2 = a.src[r], u3 = a.src[t];
                        bool f = bit_of(inf1, u0);
                        f |= bit_of(inf1, u1);
                        f |= bit_of(inf1, u2);
                        f |= bit_of(inf1, u3);
                        return f;
                    });
}

// Row i of the tile that begins at row t0, its first arc and their end.
__device__ __forceinline__ void tile_row(const StepArgs &a, int t0, int i, int &v, int &e0, int &e1)
{
    if (a.rows != nullptr) {
        const int2 r = a.rows[t0 + i];
        v = t0 + (r.y & 0xFFFF);
        e0 = r.x;
        e1 = e0 + (r.y >> 16);
    } else {
        v = t0 + i;
        e0 = a.ptr[v];
        e1 = a.ptr[v + 1];
    }
}

// Tail mode: the light rows of tile t0 .. t1 that can change at step t -- the
// candidates: themselves or an in-neighbour with an infected replicate (SI
// family) or a new activation (IC, LT) after step t-1 -- as their places in the
// tile in s_rows, in any order; returns their number to every thread of the block.
// With the out-adjacency the candidates are marked before the step; without
// it, eight lanes a row look at the row's sources, a bit a node (n / 8 bytes,
// which stay in the cache), instead of its words: a row with nothing new costs
// its arc list.  (LT, 2e5 nodes, 5 words: 97 us a step for every step.)
// A row left out keeps its state.  The buffer step t writes holds the state
// after t-2: for LT that is the same (no activation at t-1); for the SI family
// it differs only if the node had an infected replicate then (none after t-1),
// for IC (the buffer holds new activations) if it had a new activation then
// (none at t).
template <int KIND>
__device__ __forceinline__ int tail_rows(const StepArgs &a, int t0, int t1, uint16_t *s_rows)
{
    __shared__ int s_n;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const bool pull = a.cand == nullptr;
    const int lg = pull ? 3 : 0;
    const int sub = (int)threadIdx.x & ((1 << lg) - 1);
    const uint32_t *inf2 = a.ibm + (size_t)((a.step - 2u) & 3u) * a.ibm_words;
    const int per = (int)blockDim.x >> lg;
    for (int r0 = t0; r0 < t1; r0 += per) {
        const int i = r0 - t0 + ((int)threadIdx.x >> lg);
        bool in = t0 + i < t1, f = false;
        int v = 0, e0 = 0, e1 = 0;
        if (in) {
            tile_row(a, t0, i, v, e0, e1);
            in = e1 - e0 <= a.heavy;
            if (in)
                f = pull ? tail_fresh(a, v, e0, e1, sub, 8)
                         : bit_of(a.cand + (size_t)(a.step & 1u) * a.ibm_words, v);
        }
        if (pull) {
            const uint64_t m = __ballot(f);
            f = ((m >> (threadIdx.x & 56u)) & 0xFFull) != 0ull;
        }
        if (in && f && sub == 0) s_rows[atomicAdd(&s_n, 1)] = (uint16_t)i;
        if (KIND != kKindLT && in && !f && bit_of(inf2, v))
            for (int w = sub; w < a.W; w += 1 << lg) a.next[(int64_t)v * a.W + w] = 0ull;
    }
    __syncthreads();
    return s_n;
}

// Counter planes of the light rows of a job whose segments count in L planes
// (a light row has at most kBlockRow = 255 in-arcs, but see k_step_light).
constexpr int light_planes(int L) { return L < 8 ? L : 8; }

// One segment of a wide row v (more in-arcs than the light rows', see
// kBlockRow).  By a block (`by_block`): its first kSegWaves waves split the
// segment's arcs, G lanes over words and the other lanes of each wave over
// arcs, their results meet in LDS, and wave 0 either decides the row (a row of
// one segment) or writes the segment's partial result; of a row's segments the
// one that comes last merges them (combine_row).  A lane
// group would walk such a row alone for tens of microseconds while the rest of
// its tile waits; here a row of 4095 arcs of 16 words is 16 chunks of 16 arcs
// deep (SIR, 2e4 nodes, B = 1024: 37 to 25 us a step with these rows by block
// and no merge launch).  By a wave: the same with one wave, which costs a
// large graph less per row (no merge, no idle waves while wave 0 decides).
// Without WHOLE every segment is one of several (k_step_light).
template <int KIND, int L, bool TAIL, bool WHOLE>
__device__ __forceinline__ void segment_rows(const StepArgs &a, int seg, bool by_block,
                                             const WordMap &wm, const uint32_t *tl, int tl_n,
                                             const uint32_t *tcode, uint64_t *s_part, bool &any)
{
    const int lane = threadIdx.x & 63;
    const int wave = by_block ? (int)(threadIdx.x >> 6) : 0;  // of the segment's waves
    const int nw = by_block ? min((int)(blockDim.x >> 6), kSegWaves) : 1;
    const int v = a.seg_row[seg], e0 = a.seg_e0[seg], e1 = a.seg_e1[seg];
    const int indeg = a.ptr[v + 1] - a.ptr[v];
    const bool whole = WHOLE && e1 - e0 == indeg;
    // with fewer words left than word lanes, next_pow2(words) word lanes
    // and the rest over the segment's arcs (a shorter chain per lane)
    int lgG = a.lgG;
    if (wm.compact) {
        int lg = 0;
        while ((1 << lg) < wm.count) ++lg;
        lgG = lg > a.lgG ? a.lgG : lg;
    }
    const int G = 1 << lgG;
    const int S = 64 >> lgG;  // arc lanes of a wave
    const int ss = lane >> lgG;
    const int gw = lane & (G - 1);
    if (TAIL && a.ibm != nullptr && whole) {  // as a light row (tail_rows)
        bool cand;
        if (a.cand != nullptr) {
            cand = bit_of(a.cand + (size_t)(a.step & 1u) * a.ibm_words, v);
        } else {
            cand = tail_fresh(a, v, e0, e1, by_block ? (int)threadIdx.x : lane,
                              by_block ? (int)blockDim.x : 64);
            cand = by_block ? __syncthreads_or(cand) != 0 : __ballot(cand) != 0ull;
        }
        if (!cand) {
            if (KIND != kKindLT) {
                const uint32_t *inf2 = a.ibm + (size_t)((a.step - 2u) & 3u) * a.ibm_words;
                if (wave == 0 && bit_of(inf2, v))
                    for (int w = lane; w < a.W; w += 64) a.next[(int64_t)v * a.W + w] = 0ull;
            }
            return;
        }
    }
    // the lane group's arcs: a contiguous share in chunks of 16 where the
    // group is whole 16-lane rows, else every (nw S)-th arc
    const bool rows16 = G >= 16 && a.fast32;
    const int groups = nw * S, gi = wave * S + ss;
    int g0 = e0, g1 = e1, gs = gi, gS = groups;
    if (rows16) {
        const int per = ((e1 - e0 + groups - 1) / groups + 15) & ~15;
        g0 = min(e1, e0 + gi * per);
        g1 = min(e1, g0 + per);
        gs = 0;
        gS = 1;
    }
    const int passes = (wm.count + G - 1) / G;
    for (int k = 0; k < passes; ++k) {
        bool ok;
        uint64_t lm;
        const int w = word_of(wm, k, G, gw, ok, lm);
        const int64_t idx = (int64_t)v * a.W + w;
        const bool work = wave < nw;  // wave-uniform
        bool anyw = false;
        if (KIND == kKindIC) {
            const uint64_t A = ok ? a.aux[idx] : ~0ull;
            const uint64_t cand = ok ? (~A & tail_mask(w, a.B) & lm) : 0ull;
            const uint32_t tv = a.ic_prob == kIcWeightedCascade ? wc_threshold((uint32_t)indeg) : a.ic_t;
            uint64_t acc = 0;
            if (work) ic_arcs(a, G, gS, true, g0, g1, gs, w, cand, tv, acc);
            acc = or_reduce_lanes(acc, G, S);
            if (work && wave > 0 && ss == 0) s_part[(wave - 1) * 64 + gw] = acc;
            if (by_block) __syncthreads();
            if (wave == 0) {
                for (int q = 1; q < nw; ++q) acc |= s_part[(q - 1) * 64 + gw];
                if (ok && ss == 0) {
                    if (whole) {
                        a.next[idx] = acc;
                        a.aux[idx] = A | acc;
                        anyw = acc != 0ull;
                    } else {
                        a.partial[(int64_t)seg * a.W + w] = acc;
                    }
                }
            }
        } else {
            // state of the word, and the replicates whose count matters
            const uint64_t h = ok ? a.prev[idx] : 0ull;
            uint64_t r = 0, e = 0;
            if (KIND == kKindEpidemic) {
                r = ok ? a.aux[idx] : 0ull;
                e = (ok && a.lat) ? a.lat[idx] : 0ull;
            }
            const uint64_t sus = ok ? (~(h | r | e) & tail_mask(w, a.B) & lm) : 0ull;
            const uint64_t counted =
                KIND == kKindEpidemic && a.model == kSWIR ? (sus | (e & lm)) : sus;
            uint64_t c[L];
#pragma unroll
            for (int l = 0; l < L; ++l) c[l] = 0;
            if (work) {
                if (rows16)
                    count_edges_bcast<L>(a, G, true, g0, g1, w, counted != 0ull, c);
                else if (counted)
                    count_edges<L>(a, g0 + gs, g1, gS, w, c);
            }
            bs_reduce_lanes<L>(c, G, S);
            if (work && wave > 0 && ss == 0) {
#pragma unroll
                for (int l = 0; l < L; ++l) s_part[((wave - 1) * L + l) * 64 + gw] = c[l];
            }
            if (by_block) __syncthreads();
            if (wave == 0) {
                for (int q = 1; q < nw; ++q) {
                    uint64_t d[L];
#pragma unroll
                    for (int l = 0; l < L; ++l) d[l] = s_part[((q - 1) * L + l) * 64 + gw];
                    bs_add<L>(c, d);
                }
                if (!whole) {
                    if (ok && ss == 0) {
#pragma unroll
                        for (int l = 0; l < L; ++l) a.partial[((int64_t)seg * L + l) * a.W + w] = c[l];
                    }
                } else {
                    const uint64_t share = share_bits(a.goff + 64ull * (uint64_t)w, ss, S);
                    if (KIND == kKindEpidemic)
                        epi_decide<L>(a, G, S, ok, v, w, idx, h, r, e, sus, c, ss, share, tl, tl_n,
                                      tcode, anyw);
                    else
                        lt_decide<L>(a, G, S, ok, v, w, idx, h, sus, (uint32_t)indeg, c, ss, share,
                                     true, anyw);
                }
            }
        }
        if (wave == 0 && whole) {
            note_words(a, G, w, ok, anyw);
            if (TAIL && anyw && a.ibm != nullptr) mark_infected(a, v);
            any |= anyw;
        }
        if (by_block && k + 1 < passes) __syncthreads();  // s_part is written again
    }
    if (whole || wave != 0) return;
    if (!WHOLE || a.heavy_done == nullptr) return;  // merged by a launch of its own
    // The partial is out before the row's counter rises, and whoever sees the
    // count full sees every partial.
    __threadfence();
    const int j = a.seg_heavy[seg];
    bool last = false;
    if (lane == 0)
        last = atomicAdd(&a.heavy_done[j], 1u) + 1u == (uint32_t)(a.heavy_seg[j + 1] - a.heavy_seg[j]);
    if (__ballot(last) == 0ull) return;
    __threadfence();
    if (lane == 0) a.heavy_done[j] = 0u;  // for the next step
    combine_row<KIND, L, KIND == kKindIC ? 1 : kMergePlanes>(a, j, lane < a.G * merge_lanes(a), wm, tl, tl_n,
                                                             tcode, any);
}

// Work of one block of the pull step: the first blocks own segments of wide
// rows (long, so they start first), the rest light tiles.
// Returns through `any` whether a state-1 node remains.  Light rows count in
// LL planes, segments in L.
template <int KIND, int LL, int L, bool TAIL = false>
__device__ __forceinline__ void step_block(const StepArgs &a, int bid, const uint32_t *tl,
                                           int tl_n, const uint32_t *tcode, uint64_t *s_part,
                                           uint16_t *s_rows, bool &any)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int nwaves = blockDim.x >> 6;
    const int S = a.S;
    const WordMap wm = word_map(a, a.G);
    const int seg_blocks = seg_blocks_of(a.n_seg, a.n_segb, nwaves);
    if (bid < seg_blocks) {
        const bool by_block = bid < a.n_segb;
        const int seg = by_block ? bid : a.n_segb + (bid - a.n_segb) * nwaves + wave;
        if (seg < a.n_seg)  // block-uniform where the block meets at barriers
            segment_rows<KIND, L, TAIL, LL == light_planes(L)>(a, seg, by_block, wm, tl, tl_n, tcode, s_part, any);
        return;
    }
    // light rows: once fewer words are left than the row has word lanes,
    // the row gets next_pow2(words) lanes (not below 16, which keeps the
    // DPP source broadcast) and the wave takes more rows
    int lgGe = a.lgG;
    if (wm.compact) {
        int lg = 0;
        while ((1 << lg) < wm.count) ++lg;
        const int lo = a.lgG < 4 ? a.lgG : 4;
        lgGe = lg < lo ? lo : (lg > a.lgG ? a.lgG : lg);
    }
    const int Ge = 1 << lgGe;
    const int rpwe = 64 >> (lgGe + a.lgS);
    const int slote = lane >> (lgGe + a.lgS);
    const int se = (lane >> lgGe) & (S - 1);
    const int gwe = lane & (Ge - 1);
    const uint64_t share_e = S <= 16 ? share_bits(a.goff, se, S) : 0ull;
    const int passes = (wm.count + Ge - 1) / Ge;
    const int tile = bid - seg_blocks;
    const int t0 = a.tiles[2 * tile], t1 = a.tiles[2 * tile + 1];
    // LT once at most half of the words are left: thresholds are fixed,
    // so a row none of whose in-neighbours gained an activation at step
    // t-1 has the counts it was last decided on and cannot activate; it
    // takes the copy pass without counting (earlier, nearly every row
    // has such a neighbour and the test would only add loads)
    constexpr bool kTailKind = TAIL;
    const bool fresh_test = KIND == kKindLT && a.stamp != nullptr && wm.compact &&
                            wm.count * 2 <= a.W && !(kTailKind && a.ibm != nullptr);
    const int rl = 1 << (lgGe + a.lgS);  // lanes of a row
    const uint64_t rowmask = (rl == 64 ? ~0ull : ((1ull << rl) - 1ull)) << (slote * rl);
    // tail mode: only the rows that can change
    const bool tail = kTailKind && a.ibm != nullptr;
    const int nrows = tail ? tail_rows<KIND>(a, t0, t1, s_rows) : t1 - t0;
    for (int rb = wave * rpwe; rb < nrows; rb += nwaves * rpwe) {
        bool act = rb + slote < nrows;
        int v = t0, e0 = 0, e1 = 0;
        if (act) {
            tile_row(a, t0, tail ? (int)s_rows[rb + slote] : rb + slote, v, e0, e1);
            if (e1 - e0 > a.heavy) act = false;
        }
        uint64_t rowlm = ~0ull;
        if (fresh_test) {
            const uint32_t *gained = a.stamp + (size_t)((a.step - 1u) & 1u) * (size_t)a.n;
            bool f = false;
            if (act)
                for (int e = e0 + (lane & (rl - 1)); e < e1 && !f; e += rl)
                    f = gained[a.src[e]] == a.step - 1u;
            if ((__ballot(f) & rowmask) == 0ull) rowlm = 0ull;
        }
        for (int k = 0; k < passes; ++k) {
            bool ok;
            uint64_t lm;
            const int w = word_of(wm, k, Ge, gwe, ok, lm);
            bool anyw = false;
            row_word<KIND, LL>(a, Ge, S, act && ok, v, w, e0, e1, (uint32_t)(e1 - e0), se,
                              share_e, tl, tl_n, tcode, lm & rowlm, anyw);
            note_words(a, Ge, w, ok, anyw);
            // anyw: an infected replicate (SI family) or a new activation
            // (IC, LT) in this word after the step
            if (kTailKind && anyw && a.ibm != nullptr) mark_infected(a, v);
            any |= anyw;
        }
    }
}

// Tail mode: whether light-row block `bid` has nothing to do at step t -- no
// candidate row and no row infected (IC: newly activated) after t-2, whose
// buffer word must be cleared, in its tile.  The bitmap words at the tile's
// ends may hold other tiles' rows, which only makes the test keep a tile it
// could have left.
// Every wave of the block reads the same words and gets the same answer.
__device__ __forceinline__ bool tail_tile_idle(const StepArgs &a, int bid, bool zero_store)
{
    const int seg_blocks = seg_blocks_of(a.n_seg, a.n_segb, blockDim.x >> 6);
    if (bid < seg_blocks || a.cand == nullptr) return false;
    const int tile = bid - seg_blocks;
    const int t0 = a.tiles[2 * tile], t1 = a.tiles[2 * tile + 1];
    if (t1 <= t0) return true;
    const uint32_t *cand = a.cand + (size_t)(a.step & 1u) * a.ibm_words;
    const uint32_t *inf2 = a.ibm + (size_t)((a.step - 2u) & 3u) * a.ibm_words;
    bool busy = false;
    for (int i = (t0 >> 5) + (int)(threadIdx.x & 63); i <= ((t1 - 1) >> 5) && !busy; i += 64)
        busy = (cand[i] | (zero_store ? inf2[i] : 0u)) != 0u;
    return __ballot(busy) == 0ull;
}

// One synchronous step t = a.step of one job.
template <int KIND, int LL, int L, bool TAIL>
__device__ __forceinline__ void run_step(const StepArgs &a)
{
    if (a.flags[(a.step - 1) % (uint32_t)a.ring] == 0u) return;  // nothing left to change
    if (TAIL && a.ibm != nullptr) {
        // the bitmaps step t+1 sets, then whether this block has work
        uint32_t *clr = a.ibm + (size_t)((a.step + 1u) & 3u) * a.ibm_words;
        uint32_t *cclr = a.cand + (size_t)((a.step + 1u) & 1u) * a.ibm_words;
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.ibm_words;
             i += (int64_t)gridDim.x * blockDim.x) {
            clr[i] = 0u;
            if (a.cand != nullptr) cclr[i] = 0u;
        }
        if (tail_tile_idle(a, a.first + (int)blockIdx.x, KIND != kKindLT)) return;
    }
    __shared__ uint32_t s_tinf[KIND == kKindEpidemic ? kTinfLds : 1];
    __shared__ uint32_t s_code[kCodeTable];
    __shared__ uint64_t s_part[seg_lds_words<KIND, L>()];
    __shared__ uint16_t s_rows[TAIL ? kMaxTileRows : 1];
    int tl_n = 0;
    if (KIND == kKindEpidemic) {
        tl_n = a.khat + 1 < kTinfLds ? a.khat + 1 : kTinfLds;
        for (int i = threadIdx.x; i < tl_n; i += blockDim.x) s_tinf[i] = a.tinf[i];
        stage_codes(a, s_code);
        __syncthreads();
    }
    bool any = false;
    step_block<KIND, LL, L, TAIL>(a, a.first + (int)blockIdx.x, s_tinf, tl_n, s_code, s_part, s_rows, any);
    if (__ballot(any) != 0ull && (threadIdx.x & 63) == 0) a.flags[a.step % (uint32_t)a.ring] = 1u;
}

template <int KIND, int L, bool TAIL = false>
__global__ void __launch_bounds__(1024) k_step(StepArgs a)
{
    run_step<KIND, light_planes(L), L, TAIL>(a);
}

// The step of a graph whose rows of up to kLightMost in-arcs are light (see
// light_rows): they count in kLightPlanes planes, and longer ones are always
// cut, their segments merged by a launch of its own, so no wide row is decided
// here.  LT needs 161 registers for its planes: compiled for blocks of 256
// threads it keeps them, at three waves a SIMD instead of four with 92 bytes a
// lane in scratch, which is better for rows of one word (8000 rows of 600 arcs,
// 64 replicates, 30 steps: 0.90 ms, else 1.09) and worse for wider ones (8000
// of 400, 128 replicates: 1.07 and 1.03; 32,000 of 600, 300 replicates: 8.38
// and 7.00).
template <int KIND, bool TAIL, int THREADS = 1024>
__global__ void __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(THREADS == 256 ? 3 : 1)))
k_step_light(StepArgs a)
{
    run_step<KIND, kLightPlanes, kLightPlanes, TAIL>(a);
}

// The rows of every tile by decreasing in-degree (a block per tile, by
// counting; rows of the same degree in any order): the rows that share a wave
// then end together, where each wave took as long as its longest row.  Four
// rows a wave: IC, 3e5 nodes, 1000 replicates, 14.3 -> 12.9 ms; SIR, 1e6
// nodes, 1024 replicates, 87.0 -> 84.8.  Eight: LT, 2e5 nodes, 300 replicates,
// 14.2 -> 14.0 (rows of neighbouring numbers are of like degree there).
__global__ void __launch_bounds__(256) k_tile_rows(const int32_t *ptr, const int32_t *tiles, int2 *rows)
{
    __shared__ int s_at[256];
    const int t0 = tiles[2 * blockIdx.x], t1 = tiles[2 * blockIdx.x + 1];
    const int tid = (int)threadIdx.x;
    s_at[tid] = 0;
    __syncthreads();
    for (int v = t0 + tid; v < t1; v += 256) atomicAdd(&s_at[255 - min(ptr[v + 1] - ptr[v], 255)], 1);
    __syncthreads();
    const int own = s_at[tid];
    for (int k = 1; k < 256; k <<= 1) {  // inclusive sums
        const int x = tid >= k ? s_at[tid - k] : 0;
        __syncthreads();
        s_at[tid] += x;
        __syncthreads();
    }
    const int before = s_at[tid] - own;
    __syncthreads();
    s_at[tid] = before;
    __syncthreads();
    for (int v = t0 + tid; v < t1; v += 256) {
        const int e0 = ptr[v], d = ptr[v + 1] - e0;
        rows[t0 + atomicAdd(&s_at[255 - min(d, 255)], 1)] = make_int2(e0, d << 16 | (v - t0));
    }
}

// Heavy row of this lane's group in the merge launch; false where its wave has
// none at all.
__device__ __forceinline__ bool merge_group(const StepArgs &a, uint32_t block, int &j, bool &act)
{
    const int size = a.G * merge_lanes(a), per = 64 / size;  // lanes of a group, groups a wave
    const int first = ((int)block * (int)(blockDim.x >> 6) + (int)(threadIdx.x >> 6)) * per;
    j = first + (int)(threadIdx.x & 63) / size;
    act = j < a.n_heavy;
    j = act ? j : a.n_heavy - 1;
    return first < a.n_heavy;
}

// The merge of the heavy rows in a launch of its own, a lane group per row:
// where there are many segments (kMergeSegs), with k_step_light, and for graphs
// with a row of more than kMergeRow in-arcs, whose count the step kernel's
// merge has no planes for.
template <int KIND, int LP>
__global__ void __launch_bounds__(256) k_combine(StepArgs a)
{
    if (a.flags[(a.step - 1) % (uint32_t)a.ring] == 0u) return;
    __shared__ uint32_t s_code[kCodeTable];
    if (KIND == kKindEpidemic) {
        stage_codes(a, s_code);
        __syncthreads();
    }
    int j;
    bool act;
    if (!merge_group(a, blockIdx.x, j, act)) return;
    bool any = false;
    combine_row<KIND, LP, KIND == kKindIC ? 1 : 32>(a, j, act, word_map(a, a.G), nullptr, 0, s_code, any);
    if (__ballot(any) != 0ull && (threadIdx.x & 63) == 0) a.flags[a.step % (uint32_t)a.ring] = 1u;
}

// ------------------------------------------- IC, one word per node ----
// Edge-parallel variant for B <= 64 (W = 1): persistent blocks stream the
// arcs' source groups once per step, four 16-byte loads per thread per pass,
// and test each arc against the frontier: first the summary (one bit per
// group of nodes, in LDS), then, for summary hits, the source and
// its bit of the frontier bitmap (N bits, cache-resident).  Only a frontier arc reads its target row (the
// arc's entry of dst), gathers the source word, runs the arc's trials and ORs
// fired replicates into the target's words with atomics; the target joins the
// next frontier.  The step has no tiles and no block barriers, and it reads
// neither the row pointers (except a frontier arc's target degree under the
// weighted cascade) nor the words of rows that do not change.
__device__ __forceinline__ uint32_t ic_threshold(const StepArgs &a, uint32_t indeg)
{
    return a.ic_prob == kIcWeightedCascade ? wc_threshold(indeg) : a.ic_t;
}

__device__ __forceinline__ void mark_frontier(const StepArgs &a, int v)
{
    atomicOr(&a.bm_next[v >> 5], 1u << (v & 31));
    const uint32_t i = node_group((uint32_t)v);
    atomicOr(&a.sum_next[i >> 5], 1u << (i & 31));
}

// Work item k of node v whose out-arcs are oarc[o0 .. o1): (v, k, first arc,
// end of its arcs).
__device__ __forceinline__ uint4 out_item(int v, uint32_t k, int o0, int o1)
{
    const int b = o0 + (int)k * kOutChunk;
    const int e = o1 - b < kOutChunk ? o1 : b + kOutChunk;
    return make_uint4((uint32_t)v, k, (uint32_t)b, (uint32_t)e);
}

// Joins node v to the frontier of step t (its bit in the next bitmap; the
// first thread to set the bit also sets the summary bit and, with a queue,
// appends v's work items and adds its out-degree to the queue's arc count).
template <bool Q>
__device__ __forceinline__ void join_frontier(const StepArgs &a, int v)
{
    if (!Q) {
        mark_frontier(a, v);
        return;
    }
    const uint32_t bit = 1u << (v & 31);
    const uint32_t old = atomicOr(&a.bm_next[v >> 5], bit);
    if (old & bit) return;
    const uint32_t i = node_group((uint32_t)v);
    atomicOr(&a.sum_next[i >> 5], 1u << (i & 31));
    if (a.ever) atomicOr(&a.ever[v >> 5], bit);
    const int o0 = a.optr[v], o1 = a.optr[v + 1];
    const int deg = o1 - o0;
    const uint32_t nch = deg > kOutChunk ? (uint32_t)((deg + kOutChunk - 1) / kOutChunk) : 1u;
    const uint32_t at = atomicAdd(&a.qcnt[a.qi_out], nch);
    for (uint32_t k = 0; k < nch; ++k) a.q_out[at + k] = out_item(v, k, o0, o1);
    if (deg > 0) atomicAdd(&a.qarcs[a.qi_out], (unsigned long long)deg);
}

// Claims node v for the frontier of step t: sets its bit in the next bitmap
// and returns true for the one thread that set it first (which then sets
// the summary bit and must queue v).
__device__ __forceinline__ bool claim_frontier(const StepArgs &a, int v)
{
    const uint32_t bit = 1u << (v & 31);
    const uint32_t old = atomicOr(&a.bm_next[v >> 5], bit);
    if (old & bit) return false;
    const uint32_t i = node_group((uint32_t)v);
    atomicOr(&a.sum_next[i >> 5], 1u << (i & 31));
    if (a.ever) atomicOr(&a.ever[v >> 5], bit);
    return true;
}

// Queues the nodes the lanes of a wave claimed (v < 0: none), called by all
// 64 lanes together: one atomic add per wave reserves the items of all of
// them (a shuffle scan gives each lane its offset) and one adds their
// out-arcs; a node with more than 64 items has them written by the whole
// wave.
__device__ __forceinline__ void queue_claimed(const StepArgs &a, int v, int o0, int o1)
{
    const int lane = threadIdx.x & 63;
    const int deg = v >= 0 ? o1 - o0 : 0;
    const uint32_t nch = v < 0 ? 0u : (deg > kOutChunk ? (uint32_t)((deg + kOutChunk - 1) / kOutChunk) : 1u);
    if (__ballot(nch != 0u) == 0ull) return;
    uint32_t incl = nch;
    unsigned long long arcs = (unsigned long long)deg;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t x = (uint32_t)__shfl_up((int)incl, off, 64);
        if (lane >= off) incl += x;
        arcs += __shfl_xor(arcs, off, 64);
    }
    uint32_t base = 0;
    if (lane == 63) {
        base = atomicAdd(&a.qcnt[a.qi_out], incl);
        if (arcs) atomicAdd(&a.qarcs[a.qi_out], arcs);
    }
    base = (uint32_t)__shfl((int)base, 63, 64);
    const uint32_t at = base + incl - nch;
    if (nch <= 64u) {
        for (uint32_t k = 0; k < nch; ++k) a.q_out[at + k] = out_item(v, k, o0, o1);
    }
    uint64_t big = __ballot(nch > 64u);
    while (big) {
        const int l = __builtin_ctzll(big);
        big &= big - 1;
        const int bv = __shfl(v, l, 64), b0 = __shfl(o0, l, 64), b1 = __shfl(o1, l, 64);
        const uint32_t bat = (uint32_t)__shfl((int)at, l, 64), bn = (uint32_t)__shfl((int)nch, l, 64);
        for (uint32_t k = (uint32_t)lane; k < bn; k += 64) a.q_out[bat + k] = out_item(bv, k, b0, b1);
    }
}

// A frontier arc e = (u -> v): its trials, the replicates that fired into v's
// words, v into the next frontier.
template <bool Q>
__device__ __forceinline__ void ic_arc_hit(const StepArgs &a, int64_t e, int u, bool &any)
{
    const int v = a.dst[e];
    const uint32_t tv = a.edge_t ? 0u : ic_threshold(a, (uint32_t)(a.ptr[v + 1] - a.ptr[v]));
    const uint64_t cand_r = ~a.aux[v] & tail_mask(0, a.B);
    uint64_t acc = 0;
    ic_edge(a, (int)e, a.prev[u] & cand_r, a.goff, tv, acc);
    if (acc) {
        atomicOr((unsigned long long *)&a.next[v], (unsigned long long)acc);
        atomicOr((unsigned long long *)&a.aux[v], (unsigned long long)acc);
        join_frontier<Q>(a, v);
        any = true;
    }
}

// What a wave of the streaming step has found but not worked on yet, in LDS:
// candidates (arcs whose source's group holds a frontier node) and hits
// (candidates whose source is one), at most 127 of each.
struct StreamQueue {
    uint32_t cand[128];
    uint2 hit[128];  // arc, source
};

// The wave's LDS writes before this are read by its other lanes after it (a
// wave's LDS accesses execute in order).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One streaming step.  What is streamed is not the sources but their groups
// (node_group, 16 bits an arc, written when the graph is bound): the summary
// needs no more, and the stream bounds the step while the frontier is small
// (R-MAT scale 24, 2.7e8 arcs: 203 us a step with 4-byte sources, 97 with
// groups, 5.5 TB/s; scale 26, 1.1e9: 481 us, 4.5 TB/s).  A thread has 32 arcs in flight.  Candidates and hits are
// rare and scattered over the lanes, and each is a chain of dependent loads, so
// a wave collects them and works on 64 at a time: with each lane following its
// own the chain was waited for once per hit (the peak step of that run: 245 us,
// 223 collected; what is left there is the hits' own loads and atomics, and
// sources kept as their upper 8 bits beside the group took it only to 208).
template <bool Q>
__device__ __forceinline__ void ic_stream_pass(const StepArgs &a, const uint32_t *s_sum,
                                               StreamQueue *queues, bool &any)
{
    const int lane = threadIdx.x & 63;
    StreamQueue &q = queues[threadIdx.x >> 6];
    int nc = 0, nh = 0;  // entries of q.cand, q.hit (wave-uniform)
    const uint64_t below = (1ull << lane) - 1ull;
    // the last min(64, nh) hits
    auto work = [&]() {
        wave_lds_sync();
        const int k = nh < 64 ? nh : 64;
        if (lane < k) {
            const uint2 h = q.hit[nh - k + lane];
            ic_arc_hit<Q>(a, (int64_t)h.x, (int)h.y, any);
        }
        nh -= k;
        wave_lds_sync();
    };
    // the last min(64, nc) candidates
    auto test = [&]() {
        wave_lds_sync();
        const int k = nc < 64 ? nc : 64;
        bool hit = false;
        uint32_t e = 0, u = 0;
        if (lane < k) {
            e = q.cand[nc - k + lane];
            u = (uint32_t)a.src[e];
            hit = (a.bm_prev[u >> 5] >> (u & 31u)) & 1u;
        }
        nc -= k;
        const uint64_t m = __ballot(hit);
        if (hit) q.hit[nh + __popcll(m & below)] = make_uint2(e, u);
        nh += __popcll(m);
        if (nh >= 64) work();
        wave_lds_sync();
    };
    const int64_t nnz = a.nnz;
    // pass: chunk c of thread t covers arcs base + c*stride .. +7; the loop is
    // the wave's (wb: its first lane's base)
    const int64_t stride = (int64_t)gridDim.x * blockDim.x * 8;
    constexpr int kChunks = 4;
    for (int64_t wb = ((int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63u)) * 8; wb < nnz;
         wb += stride * kChunks) {
        const int64_t base = wb + 8 * lane;
        uint4 g[kChunks];
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const int64_t eb = base + c * stride;
            g[c] = make_uint4(0u, 0u, 0u, 0u);
            if (eb < nnz) g[c] = *reinterpret_cast<const uint4 *>(a.grp + eb);  // groups padded by 16 B
        }
        uint32_t cand = 0;
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const uint32_t w[4] = {g[c].x, g[c].y, g[c].z, g[c].w};
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t id = (j & 1) ? w[j >> 1] >> 16 : w[j >> 1] & 0xFFFFu;
                cand |= ((s_sum[id >> 5] >> (id & 31u)) & 1u) << (8 * c + j);
            }
        }
        if (__ballot(cand != 0u) == 0ull) continue;
        // arcs past the end of the array
#pragma unroll
        for (int c = 0; c < kChunks; ++c) {
            const int64_t left = nnz - (base + c * stride);
            const uint32_t keep = left >= 8 ? 0xFFu : (left > 0 ? (1u << left) - 1u : 0u);
            cand &= ~(0xFFu << (8 * c)) | (keep << (8 * c));
        }
        for (;;) {  // a candidate of each lane at a time
            const uint64_t m = __ballot(cand != 0u);
            if (m == 0ull) break;
            if (cand != 0u) {
                const int b = __builtin_ctz(cand);
                cand &= cand - 1u;
                q.cand[nc + __popcll(m & below)] = (uint32_t)(base + (b >> 3) * stride + (b & 7));
            }
            nc += __popcll(m);
            if (nc >= 64) test();
        }
    }
    while (nc > 0) test();
    while (nh > 0) work();
}

__global__ void __launch_bounds__(1024) k_ic_stream(StepArgs a)
{
    if (a.flags[(a.step - 1) % (uint32_t)a.ring] == 0u) return;
    __shared__ uint32_t s_sum[kSumWords];
    __shared__ StreamQueue s_queue[16];
    for (int i = threadIdx.x; i < a.sum_words; i += blockDim.x) s_sum[i] = a.sum_prev[i];
    __syncthreads();
    bool any = false;
    ic_stream_pass<false>(a, s_sum, s_queue, any);
    if (__ballot(any) != 0ull && (threadIdx.x & 63) == 0) a.flags[a.step % (uint32_t)a.ring] = 1u;
}

// Push over the out-arcs of the frontier of t-1: one wave per work item
// (a chunk of at most kOutChunk out-arcs of a frontier node u), lanes over
// the chunk's arcs.  An arc u -> v with edge id e runs the same trials the
// pull step would (keyed by e, threshold of v), for the replicates where u
// is newly active and v is not yet active.
__device__ __forceinline__ void ic_push_pass(const StepArgs &a, bool &any)
{
    const uint64_t tail = tail_mask(0, a.B);
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int64_t nitems = a.qcnt[a.qi_in];
    const bool wc = a.ic_prob == kIcWeightedCascade && !a.edge_t;
    for (int64_t i = wave; i < nitems; i += nwave) {
        // an item carries its arc range, so the chain of dependent loads
        // is: item; arc and source word; target's active word, in-degree
        // and out-arc range; then the trials and the atomics
        const uint4 it = a.q_in[i];
        const int u = (int)it.x;
        const int j = (int)it.z + lane;
        const bool has = j < (int)it.w;
        const uint64_t fu = a.prev[u] & tail;
        const int2 ve = has ? a.oarc[j] : make_int2(0, 0);
        const int v = ve.x;
        uint64_t av = ~0ull;
        int p0 = 0, p1 = 0, o0 = 0, o1 = 0;
        if (has) {
            av = a.aux[v];
            if (wc) {
                p0 = a.ptr[v];
                p1 = a.ptr[v + 1];
            }
        }
        const uint64_t cand = fu & ~av;
        int claimed = -1;
        if (cand) {
            const uint32_t tv = a.edge_t ? 0u : (wc ? wc_threshold((uint32_t)(p1 - p0)) : a.ic_t);
            uint64_t acc = 0;
            ic_edge(a, ve.y, cand, a.goff, tv, acc);
            if (acc) {
                atomicOr((unsigned long long *)&a.next[v], (unsigned long long)acc);
                atomicOr((unsigned long long *)&a.aux[v], (unsigned long long)acc);
                if (claim_frontier(a, v)) {
                    claimed = v;
                    o0 = a.optr[v];
                    o1 = a.optr[v + 1];
                }
                any = true;
            }
        }
        queue_claimed(a, claimed, o0, o1);
    }
}

// The nodes of the queue a.qi_clr leave their frontier plane and bitmap, and
// the summary is cleared; thread `r` of `nthr`.
__device__ __forceinline__ void ic_clear_pass(const StepArgs &a, int64_t r, int64_t nthr)
{
    const int64_t nclr = a.qcnt[a.qi_clr];
    for (int64_t i = r; i < nclr; i += nthr) {
        const uint4 it = a.q_clr[i];
        if (it.y == 0u) {
            a.f_clr[it.x] = 0ull;
            a.bm_clr[it.x >> 5] = 0u;  // every set bit of this bitmap is such a node
        }
    }
    for (int64_t i = r; i < a.sum_words; i += nthr) a.sum_clr[i] = 0u;
}

// One step of the frontier-driven IC path (see StepArgs): first the nodes of
// the frontier of t-2 leave their plane, bitmap and summary (buffers step t
// does not touch) and the counters of the queue of t+1 are reset; then the
// frontier of t-1 is pushed over its out-arcs when it has at most
// push_limit of them, else the step streams every source.  The choice
// depends only on counts from step t-1, so every block makes the same one.
__global__ void __launch_bounds__(512) k_ic_front(StepArgs a)
{
    if (a.flags[(a.step - 1) % (uint32_t)a.ring] == 0u) return;
    __shared__ uint32_t s_sum[kSumWords];
    __shared__ StreamQueue s_queue[8];
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nthr = (int64_t)gridDim.x * blockDim.x;
    // when pushing, the clearing takes the threads after the push items'
    // waves (still in the first blocks dispatched), so no thread's chain of
    // loads holds both
    const bool push = a.qarcs[a.qi_in] <= a.push_limit;
    // (modulo the launch: a queue of more items than the launch has waves
    // wraps around)
    const int64_t skip = push ? (int64_t)a.qcnt[a.qi_in] * 64 % nthr : 0;
    const int64_t rtid = tid >= skip ? tid - skip : tid - skip + nthr;
    ic_clear_pass(a, rtid, nthr);
    if (tid == 0) {
        a.qcnt[a.qi_rst] = 0u;
        a.qarcs[a.qi_rst] = 0ull;
    }
    bool any = false;
    if (push) {
        ic_push_pass(a, any);
    } else {
        for (int i = threadIdx.x; i < a.sum_words; i += blockDim.x) s_sum[i] = a.sum_prev[i];
        __syncthreads();
        ic_stream_pass<true>(a, s_sum, s_queue, any);
    }
    if (__ballot(any) != 0ull && (threadIdx.x & 63) == 0) a.flags[a.step % (uint32_t)a.ring] = 1u;
}

// A finalize queued before the host knew the run had ended: the first step
// of t0+1 .. t0+c whose absorption flag is clear (the run's last step), or
// -1 (the run goes on; nothing to do).  A load and a ballot per 64 steps;
// every lane of the wave gets the same answer.
__device__ __forceinline__ int64_t spec_last_step(const SpecFin &s)
{
    const int lane = (int)(threadIdx.x & 63u);
    for (int b = 0; b < s.c; b += 64) {
        const int i = b + lane;
        const bool clear =
            i < s.c && s.flags[(uint32_t)(s.t0 + 1 + i) % (uint32_t)s.ring] == 0u;
        const uint64_t m = __ballot(clear);
        if (m) return s.t0 + 1 + b + __builtin_ctzll(m);
    }
    return -1;
}

// Entry i of a 3- or 4-entry pointer array held in kernel arguments, with
// constant indices only (a run-time index would copy the arguments to
// per-lane scratch).
template <typename P>
__device__ __forceinline__ P pick3(const P (&a)[3], int i)
{
    return i == 0 ? a[0] : (i == 1 ? a[1] : a[2]);
}
template <typename P>
__device__ __forceinline__ P pick4(const P (&a)[4], int i)
{
    return i == 0 ? a[0] : (i == 1 ? a[1] : (i == 2 ? a[2] : a[3]));
}

// The planes of a speculative finalize: the frontier of the run's last step
// (empty, since that step activated nothing), or false when the run has not
// ended.
__device__ __forceinline__ bool spec_planes(FinArgs &f)
{
    if (f.spec.flags == nullptr) return true;
    const int64_t T = spec_last_step(f.spec);
    if (T < 0) return false;
    const int m = (int)(T % 3);
    f.one = pick3(f.spec.front3, m);
    f.bm = pick3(f.spec.bm3, m);
    return true;
}

// End of a frontier-driven run: the last two frontiers, which no later step
// clears, leave their buffers (one launch per frontier).
__global__ void __launch_bounds__(256) k_ic_scrub(StepArgs a)
{
    ic_clear_pass(a, (int64_t)blockIdx.x * blockDim.x + threadIdx.x,
                  (int64_t)gridDim.x * blockDim.x);
}

// The same, queued before the host knew the run had ended (SpecFin): the
// frontier of step T - 2 + which, T the run's last step; after the second
// one the tag records that the run left its buffers clear.
__global__ void __launch_bounds__(256) k_ic_scrub_spec(StepArgs a, SpecFin sp, int which,
                                                      uint64_t *tag, uint64_t tag_value)
{
    const int64_t T = spec_last_step(sp);
    if (T < 0) return;
    const int64_t t = T + which;  // the step whose clear duty this is
    const int m = (int)((t - 2) % 3);
    a.qi_clr = (int32_t)((t + 2) % 4);
    a.q_clr = pick4(sp.queue4, a.qi_clr);
    a.f_clr = pick3(sp.front3, m);
    a.bm_clr = pick3(sp.bm3, m);
    a.sum_clr = pick3(sp.sum3, m);
    ic_clear_pass(a, (int64_t)blockIdx.x * blockDim.x + threadIdx.x,
                  (int64_t)gridDim.x * blockDim.x);
    if (tag != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *tag = tag_value;
}

// Seeds of a frontier-driven run: joined to the frontier of step 0 (bitmap,
// summary, queue 0) once each, duplicates included.
__global__ void k_seed_queue(StepArgs a, const int32_t *seeds, int64_t ns)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ns;
         i += (int64_t)gridDim.x * blockDim.x)
        join_frontier<true>(a, seeds[i]);
}

// Out-adjacency of a bound graph: out-degrees, then every arc placed in its
// source's range (any order inside a range: the steps that read it combine
// with OR).
__global__ void k_out_count(const int32_t *src, int64_t nnz, int32_t *cnt)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&cnt[src[e]], 1);
}

__global__ void k_out_fill(const int32_t *src, const int32_t *dst, int64_t nnz, int32_t *cursor,
                           int2 *oarc)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int at = atomicAdd(&cursor[src[e]], 1);
        oarc[at] = make_int2(dst[e], (int)e);
    }
}

// LT thresholds of one run, bit-sliced (one thread per node word): replicate
// g = goff + 64 w + b of node v gets need = max(1, ceil(U indeg / 2^32)) with
// U = D(LT threshold, v, g, 0), the same draw the per-step path takes; v
// activates iff its count of active in-neighbours reaches need.  Nodes
// whose in-degree needs more planes than the counter has are left to the
// per-step path (they are heavy rows, merged from their segments).
__global__ void k_lt_need(StepArgs a)
{
    const int64_t total = (int64_t)a.n * a.W;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int v = (int)(i / a.W);
        const int w = (int)(i - (int64_t)v * a.W);
        const uint32_t indeg = (uint32_t)(a.ptr[v + 1] - a.ptr[v]);
        const int P = indeg ? 32 - __builtin_clz(indeg) : 0;
        if (P == 0 || P > a.Lp) continue;
        uint64_t pl[16];
#pragma unroll
        for (int p = 0; p < 16; ++p) pl[p] = 0;
        const uint64_t g0 = a.goff + 64ull * (uint64_t)w;
        U4 o = {0u, 0u, 0u, 0u};
        for (int b = 0; b < 64; ++b) {
            const uint64_t g = g0 + (uint64_t)b;
            if (b == 0 || (g & 3u) == 0u)
                o = philox10((uint32_t)v, (uint32_t)(g >> 2), 0u, kDomLtThresh << 24, a.key0, a.key1);
            const uint32_t j = (uint32_t)g & 3u;
            const uint32_t u = j == 0 ? o.x : j == 1 ? o.y : j == 2 ? o.z : o.w;
            uint64_t need = ((uint64_t)u * (uint64_t)indeg + 0xFFFFFFFFull) >> 32;
            need = need ? need : 1ull;
#pragma unroll
            for (int p = 0; p < 16; ++p) pl[p] |= ((need >> p) & 1ull) << b;
        }
        uint64_t *np = a.need + (int64_t)v * a.Lp * a.W + w;
#pragma unroll
        for (int p = 0; p < 16; ++p)
            if (p < P) np[(int64_t)p * a.W] = pl[p];
    }
}

// Target row of every arc, used once when a graph is bound.  A block takes 256
// rows, their row pointers in LDS; its threads go over the rows' arcs and find
// each arc's row by bisection, so the stores are contiguous and a long row is
// shared by the block (a thread a row: 49 ms for 2.7e8 arcs of an R-MAT graph,
// 6.9 ms like this).
__global__ void __launch_bounds__(256) k_expand_rows(const int32_t *ptr, int64_t n, int32_t *dst)
{
    __shared__ int32_t s_ptr[257];
    for (int64_t r0 = (int64_t)blockIdx.x * 256; r0 < n; r0 += (int64_t)gridDim.x * 256) {
        const int rows = n - r0 < 256 ? (int)(n - r0) : 256;
        __syncthreads();
        for (int i = threadIdx.x; i <= rows; i += 256) s_ptr[i] = ptr[r0 + i];
        __syncthreads();
        const int e1 = s_ptr[rows];
        for (int e = s_ptr[0] + (int)threadIdx.x; e < e1; e += 256) {
            int lo = 0, hi = rows - 1;  // the last row that begins at or before e
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_ptr[mid] <= e) lo = mid; else hi = mid - 1;
            }
            dst[e] = (int32_t)(r0 + lo);
        }
    }
}

// Group of every arc's source, once when a graph is bound.
__global__ void k_src_groups(const int32_t *src, int64_t nnz, uint16_t *grp)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz;
         e += (int64_t)gridDim.x * blockDim.x)
        grp[e] = (uint16_t)node_group((uint32_t)src[e]);
}

// Before a step of the edge-parallel kernel: the next-frontier bitmap still
// holds the frontier of two steps back, whose words in the next plane are the
// only nonzero ones there; zero those words (the step ORs into them), then
// clear the bitmap and its summary.
__global__ void k_ic_clear(StepArgs a)
{
    if (a.flags[(a.step - 1) % (uint32_t)a.ring] == 0u) return;
    const int64_t nw = ((int64_t)a.n + 31) >> 5;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nw;
         i += (int64_t)gridDim.x * blockDim.x) {
        uint32_t x = a.bm_next[i];
        if (x) {
            a.bm_next[i] = 0u;
            while (x) {
                const int b = __builtin_ctz(x);
                x &= x - 1u;
                a.next[i * 32 + b] = 0ull;
            }
        }
        if (i < a.sum_words) a.sum_next[i] = 0u;
    }
}

// ------------------------------------------------------------ batches ----
// One launch per synchronous step for every job of a batch: a block per step
// block of every job, so jobs of very different sizes share the chip; a block
// reads its job from a table, leaves if the job is absorbed or past its step
// cap, and runs the job's own pull-step block.  (The dispatcher hands out
// blocks at a fraction of a nanosecond each -- 262,144 blocks that leave at
// once take 65-75 us -- where persistent blocks taking items from one counter
// were held to the 14 ns of its atomic add: twelve jobs of 1e4 to 1e5 nodes
// took 168, 68 and 52 ms with tiles of 256, 1024 and 4096 arcs.)  Ordering
// between steps comes from the kernel boundaries.

template <typename T>
__device__ __forceinline__ int find_job(const T *off, int n_jobs, T item)
{
    int lo = 0, hi = n_jobs - 1;  // last job whose first item is <= item
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= item) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ StepArgs job_at_step(const BatchCtl &c, int j, uint32_t t)
{
    StepArgs a = c.jobs[j];
    const uint64_t *p0 = a.prev;
    uint64_t *p1 = a.next;
    a.prev = (t & 1u) ? p0 : p1;   // state of step t-1
    a.next = (t & 1u) ? p1 : const_cast<uint64_t *>(p0);
    a.step = t;
    if (c.tail_on[j] == 0) {  // not in the tail mode this chunk
        a.ibm = nullptr;
        a.cand = nullptr;
    }
    return a;
}

__device__ __forceinline__ bool job_live(const BatchCtl &c, const StepArgs &a, int j, uint32_t t)
{
    return t <= (uint32_t)c.max_step[j] && a.flags[(t - 1) % (uint32_t)a.ring] != 0u;
}

__global__ void __launch_bounds__(kBatchBlock) __attribute__((amdgpu_waves_per_eu(kBatchWavesPerSimd)))
k_batch_step(BatchCtl c, uint32_t t, int first)
{
    __shared__ uint32_t s_code[kCodeTable];
    __shared__ uint64_t s_part[seg_lds_words<kKindLT, 16>()];
    __shared__ uint16_t s_rows[kMaxTileRows];
    const int item = first + (int)blockIdx.x;
    const int j = __builtin_amdgcn_readfirstlane((int)c.item_job[item]);
    const StepArgs a = job_at_step(c, j, t);
    if (!job_live(c, a, j, t)) return;
    const int local = item - c.item_off[j];
    if (a.ibm != nullptr && a.cand == nullptr) {
        // without the out-adjacency no launch before the step clears the
        // bitmap step t+1 sets
        uint32_t *clr = a.ibm + (size_t)((t + 1u) & 3u) * a.ibm_words;
        const int64_t nthr = (int64_t)(c.item_off[j + 1] - c.item_off[j]) * kBatchBlock;
        for (int64_t i = (int64_t)local * kBatchBlock + (int)threadIdx.x; i < a.ibm_words; i += nthr)
            clr[i] = 0u;
    }
    // tail mode: a tile with no candidate row leaves at once (every thread of
    // the block reads the same words)
    if (a.ibm != nullptr && tail_tile_idle(a, local, c.code[j] / 32 != kKindLT)) return;
    if (c.code[j] / 32 == kKindEpidemic) {  // block-uniform
        stage_codes(a, s_code);
        __syncthreads();
    }
    bool any = false;
    switch (c.code[j]) {
    case kKindIC * 32 + 1: step_block<kKindIC, light_planes(1), 1, true>(a, local, nullptr, 0, s_code, s_part, s_rows, any); break;
    case kKindEpidemic * 32 + 2: step_block<kKindEpidemic, light_planes(2), 2, true>(a, local, nullptr, 0, s_code, s_part, s_rows, any); break;
    case kKindEpidemic * 32 + 4: step_block<kKindEpidemic, light_planes(4), 4, true>(a, local, nullptr, 0, s_code, s_part, s_rows, any); break;
    case kKindEpidemic * 32 + 8: step_block<kKindEpidemic, light_planes(8), 8, true>(a, local, nullptr, 0, s_code, s_part, s_rows, any); break;
    case kKindEpidemic * 32 + 12: step_block<kKindEpidemic, light_planes(12), 12, true>(a, local, nullptr, 0, s_code, s_part, s_rows, any); break;
    case kKindEpidemic * 32 + 16: step_block<kKindEpidemic, light_planes(16), 16, true>(a, local, nullptr, 0, s_code, s_part, s_rows, any); break;
    case kKindLT * 32 + 2: step_block<kKindLT, light_planes(2), 2, true>(a, local, nullptr, 0, s_code, s_part, s_rows, any); break;
    case kKindLT * 32 + 4: step_block<kKindLT, light_planes(4), 4, true>(a, local, nullptr, 0, s_code, s_part, s_rows, any); break;
    case kKindLT * 32 + 8: step_block<kKindLT, light_planes(8), 8, true>(a, local, nullptr, 0, s_code, s_part, s_rows, any); break;
    case kKindLT * 32 + 12: step_block<kKindLT, light_planes(12), 12, true>(a, local, nullptr, 0, s_code, s_part, s_rows, any); break;
    case kKindLT * 32 + 16: step_block<kKindLT, light_planes(16), 16, true>(a, local, nullptr, 0, s_code, s_part, s_rows, any); break;
    default: break;
    }
    if (__ballot(any) != 0ull && (threadIdx.x & 63) == 0) a.flags[t % (uint32_t)a.ring] = 1u;
}

// k_combine for the jobs of a batch (blockIdx.y: the job).
__global__ void __launch_bounds__(kBatchBlock) k_batch_combine(BatchCtl c, uint32_t t)
{
    __shared__ uint32_t s_code[kCodeTable];
    const int j = (int)blockIdx.y;
    const StepArgs a = job_at_step(c, j, t);
    if (a.heavy_done != nullptr || !job_live(c, a, j, t)) return;
    if (c.code[j] / 32 == kKindEpidemic) {  // block-uniform
        stage_codes(a, s_code);
        __syncthreads();
    }
    int row;
    bool act;
    if (!merge_group(a, blockIdx.x, row, act)) return;
    const WordMap wm = word_map(a, a.G);
    bool any = false;
    switch (c.code[j]) {
    case kKindIC * 32 + 1: combine_row<kKindIC, 1, 1>(a, row, act, wm, nullptr, 0, s_code, any); break;
    case kKindEpidemic * 32 + 2: combine_row<kKindEpidemic, 2, 32>(a, row, act, wm, nullptr, 0, s_code, any); break;
    case kKindEpidemic * 32 + 4: combine_row<kKindEpidemic, 4, 32>(a, row, act, wm, nullptr, 0, s_code, any); break;
    case kKindEpidemic * 32 + 8: combine_row<kKindEpidemic, 8, 32>(a, row, act, wm, nullptr, 0, s_code, any); break;
    case kKindEpidemic * 32 + 12: combine_row<kKindEpidemic, 12, 32>(a, row, act, wm, nullptr, 0, s_code, any); break;
    case kKindEpidemic * 32 + 16: combine_row<kKindEpidemic, 16, 32>(a, row, act, wm, nullptr, 0, s_code, any); break;
    case kKindLT * 32 + 2: combine_row<kKindLT, 2, 32>(a, row, act, wm, nullptr, 0, s_code, any); break;
    case kKindLT * 32 + 4: combine_row<kKindLT, 4, 32>(a, row, act, wm, nullptr, 0, s_code, any); break;
    case kKindLT * 32 + 8: combine_row<kKindLT, 8, 32>(a, row, act, wm, nullptr, 0, s_code, any); break;
    case kKindLT * 32 + 12: combine_row<kKindLT, 12, 32>(a, row, act, wm, nullptr, 0, s_code, any); break;
    case kKindLT * 32 + 16: combine_row<kKindLT, 16, 32>(a, row, act, wm, nullptr, 0, s_code, any); break;
    default: break;
    }
    if (__ballot(any) != 0ull && (threadIdx.x & 63) == 0) a.flags[t % (uint32_t)a.ring] = 1u;
}

// Tail mode of the batched launch, before batched step t: for every job in
// the mode, the bitmaps step t+1 sets are cleared and the nodes of bitmap
// t-1 and their out-neighbours are marked in candidate bitmap t % 2 (a wave
// per bitmap word, over the words of all jobs that can take the mode).  The
// job offsets and mode switches are staged in LDS; a wave keeps a job's
// arguments while its words follow one another, and jumps past the words of
// a job that is not in the mode or has stopped.
__global__ void __launch_bounds__(256) k_batch_expand(BatchCtl c, uint32_t t)
{
    __shared__ int32_t s_off[kMaxBatchJobs + 1];
    __shared__ int32_t s_on[kMaxBatchJobs];
    for (int i = threadIdx.x; i <= c.n_jobs; i += blockDim.x) {
        s_off[i] = c.word_off[i];
        if (i < c.n_jobs) s_on[i] = c.tail_on[i];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int64_t total = s_off[c.n_jobs];
    int jc = -1;  // the job `a` holds
    bool on = false;
    StepArgs a{};
    for (int64_t item = wave; item < total; item += nwave) {
        const int j = __builtin_amdgcn_readfirstlane(find_job(s_off, c.n_jobs, (int32_t)item));
        if (j != jc) {
            jc = j;
            on = s_on[j] != 0;
            if (on) {
                a = job_at_step(c, j, t);
                on = job_live(c, a, j, t);
            }
        }
        if (!on) {
            // the loop step then lands on this wave's first word of a later job
            item += ((int64_t)s_off[j + 1] - 1 - item) / nwave * nwave;
            continue;
        }
        const int i = (int)item - s_off[j];
        if (lane == 0) {
            a.ibm[(size_t)((t + 1u) & 3u) * a.ibm_words + i] = 0u;
            a.cand[(size_t)((t + 1u) & 1u) * a.ibm_words + i] = 0u;
        }
        uint32_t m = a.ibm[(size_t)((t - 1u) & 3u) * a.ibm_words + i];
        if (m == 0u) continue;
        uint32_t *cand = a.cand + (size_t)(t & 1u) * a.ibm_words;
        if (lane == 0) atomicOr(&cand[i], m);
        while (m) {
            const int u = 32 * i + __builtin_ctz(m);
            m &= m - 1u;
            const int o1 = a.optr[u + 1];
            for (int e = a.optr[u] + lane; e < o1; e += 64) {
                const int v = a.oarc[e].x;
                atomicOr(&cand[v >> 5], 1u << (v & 31));
            }
        }
    }
}

// Per job that can take the tail mode, the nodes with an infected replicate
// or a new activation after step t into counts[j] (zeroed by the caller): a
// nonzero word of the state plane after step t (SI family: the infected
// plane; IC: the frontier plane), or activation stamp t (LT).  A job in the tail mode has these nodes in its bitmap t % 4
// already (a node that is no candidate keeps no infected replicate and gains
// no activation), so one bit is read instead of its row; a job that did not
// run step t counts nothing (the host no longer reads its count).
__global__ void k_batch_count(BatchCtl c, uint32_t t, unsigned long long *counts)
{
    const int64_t total = c.row_off[c.n_jobs];
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
    // a wave takes 64 consecutive rows at a time, job by job within them;
    // state planes of several words a row are read with lanes over words
    // (64 / W whole rows a pass), so the loads of a pass are contiguous
    for (int64_t r0 = wave * 64; r0 < total; r0 += nwave * 64) {
        const int64_t rend = r0 + 64 < total ? r0 + 64 : total;
        for (int64_t r = r0; r < rend;) {
            const int j = __builtin_amdgcn_readfirstlane(find_job(c.row_off, c.n_jobs, r));
            const int64_t je = c.row_off[j + 1] < rend ? c.row_off[j + 1] : rend;
            const StepArgs &a = c.jobs[j];
            const int64_t v0 = r - c.row_off[j];  // first row of the job in [r, je)
            const int64_t nr = je - r;
            unsigned long long cnt = 0;
            if (job_live(c, a, j, t)) {
                if (c.tail_on[j] != 0 && a.ibm != nullptr) {
                    const int64_t v = v0 + lane;
                    const bool hit = lane < nr &&
                                     ((a.ibm[(size_t)(t & 3u) * a.ibm_words + (v >> 5)] >> (v & 31)) & 1u);
                    cnt = (unsigned long long)__popcll(__ballot(hit));
                } else if (c.code[j] / 32 == kKindLT) {
                    const int64_t v = v0 + lane;
                    const bool hit = lane < nr && a.stamp[(size_t)(t & 1u) * (size_t)a.n + (size_t)v] == t;
                    cnt = (unsigned long long)__popcll(__ballot(hit));
                } else {
                    const uint64_t *pl = (t & 1u) ? a.next : a.prev;  // state after step t
                    const int W = a.W;
                    if (W <= 64) {
                        const int R = 64 / W;  // rows a pass
                        const int slot = lane / W, w = lane - slot * W;
                        const uint64_t gmask = W == 64 ? ~0ull : ((1ull << W) - 1ull);
                        for (int64_t q = 0; q < nr; q += R) {
                            const bool in = slot < R && q + slot < nr;
                            const uint64_t x = in ? pl[(v0 + q + slot) * W + w] : 0ull;
                            const uint64_t m = __ballot(x != 0ull);
                            for (int k = 0; k < R; ++k) cnt += ((m >> (k * W)) & gmask) != 0ull ? 1ull : 0ull;
                        }
                    } else {
                        for (int64_t q = 0; q < nr; ++q) {
                            uint64_t x = 0;
                            for (int w = lane; w < W; w += 64) x |= pl[(v0 + q) * W + w];
                            cnt += __ballot(x != 0ull) != 0ull ? 1ull : 0ull;
                        }
                    }
                }
            }
            if (lane == 0 && cnt) atomicAdd(&counts[j], cnt);  // cnt is wave-uniform
            r = je;
        }
    }
}

// Before a chunk of steps that begins at step t: every flag of every job's
// ring but slot t-1 (which step t reads) is cleared, and every word flag but
// those of t-1 and t-2.  One block per job.
__global__ void __launch_bounds__(256) k_batch_ring_clear(BatchCtl c, uint32_t t)
{
    const StepArgs &a = c.jobs[blockIdx.x];
    const uint32_t keep = (t - 1u) % (uint32_t)a.ring;
    for (uint32_t i = threadIdx.x; i < (uint32_t)a.ring; i += blockDim.x)
        if (i != keep) a.flags[i] = 0u;
    if (a.wflags == nullptr) return;
    const uint32_t wr = (uint32_t)a.wring, W = (uint32_t)a.W;
    const uint32_t k1 = (t - 1u) % wr, k2 = (t + wr - 2u) % wr;
    for (uint32_t i = threadIdx.x; i < wr * W; i += blockDim.x) {
        const uint32_t sl = i / W;
        if (sl != k1 && sl != k2) a.wflags[i] = 0u;
    }
}

// ------------------------------------------------------- init / output ----

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Zeroes count16 16-byte words with non-temporal stores (the zeroed planes
// are next touched a step or more later, sparsely).
__global__ void k_zero16(u32x4 *p, int64_t count16)
{
    const u32x4 z = {0u, 0u, 0u, 0u};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count16;
         i += (int64_t)gridDim.x * blockDim.x)
        __builtin_nontemporal_store(z, p + i);
}

// Bitmaps of the tail mode for step t: bit v of bitmap (t-1) % 4 set iff
// `cur` (the state after t-1) has a nonzero word in row v, of bitmap
// (t-2) % 4 iff `old` (the state after t-2) does; bitmap t % 4 cleared.  One
// thread per bitmap word (32 rows).
__global__ void k_mark_rows(const uint64_t *cur, const uint64_t *old, uint32_t *ibm, uint32_t *cand,
                            int32_t ibm_words, int64_t n, int64_t W, uint32_t t)
{
    uint32_t *b1 = ibm + (size_t)((t - 1u) & 3u) * ibm_words;
    uint32_t *b2 = ibm + (size_t)((t - 2u) & 3u) * ibm_words;
    uint32_t *b0 = ibm + (size_t)(t & 3u) * ibm_words;
    uint32_t *c0 = cand + (size_t)(t & 1u) * ibm_words;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ibm_words;
         i += (int64_t)gridDim.x * blockDim.x) {
        uint32_t m1 = 0, m2 = 0;
        for (int j = 0; j < 32; ++j) {
            const int64_t v = 32 * i + j;
            if (v >= n) break;
            uint64_t c = 0, o = 0;
            for (int64_t w = 0; w < W; ++w) {
                c |= cur[v * W + w];
                o |= old[v * W + w];
            }
            m1 |= (c ? 1u : 0u) << j;
            m2 |= (o ? 1u : 0u) << j;
        }
        b1[i] = m1;
        b2[i] = m2;
        b0[i] = 0u;
        c0[i] = 0u;
    }
}

// Candidates of tail-mode step t: every node with an infected replicate
// after t-1 (bitmap t-1) and its out-neighbours are marked in candidate
// bitmap t % 2.  Wave k takes bitmap words k, k + waves, ...; each set bit is
// a node whose out-arcs the wave's lanes mark.
__global__ void __launch_bounds__(256) k_tail_expand(StepArgs a)
{
    if (a.flags[(a.step - 1) % (uint32_t)a.ring] == 0u) return;  // as the step: nothing left
    const uint32_t *inf1 = a.ibm + (size_t)((a.step - 1u) & 3u) * a.ibm_words;
    uint32_t *cand = a.cand + (size_t)(a.step & 1u) * a.ibm_words;
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t i = wave; i < a.ibm_words; i += nwave) {
        uint32_t m = inf1[i];
        if (m == 0u) continue;
        if (lane == 0) atomicOr(&cand[i], m);
        while (m) {
            const int u = (int)(32 * i) + __builtin_ctz(m);
            m &= m - 1u;
            const int o1 = a.optr[u + 1];
            for (int e = a.optr[u] + lane; e < o1; e += 64) {
                const int v = a.oarc[e].x;
                atomicOr(&cand[v >> 5], 1u << (v & 31));
            }
        }
    }
}

// The same for LT from its activation stamps: bitmap (t-1) % 4 marks the
// nodes with a new activation at t-1, bitmap (t-2) % 4 those at t-2.
__global__ void k_mark_gained(const uint32_t *stamp, uint32_t *ibm, uint32_t *cand,
                              int32_t ibm_words, int64_t n, uint32_t t)
{
    const uint32_t *s1 = stamp + (size_t)((t - 1u) & 1u) * (size_t)n;
    const uint32_t *s2 = stamp + (size_t)(t & 1u) * (size_t)n;
    uint32_t *b1 = ibm + (size_t)((t - 1u) & 3u) * ibm_words;
    uint32_t *b2 = ibm + (size_t)((t - 2u) & 3u) * ibm_words;
    uint32_t *b0 = ibm + (size_t)(t & 3u) * ibm_words;
    uint32_t *c0 = cand + (size_t)(t & 1u) * ibm_words;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ibm_words;
         i += (int64_t)gridDim.x * blockDim.x) {
        uint32_t m1 = 0, m2 = 0;
        for (int j = 0; j < 32; ++j) {
            const int64_t v = 32 * i + j;
            if (v >= n) break;
            m1 |= (s1[v] == t - 1u ? 1u : 0u) << j;
            m2 |= (s2[v] == t - 2u ? 1u : 0u) << j;
        }
        b1[i] = m1;
        b2[i] = m2;
        b0[i] = 0u;
        c0[i] = 0u;
    }
}

// Number of LT nodes with a new activation at step t (stamp t in array t & 1).
__global__ void k_count_stamped(const uint32_t *stamp, int64_t n, uint32_t t, unsigned long long *count)
{
    const uint32_t *s = stamp + (size_t)(t & 1u) * (size_t)n;
    unsigned long long c = 0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x)
        c += s[v] == t ? 1ull : 0ull;
    for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
    if ((threadIdx.x & 63) == 0 && c) atomicAdd(count, c);
}

// Nodes with a nonzero word in `plane` ([n][W]) into *count (zeroed by the
// caller).  Lanes go over words so that a wave's loads are contiguous: with
// W <= 64 a pass of the wave takes 64 / W whole rows (R W consecutive words)
// and counts the rows whose W-bit group of the ballot is nonzero; wider rows
// take a wave each, its lanes striding over the row.
__global__ void k_count_rows(const uint64_t *plane, int64_t n, int64_t W, unsigned long long *count)
{
    const int lane = (int)(threadIdx.x & 63u);
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
    unsigned long long c = 0;
    if (W <= 64) {
        const int Wi = (int)W;
        const int R = 64 / Wi;  // rows per pass
        const int slot = lane / Wi, w = lane - slot * Wi;
        const uint64_t gmask = Wi == 64 ? ~0ull : ((1ull << Wi) - 1ull);
        for (int64_t r0 = wave * R; r0 < n; r0 += nwave * R) {
            const int64_t v = r0 + slot;
            const uint64_t x = (slot < R && v < n) ? plane[v * W + w] : 0ull;
            const uint64_t m = __ballot(x != 0ull);
            if (Wi == 1) {
                c += (unsigned long long)__popcll(m);
            } else {
                for (int k = 0; k < R; ++k) c += ((m >> (k * Wi)) & gmask) != 0ull ? 1ull : 0ull;
            }
        }
    } else {
        for (int64_t v = wave; v < n; v += nwave) {
            uint64_t x = 0;
            for (int64_t w = lane; w < W; w += 64) x |= plane[v * W + w];
            c += __ballot(x != 0ull) != 0ull ? 1ull : 0ull;
        }
    }
    if (lane == 0 && c) atomicAdd(count, c);  // c is the same in every lane of the wave
}

__global__ void k_zero16_unless(u32x4 *p, int64_t count16, const uint64_t *tag, uint64_t expect)
{
    if (*tag == expect) return;
    const u32x4 z = {0u, 0u, 0u, 0u};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count16;
         i += (int64_t)gridDim.x * blockDim.x)
        __builtin_nontemporal_store(z, p + i);
}

__global__ void k_fill64(uint64_t *p, int64_t count, uint64_t value)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

__global__ void k_stamp_seeds(uint32_t *stamp, const int32_t *seeds, int64_t ns)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ns;
         i += (int64_t)gridDim.x * blockDim.x)
        stamp[seeds[i]] = 0u;
}

__global__ void k_fill32(uint32_t *p, int64_t count, uint32_t value)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

// Clears every absorption flag of the ring except slot `keep` (the step
// before the next chunk).
// With word flags, the slots of steps t and t-1 are kept (the next step
// reads both).
__global__ void k_ring_clear(uint32_t *flags, int32_t ring, int32_t keep, uint32_t *wflags,
                             int32_t W, int32_t wring, int64_t t)
{
    for (int i = threadIdx.x; i < ring; i += blockDim.x)
        if (i != keep) flags[i] = 0u;
    if (wflags == nullptr) return;
    const int64_t k1 = t % wring, k2 = (t + wring - 1) % wring;
    for (int64_t i = threadIdx.x; i < (int64_t)wring * W; i += blockDim.x) {
        const int64_t sl = i / W;
        if (sl != k1 && sl != k2) wflags[i] = 0u;
    }
}

// Seeds are in state 1 in every replicate (Algorithm 1, initial states).
__global__ void k_seed(uint64_t *p1, uint64_t *p2, const int32_t *seeds, int64_t ns, int32_t W,
                       int64_t B, uint32_t *flag0, uint32_t *bm, uint32_t *sum)
{
    const int64_t total = ns * W;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = i / W;
        const int w = (int)(i - k * W);
        const int64_t idx = (int64_t)seeds[k] * W + w;
        const uint64_t m = tail_mask(w, B);
        p1[idx] = m;
        if (p2) p2[idx] = m;
        if (bm && w == 0) {
            const int u = seeds[k];
            const uint32_t i = node_group((uint32_t)u);
            atomicOr(&bm[u >> 5], 1u << (u & 31));
            atomicOr(&sum[i >> 5], 1u << (i & 31));
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && ns > 0) flag0[0] = 1u;
}

// Packed planes -> uint8 states [n][B] and per-node counts: any B and any
// alignment of the states (byte stores; launch_finalize uses it for the states
// only where they are not 16-byte aligned, and otherwise for the counts).
__global__ void __launch_bounds__(256) k_finalize(FinArgs f)
{
    if (!spec_planes(f)) return;
    const int lane = threadIdx.x & 63;
    const int G = f.G;
    const int rpw = 64 >> f.lgG;
    const int gw = lane & (G - 1);
    const int64_t gwave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwave_total = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t rb = gwave * rpw; rb < f.n; rb += nwave_total * rpw) {
        const int64_t v = rb + (lane >> f.lgG);
        const bool act = v < f.n;
        uint32_t cnt = 0;
        for (int w0 = 0; w0 < f.W; w0 += G) {
            const int w = w0 + gw;
            if (!act || w >= f.W) continue;
            const int64_t idx = v * f.W + w;
            const uint64_t tail = tail_mask(w, f.B);
            const bool live = !f.bm || ((f.bm[v >> 5] >> (v & 31)) & 1u);
            const bool live2 = f.two && (!f.two_bm || ((f.two_bm[v >> 5] >> (v & 31)) & 1u));
            const uint64_t one = live ? (f.one[idx] & tail) : 0ull;
            const uint64_t two = live2 ? (f.two[idx] & tail) : 0ull;
            const uint64_t three = f.three ? (f.three[idx] & tail) : 0ull;
            if (f.scrub && live2) f.two[idx] = 0ull;
            cnt += (uint32_t)__popcll(f.model == kSIS ? one : (one | two | three));
            if (!f.states) continue;
            // state codes: with a latent plane E 1, I 2, R 3 (the planes are
            // disjoint); else 1 for the first plane, 2 for the second only
            const uint32_t m1 = f.three ? 2u : 1u, m2 = f.three ? 3u : 2u;
            uint8_t *dst = f.states + v * f.B + 64ll * w;
            const int64_t nb = f.B - 64ll * w < 64 ? f.B - 64ll * w : 64;
            for (int j = 0; j < nb; ++j) {
                const uint32_t s1 = (uint32_t)(one >> j) & 1u;
                const uint32_t s2 = (uint32_t)(two >> j) & 1u & ~s1;
                const uint32_t s3 = (uint32_t)(three >> j) & 1u;
                dst[j] = (uint8_t)(s1 * m1 + s2 * m2 + s3);
            }
        }
        for (int off = 1; off < G; off <<= 1) cnt += __shfl_xor(cnt, off, 64);
        if (act && gw == 0 && f.counts) f.counts[v] = cnt;
        // scrubbing runs have one word per node (G = 1), so the wave's 64
        // nodes cover whole bitmap words, all read above
        if (f.scrub && act && (v & 31) == 0) f.two_bm[v >> 5] = 0u;
    }
}

// States alone for any B, the array 16-byte aligned: [n][B] is written as flat
// bytes, 16 a lane and 1 KB a store instruction, whatever B is; a lane finds
// the row and replicate its bytes start at and takes up to 16 bits of each
// plane from there, going on in the next rows where a row ends.  Bound by the
// writes: 3e5 nodes at B = 1000 (300 MB) took 335 us with each lane storing
// its word's 64 bytes one by one, 85 us (3.5 TB/s) and 27 for the counts.
constexpr int kFlatKb = 4;  // consecutive KB a wave writes

__device__ __forceinline__ uint32_t bits16(const uint64_t *p, int64_t base, int W, uint32_t r)
{
    const uint32_t w = r >> 6, sh = r & 63u;
    uint64_t x = p[base + w] >> sh;
    if (sh > 48u && (int)w + 1 < W) x |= p[base + w + 1] << (64u - sh);
    return (uint32_t)x & 0xFFFFu;
}

__global__ void __launch_bounds__(256) k_finalize_flat(FinArgs f)
{
    if (!spec_planes(f)) return;
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t total = (int64_t)f.n * f.B;
    const int64_t o0 = wave * (kFlatKb * 1024);
    if (o0 >= total) return;
    // (v, r): row and replicate of this lane's first byte, then 1 KB on
    const uint32_t B = (uint32_t)f.B;
    const int64_t v0 = o0 / f.B;
    const uint32_t off = (uint32_t)(o0 - v0 * f.B) + 16u * (uint32_t)lane;
    int64_t v = v0 + (int64_t)(off / B);
    uint32_t r = off % B;
    const uint32_t dq = 1024u / B, dr = 1024u - dq * B;
    const uint32_t m1 = f.three ? 2u : 1u, m2 = f.three ? 3u : 2u;
#pragma unroll
    for (int k = 0; k < kFlatKb; ++k) {
        const int64_t o = o0 + 1024 * k + 16 * lane;
        if (o < total) {
            uint32_t h1 = 0, h2 = 0, h3 = 0, filled = 0, rr = r;
            int64_t vv = v;
            do {
                const uint32_t m = min(16u - filled, B - rr);
                const uint32_t keep = (1u << m) - 1u;
                const int64_t base = vv * f.W;
                const bool live = !f.bm || ((f.bm[vv >> 5] >> (vv & 31)) & 1u);
                const bool live2 = f.two && (!f.two_bm || ((f.two_bm[vv >> 5] >> (vv & 31)) & 1u));
                if (live) h1 |= (bits16(f.one, base, f.W, rr) & keep) << filled;
                if (live2) h2 |= (bits16(f.two, base, f.W, rr) & keep) << filled;
                if (f.three) h3 |= (bits16(f.three, base, f.W, rr) & keep) << filled;
                filled += m;
                ++vv;
                rr = 0;
            } while (filled < 16u && vv < f.n);
            h2 &= ~h1;
            uint32_t wd[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t n1 = (h1 >> (4 * q)) & 0xFu, n2 = (h2 >> (4 * q)) & 0xFu,
                               n3 = (h3 >> (4 * q)) & 0xFu;
                wd[q] = spread4(n1, 0x204081u, 0x01010101u) * m1 +
                        spread4(n2, 0x204081u, 0x01010101u) * m2 + spread4(n3, 0x204081u, 0x01010101u);
            }
            if (o + 16 <= total) {
                const u32x4 out = {wd[0], wd[1], wd[2], wd[3]};
                __builtin_nontemporal_store(out, reinterpret_cast<u32x4 *>(f.states + o));
            } else {  // the array's last bytes
                for (int64_t j = 0; o + j < total; ++j) {
                    const uint32_t x = j < 4 ? wd[0] : (j < 8 ? wd[1] : (j < 12 ? wd[2] : wd[3]));
                    f.states[o + j] = (uint8_t)(x >> (8 * (j & 3)));
                }
            }
        }
        v += dq;
        r += dr;
        if (r >= B) {
            r -= B;
            ++v;
        }
    }
}

// The same when B = 64 W and W is a power of two up to 64 (so G = W and a
// wave holds one word per lane): the uint8 states of a wave's 64 words form
// one contiguous 4 KB block, and each store instruction writes 1 KB of it
// (pass q, lane l: bytes 16 (64 q + l) .. +15 of the block, whose word is
// held by lane 16 q + l / 4 and reaches lane l by shuffle), instead of 16
// bytes at a 64-byte stride per lane.  Needs a 16-byte aligned state array.
__device__ __forceinline__ uint64_t shfl64(uint64_t x, int src)
{
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)x, src, 64);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(x >> 32), src, 64);
    return ((uint64_t)hi << 32) | lo;
}

// Loads the packed words of lane's node word for the dense finalize.
struct DenseWords {
    uint64_t one, two, three;
    bool act;
};

__device__ __forceinline__ DenseWords dense_words(const FinArgs &f, int64_t rb, int lane)
{
    DenseWords d = {0ull, 0ull, 0ull, false};
    const int64_t v = rb + (lane >> f.lgG);
    d.act = v < f.n;
    if (d.act) {
        const int64_t idx = v * f.W + (lane & (f.G - 1));
        const bool live = !f.bm || ((f.bm[v >> 5] >> (v & 31)) & 1u);
        const bool live2 = f.two && (!f.two_bm || ((f.two_bm[v >> 5] >> (v & 31)) & 1u));
        d.one = live ? f.one[idx] : 0ull;
        d.two = live2 ? f.two[idx] : 0ull;
        d.three = f.three ? f.three[idx] : 0ull;
        if (f.scrub && live2) f.two[idx] = 0ull;
    }
    return d;
}

// Counts and states of one wave's 64 words (rows rb .. rb + 64 / G - 1).
__device__ __forceinline__ void dense_out(const FinArgs &f, int64_t rb, int lane,
                                          const DenseWords &d)
{
    const int G = f.G;
    uint32_t cnt = (uint32_t)__popcll(f.model == kSIS ? d.one : (d.one | d.two | d.three));
    for (int off = 1; off < G; off <<= 1) cnt += __shfl_xor(cnt, off, 64);
    if (d.act && (lane & (G - 1)) == 0 && f.counts) f.counts[rb + (lane >> f.lgG)] = cnt;
    if (!f.states) return;
    // state byte = s1 m1 + s2 m2 + s3 (at most 3, so bytes never carry)
    const uint32_t m1 = f.three ? 2u : 1u, m2 = f.three ? 3u : 2u;
    uint8_t *blk = f.states + rb * f.B;
    const int64_t limit = (f.n - rb) * f.B;  // bytes of the block inside the array
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int src = 16 * q + (lane >> 2);
        const uint64_t o1 = shfl64(d.one, src), o2 = shfl64(d.two, src), o3 = shfl64(d.three, src);
        const int sh = 16 * (lane & 3);
        const uint32_t h1 = (uint32_t)(o1 >> sh) & 0xFFFFu, h2 = (uint32_t)(o2 >> sh) & 0xFFFFu & ~h1,
                       h3 = (uint32_t)(o3 >> sh) & 0xFFFFu;
        uint32_t wd[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t n1 = (h1 >> (4 * k)) & 0xFu, n2 = (h2 >> (4 * k)) & 0xFu,
                           n3 = (h3 >> (4 * k)) & 0xFu;
            wd[k] = spread4(n1, 0x204081u, 0x01010101u) * m1 +
                    spread4(n2, 0x204081u, 0x01010101u) * m2 + spread4(n3, 0x204081u, 0x01010101u);
        }
        const int64_t byte = 16 * (64 * q + lane);
        if (byte < limit) {
            const u32x4 o = {wd[0], wd[1], wd[2], wd[3]};
            __builtin_nontemporal_store(o, reinterpret_cast<u32x4 *>(blk + byte));
        }
    }
}

// Two blocks of 64 words per pass, their loads issued before either's stores.
__global__ void __launch_bounds__(256) k_finalize_dense(FinArgs f)
{
    if (!spec_planes(f)) return;
    const int lane = threadIdx.x & 63;
    const int rpw = 64 >> f.lgG;
    const int64_t gwave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwave_total = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int64_t stride = nwave_total * rpw;
    for (int64_t rb = gwave * rpw; rb < f.n; rb += 2 * stride) {
        const DenseWords d0 = dense_words(f, rb, lane);
        const bool two_blocks = rb + stride < f.n;
        const DenseWords d1 = two_blocks ? dense_words(f, rb + stride, lane)
                                         : DenseWords{0ull, 0ull, 0ull, false};
        if (f.scrub) {  // one word per node: a wave's 64 nodes are two whole bitmap words
            const int64_t v = rb + lane;
            if (d0.act && (v & 31) == 0) f.two_bm[v >> 5] = 0u;
            if (d1.act && ((v + stride) & 31) == 0) f.two_bm[(v + stride) >> 5] = 0u;
        }
        dense_out(f, rb, lane, d0);
        if (two_blocks) dense_out(f, rb + stride, lane, d1);
    }
}

// State tally after a step (per-step trajectories): popcounts of the state
// planes summed over nodes and replicates into tally[0..2] (zeroed by the
// caller); integer atomics, so the totals are exact and independent of the
// order.  Lanes go over words (64 / W whole rows a pass), the waves of a block
// meet in LDS and at most 512 blocks add to the totals: one atomic a wave on
// the same line bounded the kernel before (1e5 nodes of 4 words: 198 us a
// step with 6250 waves adding, 15 us).
__global__ void __launch_bounds__(256) k_tally(FinArgs f)
{
    if (f.flags && f.step > 1u && f.flags[(f.step - 1u) % (uint32_t)f.ring] == 0u) {
        if (blockIdx.x == 0 && threadIdx.x < 3) f.tally[threadIdx.x] = f.tally[(int)threadIdx.x - 3];
        return;
    }
    unsigned long long c1 = 0, c2 = 0, c3 = 0;
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
    auto add = [&](int64_t v, int w, uint64_t tail) {
        const int64_t i = v * f.W + w;
        const bool live = !f.bm || ((f.bm[v >> 5] >> (v & 31)) & 1u);
        const uint64_t one = live ? (f.one[i] & tail) : 0ull;
        const uint64_t two = f.two ? (f.two[i] & tail & ~one) : 0ull;
        if (f.three) {  // E 1, I 2, R 3
            c1 += (unsigned long long)__popcll(f.three[i] & tail);
            c2 += (unsigned long long)__popcll(one);
            c3 += (unsigned long long)__popcll(two);
        } else {
            c1 += (unsigned long long)__popcll(one);
            c2 += (unsigned long long)__popcll(two);
        }
    };
    if (f.W <= 64) {
        const int R = 64 / f.W, slot = lane / f.W, w = lane - slot * f.W;
        const uint64_t tail = tail_mask(w, f.B);
        for (int64_t r0 = wave * R; r0 < f.n; r0 += nwave * R)
            if (slot < R && r0 + slot < f.n) add(r0 + slot, w, tail);
    } else {
        for (int64_t v = wave; v < f.n; v += nwave)
            for (int w = lane; w < f.W; w += 64) add(v, w, tail_mask(w, f.B));
    }
    for (int off = 32; off > 0; off >>= 1) {
        c1 += __shfl_xor(c1, off, 64);
        c2 += __shfl_xor(c2, off, 64);
        c3 += __shfl_xor(c3, off, 64);
    }
    __shared__ unsigned long long s_c[4][3];
    if (lane == 0) {
        s_c[threadIdx.x >> 6][0] = c1;
        s_c[threadIdx.x >> 6][1] = c2;
        s_c[threadIdx.x >> 6][2] = c3;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const unsigned long long t = s_c[0][threadIdx.x] + s_c[1][threadIdx.x] +
                                     s_c[2][threadIdx.x] + s_c[3][threadIdx.x];
        if (t) atomicAdd(&f.tally[threadIdx.x], t);
    }
}

__global__ void k_philox(const uint32_t *ctr, uint32_t k0, uint32_t k1, uint32_t *out,
                         int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x) {
        const U4 o = philox10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], k0, k1);
        out[4 * i] = o.x;
        out[4 * i + 1] = o.y;
        out[4 * i + 2] = o.z;
        out[4 * i + 3] = o.w;
    }
}

// ------------------------------------------------------------ launchers ----

static unsigned grid_for(int64_t work, int block)
{
    int64_t g = (work + block - 1) / block;
    if (g < 1) g = 1;
    if (g > 65536) g = 65536;
    return (unsigned)g;
}

// Most blocks of a launch: its threads are counted in 32 bits.
static int most_blocks(int block) { return (int)(0xFFFFFFFFu / (unsigned)block); }

hipError_t launch_zero(void *p, size_t bytes, hipStream_t s)
{
    // 16-byte words first (p is 256-byte aligned), the last 8 bytes if any
    const int64_t n16 = (int64_t)(bytes / 16);
    if (n16 > 0) {
        hipLaunchKernelGGL(k_zero16, dim3(grid_for(n16, 256)), dim3(256), 0, s, (u32x4 *)p, n16);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (bytes % 16 >= 8) return launch_fill64((uint64_t *)((char *)p + 16 * n16), 1, 0ull, s);
    return hipSuccess;
}

hipError_t launch_zero_unless(void *p, size_t bytes, const uint64_t *tag, uint64_t expect,
                              hipStream_t s)
{
    // whole 16-byte words only: callers pass regions of 256-byte multiples
    const int64_t n16 = (int64_t)(bytes / 16);
    if (n16 <= 0) return hipSuccess;
    // a grid of at most 1024 blocks: when the tag is there every block only
    // reads it, and a larger grid costs more to dispatch than that
    const unsigned g = std::min<unsigned>(grid_for(n16, 256), 1024u);
    hipLaunchKernelGGL(k_zero16_unless, dim3(g), dim3(256), 0, s, (u32x4 *)p, n16, tag, expect);
    return hipGetLastError();
}

hipError_t launch_mark_rows(const uint64_t *cur, const uint64_t *old, uint32_t *ibm, uint32_t *cand,
                            int32_t ibm_words, int64_t n, int64_t W, uint32_t t, hipStream_t s)
{
    if (ibm_words <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mark_rows, dim3(grid_for(ibm_words, 64)), dim3(64), 0, s, cur, old, ibm,
                       cand, ibm_words, n, W, t);
    return hipGetLastError();
}

hipError_t launch_mark_gained(const uint32_t *stamp, uint32_t *ibm, uint32_t *cand, int32_t ibm_words,
                              int64_t n, uint32_t t, hipStream_t s)
{
    if (ibm_words <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mark_gained, dim3(grid_for(ibm_words, 64)), dim3(64), 0, s, stamp, ibm, cand,
                       ibm_words, n, t);
    return hipGetLastError();
}

hipError_t launch_count_stamped(const uint32_t *stamp, int64_t n, uint32_t t,
                                unsigned long long *count, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill64, dim3(1), dim3(64), 0, s, (uint64_t *)count, (int64_t)1, 0ull);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n <= 0) return e;
    hipLaunchKernelGGL(k_count_stamped, dim3(std::min<unsigned>(grid_for(n, 256), 2048u)), dim3(256),
                       0, s, stamp, n, t, count);
    return hipGetLastError();
}

hipError_t launch_tail_expand(const StepArgs &a, hipStream_t s)
{
    // a wave per bitmap word, at most 1024 blocks of four waves
    const unsigned g = std::min<unsigned>(grid_for((int64_t)a.ibm_words * 64, 256), 1024u);
    hipLaunchKernelGGL(k_tail_expand, dim3(g), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_count_rows(const uint64_t *plane, int64_t n, int64_t W, unsigned long long *count,
                             hipStream_t s)
{
    hipLaunchKernelGGL(k_fill64, dim3(1), dim3(64), 0, s, (uint64_t *)count, (int64_t)1, 0ull);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n <= 0) return e;
    hipLaunchKernelGGL(k_count_rows, dim3(std::min<unsigned>(grid_for(n, 256), 2048u)), dim3(256), 0,
                       s, plane, n, W, count);
    return hipGetLastError();
}

hipError_t launch_ic_scrub(const StepArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_ic_scrub, dim3(256), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_ic_scrub_spec(const StepArgs &a, const SpecFin &sp, int which, uint64_t *tag,
                                uint64_t tag_value, hipStream_t s)
{
    hipLaunchKernelGGL(k_ic_scrub_spec, dim3(256), dim3(256), 0, s, a, sp, which, tag, tag_value);
    return hipGetLastError();
}

hipError_t launch_fill64(uint64_t *p, int64_t count, uint64_t value, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill64, dim3(grid_for(count, 256)), dim3(256), 0, s, p, count, value);
    return hipGetLastError();
}

hipError_t launch_stamp_seeds(uint32_t *stamp, const int32_t *seeds, int64_t ns, hipStream_t s)
{
    if (ns <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_stamp_seeds, dim3(grid_for(ns, 256)), dim3(256), 0, s, stamp, seeds, ns);
    return hipGetLastError();
}

hipError_t launch_fill32(uint32_t *p, int64_t count, uint32_t value, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill32, dim3(grid_for(count, 256)), dim3(256), 0, s, p, count, value);
    return hipGetLastError();
}

hipError_t launch_lt_need(const StepArgs &a, hipStream_t s)
{
    const int64_t total = (int64_t)a.n * a.W;
    hipLaunchKernelGGL(k_lt_need, dim3(grid_for(total, 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_ring_clear(uint32_t *flags, int32_t ring, int32_t keep, hipStream_t s,
                             uint32_t *wflags, int32_t W, int32_t wring, int64_t t)
{
    hipLaunchKernelGGL(k_ring_clear, dim3(1), dim3(256), 0, s, flags, ring, keep, wflags, W,
                       wring, t);
    return hipGetLastError();
}

hipError_t launch_ic_front(const StepArgs &a, int grid, int block, hipStream_t s)
{
    // enough blocks for the larger of the two passes (8 arcs a thread when
    // streaming; a wave per work item when pushing), at most `grid`
    const int64_t work = std::max<int64_t>((a.nnz + 7) / 8, (int64_t)a.n * 64);
    const int64_t g = std::max<int64_t>(1, std::min<int64_t>((work + block - 1) / block, grid));
    hipLaunchKernelGGL(k_ic_front, dim3((unsigned)g), dim3((unsigned)block), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_seed_queue(const StepArgs &a, const int32_t *seeds, int64_t ns, hipStream_t s)
{
    if (ns <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_seed_queue, dim3(grid_for(ns, 256)), dim3(256), 0, s, a, seeds, ns);
    return hipGetLastError();
}

hipError_t launch_out_count(const int32_t *src, int64_t nnz, int32_t *cnt, hipStream_t s)
{
    if (nnz <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_out_count, dim3(grid_for(nnz, 256)), dim3(256), 0, s, src, nnz, cnt);
    return hipGetLastError();
}

hipError_t launch_out_fill(const int32_t *src, const int32_t *dst, int64_t nnz, int32_t *cursor,
                           int2 *oarc, hipStream_t s)
{
    if (nnz <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_out_fill, dim3(grid_for(nnz, 256)), dim3(256), 0, s, src, dst, nnz,
                       cursor, oarc);
    return hipGetLastError();
}

hipError_t launch_seed(uint64_t *p1, uint64_t *p2, const int32_t *seeds, int64_t ns, int32_t W,
                       int64_t B, uint32_t *flag0, uint32_t *bm, uint32_t *sum, hipStream_t s)
{
    if (ns <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_seed, dim3(grid_for(ns * W, 256)), dim3(256), 0, s, p1, p2, seeds, ns, W,
                       B, flag0, bm, sum);
    return hipGetLastError();
}

int counter_planes_for(int64_t max_count)
{
    int bits = 1;
    while (bits < 32 && (max_count >> bits) != 0) ++bits;
    if (bits <= 2) return 2;
    if (bits <= 4) return 4;
    if (bits <= 8) return 8;
    if (bits <= 12) return 12;
    return 16;
}

template <int KIND, bool TAIL>
static hipError_t step_kind(const StepArgs &a, int L, dim3 grid, dim3 block, hipStream_t s)
{
    if (a.heavy > kBlockRow) {
        if (L != kLightPlanes) return hipErrorInvalidValue;
        if (KIND == kKindLT && a.W == 1 && block.x <= 256)
            hipLaunchKernelGGL((k_step_light<KIND, TAIL, KIND == kKindLT ? 256 : 1024>), grid, block, 0, s, a);
        else
            hipLaunchKernelGGL((k_step_light<KIND, TAIL>), grid, block, 0, s, a);
        return hipGetLastError();
    }
    switch (L) {
    case 2: hipLaunchKernelGGL((k_step<KIND, 2, TAIL>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((k_step<KIND, 4, TAIL>), grid, block, 0, s, a); break;
    case 8: hipLaunchKernelGGL((k_step<KIND, 8, TAIL>), grid, block, 0, s, a); break;
    case 12: hipLaunchKernelGGL((k_step<KIND, 12, TAIL>), grid, block, 0, s, a); break;
    case 16: hipLaunchKernelGGL((k_step<KIND, 16, TAIL>), grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

static hipError_t step_part(const StepArgs &a, int kind, int L, dim3 grid, dim3 blk, hipStream_t s)
{
    // the tail-mode row test in its own instantiation: the other kernels
    // keep their register allocation
    if (kind == kKindIC) {
        if (a.ibm != nullptr)
            hipLaunchKernelGGL((k_step<kKindIC, 1, true>), grid, blk, 0, s, a);
        else
            hipLaunchKernelGGL((k_step<kKindIC, 1>), grid, blk, 0, s, a);
        return hipGetLastError();
    }
    if (kind == kKindEpidemic && a.ibm != nullptr)
        return step_kind<kKindEpidemic, true>(a, L, grid, blk, s);
    if (kind == kKindEpidemic) return step_kind<kKindEpidemic, false>(a, L, grid, blk, s);
    if (a.ibm != nullptr) return step_kind<kKindLT, true>(a, L, grid, blk, s);
    return step_kind<kKindLT, false>(a, L, grid, blk, s);
}

hipError_t launch_step(const StepArgs &a, int kind, int L, int block, hipStream_t s)
{
    const int nblocks = step_blocks(a, block), most = most_blocks(block);
    if (nblocks <= most)
        return nblocks > 0 ? step_part(a, kind, L, dim3((unsigned)nblocks), dim3((unsigned)block), s)
                           : hipSuccess;
    StepArgs part = a;
    for (int64_t first = 0; first < nblocks; first += most) {
        part.first = (int32_t)first;
        const dim3 grid((unsigned)std::min<int64_t>(most, nblocks - first));
        const hipError_t e = step_part(part, kind, L, grid, dim3((unsigned)block), s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_tile_rows(const int32_t *ptr, const int32_t *tiles, int32_t n_tiles, int2 *rows,
                            hipStream_t s)
{
    const int most = most_blocks(256);
    for (int64_t first = 0; first < n_tiles; first += most) {
        hipLaunchKernelGGL(k_tile_rows, dim3((unsigned)std::min<int64_t>(most, n_tiles - first)),
                           dim3(256), 0, s, ptr, tiles + 2 * first, rows);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_combine(const StepArgs &a, int kind, hipStream_t s)
{
    if (a.n_heavy <= 0) return hipSuccess;
    const int rows = 4 * (64 / (a.G * std::min(64 >> a.lgG, 16)));  // of a block
    const dim3 grid((unsigned)((a.n_heavy + rows - 1) / rows)), blk(256);
#define FSG_COMBINE(K)                                                              \
    switch (a.Lp) {                                                                 \
    case 2: hipLaunchKernelGGL((k_combine<K, 2>), grid, blk, 0, s, a); break;       \
    case 4: hipLaunchKernelGGL((k_combine<K, 4>), grid, blk, 0, s, a); break;       \
    case 8: hipLaunchKernelGGL((k_combine<K, 8>), grid, blk, 0, s, a); break;       \
    case 12: hipLaunchKernelGGL((k_combine<K, 12>), grid, blk, 0, s, a); break;     \
    case 16: hipLaunchKernelGGL((k_combine<K, 16>), grid, blk, 0, s, a); break;     \
    default: return hipErrorInvalidValue;                                           \
    }
    if (kind == kKindIC) {
        hipLaunchKernelGGL((k_combine<kKindIC, 1>), grid, blk, 0, s, a);
    } else if (kind == kKindEpidemic) {
        FSG_COMBINE(kKindEpidemic)
    } else {
        FSG_COMBINE(kKindLT)
    }
#undef FSG_COMBINE
    return hipGetLastError();
}

hipError_t launch_ic_stream(const StepArgs &a, int grid, int block, hipStream_t s)
{
    if (a.nnz <= 0) return hipSuccess;
    const int64_t need = (a.nnz + 8 * (int64_t)block - 1) / (8 * (int64_t)block);
    const int64_t g = std::max<int64_t>(1, std::min<int64_t>(need, grid));
    hipLaunchKernelGGL(k_ic_stream, dim3((unsigned)g), dim3((unsigned)block), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_ic_clear(const StepArgs &a, hipStream_t s)
{
    const int64_t work = ((int64_t)a.n + 31) >> 5;
    hipLaunchKernelGGL(k_ic_clear, dim3(grid_for(work, 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_src_groups(const int32_t *src, int64_t nnz, uint16_t *grp, hipStream_t s)
{
    if (nnz <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_src_groups, dim3(grid_for(nnz, 256)), dim3(256), 0, s, src, nnz, grp);
    return hipGetLastError();
}

hipError_t launch_expand_rows(const int32_t *ptr, int64_t n, int32_t *dst, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_expand_rows, dim3(grid_for(n, 256)), dim3(256), 0, s, ptr, n, dst);
    return hipGetLastError();
}

int step_blocks(const StepArgs &a, int block)
{
    return seg_blocks_of(a.n_seg, a.n_segb, block / 64) + a.n_tiles;
}

hipError_t launch_batch_step(const BatchCtl &c, uint32_t t, int items, hipStream_t s)
{
    const int most = most_blocks(kBatchBlock);
    for (int64_t first = 0; first < items; first += most) {
        hipLaunchKernelGGL(k_batch_step, dim3((unsigned)std::min<int64_t>(most, items - first)),
                           dim3(kBatchBlock), 0, s, c, t, (int)first);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_batch_combine(const BatchCtl &c, uint32_t t, int rows, hipStream_t s)
{
    const int per = kBatchBlock / 64;
    hipLaunchKernelGGL(k_batch_combine, dim3((unsigned)((rows + per - 1) / per), (unsigned)c.n_jobs),
                       dim3(kBatchBlock), 0, s, c, t);
    return hipGetLastError();
}

hipError_t launch_batch_ring_clear(const BatchCtl &c, uint32_t t, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_ring_clear, dim3((unsigned)c.n_jobs), dim3(256), 0, s, c, t);
    return hipGetLastError();
}

hipError_t launch_batch_expand(const BatchCtl &c, uint32_t t, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_expand, dim3(1024), dim3(256), 0, s, c, t);
    return hipGetLastError();
}

hipError_t launch_batch_count(const BatchCtl &c, uint32_t t, unsigned long long *counts, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_count, dim3(2048), dim3(256), 0, s, c, t, counts);
    return hipGetLastError();
}

hipError_t launch_finalize(const FinArgs &f, hipStream_t s)
{
    // a wave per 64 words, as many as that takes: the finalize mostly writes
    // (R-MAT scale 26 at B = 64: 0.771 ms with 262,144 blocks, 0.82 with
    // the 65,536 of two 64-word blocks a wave, 0.85 with 16,384)
    const int64_t waves = ((int64_t)f.n * f.G + 63) / 64;
    int64_t blocks = (waves + 3) / 4;
    if (blocks < 1) blocks = 1;
    if (blocks > (1 << 22)) blocks = 1 << 22;
    const bool dense = f.G == f.W && f.B == 64ll * f.W &&
                       ((uintptr_t)f.states & 15u) == 0;
    if (dense) {
        hipLaunchKernelGGL(k_finalize_dense, dim3((unsigned)blocks), dim3(256), 0, s, f);
        return hipGetLastError();
    }
    FinArgs rest = f;
    const int64_t flat = ((int64_t)f.n * f.B + 4 * kFlatKb * 1024 - 1) / (4 * kFlatKb * 1024);
    if (f.states && ((uintptr_t)f.states & 15u) == 0 && flat <= INT32_MAX) {
        hipLaunchKernelGGL(k_finalize_flat, dim3((unsigned)flat), dim3(256), 0, s, f);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        rest.states = nullptr;
    }
    if (rest.states || rest.counts || rest.scrub)  // (the scrub clears what the flat pass read)
        hipLaunchKernelGGL(k_finalize, dim3((unsigned)blocks), dim3(256), 0, s, rest);
    return hipGetLastError();
}

hipError_t launch_tally(const FinArgs &f, hipStream_t s)
{
    // two passes a wave or more, at most 512 blocks of four waves
    const int64_t passes = f.W <= 64 ? (int64_t)f.n / (64 / f.W) + 1 : (int64_t)f.n;
    const unsigned g = (unsigned)std::min<int64_t>(512, passes / 8 + 1);
    hipLaunchKernelGGL(k_tally, dim3(g), dim3(256), 0, s, f);
    return hipGetLastError();
}

hipError_t launch_philox(const uint32_t *ctr, uint32_t k0, uint32_t k1, uint32_t *out,
                         int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_philox, dim3(grid_for(count, 256)), dim3(256), 0, s, ctr, k0, k1, out,
                       count);
    return hipGetLastError();
}

}  // namespace fsg
