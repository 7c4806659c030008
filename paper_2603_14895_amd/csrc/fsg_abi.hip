// fsg_abi.hip -- host side of libfsg: argument validation, FP64 threshold
// tables, the row-tile planner, workspace layout and the step loop.
// Declarations and contracts: include/fsg.h.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <functional>
#include <fstream>
#include <sstream>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/fsg.h"
#include "fsg_internal.hpp"

using namespace fsg;

namespace {

thread_local std::string g_err = "no error";

int fail(int code, const std::string &msg)
{
    g_err = msg;
    return code;
}

#define HIP_TRY(expr)                                                                       \
    do {                                                                                    \
        if (fsg::inject_device_fault())                                                     \
            return fail(FSG_EDEVICE, std::string(#expr) + ": injected fault");              \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess)                                                               \
            return fail(FSG_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_));    \
    } while (0)

// FSG_FAULT_INJECT: the call numbers at which a guarded allocation or a
// checked HIP call fails (0: never), parsed on first use.
struct FaultPlan {
    long alloc_at = 0, device_at = 0;
    std::atomic<long> allocs{0}, devices{0};
    FaultPlan()
    {
        const char *env = getenv("FSG_FAULT_INJECT");
        if (!env) return;
        std::string spec(env);
        size_t pos = 0;
        while (pos <= spec.size()) {
            size_t end = spec.find(',', pos);
            if (end == std::string::npos) end = spec.size();
            const std::string item = spec.substr(pos, end - pos);
            const size_t c = item.find(':');
            if (c != std::string::npos) {
                const long at = atol(item.c_str() + c + 1);
                if (item.compare(0, c, "alloc") == 0) alloc_at = at;
                if (item.compare(0, c, "device") == 0) device_at = at;
            }
            pos = end + 1;
        }
    }
};

FaultPlan &fault_plan()
{
    static FaultPlan plan;
    return plan;
}

// Probability -> uint32 threshold (the Bernoulli fires iff t == 2^32-1 or
// draw < t).  Scaling by 2^32 is exact in FP64.
uint32_t threshold_of(double p)
{
    if (!(p > 0.0)) return 0u;
    if (p >= 1.0) return 0xFFFFFFFFu;
    double x = floor(p * 4294967296.0);
    return x > 4294967294.0 ? 0xFFFFFFFEu : (uint32_t)x;
}

// Appendix A.1: with k infected in-neighbours the infection probability is
// 1 - exp(k log(1-beta)) = 1 - (1-beta)^k.  The survival power is built by
// repeated FP64 multiplication; the table stops where it saturates.
std::vector<uint32_t> infection_table(double beta, int64_t max_k)
{
    std::vector<uint32_t> t;
    t.reserve((size_t)std::min<int64_t>(max_k + 1, 1 << 16));
    volatile double surv = 1.0;
    for (int64_t k = 0; k <= max_k; ++k) {
        if (k > 0) surv = surv * (1.0 - beta);
        const uint32_t x = threshold_of(1.0 - surv);
        t.push_back(x);
        if (x == 0xFFFFFFFFu) break;  // every later entry is "always" too
    }
    return t;
}

bool bad_prob(double p) { return !(p >= 0.0 && p <= 1.0); }

int64_t next_pow2(int64_t x)
{
    int64_t p = 1;
    while (p < x) p <<= 1;
    return p;
}

int ilog2(int64_t x)
{
    int l = 0;
    while ((1ll << l) < x) ++l;
    return l;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Largest arc count: arc indices are int32 in the kernels.  The 256 below 2^31
// are for the loops that count in int32 and step by up to 256 from an arc of a
// row (lanes past a row's end); the walks that look further count in uint32
// (walk_arcs, any_arcs).
constexpr int64_t kMaxNnz = ((int64_t)1 << 31) - 256;

struct Plan {
    std::vector<int32_t> tiles;      // (row_begin, row_end) pairs; light rows only
    std::vector<int32_t> heavy_rows; // rows of several segments
    std::vector<int32_t> heavy_seg;  // [n_heavy + 1] first segment of each heavy row
    std::vector<int32_t> seg_heavy;  // the heavy row of each of their segments
    // segments of the heavy rows, then the other rows above `cut` in-arcs,
    // longest first, as one segment each
    std::vector<int32_t> seg_row, seg_e0, seg_e1;
    int64_t n_segb = 0;              // segments that take a block each (the first ones)
    int64_t cut = 0;                 // most in-arcs of a light row
    int64_t max_light = 0;           // largest light in-degree
    int64_t max_seg = 0;             // longest segment
};

}  // namespace

struct fsg_graph {
    int64_t n = 0, nnz = 0, max_indeg = 0;
    int64_t mid = 0, mid_arcs = 0;  // rows of kBlockRow + 1 .. kLightMost in-arcs, and those arcs
    std::vector<int64_t> ptr;
    const int32_t *src_host = nullptr;
    bool bound = false;
    int32_t *d_ptr = nullptr;
    int32_t *d_src = nullptr;
    int32_t *d_dst = nullptr;  // target row of every arc (built on the device at bind)
    std::vector<int32_t> wide;  // rows with more than kWideRow in-arcs, largest first
    int64_t wide_arcs = 0;      // their arcs
    int32_t *d_wide = nullptr;
    std::vector<int32_t> order;  // the other rows by decreasing in-degree
    int32_t *d_order = nullptr;
    uint16_t *d_grp = nullptr;  // group of every arc's source (built on the device at bind)
    // out-adjacency (fsg_graph_bind_out): arcs grouped by source
    bool has_out = false;
    int32_t *d_optr = nullptr;
    int2 *d_oarc = nullptr;
    int64_t out_items = 0;  // sum over nodes of max(1, ceil(outdeg / kOutChunk))
    // plans made so far; runs of one graph on several threads share them (an
    // entry stays where it is once it is there)
    std::map<std::tuple<int64_t, int64_t, bool, bool>, Plan> plans;
    std::mutex plans_mu;
};

namespace fsg {

int set_error(int code, const char *msg) { return fail(code, msg); }

void inject_alloc_fault()
{
    FaultPlan &f = fault_plan();
    if (f.alloc_at > 0 && f.allocs.fetch_add(1) + 1 == f.alloc_at) throw std::bad_alloc();
}

bool inject_device_fault()
{
    FaultPlan &f = fault_plan();
    return f.device_at > 0 && f.devices.fetch_add(1) + 1 == f.device_at;
}

bool graph_view(const fsg_graph *g, int64_t *n, int64_t *nnz, int64_t *max_indeg,
                const int32_t **ptr, const int32_t **src, const int32_t **wide, int64_t *n_wide,
                const int32_t **order, int64_t *wide_arcs)
{
    if (!g || !g->bound) return false;
    *wide = g->d_wide;
    *order = g->d_order;
    *n_wide = (int64_t)g->wide.size();
    *wide_arcs = g->wide_arcs;
    *n = g->n;
    *nnz = g->nnz;
    *max_indeg = g->max_indeg;
    *ptr = g->d_ptr;
    *src = g->d_src;
    return true;
}

}  // namespace fsg

// Target-node partition by prefix sums (Sec. 3.2, Definition "Target-Node-
// Based Partitioning"): node i with prefix load C_i goes to part
// ceil(d C_i / W_total); here the nodes keep their CSR order so each part is
// a contiguous row range owned by one workgroup.  Load of a row: in-degree
// (0 for heavy rows, which are processed as segments) plus row_cost.
extern "C" int fsg_plan_row_tiles(const int64_t *in_ptr, int64_t n, int64_t heavy,
                                  int64_t row_cost, int64_t n_parts, int64_t *bounds_out,
                                  int64_t *n_out)
{
    if (!in_ptr || !bounds_out || !n_out || n < 1 || n_parts < 1 || row_cost < 0)
        return fail(FSG_EINVAL, "fsg_plan_row_tiles: bad arguments");
    unsigned __int128 total = 0;
    for (int64_t v = 0; v < n; ++v) {
        const int64_t d = in_ptr[v + 1] - in_ptr[v];
        total += (unsigned __int128)((d > heavy ? 0 : d) + row_cost);
    }
    int64_t nb = 0;
    bounds_out[nb++] = 0;
    if (total == 0) {
        bounds_out[nb++] = n;
        *n_out = nb - 1;
        return FSG_OK;
    }
    unsigned __int128 c = 0;
    int64_t cur = 1;  // part of the rows seen so far
    for (int64_t v = 0; v < n; ++v) {
        const int64_t d = in_ptr[v + 1] - in_ptr[v];
        c += (unsigned __int128)((d > heavy ? 0 : d) + row_cost);
        const unsigned __int128 num = (unsigned __int128)n_parts * c;
        int64_t q = (int64_t)((num + total - 1) / total);
        if (q < 1) q = 1;
        if (q > cur) {
            // row v opens part q: close the previous one before v (if non-empty)
            if (v > bounds_out[nb - 1]) bounds_out[nb++] = v;
            cur = q;
        }
    }
    if (bounds_out[nb - 1] != n) bounds_out[nb++] = n;
    *n_out = nb - 1;
    return FSG_OK;
}

namespace {

constexpr int64_t kRowCost = 4;

// `light`: rows of up to `heavy` in-arcs are light rows.  `narrow`: a row is one or two words and its arcs are counted.
const Plan &get_plan(fsg_graph *g, int64_t heavy, int64_t tile_edges, bool light, bool narrow)
{
    std::lock_guard<std::mutex> lock(g->plans_mu);
    auto key = std::make_tuple(heavy, tile_edges, light, narrow);
    auto it = g->plans.find(key);
    if (it != g->plans.end()) return it->second;
    Plan p;
    const int64_t n = g->n;
    const int64_t *ptr = g->ptr.data();
    const int64_t cut = light ? heavy : std::min<int64_t>(heavy, kBlockRow);
    p.cut = cut;
    unsigned __int128 total = 0;
    std::vector<int32_t> single;  // rows of one segment
    for (int64_t v = 0; v < n; ++v) {
        const int64_t d = ptr[v + 1] - ptr[v];
        total += (unsigned __int128)((d > cut ? 0 : d) + kRowCost);
        if (d > heavy) {
            p.heavy_rows.push_back((int32_t)v);
            p.heavy_seg.push_back((int32_t)p.seg_row.size());
            const int64_t per = (d + (d + heavy - 1) / heavy - 1) / ((d + heavy - 1) / heavy);
            for (int64_t e = ptr[v]; e < ptr[v + 1]; e += per) {  // segments of like length
                p.seg_row.push_back((int32_t)v);
                p.seg_e0.push_back((int32_t)e);
                p.seg_e1.push_back((int32_t)std::min(ptr[v + 1], e + per));
                p.seg_heavy.push_back((int32_t)p.heavy_rows.size() - 1);
            }
        } else if (d > cut) {
            single.push_back((int32_t)v);
        } else {
            p.max_light = std::max(p.max_light, d);
        }
        if (d > cut) p.max_seg = std::max(p.max_seg, std::min(d, heavy));
    }
    if (p.max_light <= kBlockRow) p.cut = std::min<int64_t>(cut, kBlockRow);
    p.heavy_seg.push_back((int32_t)p.seg_row.size());
    std::stable_sort(single.begin(), single.end(), [&](int32_t x, int32_t y) {
        return ptr[x + 1] - ptr[x] > ptr[y + 1] - ptr[y];
    });
    // Long segments take a block, the others a wave.  A block shortens the
    // chain of a long row, which bounds the step of a small graph; a large one
    // has other blocks to run meanwhile and pays for the waves that wait (SIR,
    // 1e6 nodes, load 2.4e7: all rows above 255 arcs by block 96.0 ms a run,
    // above 1464 93.4).  And blocks are for few: the i-th longest takes one
    // while its length is well above i, since beyond a thousand or so they
    // queue, four waves for one row (40 steps of SIR over 300 replicates, all
    // by block and all by wave: 1500 rows of 2000 to 4000 arcs 1.72 and 2.89 ms,
    // 4000 of 1000 to 2000 2.62 and 2.00, 4000 of 300 1.95 and 1.07; a
    // Chung-Lu graph of 2e4 nodes of mean degree 100, 950 rows above 255, LT 1.63
    // and 2.83).  With one or two
    // words a row the wave's 64 lanes share its arcs already (1500 rows of 2000 to
    // 4000, 64 replicates: 1.26 and 0.95).  Where the lengths are alike a few
    // blocks shorten nothing: most of the rows take one or none does.
    const int64_t by_block =
        std::max<int64_t>(kBlockRow, std::min<int64_t>(2048, (g->nnz + kRowCost * n) >> 14));
    std::vector<int64_t> lens;  // of the segments above it: the heavy rows', then the single ones'
    for (size_t i = 0; i < p.seg_row.size(); ++i)
        if (p.seg_e1[i] - p.seg_e0[i] > by_block) lens.push_back(p.seg_e1[i] - p.seg_e0[i]);
    const int64_t heavy_long = (int64_t)lens.size();
    std::sort(lens.begin(), lens.end(), std::greater<int64_t>());
    for (int32_t v : single)
        if (ptr[v + 1] - ptr[v] > by_block) lens.push_back(ptr[v + 1] - ptr[v]);
    const int64_t most = (int64_t)lens.size();
    int64_t blocks = 0;
    while (blocks < most && blocks * (narrow ? 16 : 1) < lens[(size_t)blocks] - kBlockRow) ++blocks;
    std::sort(lens.begin(), lens.end(), std::greater<int64_t>());
    if (most > 0 && lens[0] < 2 * lens[(size_t)(most / 2)]) blocks = blocks * 4 >= most * 3 ? most : 0;
    // (the segments of the heavy rows come first, long or not)
    p.n_segb = blocks == 0 ? 0
               : blocks < heavy_long ? blocks
                                     : (int64_t)p.seg_row.size() + blocks - heavy_long;
    for (int32_t v : single) {
        p.seg_row.push_back(v);
        p.seg_e0.push_back((int32_t)ptr[v]);
        p.seg_e1.push_back((int32_t)ptr[v + 1]);
    }
    int64_t parts = (int64_t)((total + (unsigned __int128)tile_edges - 1) / (unsigned __int128)tile_edges);
    parts = std::max<int64_t>(1, std::min<int64_t>(parts, n));
    std::vector<int64_t> b((size_t)n + 2);
    int64_t nt = 0;
    fsg_plan_row_tiles(ptr, n, cut, kRowCost, parts, b.data(), &nt);
    // wider rows are cut out of the parts (their segments are separate work
    // items) and no tile holds more than kMaxTileRows rows
    for (int64_t i = 0; i < nt; ++i) {
        int64_t r = b[(size_t)i];
        const int64_t end = b[(size_t)i + 1];
        while (r < end) {
            while (r < end && ptr[r + 1] - ptr[r] > cut) ++r;
            int64_t q = r;
            while (q < end && q - r < kMaxTileRows && ptr[q + 1] - ptr[q] <= cut) ++q;
            if (q > r) {
                p.tiles.push_back((int32_t)r);
                p.tiles.push_back((int32_t)q);
            }
            r = q;
        }
    }
    if (p.tiles.empty()) {  // no light row: one empty tile keeps the grid valid
        p.tiles.push_back(0);
        p.tiles.push_back(0);
    }
    return g->plans.emplace(key, std::move(p)).first->second;
}

int model_kind(int model)
{
    if (model == kIC) return kKindIC;
    if (model == kLT) return kKindLT;
    return kKindEpidemic;
}

int check_params(const fsg_graph *g, const fsg_params *prm, int64_t B)
{
    if (!g) return fail(FSG_EINVAL, "graph is NULL");
    if (!prm) return fail(FSG_EINVAL, "params is NULL");
    if (prm->model < FSG_IC || prm->model > FSG_SWIR) return fail(FSG_EINVAL, "unknown model");
    if (B < 1) return fail(FSG_EINVAL, "B must be >= 1");
    if (B > (int64_t)1 << 31) return fail(FSG_EUNSUPPORTED, "B above 2^31");
    const bool swir = prm->model == FSG_SWIR;
    const bool latent = prm->model == FSG_SEIR || prm->model == FSG_SEIS || swir;
    const bool epi = prm->model == FSG_SI || prm->model == FSG_SIS || prm->model == FSG_SIR || latent;
    if (epi && !swir && prm->max_steps < 0)
        return fail(FSG_EINVAL, "SI/SIS/SIR/SEIR/SEIS need max_steps >= 0");
    if (prm->max_steps > 0x7FFFFFFF) return fail(FSG_EUNSUPPORTED, "max_steps above 2^31-1");
    if (prm->model == FSG_IC) {
        if (prm->ic_prob < FSG_IC_UNIFORM || prm->ic_prob > FSG_IC_PER_EDGE)
            return fail(FSG_EINVAL, "unknown ic_prob");
        if (prm->ic_prob == FSG_IC_UNIFORM && bad_prob(prm->p))
            return fail(FSG_EINVAL, "p must be in [0, 1]");
        if (prm->ic_prob == FSG_IC_PER_EDGE) {
            if (g->nnz > 0 && !prm->edge_p) return fail(FSG_EINVAL, "edge_p is NULL");
            for (int64_t e = 0; e < g->nnz; ++e)
                if (bad_prob(prm->edge_p[e])) return fail(FSG_EINVAL, "edge_p[e] outside [0, 1]");
        }
    }
    if (epi) {
        if (bad_prob(prm->beta)) return fail(FSG_EINVAL, "beta must be in [0, 1]");
        if (prm->model != FSG_SI && bad_prob(prm->gamma))
            return fail(FSG_EINVAL, "gamma must be in [0, 1]");
        if (latent && bad_prob(prm->alpha)) return fail(FSG_EINVAL, "alpha must be in [0, 1]");
        if (swir && !(prm->beta + prm->alpha <= 1.0))
            return fail(FSG_EINVAL, "SWIR needs beta + alpha <= 1 (kappa + mu)");
    }
    return FSG_OK;
}

struct Sched {
    int G, S, lgG, lgS, block, tile_edges, heavy, sync, timed;
    bool edge1;  // edge-parallel IC kernel (frontier bitmap and summary)
    bool push;   // frontier-driven IC: work queues, push over out-arcs or stream
    bool wide;   // 64-bit offsets in the row-group kernels even where 32-bit ones fit
    bool count;  // count the generator calls of the SI-family decisions
    bool reuse;  // the caller vouches for the workspace (FSG_OPT_REUSE_WORKSPACE)
    bool tail;   // SI family, LT, pull-step IC: tail mode allowed
    bool light;  // rows of up to kLightMost in-arcs are light (light_rows)
    bool compact; // the smallest workspace (Room::kCompact)
    bool narrow; // one or two words a row, counted
    bool rows;   // several rows share a wave: those of a tile are taken by decreasing in-degree
    bool tail_always;  // ... and taken from the second chunk on (FSG_OPT_TAIL_ALWAYS)
};

// How much work shares a launch: rows and load (arcs + kRowCost per row) of
// one job, or of all the jobs of a batch.
struct Fill {
    int64_t rows, load;
};

Fill fill_of(const fsg_graph *g) { return Fill{g->n, g->nnz + kRowCost * g->n}; }

double mean_row(const fsg_graph *g) { return (double)fill_of(g).load / (double)g->n; }

// Whether rows of kBlockRow + 1 to kLightMost in-arcs are light rows, a lane
// group of a tile each, rather than a wave's or a block's own.  In a graph
// with many of them a wave a row fills the chip several times over and repeats
// the sum over its 64 lanes and the decision's bookkeeping in each, which pays
// only where the row is long and wide.  40 steps, light and by wave, ms: SIR,
// one word, 4000 rows of 300 arcs 0.79 and 1.00, 16,000 1.37 and 2.55, of 600
// 1.86 and 2.73; two words, 8000 of 400 1.15 and 1.54; four words, 8000 of 300
// 1.26 and 1.52, of 600 1.86 and 1.79; 16 words, 8000 of 300 2.41 and 2.11.  LT
// (30 steps), 16 words, 8000 of 300 1.59 and 1.85.  Fewer than 6000 rows of
// more than two words leave room on the chip (four words, 4000 of 300: 1.10
// and 0.97), and beside many short rows they unbalance the tiles.  IC has no
// counts to sum (always a wave or block: 8000 of 300, one word 1.19 and 0.88).
bool light_rows(const fsg_graph *g, int kind, int64_t W)
{
    if (kind == kKindIC || g->mid == 0) return false;
    if (W <= 2) return g->mid * 8 >= g->n;
    const double work = (double)g->mid_arcs / (double)g->mid * (double)W;
    return g->mid * 2 >= g->n && g->mid >= 6000 && work <= (kind == kKindLT ? 4800.0 : 2400.0);
}

// The steps of a graph of a smaller load take little more than their launch:
// sorting its rows, or counting what the tail mode without the out-adjacency
// is decided by, does not pay (each is a launch of 5 us; 1e3 nodes, 1e4 arcs
// take 0.46 ms a run).
constexpr int64_t kSmallLoad = 100000;

// Lanes per row of a job of W words on a launch of `rows` rows.  G lanes go
// over the words; more lanes split the row's arcs, which shortens the chain of
// gathers a lane walks but repeats the decision's bookkeeping and, below 16
// lanes, costs rows in flight.  So the arcs are split only while the rows are
// too few to fill the chip (4096 waves of 64 lanes; the lanes a row wants
// before it stops paying depend on what a lane does per arc).  Measured on
// Chung-Lu graphs of 1.5e3 to 4e5 nodes and 1 to 48 words, 1 to 64 lanes:
// SIR at 4e5 nodes, 4 words, 40 steps: 11.0 ms with 16 lanes, 6.4 with 4; at
// 2e4 nodes 1.77 with 16, 2.6 with 4.  LT at 4e5 nodes, 2 words: 33.4 with
// 16, 16.0 with 4.  IC at 1e5 nodes, 2 words: 1.61 with 16, 1.80 with 8.
// Graphs of long rows (`row`: their mean load) keep 16 lanes for the SI family
// (32,000 rows of 400 arcs, 8 words, 40 steps: 8.8 ms with 8 lanes, 6.2 with 16).
int default_lanes(int kind, int64_t W, int64_t rows, double row)
{
    const int64_t G = std::min<int64_t>(next_pow2(W), 64);
    if (G > 16) {
        // SI-family rows of 33-48 words: three 16-lane passes fill 48 lane
        // slots where one 64-lane pass leaves up to 31 idle through the
        // draws; with too few rows for that, one pass is the shorter chain
        // (2e4 nodes, 48 words: 64 lanes 4.4 ms, 16 lanes 5.9; 1e5 nodes:
        // 15.1 and 14.3)
        if (kind == kKindEpidemic && W > 32 && W <= 48 && rows >= (1 << 16)) return 16;
        return (int)G;
    }
    int64_t want, least = G;
    if (kind == kKindIC) {
        want = 2000000;
    } else if (kind == kKindEpidemic) {
        want = row > kBlockRow ? INT64_MAX : 160000;
    } else {
        want = G >= 8 ? 1200000 : 600000;
        if (G < 8) least = 2 * G;
    }
    int64_t lanes = least;
    while (lanes < 16 && rows < want / lanes) lanes *= 2;
    return (int)lanes;
}

// Arcs per tile (a block's share of the light rows) for rows of `lanes`
// lanes on a launch of `load`.  A tile as large as the load allows amortises
// the block's set-up; small tiles give small graphs blocks enough to fill the
// chip and cut the chain of rows a wave walks.  The best size grows with the
// square root of the load, and with fewer lanes per row (more rows in flight
// per wave) with that of 16 / lanes.  Measured as above: 16 lanes, SIR of 16
// words: load 2e4: 64 to 128 arcs; 1.4e5: 128; 4.8e5: 512 (2e4 nodes, B =
// 1024, 169 steps: 16.8 ms with 4096 arcs, 6.3); 2.4e6: 512 to 1024; 2.4e7
// (1e6 nodes): 2048 to 4096.  Those are graphs of mean degree 20; with longer
// rows a tile of that size holds fewer than the block's 256 / lanes lane groups
// (`row`: mean load of a row), so where there are tiles enough (512) it holds
// one for each (40 steps of SIR, 64 replicates, rows of 150 to 240 arcs: 4000
// rows 1.15 ms without, 0.71 with it; 16,000 1.88 and 1.12).
int default_tile(int64_t load, double row, int lanes, int most)
{
    const double x = std::max(sqrt((double)std::max<int64_t>(load, 1) * 16.0 / (double)lanes) / 3.0,
                              std::min(256.0 / lanes * row, (double)load / 512.0));
    int t = 64;
    while (t < most && (double)t * 1.4142135623730951 < x) t *= 2;
    return t;
}

constexpr int kMaxDefaultTile = 4096;

// Longest segment by default: a block's lane groups (256 threads, `lanes` of
// a row's words each) take at most 256 arcs of it each, and the count of a
// segment fits 12 planes.
int default_heavy(int64_t W)
{
    const int64_t G = std::min<int64_t>(next_pow2(W), 64);
    return (int)std::min<int64_t>(4095, 256 * (256 / G));
}

void default_sched(const fsg_graph *g, const fsg_params *prm, int64_t B, fsg_schedule *o)
{
    const int64_t W = (B + 63) / 64;
    const Fill f = fill_of(g);
    memset(o, 0, sizeof(*o));
    o->row_lanes = default_lanes(model_kind(prm->model), W, f.rows, mean_row(g));
    o->block_threads = 256;
    o->tile_edges = default_tile(f.load, mean_row(g), o->row_lanes, kMaxDefaultTile);
    o->heavy_threshold = default_heavy(W);
    o->steps_per_sync = 16;
    o->kernel_variant = (prm->model == FSG_IC && W == 1) ? (g && g->has_out ? 3 : 2) : 1;
    if (o->kernel_variant >= 2) {  // measured best on R-MAT scale 26 at B = 64
        o->block_threads = 512;
        o->tile_edges = 16384;
        o->heavy_threshold = 32768;
    }
    // frontier-driven steps take microseconds and go back to back; a poll
    // of the absorption flags (a host round trip with the GPU idle) costs
    // more than the early-exit launches after absorption that longer chunks
    // leave (web-scale run, 18 steps: 1.40 / 1.40 / 1.34 ms per run with
    // chunks of 8 / 16 / 32)
    if (o->kernel_variant == 3) o->steps_per_sync = 32;
}

// Workspace of a run: all of it; without the row table; or the least a run can
// do with: no row table, no wide rows of their own (rows of up to the heavy cut
// are light), merges by a launch, the largest default tiles, half the seed
// staging.  The last two are for the static scratch, where a run near its
// limit goes slower rather than not at all.
enum class Room { kAll, kNoRows, kCompact };

// Most in-arcs of a light row in kLightPlanes planes.
constexpr int kLightCount = (1 << kLightPlanes) - 1;

int resolve_sched(const fsg_graph *g, const fsg_params *prm, int64_t B, const fsg_schedule *in,
                  Sched *s, bool light_ok = true, Room room = Room::kAll)
{
    fsg_schedule d;
    default_sched(g, prm, B, &d);
    const bool compact = room == Room::kCompact;
    if (compact && d.kernel_variant < 2) {
        d.tile_edges = kMaxDefaultTile;
        d.heavy_threshold = kLightMost;
    }
    fsg_schedule u = in ? *in : d;
    if (u.row_lanes == 0) u.row_lanes = d.row_lanes;
    if (u.block_threads == 0) u.block_threads = d.block_threads;
    if (u.tile_edges == 0) u.tile_edges = d.tile_edges;
    if (u.heavy_threshold == 0) u.heavy_threshold = d.heavy_threshold;
    if (u.steps_per_sync == 0) u.steps_per_sync = d.steps_per_sync;
    if (u.kernel_variant == 0) u.kernel_variant = d.kernel_variant;
    if (u.kernel_variant < 1 || u.kernel_variant > 3)
        return fail(FSG_EINVAL, "kernel_variant must be 0, 1, 2 or 3");
    if (u.kernel_variant >= 2 && !(prm->model == FSG_IC && B <= 64))
        return fail(FSG_EINVAL, "kernel_variants 2 and 3 need IC with B <= 64");
    if (u.kernel_variant == 3 && !g->has_out)
        return fail(FSG_EINVAL, "kernel_variant 3 needs the graph's out-adjacency (fsg_graph_bind_out)");
    if (u.row_lanes < 1 || u.row_lanes > 64 || (u.row_lanes & (u.row_lanes - 1)))
        return fail(FSG_EINVAL, "row_lanes must be a power of two in [1, 64]");
    if (u.block_threads < 64 || u.block_threads > 1024 || (u.block_threads & (u.block_threads - 1)))
        return fail(FSG_EINVAL, "block_threads must be a power of two in [64, 1024]");
    if (u.tile_edges < 1) return fail(FSG_EINVAL, "tile_edges must be >= 1");
    if (u.heavy_threshold < 1 || u.heavy_threshold > 65535)
        return fail(FSG_EINVAL, "heavy_threshold must be in [1, 65535]");
    if (u.steps_per_sync < 1 || u.steps_per_sync > 4096)
        return fail(FSG_EINVAL, "steps_per_sync must be in [1, 4096]");
    const int64_t W = (B + 63) / 64;
    const int64_t G = std::min<int64_t>(u.row_lanes, std::min<int64_t>(next_pow2(W), 64));
    s->G = (int)G;
    s->S = (int)(u.row_lanes / G);
    s->lgG = ilog2(s->G);
    s->lgS = ilog2(s->S);
    s->block = u.block_threads;
    s->tile_edges = u.tile_edges;
    s->heavy = u.heavy_threshold;
    s->sync = u.steps_per_sync;
    s->timed = u.time_kernels != 0;
    s->edge1 = u.kernel_variant >= 2;
    s->push = u.kernel_variant == 3;
    if (s->push) s->block = 512;
    if (u.options & ~(FSG_OPT_WIDE_OFFSETS | FSG_OPT_COUNT_DRAWS | FSG_OPT_REUSE_WORKSPACE |
                      FSG_OPT_TAIL_OFF | FSG_OPT_TAIL_ALWAYS))
        return fail(FSG_EINVAL, "unknown schedule option bits");
    if ((u.options & FSG_OPT_TAIL_OFF) && (u.options & FSG_OPT_TAIL_ALWAYS))
        return fail(FSG_EINVAL, "FSG_OPT_TAIL_OFF and FSG_OPT_TAIL_ALWAYS together");
    s->wide = (u.options & FSG_OPT_WIDE_OFFSETS) != 0;
    s->count = (u.options & FSG_OPT_COUNT_DRAWS) != 0;
    s->reuse = (u.options & FSG_OPT_REUSE_WORKSPACE) != 0;
    // the tail mode: SI, SIS, SIR (no latent plane), LT, and IC on the pull
    // step (the edge-parallel IC steps find their frontier themselves)
    s->tail = (prm->model == FSG_SI || prm->model == FSG_SIS || prm->model == FSG_SIR ||
               prm->model == FSG_LT || (prm->model == FSG_IC && !s->edge1)) &&
              !(u.options & FSG_OPT_TAIL_OFF);
    s->tail_always = s->tail && (u.options & FSG_OPT_TAIL_ALWAYS) != 0;
    s->light = light_ok && !s->edge1 && s->heavy > kBlockRow && light_rows(g, model_kind(prm->model), W);
    if (s->light) s->heavy = std::min<int64_t>(s->heavy, kLightMost);
    s->compact = compact;
    if (compact) {
        s->light = s->heavy > kBlockRow;
        if (s->light && !s->edge1) s->heavy = std::min<int64_t>(s->heavy, kLightCount);
    }
    s->narrow = W <= 2 && model_kind(prm->model) != kKindIC;
    s->rows = !s->edge1 && !s->light && room == Room::kAll && s->G * s->S < 64 &&
              fill_of(g).load >= kSmallLoad;
    return FSG_OK;
}

struct Layout {
    size_t planes[4];
    int n_planes;
    size_t flags, wflags, tiles, heavy_rows, heavy_seg, seg_row, seg_e0, seg_e1, seg_heavy,
        heavy_done, partial, tinf, edge_t,
        seeds, bm[3], sum[3], ever, need, stamp, ibm, icount, queue[4], qctl, draws, tag, rows, total;
    int sum_words;
    int64_t W, plane_words, n_tinf, n_seed_stage;
    int L;
};

constexpr int64_t kSeedStage = 65536;

// HIP events for optional per-step timing, released on scope exit.
// Events of a timed call come from a per-thread list of released ones, so a
// run does not create and destroy its events (a timed SIR run polls 25 times,
// with 16 events a poll).  Each entry remembers its device; the list is never
// torn down (its events live until the process ends).
struct CachedEvent {
    int dev;
    hipEvent_t ev;
};
constexpr size_t kEventCacheMax = 4096;
std::vector<CachedEvent> &event_cache()
{
    thread_local std::vector<CachedEvent> *c = new std::vector<CachedEvent>();
    return *c;
}

struct EventPool {
    EventPool() = default;
    EventPool(const EventPool &) = delete;
    EventPool &operator=(const EventPool &) = delete;
    std::vector<hipEvent_t> e;
    int dev = -1;
    hipError_t init(size_t count)
    {
        release();
        hipError_t r = hipGetDevice(&dev);
        if (r != hipSuccess) return r;
        std::vector<CachedEvent> &c = event_cache();
        e.assign(count, nullptr);
        for (auto &x : e) {
            for (size_t i = c.size(); i-- > 0;)
                if (c[i].dev == dev) {
                    x = c[i].ev;
                    c[i] = c.back();
                    c.pop_back();
                    break;
                }
            if (!x) {
                r = hipEventCreate(&x);
                if (r != hipSuccess) return r;
            }
        }
        return hipSuccess;
    }
    void release()
    {
        std::vector<CachedEvent> &c = event_cache();
        for (auto x : e) {
            if (!x) continue;
            if (c.size() < kEventCacheMax)
                c.push_back({dev, x});
            else
                (void)hipEventDestroy(x);
        }
        e.clear();
    }
    ~EventPool() { release(); }
};

int layout(fsg_graph *g, const fsg_params *prm, int64_t B, const Sched &s, const Plan &p,
           Layout *L)
{
    const int kind = model_kind(prm->model);
    L->W = (B + 63) / 64;
    // one extra all-zero row (index n): gathers of padding lanes read it
    L->plane_words = (g->n + 1) * L->W;
    const bool latent = prm->model == FSG_SEIR || prm->model == FSG_SEIS || prm->model == FSG_SWIR;
    // frontier-driven IC keeps a third frontier plane (index 3)
    L->n_planes = kind == kKindLT ? 2 : ((latent || s.push) ? 4 : 3);
    L->L = kind == kKindIC ? 1 : counter_planes_for(std::max(p.max_light, p.max_seg));
    // room for the longest table (it stops early once it saturates), so the
    // workspace size does not depend on beta
    // SWIR keeps three tables (S -> I, S -> I or W, W -> I) of that length
    L->n_tinf = (kind == kKindEpidemic ? g->max_indeg + 1 : 1) * (prm->model == FSG_SWIR ? 3 : 1);
    L->n_seed_stage = std::min<int64_t>(g->n, kSeedStage);
    if (s.compact) L->n_seed_stage = (L->n_seed_stage + 1) / 2;
    size_t off = 0;
    for (int i = 0; i < L->n_planes; ++i) {
        L->planes[i] = off;
        off = align256(off + (size_t)L->plane_words * 8);
    }
    const int ring = s.sync + 1;
    L->flags = off; off = align256(off + (size_t)ring * 4);
    L->wflags = off;  // per-word flags [ring + 1][W] when 16 < W <= 64
    if (L->W > 16 && L->W <= 64) off = align256(off + (size_t)(ring + 1) * (size_t)L->W * 4);
    L->tiles = off; off = align256(off + p.tiles.size() * 4);
    L->heavy_rows = off; off = align256(off + (p.heavy_rows.size() + 1) * 4);
    L->heavy_seg = off; off = align256(off + p.heavy_seg.size() * 4);
    L->seg_row = off; off = align256(off + (p.seg_row.size() + 1) * 4);
    L->seg_e0 = off; off = align256(off + (p.seg_e0.size() + 1) * 4);
    L->seg_e1 = off; off = align256(off + (p.seg_e1.size() + 1) * 4);
    L->seg_heavy = off;  // (the merge in the step)
    if (!s.compact) off = align256(off + p.seg_heavy.size() * 4);
    L->heavy_done = off;
    if (!s.compact) off = align256(off + p.heavy_rows.size() * 4);
    L->partial = off; off = align256(off + p.seg_heavy.size() * (size_t)L->L * (size_t)L->W * 8);
    L->tinf = off; off = align256(off + (size_t)L->n_tinf * 4);
    L->edge_t = off;
    if (prm->model == FSG_IC && prm->ic_prob == FSG_IC_PER_EDGE)
        off = align256(off + (size_t)g->nnz * 4);
    L->seeds = off; off = align256(off + (size_t)L->n_seed_stage * 4);
    L->need = off;
    if (kind == kKindLT)  // bit-sliced thresholds [n][L][W]
        off = align256(off + (size_t)g->n * (size_t)L->L * (size_t)L->W * 8);
    L->stamp = off;
    if (kind == kKindLT) off = align256(off + (size_t)g->n * 8);  // gain steps, two arrays
    L->ibm = off;  // tail mode: four infected-node (IC, LT: new-activation) and two candidate bitmaps
    if (s.tail) off = align256(off + 6 * (size_t)((g->n + 31) / 32) * 4);
    L->icount = off;  // nodes with an infected replicate (tail-mode decisions)
    if (s.tail) off = align256(off + 8);
    for (int i = 0; i < 3; ++i) L->bm[i] = L->sum[i] = 0;
    for (int i = 0; i < 4; ++i) L->queue[i] = 0;
    L->qctl = 0;
    L->sum_words = 0;
    if (s.edge1) {
        const int nbuf = s.push ? 3 : 2;
        const size_t bmb = (size_t)((g->n + 31) / 32) * 4;
        for (int i = 0; i < nbuf; ++i) {
            L->bm[i] = off;
            off = align256(off + bmb);
        }
        L->sum_words = (int)std::min<int64_t>(kSumWords, (g->n + 31) / 32);
        for (int i = 0; i < nbuf; ++i) {
            L->sum[i] = off;
            off = align256(off + (size_t)L->sum_words * 4);
        }
    }
    L->ever = off;  // frontier-driven IC: bit per node ever in a frontier
    if (s.push) off = align256(off + (size_t)((g->n + 31) / 32) * 4);
    L->draws = off;  // generator-call counter (counting runs)
    off = align256(off + 8);
    if (s.push) {  // four queues of 16-byte items; counters: uint32 [4], uint64 [4]
        for (int i = 0; i < 4; ++i) {
            L->queue[i] = off;
            off = align256(off + (size_t)std::max<int64_t>(g->out_items, 1) * 16);
        }
        L->qctl = off;
        off = align256(off + 64);
    }
    L->tag = off;  // frontier-driven IC: which layout last left its buffers clear
    if (s.push) off = align256(off + 8);
    L->rows = off;  // the tiles' rows by decreasing in-degree
    if (s.rows) off = align256(off + (size_t)g->n * 8);
    L->total = off;
    return FSG_OK;
}

}  // namespace

namespace {

int validate_run(fsg_graph *g, const fsg_params *prm, const int32_t *seeds, int64_t n_seeds,
                 int64_t B, int64_t replicate_offset)
{
    int rc = check_params(g, prm, B);
    if (rc) return rc;
    if (!g->bound) return fail(FSG_EINVAL, "graph is not bound to device memory");
    if (replicate_offset < 0 || replicate_offset + B > ((int64_t)1 << 34))
        return fail(FSG_EINVAL, "replicate_offset + B must lie in [0, 2^34]");
    if (n_seeds < 0 || (n_seeds > 0 && !seeds)) return fail(FSG_EINVAL, "bad seed array");
    for (int64_t i = 0; i < n_seeds; ++i)
        if (seeds[i] < 0 || (int64_t)seeds[i] >= g->n)
            return fail(FSG_EINVAL, "seed out of range at index " + std::to_string(i));
    return FSG_OK;
}

// Tag a frontier-driven IC run writes into its workspace once it has left
// its planes, bitmaps and summaries clear: a hash of the layout, the graph,
// the parameters and the workspace address, never 0 (the value a run in
// progress leaves there).
uint64_t clean_tag(const fsg_graph *g, const fsg_params *prm, int64_t B, const struct Layout &L,
                   const char *base)
{
    uint64_t h = 0x6A09E667F3BCC908ull;
    auto mix = [&](uint64_t x) {
        h ^= x + 0x9E3779B97F4A7C15ull + (h << 6) + (h >> 2);
        h *= 0xBF58476D1CE4E5B9ull;
        h ^= h >> 31;
    };
    mix((uint64_t)(uintptr_t)base);
    mix((uint64_t)g->n);
    mix((uint64_t)g->nnz);
    mix((uint64_t)B);
    mix((uint64_t)prm->model);
    mix((uint64_t)L.total);
    mix((uint64_t)L.planes[0]);
    mix((uint64_t)L.bm[0]);
    mix((uint64_t)L.tag);
    return h ? h : 1ull;
}

// One job on the device: its planes, tables and launch arguments.
struct Job {
    StepArgs a;
    Layout L;
    Sched s;
    int kind = 0;
    int ring = 0;
    int64_t K = 0;
    int64_t n = 0;
    int64_t B = 0;
    int model = 0;
    uint64_t *pl[4] = {nullptr, nullptr, nullptr, nullptr};
    uint32_t *bm[3] = {nullptr, nullptr, nullptr};
    uint32_t *sum[3] = {nullptr, nullptr, nullptr};
    uint4 *queue[4] = {nullptr, nullptr, nullptr, nullptr};
    std::vector<uint32_t> tinf_h, edge_t_h;  // host tables the set-up uploads
    uint32_t *ever = nullptr;                // frontier-driven IC: ever-in-a-frontier bitmap
    uint32_t *ibm = nullptr;                 // tail mode: infected-node and candidate bitmaps
    bool tail = false;                       // the tail mode can be taken
    bool tail_out = false;                   // ... with the out-adjacency
    unsigned long long *icount = nullptr;    // tail mode: nodes infected (IC, LT: newly activated)
    uint64_t *tag = nullptr;                 // frontier-driven IC: clean-buffers tag
    uint64_t tag_value = 0;                  // the tag this job's layout writes
    // frontier plane (state 1) and its bitmap after step t: the planes
    // alternate, or rotate over three in the frontier-driven IC path
    static int mod3(int64_t t) { return (int)(((t % 3) + 3) % 3); }
    uint64_t *front(int64_t t) const
    {
        return s.push ? pl[mod3(t) == 2 ? 3 : mod3(t)] : pl[t & 1];
    }
    uint32_t *front_bm(int64_t t) const
    {
        return s.edge1 ? (s.push ? bm[mod3(t)] : bm[t & 1]) : nullptr;
    }
    uint32_t *front_sum(int64_t t) const { return s.push ? sum[mod3(t)] : sum[t & 1]; }
};

// Uploads the job's tables into `base`, clears its planes and seeds them
// (every replicate starts with the seeds in state 1).  `flags` is the job's
// absorption ring.  Returns after the stream has drained.
int setup_job(fsg_graph *g, const fsg_params *prm, const int32_t *seeds, int64_t n_seeds,
              int64_t B, int64_t replicate_offset, uint64_t rng_key, const Sched &s,
              const Plan &p, const Layout &L, char *base, uint32_t *flags, hipStream_t st,
              Job *jb)
{
    const int kind = model_kind(prm->model);
    jb->L = L;
    jb->s = s;
    jb->kind = kind;
    jb->ring = s.sync + 1;
    jb->K = prm->max_steps < 0 ? g->n : prm->max_steps;
    jb->n = g->n;
    jb->B = B;
    jb->model = prm->model;
    // plane roles: IC {F0, F1, A}; epidemic {h0, h1, r}, SEIR / SEIS also
    // the latent plane e; LT {act0, act1}
    for (int i = 0; i < 4; ++i)
        jb->pl[i] = i < L.n_planes ? (uint64_t *)(base + L.planes[i]) : nullptr;
    const int ring = jb->ring;

    // host tables stay in the job until the run ends: the copies below are
    // not waited for
    std::vector<uint32_t> &tinf = jb->tinf_h;
    tinf.assign(1, 0u);
    if (kind == kKindEpidemic) tinf = infection_table(prm->beta, g->max_indeg);
    // SWIR: kappa = beta (S -> I), mu = alpha (S -> W), nu = gamma (W -> I);
    // S -> I or W with 1 - (1 - kappa - mu)^k, the sum formed in FP64
    const bool swir = prm->model == FSG_SWIR;
    const size_t n_si = tinf.size();
    size_t n_siw = 0, n_wi = 0;
    if (swir) {
        const std::vector<uint32_t> siw = infection_table(prm->beta + prm->alpha, g->max_indeg);
        const std::vector<uint32_t> wi = infection_table(prm->gamma, g->max_indeg);
        n_siw = siw.size();
        n_wi = wi.size();
        tinf.insert(tinf.end(), siw.begin(), siw.end());
        tinf.insert(tinf.end(), wi.begin(), wi.end());
    }
    std::vector<uint32_t> &edge_t = jb->edge_t_h;
    edge_t.clear();
    if (prm->model == FSG_IC && prm->ic_prob == FSG_IC_PER_EDGE) {
        edge_t.resize((size_t)g->nnz);
        for (int64_t e = 0; e < g->nnz; ++e) edge_t[(size_t)e] = threshold_of(prm->edge_p[e]);
    }
    auto up = [&](size_t off, const void *src, size_t bytes) -> hipError_t {
        if (bytes == 0) return hipSuccess;
        return hipMemcpyAsync(base + off, src, bytes, hipMemcpyHostToDevice, st);
    };
    if (!s.push) {  // the frontier-driven IC step reads no row tiles, segments or tables
        HIP_TRY(up(L.tiles, p.tiles.data(), p.tiles.size() * 4));
        if (s.rows)
            HIP_TRY(launch_tile_rows(g->d_ptr, (const int32_t *)(base + L.tiles),
                                     (int32_t)(p.tiles.size() / 2), (int2 *)(base + L.rows), st));
        HIP_TRY(up(L.heavy_rows, p.heavy_rows.data(), p.heavy_rows.size() * 4));
        HIP_TRY(up(L.heavy_seg, p.heavy_seg.data(), p.heavy_seg.size() * 4));
        HIP_TRY(up(L.seg_row, p.seg_row.data(), p.seg_row.size() * 4));
        HIP_TRY(up(L.seg_e0, p.seg_e0.data(), p.seg_e0.size() * 4));
        HIP_TRY(up(L.seg_e1, p.seg_e1.data(), p.seg_e1.size() * 4));
        if (!s.compact) {
            HIP_TRY(up(L.seg_heavy, p.seg_heavy.data(), p.seg_heavy.size() * 4));
            HIP_TRY(launch_fill32((uint32_t *)(base + L.heavy_done), (int64_t)p.heavy_rows.size(), 0u, st));
        }
        HIP_TRY(up(L.tinf, tinf.data(), tinf.size() * 4));
    }
    HIP_TRY(up(L.edge_t, edge_t.data(), edge_t.size() * 4));

    // the planes lie back to back (256-byte aligned): one zeroing launch.
    // A frontier-driven IC run clears what it wrote before it ends; with
    // FSG_OPT_REUSE_WORKSPACE the planes, bitmaps and summaries are cleared
    // only if the tag of this layout is not in the workspace.
    const size_t plane_bytes = L.planes[L.n_planes - 1] + (size_t)L.plane_words * 8 - L.planes[0];
    if (s.push) {
        jb->tag = (uint64_t *)(base + L.tag);
        jb->ever = (uint32_t *)(base + L.ever);
        jb->tag_value = clean_tag(g, prm, B, L, base);
        const size_t bm_bytes = align256(L.ever + (size_t)((g->n + 31) / 32) * 4) - L.bm[0];
        if (s.reuse) {
            HIP_TRY(launch_zero_unless(base + L.planes[0], align256(plane_bytes), jb->tag,
                                       jb->tag_value, st));
            HIP_TRY(launch_zero_unless(base + L.bm[0], bm_bytes, jb->tag, jb->tag_value, st));
        } else {
            HIP_TRY(launch_zero(base + L.planes[0], plane_bytes, st));
            HIP_TRY(launch_zero(base + L.bm[0], bm_bytes, st));
        }
        HIP_TRY(launch_fill64(jb->tag, 1, 0ull, st));  // dirty until the run has cleared up
    } else {
        HIP_TRY(launch_zero(base + L.planes[0], plane_bytes, st));
    }
    HIP_TRY(launch_fill32(flags, ring, 0u, st));
    uint32_t *wflags = (L.W > 16 && L.W <= 64) ? (uint32_t *)(base + L.wflags) : nullptr;
    if (wflags) {  // every word is live before step 1 (slot 0); the others clear
        HIP_TRY(launch_fill32(wflags, L.W, 1u, st));
        HIP_TRY(launch_fill32(wflags + L.W, (int64_t)ring * L.W, 0u, st));
    }
    if (s.edge1) {
        for (int i = 0; i < (s.push ? 3 : 2); ++i) {
            jb->bm[i] = (uint32_t *)(base + L.bm[i]);
            jb->sum[i] = (uint32_t *)(base + L.sum[i]);
            if (s.push) continue;  // cleared above with the planes
            HIP_TRY(launch_fill32(jb->bm[i], (g->n + 31) / 32, 0u, st));
            HIP_TRY(launch_fill32(jb->sum[i], L.sum_words, 0u, st));
        }
    }
    uint32_t *qcnt = nullptr;
    unsigned long long *qarcs = nullptr;
    if (s.push) {
        for (int i = 0; i < 4; ++i) jb->queue[i] = (uint4 *)(base + L.queue[i]);
        qcnt = (uint32_t *)(base + L.qctl);
        qarcs = (unsigned long long *)(base + L.qctl + 32);
        HIP_TRY(launch_fill32(qcnt, 16, 0u, st));  // counters and arc sums of the four queues
    }
    StepArgs sq;  // seeds join the frontier of step 0 (queue 0)
    memset(&sq, 0, sizeof(sq));
    if (s.push) {
        sq.ever = jb->ever;
        sq.bm_next = jb->bm[0];
        sq.sum_next = jb->sum[0];
        sq.optr = g->d_optr;
        sq.q_out = jb->queue[0];
        sq.qcnt = qcnt;
        sq.qarcs = qarcs;
        sq.qi_out = 0;
    }
    int32_t *dseeds = (int32_t *)(base + L.seeds);
    if (kind == kKindLT) HIP_TRY(launch_fill32((uint32_t *)(base + L.stamp), 2 * g->n, 0xFFFFFFFFu, st));
    if (s.tail) {
        jb->ibm = (uint32_t *)(base + L.ibm);
        jb->icount = (unsigned long long *)(base + L.icount);
    }
    // candidates come from the out-adjacency, or from the rows' sources (not
    // where the rows are long: hardly any is without a new source then, and
    // the look at them costs what the gather does)
    jb->tail_out = s.tail && g->has_out;
    jb->tail = jb->tail_out ||
               (s.tail && (s.tail_always ||
                           (fill_of(g).load >= kSmallLoad && mean_row(g) <= kBlockRow)));
    for (int64_t i0 = 0; i0 < n_seeds; i0 += L.n_seed_stage) {
        const int64_t cnt = std::min<int64_t>(L.n_seed_stage, n_seeds - i0);
        HIP_TRY(hipMemcpyAsync(dseeds, seeds + i0, (size_t)cnt * 4, hipMemcpyHostToDevice, st));
        uint64_t *second = kind == kKindIC ? jb->pl[2] : nullptr;  // IC: A too
        if (kind == kKindLT) HIP_TRY(launch_stamp_seeds((uint32_t *)(base + L.stamp), dseeds, cnt, st));
        if (s.push) HIP_TRY(launch_seed_queue(sq, dseeds, cnt, st));
        HIP_TRY(launch_seed(jb->pl[0], second, dseeds, cnt, (int32_t)L.W, B, flags, jb->bm[0],
                            jb->sum[0], st));
        // the staging array is reused by the next chunk of seeds
        if (i0 + cnt < n_seeds) HIP_TRY(hipStreamSynchronize(st));
    }

    StepArgs &a = jb->a;
    memset(&a, 0, sizeof(a));
    a.ptr = g->d_ptr;
    a.src = g->d_src;
    a.n = (int32_t)g->n;
    a.W = (int32_t)L.W;
    a.B = B;
    a.goff = (uint64_t)replicate_offset;
    a.key0 = (uint32_t)rng_key;
    a.key1 = (uint32_t)(rng_key >> 32);
    a.prev = jb->pl[0];
    a.next = jb->pl[1];
    a.aux = jb->pl[2];
    a.model = prm->model;
    a.ic_prob = prm->ic_prob;
    a.ic_t = threshold_of(prm->p);
    a.edge_t = edge_t.empty() ? nullptr : (const uint32_t *)(base + L.edge_t);
    a.tinf = (const uint32_t *)(base + L.tinf);
    a.khat = (int32_t)n_si - 1;
    a.tsiw = swir ? a.tinf + n_si : nullptr;
    a.twi = swir ? a.tinf + n_si + n_siw : nullptr;
    a.khat_siw = swir ? (int32_t)n_siw - 1 : 0;
    a.khat_wi = swir ? (int32_t)n_wi - 1 : 0;
    a.trec = prm->model == FSG_SI ? 0u : threshold_of(prm->gamma);
    const bool latent = prm->model == FSG_SEIR || prm->model == FSG_SEIS || swir;
    a.talpha = (latent && !swir) ? threshold_of(prm->alpha) : 0u;
    a.lat = latent ? jb->pl[3] : nullptr;
    a.G = s.G;
    a.S = s.S;
    a.lgG = s.lgG;
    a.lgS = s.lgS;
    a.heavy = (int32_t)p.cut;
    a.fast32 = (!s.wide && g->n + 1 < (1 << 24) && L.W < (1 << 21) &&
                (g->n + 1) * L.W < (1 << 29) && g->nnz < (1 << 30)) ? 1 : 0;
    a.tiles = (const int32_t *)(base + L.tiles);
    a.n_tiles = (int32_t)(p.tiles.size() / 2);
    a.rows = s.rows ? (const int2 *)(base + L.rows) : nullptr;
    a.seg_row = (const int32_t *)(base + L.seg_row);
    a.seg_e0 = (const int32_t *)(base + L.seg_e0);
    a.seg_e1 = (const int32_t *)(base + L.seg_e1);
    a.n_seg = (int32_t)p.seg_row.size();
    a.n_segb = (int32_t)p.n_segb;
    a.heavy_rows = (const int32_t *)(base + L.heavy_rows);
    a.heavy_seg = (const int32_t *)(base + L.heavy_seg);
    a.n_heavy = (int32_t)p.heavy_rows.size();
    a.seg_heavy = (const int32_t *)(base + L.seg_heavy);
    const bool merged = !s.light && !s.compact && (int64_t)p.seg_heavy.size() <= kMergeSegs &&
                        (kind == kKindIC || g->max_indeg <= kMergeRow);
    a.heavy_done = merged ? (uint32_t *)(base + L.heavy_done) : nullptr;
    a.partial = (uint64_t *)(base + L.partial);
    a.Lp = L.L;
    a.flags = flags;
    a.ring = ring;
    a.wflags = wflags;
    a.wring = ring + 1;
    a.dst = g->d_dst;
    a.grp = g->d_grp;
    a.nnz = g->nnz;
    a.sum_words = L.sum_words;
    a.need = nullptr;
    a.stamp = kind == kKindLT ? (uint32_t *)(base + L.stamp) : nullptr;
    a.draws = nullptr;
    if (s.count) {
        a.draws = (unsigned long long *)(base + L.draws);
        HIP_TRY(launch_fill64((uint64_t *)a.draws, 1, 0ull, st));
    }
    if (jb->tail_out) {
        a.optr = g->d_optr;
        a.oarc = g->d_oarc;
    }
    if (s.push) {
        a.ever = jb->ever;
        a.optr = g->d_optr;
        a.oarc = g->d_oarc;
        a.qcnt = qcnt;
        a.qarcs = qarcs;
        // push while the frontier's out-arcs are at most 1/16 of all arcs:
        // a pushed arc costs a random read of its target's word and more
        // address traffic than a streamed source (4 bytes)
        a.push_limit = (unsigned long long)(g->nnz / 16);
    }
    if (kind == kKindLT && g->n > 0) {
        a.need = (uint64_t *)(base + L.need);
        HIP_TRY(launch_lt_need(a, st));
        HIP_TRY(hipStreamSynchronize(st));
    }
    return FSG_OK;
}

// End of a frontier-driven IC run whose finalize clears the ever-active
// plane: the frontiers of the last two steps leave their buffers (every
// earlier one was cleared by the step two after it), then the tag records
// that the run left its buffers clear.  Enqueued only.
hipError_t scrub_frontiers(const Job &jb, int64_t steps_run, hipStream_t st)
{
    StepArgs a = jb.a;
    for (int64_t t = steps_run + 1; t <= steps_run + 2; ++t) {
        a.qi_clr = (int32_t)((t + 2) % 4);
        a.q_clr = jb.queue[a.qi_clr];
        a.f_clr = jb.front(t - 2);
        a.bm_clr = jb.front_bm(t - 2);
        a.sum_clr = jb.front_sum(t - 2);
        hipError_t e = launch_ic_scrub(a, st);
        if (e != hipSuccess) return e;
    }
    return launch_fill64(jb.tag, 1, jb.tag_value, st);
}

// Packed planes of the step `steps_run` -> uint8 states and counts; with
// `scrub` (frontier-driven IC, one word per node) the run's buffers are left
// clear as well.
FinArgs fin_args(const Job &jb, int64_t steps_run, uint8_t *final_states, uint32_t *counts,
                 bool scrub)
{
    FinArgs f;
    memset(&f, 0, sizeof(f));
    f.n = (int32_t)jb.n;
    f.W = (int32_t)jb.L.W;
    f.G = (int)std::min<int64_t>(next_pow2(jb.L.W), 64);
    f.lgG = ilog2(f.G);
    f.B = jb.B;
    f.model = jb.model;
    f.one = jb.front(steps_run);
    f.two = jb.kind == kKindLT ? nullptr : jb.pl[2];
    if (jb.model == FSG_SIS || jb.model == FSG_SI || jb.model == FSG_SEIS) f.two = nullptr;
    f.three = jb.kind == kKindEpidemic ? jb.pl[3] : nullptr;
    f.states = final_states;
    f.counts = counts;
    f.bm = jb.front_bm(steps_run);
    if (jb.s.push) {  // the ever-active plane is nonzero only where the bitmap says so
        f.two_bm = jb.ever;
        f.scrub = (scrub && f.W == 1) ? 1 : 0;
    }
    return f;
}

int finalize_job(const Job &jb, int64_t steps_run, uint8_t *final_states, uint32_t *counts,
                 hipStream_t st, double *ms_out = nullptr, bool scrub = false)
{
    if (!final_states && !counts) return FSG_OK;
    const FinArgs f = fin_args(jb, steps_run, final_states, counts, scrub);
    EventPool ev;
    if (ms_out) {
        HIP_TRY(ev.init(2));
        HIP_TRY(hipEventRecord(ev.e[0], st));
    }
    HIP_TRY(launch_finalize(f, st));
    if (ms_out) HIP_TRY(hipEventRecord(ev.e[1], st));
    if (f.scrub) HIP_TRY(scrub_frontiers(jb, steps_run, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (ms_out) {
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, ev.e[0], ev.e[1]));
        *ms_out = ms;
    }
    return FSG_OK;
}

// Frontier-driven IC through fsg_simulate: the finalize, the clearing of the
// last two frontiers and the tag are queued right after the run's first
// chunk of steps, before the host reads the absorption flags; on the device
// they act only if the chunk ended the run (SpecFin), so the finalize follows
// the last step without a host round trip.  When they do not act, the finalize
// has still dispatched its whole grid (65-75 us at web scale), so later
// chunks are not followed by one: a run that outlives its first chunk pays
// that once and is finalized after the host has seen its end.  `done` tells
// the caller the outputs are written.
struct SpecOut {
    uint8_t *states = nullptr;
    uint32_t *counts = nullptr;
    bool done = false;
    double ms = 0.0;  // finalize kernel time (timed schedules)
    EventPool ev;
};

SpecFin spec_of(const Job &jb, int64_t t0, int64_t c)
{
    SpecFin sp;
    memset(&sp, 0, sizeof(sp));
    sp.flags = jb.a.flags;
    sp.ring = jb.ring;
    sp.c = (int32_t)c;
    sp.t0 = t0;
    for (int i = 0; i < 3; ++i) {  // front(t) and its bitmap and summary depend on t mod 3
        sp.front3[i] = jb.front(i);
        sp.bm3[i] = jb.front_bm(i);
        sp.sum3[i] = jb.front_sum(i);
    }
    for (int i = 0; i < 4; ++i) sp.queue4[i] = jb.queue[i];
    return sp;
}

hipError_t queue_spec_finalize(const Job &jb, int64_t t0, int64_t c, SpecOut &so, hipStream_t st)
{
    const SpecFin sp = spec_of(jb, t0, c);
    FinArgs f = fin_args(jb, t0 + 1, so.states, so.counts, true);
    f.spec = sp;
    if (jb.s.timed) {
        hipError_t e = hipEventRecord(so.ev.e[0], st);
        if (e != hipSuccess) return e;
    }
    hipError_t e = launch_finalize(f, st);
    if (e != hipSuccess) return e;
    if (jb.s.timed) {
        e = hipEventRecord(so.ev.e[1], st);
        if (e != hipSuccess) return e;
    }
    e = launch_ic_scrub_spec(jb.a, sp, 1, nullptr, 0ull, st);
    if (e != hipSuccess) return e;
    return launch_ic_scrub_spec(jb.a, sp, 2, jb.tag, jb.tag_value, st);
}

// A run in progress: the job on the caller's workspace, its schedule, and
// how far it has got.
struct Session {
    Job jb;
    int edge_grid = 0;
    int push_grid = 0;      // frontier-driven IC: grid of a chunk that starts with a push
    bool push_next = true;  // ... whether it does (the frontier's arcs at the last poll)
    int64_t steps_run = 0;  // steps executed so far
    bool absorbed = false;
    double kernel_ms = 0.0;
    int64_t timed_steps = 0;
    bool tail_on = false;                    // the last chunk ran in the tail mode
    int64_t tail_steps = 0;                  // live steps run in the tail mode
    int64_t infected_rows = -1;              // nodes with an infected replicate at the last poll
    double setup_ms = 0.0, finalize_ms = 0.0;
    EventPool setup_ev;  // around the set-up, read once the stream has passed them
    int64_t philox_calls = 0;
};

int begin_session(fsg_graph *g, const fsg_params *prm, const int32_t *seeds, int64_t n_seeds,
                  int64_t B, int64_t replicate_offset, uint64_t rng_key, const fsg_schedule *sched,
                  void *dev_ws, size_t ws_bytes, hipStream_t st, Session *ss, Room room = Room::kAll)
{
    int rc = validate_run(g, prm, seeds, n_seeds, B, replicate_offset);
    if (rc) return rc;
    Sched s;
    rc = resolve_sched(g, prm, B, sched, &s, true, room);
    if (rc) return rc;
    const Plan &p = get_plan(g, s.heavy, s.tile_edges, s.light, s.narrow);
    Layout L;
    layout(g, prm, B, s, p, &L);
    if (!dev_ws || ws_bytes < L.total)
        return fail(FSG_EWORKSPACE, "simulation workspace too small");
    if (((uintptr_t)dev_ws & 255) != 0) return fail(FSG_EWORKSPACE, "workspace not 256-byte aligned");
    char *base = (char *)dev_ws;
    // timing events are read after the next synchronisation (run_steps)
    EventPool &ev = ss->setup_ev;
    if (s.timed) {
        HIP_TRY(ev.init(2));
        HIP_TRY(hipEventRecord(ev.e[0], st));
    }
    rc = setup_job(g, prm, seeds, n_seeds, B, replicate_offset, rng_key, s, p, L, base,
                   (uint32_t *)(base + L.flags), st, &ss->jb);
    if (rc) return rc;
    ss->setup_ms = 0.0;
    ss->finalize_ms = 0.0;
    if (s.timed) HIP_TRY(hipEventRecord(ev.e[1], st));
    ss->edge_grid = 0;
    if (s.edge1) {
        int dev = 0, ncu = 0;
        HIP_TRY(hipGetDevice(&dev));
        HIP_TRY(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
        // streaming: four times more blocks than fit at once, so blocks that finish early are replaced, which evens out
        // the uneven work of frontier arcs (measured best on R-MAT scale 26 at
        // B = 64).  Pushing over a small frontier, the blocks beyond one
        // resident round only add dispatch time: R-MAT scale 26, 18 pushing
        // steps and 14 steps after absorption take 0.39 ms with 16 blocks per
        // CU, 0.24 ms with 2 or 4 (the streaming step slows 8% with 4)
        ss->edge_grid = 16 * std::max(ncu, 1);
        ss->push_grid = 4 * std::max(ncu, 1);
    }
    ss->push_next = true;  // the seeds' frontier is taken to be small
    ss->steps_run = 0;
    ss->absorbed = n_seeds == 0;
    ss->kernel_ms = 0.0;
    ss->timed_steps = 0;
    return FSG_OK;
}

// Tally arguments for the state after step `step` (0: the current state,
// no absorption check).
FinArgs tally_args(const Session &ss, unsigned long long *out, uint32_t step)
{
    const Job &jb = ss.jb;
    const int64_t t = step ? (int64_t)step : ss.steps_run;
    FinArgs f;
    memset(&f, 0, sizeof(f));
    f.n = (int32_t)jb.n;
    f.W = (int32_t)jb.L.W;
    f.B = jb.B;
    f.model = jb.model;
    f.one = jb.front(t);
    f.two = jb.kind == kKindLT ? nullptr : jb.pl[2];
    if (jb.model == FSG_SIS || jb.model == FSG_SI || jb.model == FSG_SEIS) f.two = nullptr;
    f.three = jb.kind == kKindEpidemic ? jb.pl[3] : nullptr;
    f.bm = jb.front_bm(t);
    f.tally = out;
    f.flags = step ? jb.a.flags : nullptr;
    f.ring = jb.ring;
    f.step = step;
    return f;
}

// The generator-call counter of a counting run into the session.
int read_draws(Session &ss, hipStream_t st)
{
    if (!ss.jb.a.draws) return FSG_OK;
    unsigned long long calls = 0;
    HIP_TRY(hipMemcpyAsync(&calls, ss.jb.a.draws, 8, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    ss.philox_calls = (int64_t)calls;
    return FSG_OK;
}

void fill_info(const Session &ss, fsg_run_info *info)
{
    info->steps_run = ss.steps_run;
    info->absorbed = ss.absorbed ? 1 : 0;
    info->tail_steps = (int32_t)std::min<int64_t>(ss.tail_steps, INT32_MAX);
    info->step_kernel_ms = ss.kernel_ms;
    info->step_launches = ss.timed_steps;
    info->setup_ms = ss.setup_ms;
    info->finalize_ms = ss.finalize_ms;
    info->philox_calls = ss.philox_calls;
}

// Up to n_more further steps (never past the job's step cap), in chunks of
// Tail mode: taken for a chunk when the nodes holding an infected replicate
// (IC, LT: a new activation), times the mean in-degree, are at most this many
// times n (without the out-adjacency, LT at 2e5 nodes: 13.7 ms with 1, 14.0
// with 2, 14.4 with 4).
constexpr double kTailFactor = 1.0;

// The set-up time of a timed session, once the stream has passed its events.
hipError_t take_setup_time(Session &ss)
{
    if (ss.setup_ev.e.size() != 2) return hipSuccess;
    float ms = 0.f;
    hipError_t e = hipEventElapsedTime(&ms, ss.setup_ev.e[0], ss.setup_ev.e[1]);
    if (e != hipSuccess) return e;
    ss.setup_ms = ms;
    ss.setup_ev.release();
    return hipSuccess;
}

// `sync` steps with one poll of the absorption flags per chunk.  With
// dev_tally, row i receives the state tally after the i-th step of this call.
int run_steps(Session &ss, int64_t n_more, uint64_t *dev_tally, hipStream_t st,
              SpecOut *so = nullptr)
{
    Job &jb = ss.jb;
    const Sched &s = jb.s;
    StepArgs &a = jb.a;
    const int kind = jb.kind;
    const int ring = jb.ring;
    uint32_t *flags = a.flags;
    const int64_t t_begin = ss.steps_run;
    const int64_t K = std::min<int64_t>(jb.K, t_begin + n_more);
    std::vector<uint32_t> hflags((size_t)ring);
    unsigned long long hqarcs = 0ull;  // frontier-driven IC: the last frontier's out-arcs
    EventPool ev;  // a pair per step, or one pair per chunk for the frontier-driven IC step
    if (s.timed) HIP_TRY(ev.init(s.push ? 2 : 2 * (size_t)s.sync));
    int64_t t = t_begin;
    std::vector<uint32_t> htail(2);
    while (!ss.absorbed && t < K) {
        const int64_t c = std::min<int64_t>(s.sync, K - t);
        HIP_TRY(launch_ring_clear(flags, ring, (int32_t)(t % ring), st, a.wflags, a.W, a.wring, t));
        if (jb.tail) {
            // tail mode for this chunk: when few nodes hold an infected
            // replicate (a row can only change if it or an in-neighbour
            // does); the stamps of steps t and t-1 are written on entry
            const double n = (double)jb.n, deg = (double)a.nnz / std::max(n, 1.0);
            const bool want = t >= 1 && (s.tail_always ||
                                         (ss.infected_rows >= 0 &&
                                          (double)ss.infected_rows * deg <= n * kTailFactor));
            a.ibm_words = (int32_t)((jb.n + 31) / 32);
            uint32_t *cand = jb.ibm + 4 * (size_t)a.ibm_words;
            if (want && !ss.tail_on) {
                if (kind == kKindLT)
                    HIP_TRY(launch_mark_gained(a.stamp, jb.ibm, cand, a.ibm_words, jb.n,
                                               (uint32_t)(t + 1), st));
                else
                    HIP_TRY(launch_mark_rows(jb.front(t), jb.front(t + 1), jb.ibm, cand, a.ibm_words,
                                             jb.n, jb.L.W, (uint32_t)(t + 1), st));
            }
            ss.tail_on = want;
            a.ibm = want ? jb.ibm : nullptr;
            a.cand = want && jb.tail_out ? cand : nullptr;
        }
        for (int64_t i = 1; i <= c; ++i) {
            const int64_t step = t + i;
            a.step = (uint32_t)step;
            a.prev = jb.front(step - 1);
            a.next = jb.front(step);
            // timed: the dominant kernel of the step alone (the pull step,
            // without the bitmap clear or a merge of its own)
            if (s.push) {
                a.bm_prev = jb.front_bm(step - 1);
                a.bm_next = jb.front_bm(step);
                a.sum_prev = jb.front_sum(step - 1);
                a.sum_next = jb.front_sum(step);
                a.f_clr = jb.front(step - 2);
                a.bm_clr = jb.front_bm(step - 2);
                a.sum_clr = jb.front_sum(step - 2);
                a.qi_in = (int32_t)((step + 3) % 4);
                a.qi_out = (int32_t)(step % 4);
                a.qi_clr = (int32_t)((step + 2) % 4);
                a.qi_rst = (int32_t)((step + 1) % 4);
                a.q_in = jb.queue[a.qi_in];
                a.q_out = jb.queue[a.qi_out];
                a.q_clr = jb.queue[a.qi_clr];
                // one kernel a step, back to back: timed per chunk (events
                // between the launches would hold each one back)
                if (s.timed && i == 1) HIP_TRY(hipEventRecord(ev.e[0], st));
                HIP_TRY(launch_ic_front(a, ss.push_next ? ss.push_grid : ss.edge_grid, s.block, st));
                if (s.timed && i == c) HIP_TRY(hipEventRecord(ev.e[1], st));
            } else if (s.edge1) {
                a.bm_prev = jb.bm[(step - 1) & 1];
                a.bm_next = jb.bm[step & 1];
                a.sum_prev = jb.sum[(step - 1) & 1];
                a.sum_next = jb.sum[step & 1];
                HIP_TRY(launch_ic_clear(a, st));
                if (s.timed) HIP_TRY(hipEventRecord(ev.e[2 * (i - 1)], st));
                HIP_TRY(launch_ic_stream(a, ss.edge_grid, s.block, st));
                if (s.timed) HIP_TRY(hipEventRecord(ev.e[2 * (i - 1) + 1], st));
            } else {
                if (s.timed) HIP_TRY(hipEventRecord(ev.e[2 * (i - 1)], st));
                if (a.cand) HIP_TRY(launch_tail_expand(a, st));
                HIP_TRY(launch_step(a, kind, jb.L.L, s.block, st));
                if (s.timed) HIP_TRY(hipEventRecord(ev.e[2 * (i - 1) + 1], st));
                if (a.heavy_done == nullptr) HIP_TRY(launch_combine(a, kind, st));
            }
            if (dev_tally) {
                FinArgs f = tally_args(ss, (unsigned long long *)dev_tally + 3 * (step - t_begin - 1),
                                       (uint32_t)step);
                HIP_TRY(launch_tally(f, st));
            }
        }
        const bool spec = so != nullptr && t == t_begin;  // the run's first chunk only
        if (spec) HIP_TRY(queue_spec_finalize(jb, t, c, *so, st));
        if (s.push)  // out-arcs of the frontier the next step starts from (queue of step t+c)
            HIP_TRY(hipMemcpyAsync(&hqarcs, a.qarcs + (t + c) % 4, 8, hipMemcpyDeviceToHost, st));
        if (jb.tail) {  // nodes with an infected replicate (LT: a new activation) after the chunk
            if (kind == kKindLT)
                HIP_TRY(launch_count_stamped(a.stamp, jb.n, (uint32_t)(t + c), jb.icount, st));
            else
                HIP_TRY(launch_count_rows(jb.front(t + c), jb.n, jb.L.W, jb.icount, st));
            HIP_TRY(hipMemcpyAsync(htail.data(), jb.icount, 8, hipMemcpyDeviceToHost, st));
        }
        HIP_TRY(hipMemcpyAsync(hflags.data(), flags, (size_t)ring * 4, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        HIP_TRY(take_setup_time(ss));
        if (jb.tail) ss.infected_rows = (int64_t)((uint64_t)htail[0] | ((uint64_t)htail[1] << 32));
        if (s.push) ss.push_next = hqarcs <= a.push_limit;
        if (s.timed && s.push) {
            float ms = 0.f;
            HIP_TRY(hipEventElapsedTime(&ms, ev.e[0], ev.e[1]));
            ss.kernel_ms += ms;
            ss.timed_steps += c;
        } else if (s.timed) {
            for (int64_t i = 1; i <= c; ++i) {
                // steps after absorption return at once; count only live ones
                if (i > 1 && hflags[(size_t)((t + i - 1) % ring)] == 0u) break;
                float ms = 0.f;
                HIP_TRY(hipEventElapsedTime(&ms, ev.e[2 * (i - 1)], ev.e[2 * (i - 1) + 1]));
                ss.kernel_ms += ms;
                ++ss.timed_steps;
            }
        }
        ss.steps_run = t + c;
        for (int64_t i = 1; i <= c; ++i)
            if (hflags[(size_t)((t + i) % ring)] == 0u) {
                ss.steps_run = t + i;
                ss.absorbed = true;
                break;
            }
        if (spec && ss.absorbed) {  // the queued finalize acted (the same first clear flag)
            so->done = true;
            if (s.timed) {
                float ms = 0.f;
                HIP_TRY(hipEventElapsedTime(&ms, so->ev.e[0], so->ev.e[1]));
                so->ms = ms;
            }
        }
        if (ss.tail_on) ss.tail_steps += ss.steps_run - t;
        t += c;
    }
    return FSG_OK;
}

}  // namespace

struct fsg_session {
    Session s;
};

namespace {

// Workspace of a run.
int sim_size(const fsg_graph *g_, const fsg_params *prm, int64_t B, const fsg_schedule *sched,
             Room room, size_t *bytes)
{
    try {
        int rc = check_params(g_, prm, B);
        if (rc) return rc;
        fsg_graph *g = const_cast<fsg_graph *>(g_);
        Sched s;
        rc = resolve_sched(g, prm, B, sched, &s, true, room);
        if (rc) return rc;
        const Plan &p = get_plan(g, s.heavy, s.tile_edges, s.light, s.narrow);
        Layout L;
        layout(g, prm, B, s, p, &L);
        *bytes = L.total;
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

int simulate(const fsg_graph *g_, const fsg_params *prm, const int32_t *seeds, int64_t n_seeds,
             int64_t B, int64_t replicate_offset, uint64_t rng_key, const fsg_schedule *sched,
             void *dev_ws, size_t ws_bytes, uint8_t *final_states, uint32_t *infected_counts,
             fsg_run_info *info, void *stream, Room room = Room::kAll)
{
    try {
        Session ss;
        int rc = begin_session(const_cast<fsg_graph *>(g_), prm, seeds, n_seeds, B,
                               replicate_offset, rng_key, sched, dev_ws, ws_bytes,
                               (hipStream_t)stream, &ss, room);
        if (rc) return rc;
        const bool scrub = ss.jb.s.push && (final_states || infected_counts);
        SpecOut so;
        if (scrub) {  // frontier-driven IC: the finalize goes in right behind the steps
            so.states = final_states;
            so.counts = infected_counts;
            if (ss.jb.s.timed) HIP_TRY(so.ev.init(2));
        }
        rc = run_steps(ss, ss.jb.K, nullptr, (hipStream_t)stream, scrub ? &so : nullptr);
        if (rc) return rc;
        if (so.done) {
            ss.finalize_ms = so.ms;
        } else {  // the run outlived its first chunk, stopped at its step cap, or has no seeds
            rc = finalize_job(ss.jb, ss.steps_run, final_states, infected_counts, (hipStream_t)stream,
                              ss.jb.s.timed ? &ss.finalize_ms : nullptr, scrub);
            if (rc) return rc;
        }
        HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
        HIP_TRY(take_setup_time(ss));
        rc = read_draws(ss, (hipStream_t)stream);
        if (rc) return rc;
        if (info) fill_info(ss, info);
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

}  // namespace


extern "C" {

int fsg_abi_version(void) { return FSG_ABI_VERSION; }

const char *fsg_last_error(void) { return g_err.c_str(); }

int fsg_graph_create(int64_t n, int64_t nnz, const int64_t *in_ptr, const int32_t *in_src,
                     fsg_graph **out)
{
    try {
        if (!out) return fail(FSG_EINVAL, "out is NULL");
        *out = nullptr;
        if (n < 1) return fail(FSG_EINVAL, "n must be >= 1");
        if (n > 0x7FFFFFFF - 1) return fail(FSG_EUNSUPPORTED, "n above 2^31-2");
        if (nnz < 0) return fail(FSG_EINVAL, "nnz must be >= 0");
        if (nnz > kMaxNnz) return fail(FSG_EUNSUPPORTED, "nnz above 2^31 - 256");
        if (!in_ptr) return fail(FSG_EINVAL, "in_ptr is NULL");
        if (nnz > 0 && !in_src) return fail(FSG_EINVAL, "in_src is NULL");
        if (in_ptr[0] != 0) return fail(FSG_EINVAL, "in_ptr[0] must be 0");
        if (in_ptr[n] != nnz) return fail(FSG_EINVAL, "in_ptr[n] must equal nnz");
        int64_t dmax = 0;
        for (int64_t v = 0; v < n; ++v) {
            const int64_t d = in_ptr[v + 1] - in_ptr[v];
            if (d < 0) return fail(FSG_EINVAL, "in_ptr must be non-decreasing");
            dmax = std::max(dmax, d);
        }
        for (int64_t e = 0; e < nnz; ++e)
            if (in_src[e] < 0 || (int64_t)in_src[e] >= n)
                return fail(FSG_EINVAL, "in_src entry out of range at edge " + std::to_string(e));
        fsg::inject_alloc_fault();
        std::unique_ptr<fsg_graph> g(new fsg_graph);
        g->n = n;
        g->nnz = nnz;
        g->max_indeg = dmax;
        g->ptr.assign(in_ptr, in_ptr + n + 1);
        for (int64_t v = 0; v < n; ++v)
            if (in_ptr[v + 1] - in_ptr[v] > kWideRow) g->wide.push_back((int32_t)v);
        // largest rows first: kernels that give each wide row its own block
        // then start the longest ones at the head of the grid
        std::stable_sort(g->wide.begin(), g->wide.end(), [&](int32_t a, int32_t b) {
            return in_ptr[a + 1] - in_ptr[a] > in_ptr[b + 1] - in_ptr[b];
        });
        // the others by decreasing in-degree (a counting sort; equal rows in
        // node order)
        std::vector<int32_t> at((size_t)kWideRow + 2, 0);
        for (int64_t v = 0; v < n; ++v) {
            const int64_t d = in_ptr[v + 1] - in_ptr[v];
            if (d > kBlockRow && d <= kLightMost) {
                ++g->mid;
                g->mid_arcs += d;
            }
            if (d > kWideRow) g->wide_arcs += d;
            if (d <= kWideRow) ++at[(size_t)(kWideRow - d) + 1];
        }
        for (size_t i = 1; i < at.size(); ++i) at[i] += at[i - 1];
        g->order.resize((size_t)n - g->wide.size());
        for (int64_t v = 0; v < n; ++v) {
            const int64_t d = in_ptr[v + 1] - in_ptr[v];
            if (d <= kWideRow) g->order[(size_t)at[(size_t)(kWideRow - d)]++] = (int32_t)v;
        }
        g->src_host = in_src;
        *out = g.release();
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    } catch (...) {
        return fail(FSG_EINVAL, "unexpected host exception");
    }
}

int fsg_graph_workspace_size(const fsg_graph *g, size_t *bytes)
{
    if (!g || !bytes) return fail(FSG_EINVAL, "NULL argument");
    // sources are padded by 16 bytes: kernels read them with 16-byte loads;
    // then the target row of every arc, the wide rows, the others by degree, and
    // the groups of the sources
    *bytes = align256((size_t)(g->n + 1) * 4) + align256((size_t)std::max<int64_t>(g->nnz, 1) * 4 + 16) +
             align256((size_t)std::max<int64_t>(g->nnz, 1) * 4) + align256((g->wide.size() + 1) * 4) +
             align256((size_t)g->n * 4) + align256((size_t)std::max<int64_t>(g->nnz, 1) * 2 + 16);
    return FSG_OK;
}

int fsg_graph_bind(fsg_graph *g, void *dev_ws, size_t ws_bytes, void *stream)
{
    try {
        if (!g) return fail(FSG_EINVAL, "graph is NULL");
        size_t need = 0;
        fsg_graph_workspace_size(g, &need);
        if (!dev_ws || ws_bytes < need) return fail(FSG_EWORKSPACE, "graph workspace too small");
        if (((uintptr_t)dev_ws & 255) != 0) return fail(FSG_EWORKSPACE, "workspace not 256-byte aligned");
        if (g->nnz > 0 && !g->src_host) return fail(FSG_EINVAL, "graph already bound; sources released");
        hipStream_t s = (hipStream_t)stream;
        char *base = (char *)dev_ws;
        int32_t *dptr = (int32_t *)base;
        int32_t *dsrc = (int32_t *)(base + align256((size_t)(g->n + 1) * 4));
        int32_t *ddst = (int32_t *)((char *)dsrc + align256((size_t)std::max<int64_t>(g->nnz, 1) * 4 + 16));
        int32_t *dwide = (int32_t *)((char *)ddst + align256((size_t)std::max<int64_t>(g->nnz, 1) * 4));
        if (!g->wide.empty())
            HIP_TRY(hipMemcpyAsync(dwide, g->wide.data(), g->wide.size() * 4, hipMemcpyHostToDevice, s));
        int32_t *dorder = (int32_t *)((char *)dwide + align256((g->wide.size() + 1) * 4));
        if (!g->order.empty())
            HIP_TRY(hipMemcpyAsync(dorder, g->order.data(), g->order.size() * 4, hipMemcpyHostToDevice, s));
        std::vector<int32_t> p32(g->ptr.begin(), g->ptr.end());
        HIP_TRY(hipMemcpyAsync(dptr, p32.data(), p32.size() * 4, hipMemcpyHostToDevice, s));
        if (g->nnz > 0)
            HIP_TRY(hipMemcpyAsync(dsrc, g->src_host, (size_t)g->nnz * 4, hipMemcpyHostToDevice, s));
        uint16_t *dgrp = (uint16_t *)((char *)dorder + align256((size_t)g->n * 4));
        if (g->nnz > 0) HIP_TRY(launch_expand_rows(dptr, g->n, ddst, s));
        if (g->nnz > 0) HIP_TRY(launch_src_groups(dsrc, g->nnz, dgrp, s));
        HIP_TRY(hipStreamSynchronize(s));
        g->d_ptr = dptr;
        g->d_src = dsrc;
        g->d_dst = ddst;
        g->d_wide = dwide;
        g->d_order = dorder;
        g->d_grp = dgrp;
        g->bound = true;
        g->src_host = nullptr;
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

namespace {
struct OutLayout {
    size_t optr, oarc, cursor, total;
};
OutLayout out_layout(const fsg_graph *g)
{
    OutLayout o;
    size_t off = 0;
    o.optr = off; off = align256(off + (size_t)(g->n + 1) * 4);
    o.oarc = off; off = align256(off + (size_t)std::max<int64_t>(g->nnz, 1) * 8);
    o.cursor = off; off = align256(off + (size_t)g->n * 4);
    o.total = off;
    return o;
}
}  // namespace

int fsg_graph_out_workspace_size(const fsg_graph *g, size_t *bytes)
{
    if (!g || !bytes) return fail(FSG_EINVAL, "NULL argument");
    *bytes = out_layout(g).total;
    return FSG_OK;
}

int fsg_graph_bind_out(fsg_graph *g, void *dev_ws, size_t ws_bytes, void *stream)
{
    try {
        if (!g) return fail(FSG_EINVAL, "graph is NULL");
        if (!g->bound) return fail(FSG_EINVAL, "graph is not bound to device memory");
        const OutLayout o = out_layout(g);
        if (!dev_ws || ws_bytes < o.total) return fail(FSG_EWORKSPACE, "out-adjacency workspace too small");
        if (((uintptr_t)dev_ws & 255) != 0) return fail(FSG_EWORKSPACE, "workspace not 256-byte aligned");
        hipStream_t s = (hipStream_t)stream;
        char *base = (char *)dev_ws;
        int32_t *optr = (int32_t *)(base + o.optr);
        int2 *oarc = (int2 *)(base + o.oarc);
        int32_t *cursor = (int32_t *)(base + o.cursor);
        const int64_t n = g->n;
        // out-degrees on the device, prefix sums on the host
        HIP_TRY(launch_fill32((uint32_t *)cursor, n, 0u, s));
        HIP_TRY(launch_out_count(g->d_src, g->nnz, cursor, s));
        std::vector<int32_t> deg((size_t)n), p32((size_t)n + 1);
        HIP_TRY(hipMemcpyAsync(deg.data(), cursor, (size_t)n * 4, hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        int64_t acc = 0, items = 0;
        for (int64_t u = 0; u < n; ++u) {
            p32[(size_t)u] = (int32_t)acc;
            acc += deg[(size_t)u];
            items += deg[(size_t)u] > kOutChunk ? (deg[(size_t)u] + kOutChunk - 1) / kOutChunk : 1;
        }
        p32[(size_t)n] = (int32_t)acc;
        if (acc != g->nnz) return fail(FSG_EDEVICE, "out-degree count does not add up to nnz");
        HIP_TRY(hipMemcpyAsync(optr, p32.data(), p32.size() * 4, hipMemcpyHostToDevice, s));
        HIP_TRY(hipMemcpyAsync(cursor, p32.data(), (size_t)n * 4, hipMemcpyHostToDevice, s));
        HIP_TRY(launch_out_fill(g->d_src, g->d_dst, g->nnz, cursor, oarc, s));
        HIP_TRY(hipStreamSynchronize(s));
        g->d_optr = optr;
        g->d_oarc = oarc;
        g->out_items = items;
        g->has_out = true;
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

int fsg_graph_stats(const fsg_graph *g, int64_t *n, int64_t *nnz, int64_t *max_indeg)
{
    if (!g) return fail(FSG_EINVAL, "graph is NULL");
    if (n) *n = g->n;
    if (nnz) *nnz = g->nnz;
    if (max_indeg) *max_indeg = g->max_indeg;
    return FSG_OK;
}

int fsg_graph_destroy(fsg_graph *g)
{
    delete g;
    return FSG_OK;
}

int fsg_default_schedule(const fsg_graph *g, const fsg_params *prm, int64_t B, fsg_schedule *out)
{
    if (!out) return fail(FSG_EINVAL, "out is NULL");
    int rc = check_params(g, prm, B);
    if (rc) return rc;
    default_sched(g, prm, B, out);
    return FSG_OK;
}

int fsg_sim_workspace_size(const fsg_graph *g, const fsg_params *prm, int64_t B,
                           const fsg_schedule *sched, size_t *bytes)
{
    if (!bytes) return fail(FSG_EINVAL, "bytes is NULL");
    return sim_size(g, prm, B, sched, Room::kAll, bytes);
}

int fsg_simulate(const fsg_graph *g, const fsg_params *prm, const int32_t *seeds, int64_t n_seeds,
                 int64_t B, int64_t replicate_offset, uint64_t rng_key, const fsg_schedule *sched,
                 void *dev_ws, size_t ws_bytes, uint8_t *final_states, uint32_t *infected_counts,
                 fsg_run_info *info, void *stream)
{
    return simulate(g, prm, seeds, n_seeds, B, replicate_offset, rng_key, sched, dev_ws, ws_bytes,
                    final_states, infected_counts, info, stream);
}

int fsg_session_begin(const fsg_graph *g, const fsg_params *prm, const int32_t *seeds,
                      int64_t n_seeds, int64_t B, int64_t replicate_offset, uint64_t rng_key,
                      const fsg_schedule *sched, void *dev_ws, size_t ws_bytes, void *stream,
                      fsg_session **out)
{
    try {
        if (!out) return fail(FSG_EINVAL, "out is NULL");
        *out = nullptr;
        std::unique_ptr<fsg_session> ss(new fsg_session);
        int rc = begin_session(const_cast<fsg_graph *>(g), prm, seeds, n_seeds, B, replicate_offset,
                               rng_key, sched, dev_ws, ws_bytes, (hipStream_t)stream, &ss->s);
        if (rc) return rc;
        *out = ss.release();
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

int fsg_session_step(fsg_session *ss, int64_t n_steps, uint64_t *dev_tally, fsg_run_info *info,
                     void *stream)
{
    try {
        if (!ss) return fail(FSG_EINVAL, "session is NULL");
        if (n_steps < 0) return fail(FSG_EINVAL, "n_steps must be >= 0");
        Session &s = ss->s;
        const hipStream_t st = (hipStream_t)stream;
        const int64_t t0 = s.steps_run;
        if (dev_tally) HIP_TRY(launch_fill64(dev_tally, 3 * n_steps, 0ull, st));
        int rc = run_steps(s, n_steps, dev_tally, st);
        if (rc) return rc;
        if (dev_tally) {
            // rows of steps that were not run (absorbed, or past max_steps)
            // repeat the final state's tally
            for (int64_t i = s.steps_run - t0; i < n_steps; ++i) {
                FinArgs f = tally_args(s, (unsigned long long *)dev_tally + 3 * i, 0u);
                HIP_TRY(launch_tally(f, st));
            }
            HIP_TRY(hipStreamSynchronize(st));
        }
        rc = read_draws(s, st);
        if (rc) return rc;
        if (info) fill_info(s, info);
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

int fsg_session_read(fsg_session *ss, uint8_t *states, uint32_t *counts, uint64_t *dev_tally,
                     void *stream)
{
    if (!ss) return fail(FSG_EINVAL, "session is NULL");
    const Session &s = ss->s;
    const hipStream_t st = (hipStream_t)stream;
    int rc = finalize_job(s.jb, s.steps_run, states, counts, st);
    if (rc) return rc;
    if (dev_tally) {
        FinArgs f = tally_args(s, (unsigned long long *)dev_tally, 0u);
        HIP_TRY(launch_fill64(dev_tally, 3, 0ull, st));
        HIP_TRY(launch_tally(f, st));
        HIP_TRY(hipStreamSynchronize(st));
    }
    return FSG_OK;
}

int fsg_session_end(fsg_session *ss)
{
    delete ss;
    return FSG_OK;
}

}  // extern "C"

// ---- fsg_simulate without a caller workspace: the workspace is a static
// device array of kScratchBytes, one per GPU, held until the process ends.
namespace {
constexpr size_t kScratchBytes = (size_t)64 << 20;
}  // namespace

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

std::mutex g_scratch_mu;
std::map<int, void *> g_scratch_at;  // device -> address of that device's copy of scratch

// Device address of the current device's copy of scratch, looked up once per
// device (the host-side name of the array is not a device address).
int scratch_address(void **out)
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    auto it = g_scratch_at.find(dev);
    if (it == g_scratch_at.end()) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || ((uintptr_t)p & 255) != 0) return fail(FSG_EDEVICE, "scratch array misplaced");
        it = g_scratch_at.emplace(dev, p).first;
    }
    *out = it->second;
    return FSG_OK;
}

}  // namespace

extern "C" {

size_t fsg_simulate_noalloc_limit(void) { return kScratchBytes; }

int fsg_simulate_noalloc(const fsg_graph *g, const fsg_params *prm, const int32_t *seeds,
                         int64_t n_seeds, int64_t B, int64_t replicate_offset, uint64_t rng_key,
                         const fsg_schedule *sched, uint8_t *final_states,
                         uint32_t *infected_counts, fsg_run_info *info, void *stream)
{
    try {
        fsg_schedule s;
        if (sched) {
            s = *sched;
        } else {
            memset(&s, 0, sizeof(s));
        }
        s.time_kernels = 0;  // no HIP events
        // as much of the workspace as the array holds; with the largest default
        // tile (the tiles of a small graph are many) before the smallest room
        size_t need = 0;
        Room room = Room::kAll;
        fsg_schedule few = s;
        if (s.tile_edges == 0 && s.kernel_variant < 2) few.tile_edges = kMaxDefaultTile;
        const struct {
            const fsg_schedule *sched;
            Room room;
        } tries[] = {{&s, Room::kAll}, {&s, Room::kNoRows}, {&few, Room::kNoRows}, {&s, Room::kCompact}};
        fsg_schedule use = s;
        for (const auto &t : tries) {
            const int rc = sim_size(g, prm, B, t.sched, t.room, &need);
            if (rc) return rc;
            use = *t.sched;
            room = t.room;
            if (need <= kScratchBytes) break;
        }
        if (need > kScratchBytes)
            return fail(FSG_EWORKSPACE, "this run needs " + std::to_string(need) +
                                            " bytes of workspace; the static scratch holds " +
                                            std::to_string(kScratchBytes));
        void *ws = nullptr;
        const int rc = scratch_address(&ws);
        if (rc) return rc;
        return simulate(g, prm, seeds, n_seeds, B, replicate_offset, rng_key, &use, ws, kScratchBytes,
                        final_states, infected_counts, info, stream, room);
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

int fsg_philox4x32_10(const uint32_t *dev_ctr, uint32_t key0, uint32_t key1, uint32_t *dev_out,
                      int64_t count, void *stream)
{
    if (count < 0 || (count > 0 && (!dev_ctr || !dev_out)))
        return fail(FSG_EINVAL, "bad philox arguments");
    HIP_TRY(launch_philox(dev_ctr, key0, key1, dev_out, count, (hipStream_t)stream));
    return FSG_OK;
}

}  // extern "C"

// ------------------------------------------------------------------ batches

struct fsg_plan {
    std::vector<fsg_job> jobs;
    std::vector<Sched> sched;
    std::vector<const Plan *> plans;
    std::vector<Layout> layouts;
    std::vector<size_t> job_off;  // workspace offset of each job
    size_t ctl_off = 0, total = 0;
    int64_t items = 0;  // blocks of a batched step
    int sync = 16;
    int blocks_per_cu = 4;  // as set; the batched kernels launch a block per work item
};

namespace {

// Largest default tile of a job in the batched launch (larger than a job's
// alone, since the other jobs already fill the GPU: the batch autotuner chose
// 8192 arcs for every model class of 64 jobs of 3.45e8 arcs).
constexpr int kMaxBatchTile = 8192;

int resolve_batch_sched(const fsg_job &j, const Fill &fill, Sched *s)
{
    fsg_schedule u = j.sched;
    if (u.kernel_variant >= 2) return fail(FSG_EINVAL, "batched jobs use kernel_variant 0 or 1");
    u.kernel_variant = 1;
    u.block_threads = kBatchBlock;
    const int64_t W = (j.B + 63) / 64;
    const int lanes =
        u.row_lanes > 0 ? u.row_lanes : default_lanes(model_kind(j.prm.model), W, fill.rows, mean_row(j.g));
    if (u.row_lanes == 0) u.row_lanes = lanes;
    if (u.tile_edges == 0) u.tile_edges = default_tile(fill.load, mean_row(j.g), lanes, kMaxBatchTile);
    if (u.heavy_threshold == 0) u.heavy_threshold = default_heavy(W);
    // (the batched kernel counts light rows in 8 planes)
    return resolve_sched(j.g, &j.prm, j.B, &u, s, /*light_ok=*/false);
}

// The jobs share the launch.
Fill batch_fill(const fsg_job *jobs, int32_t n_jobs)
{
    Fill fill{0, 0};
    for (int32_t i = 0; i < n_jobs; ++i)
        if (jobs[i].g) {
            const Fill f = fill_of(jobs[i].g);
            fill.rows += f.rows;
            fill.load += f.load;
        }
    return fill;
}

// Step blocks of a job.
int64_t batch_items(const Plan &p)
{
    return seg_blocks_of((int)p.seg_row.size(), (int)p.n_segb, kBatchBlock / 64) +
           (int64_t)(p.tiles.size() / 2);
}

// Control area of a batch: one image, built on the host and copied whole,
// then what the device writes.
struct CtlLayout {
    size_t jobs, item_off, code, max_step, word_off, row_off, item_job, image;
    size_t tail_on, flags, counts, total;
};

CtlLayout ctl_layout(size_t n, size_t ring, size_t items)
{
    CtlLayout c;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align256(off + bytes);
        return o;
    };
    c.jobs = take(n * sizeof(StepArgs));
    c.item_off = take((n + 1) * 4);
    c.code = take(n * 4);
    c.max_step = take(n * 4);
    c.word_off = take((n + 1) * 4);
    c.row_off = take((n + 1) * 8);
    c.item_job = take(items * 2);
    c.image = off;
    c.tail_on = take(n * 4);
    c.flags = take(n * ring * 4);
    c.counts = take(n * 8);
    c.total = off;
    return c;
}

}  // namespace

extern "C" {

int fsg_batch_plan(const fsg_job *jobs, int32_t n_jobs, int32_t steps_per_sync, fsg_plan **out,
                   size_t *ws_bytes)
{
    try {
        if (!out || !ws_bytes) return fail(FSG_EINVAL, "NULL output");
        *out = nullptr;
        if (!jobs || n_jobs < 1 || n_jobs > kMaxBatchJobs)
            return fail(FSG_EINVAL, "n_jobs must be in [1, 1024]");
        if (steps_per_sync < 1 || steps_per_sync > 4096)
            return fail(FSG_EINVAL, "steps_per_sync must be in [1, 4096]");
        fsg::inject_alloc_fault();
        std::unique_ptr<fsg_plan> pl(new fsg_plan);
        pl->sync = steps_per_sync;
        size_t off = 0;
        const Fill fill = batch_fill(jobs, n_jobs);
        for (int32_t i = 0; i < n_jobs; ++i) {
            const fsg_job &j = jobs[i];
            fsg_graph *g = const_cast<fsg_graph *>(j.g);
            int rc = validate_run(g, &j.prm, j.seeds, j.n_seeds, j.B, j.replicate_offset);
            if (rc) return fail(rc, "job " + std::to_string(i) + ": " + g_err);
            Sched s;
            rc = resolve_batch_sched(j, fill, &s);
            if (rc) return fail(rc, "job " + std::to_string(i) + ": " + g_err);
            s.sync = steps_per_sync;
            const Plan &p = get_plan(g, s.heavy, s.tile_edges, s.light, s.narrow);
            Layout L;
            layout(g, &j.prm, j.B, s, p, &L);
            pl->jobs.push_back(j);
            pl->sched.push_back(s);
            pl->plans.push_back(&p);
            pl->layouts.push_back(L);
            pl->job_off.push_back(off);
            off = align256(off + L.total);
            pl->items += batch_items(p);
        }
        if (pl->items > INT32_MAX)
            return fail(FSG_EUNSUPPORTED, "too many work items in the batch");
        pl->ctl_off = off;
        off = align256(off + ctl_layout((size_t)n_jobs, (size_t)steps_per_sync + 1,
                                        (size_t)pl->items).total);
        pl->total = off;
        *ws_bytes = off;
        *out = pl.release();
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

int fsg_batch_set_launch(fsg_plan *plan, int32_t blocks_per_cu)
{
    if (!plan) return fail(FSG_EINVAL, "plan is NULL");
    if (blocks_per_cu < 1 || blocks_per_cu > 32)
        return fail(FSG_EINVAL, "blocks_per_cu must be in [1, 32]");
    plan->blocks_per_cu = blocks_per_cu;
    return FSG_OK;
}

int fsg_plan_destroy(fsg_plan *plan)
{
    delete plan;
    return FSG_OK;
}

int fsg_batch_run(fsg_plan *pl, void *dev_ws, size_t ws_bytes, fsg_run_info *infos,
                  double *total_ms, void *stream)
{
    try {
        if (!pl) return fail(FSG_EINVAL, "plan is NULL");
        if (!dev_ws || ws_bytes < pl->total) return fail(FSG_EWORKSPACE, "batch workspace too small");
        if (((uintptr_t)dev_ws & 255) != 0) return fail(FSG_EWORKSPACE, "workspace not 256-byte aligned");
        hipStream_t st = (hipStream_t)stream;
        char *base = (char *)dev_ws;
        const int n = (int)pl->jobs.size();
        const int ring = pl->sync + 1;
        char *ctl = base + pl->ctl_off;
        const CtlLayout cl = ctl_layout((size_t)n, (size_t)ring, (size_t)pl->items);
        uint32_t *d_flags = (uint32_t *)(ctl + cl.flags);
        int32_t *d_tail_on = (int32_t *)(ctl + cl.tail_on);
        unsigned long long *d_counts = (unsigned long long *)(ctl + cl.counts);

        std::vector<Job> jb((size_t)n);
        std::vector<char> image(cl.image, 0);
        StepArgs *h_jobs = (StepArgs *)(image.data() + cl.jobs);
        int32_t *item_off = (int32_t *)(image.data() + cl.item_off);
        int32_t *code = (int32_t *)(image.data() + cl.code);
        int32_t *max_step = (int32_t *)(image.data() + cl.max_step);
        int32_t *word_off = (int32_t *)(image.data() + cl.word_off);
        int64_t *row_off = (int64_t *)(image.data() + cl.row_off);
        uint16_t *item_job = (uint16_t *)(image.data() + cl.item_job);
        std::vector<int32_t> tail_on((size_t)n, 0);
        bool any_tail = false, any_out = false;
        int merge_rows = 0;  // most heavy rows of a job whose merge takes a launch
        for (int i = 0; i < n; ++i) {
            const fsg_job &j = pl->jobs[(size_t)i];
            fsg_graph *g = const_cast<fsg_graph *>(j.g);
            int rc = setup_job(g, &j.prm, j.seeds, j.n_seeds, j.B, j.replicate_offset, j.rng_key,
                               pl->sched[(size_t)i], *pl->plans[(size_t)i], pl->layouts[(size_t)i],
                               base + pl->job_off[(size_t)i], d_flags + (size_t)i * ring, st,
                               &jb[(size_t)i]);
            if (rc) return rc;
            StepArgs &a = jb[(size_t)i].a;
            if (jb[(size_t)i].tail) {  // the tail mode's bitmaps (used while tail_on)
                a.ibm_words = (int32_t)((a.n + 31) / 32);
                a.ibm = jb[(size_t)i].ibm;
                if (jb[(size_t)i].tail_out) a.cand = a.ibm + 4 * (size_t)a.ibm_words;
                any_tail = true;
                any_out |= jb[(size_t)i].tail_out;
            }
            if (a.heavy_done == nullptr) merge_rows = std::max(merge_rows, a.n_heavy);
            word_off[i + 1] = word_off[i] + (jb[(size_t)i].tail_out ? a.ibm_words : 0);
            row_off[i + 1] = row_off[i] + (jb[(size_t)i].tail ? a.n : 0);
            memcpy(&h_jobs[i], &a, sizeof(a));  // prev/next hold planes 0 and 1
            item_off[i + 1] = item_off[i] + (int32_t)batch_items(*pl->plans[(size_t)i]);
            std::fill(item_job + item_off[i], item_job + item_off[i + 1], (uint16_t)i);
            code[i] = jb[(size_t)i].kind * 32 + (jb[(size_t)i].kind == kKindIC ? 1 : a.Lp);
            max_step[i] = (int32_t)std::min<int64_t>(jb[(size_t)i].K, 0x7FFFFFFF);
        }
        HIP_TRY(hipMemcpyAsync(ctl, image.data(), image.size(), hipMemcpyHostToDevice, st));
        HIP_TRY(launch_fill32((uint32_t *)d_tail_on, n, 0u, st));
        HIP_TRY(hipStreamSynchronize(st));

        BatchCtl c;
        c.jobs = (const StepArgs *)(ctl + cl.jobs);
        c.item_off = (const int32_t *)(ctl + cl.item_off);
        c.code = (const int32_t *)(ctl + cl.code);
        c.max_step = (const int32_t *)(ctl + cl.max_step);
        c.item_job = (const uint16_t *)(ctl + cl.item_job);
        c.n_jobs = n;
        c.ring = ring;
        c.tail_on = d_tail_on;
        c.word_off = (const int32_t *)(ctl + cl.word_off);
        c.row_off = (const int64_t *)(ctl + cl.row_off);
        const int items = (int)pl->items;

        std::vector<uint32_t> hf((size_t)n * ring);
        std::vector<int64_t> steps_run((size_t)n, 0);
        std::vector<int> done((size_t)n, 0), absorbed((size_t)n, 0);
        int remaining = 0;
        for (int i = 0; i < n; ++i) {
            const fsg_job &j = pl->jobs[(size_t)i];
            if (j.n_seeds == 0 || jb[(size_t)i].K == 0) {
                done[(size_t)i] = 1;
                absorbed[(size_t)i] = j.n_seeds == 0;
            } else {
                ++remaining;
            }
        }
        EventPool ev;
        HIP_TRY(ev.init(2));
        double kernel_ms = 0.0;
        int64_t t0 = 0;
        // tail mode per job: nodes with an infected replicate (LT: a new
        // activation) at the last poll, -1 before the first
        std::vector<int64_t> icount((size_t)n, -1), tail_steps((size_t)n, 0);
        std::vector<unsigned long long> hcount((size_t)n, 0);
        while (remaining > 0) {
            if (any_tail) {
                bool changed = false;
                for (int i = 0; i < n; ++i) {
                    const Job &J = jb[(size_t)i];
                    if (!J.tail || done[(size_t)i]) continue;
                    const double nn = (double)J.n, deg = (double)J.a.nnz / std::max(nn, 1.0);
                    const bool want = t0 >= 1 && (pl->sched[(size_t)i].tail_always ||
                                                  (icount[(size_t)i] >= 0 &&
                                                   (double)icount[(size_t)i] * deg <= nn * kTailFactor));
                    if (want && !tail_on[(size_t)i]) {  // the bitmaps of steps t0 and t0-1
                        const StepArgs &a = h_jobs[(size_t)i];
                        const uint32_t t = (uint32_t)(t0 + 1);
                        uint32_t *cand = a.ibm + 4 * (size_t)a.ibm_words;
                        if (J.kind == kKindLT) {
                            HIP_TRY(launch_mark_gained(a.stamp, a.ibm, cand, a.ibm_words, a.n, t, st));
                        } else {
                            // base planes: prev holds odd steps' inputs (state of even steps)
                            const uint64_t *p0 = a.prev, *p1 = a.next;
                            const uint64_t *cur = (t & 1u) ? p0 : p1, *old = (t & 1u) ? p1 : p0;
                            HIP_TRY(launch_mark_rows(cur, old, a.ibm, cand, a.ibm_words, a.n, a.W, t,
                                                     st));
                        }
                    }
                    if (want != (tail_on[(size_t)i] != 0)) changed = true;
                    tail_on[(size_t)i] = want ? 1 : 0;
                }
                if (changed)
                    HIP_TRY(hipMemcpyAsync(d_tail_on, tail_on.data(), (size_t)n * 4,
                                           hipMemcpyHostToDevice, st));
            }
            HIP_TRY(hipEventRecord(ev.e[0], st));
            HIP_TRY(launch_batch_ring_clear(c, (uint32_t)(t0 + 1), st));
            for (int k = 1; k <= pl->sync; ++k) {
                const uint32_t t = (uint32_t)(t0 + k);
                if (any_out) HIP_TRY(launch_batch_expand(c, t, st));
                HIP_TRY(launch_batch_step(c, t, items, st));
                if (merge_rows > 0) HIP_TRY(launch_batch_combine(c, t, merge_rows, st));
            }
            HIP_TRY(hipEventRecord(ev.e[1], st));
            if (any_tail) {
                HIP_TRY(launch_fill64((uint64_t *)d_counts, n, 0ull, st));
                HIP_TRY(launch_batch_count(c, (uint32_t)(t0 + pl->sync), d_counts, st));
                HIP_TRY(hipMemcpyAsync(hcount.data(), d_counts, (size_t)n * 8, hipMemcpyDeviceToHost, st));
            }
            HIP_TRY(hipMemcpyAsync(hf.data(), d_flags, hf.size() * 4, hipMemcpyDeviceToHost, st));
            HIP_TRY(hipStreamSynchronize(st));
            if (any_tail)
                for (int i = 0; i < n; ++i) icount[(size_t)i] = (int64_t)hcount[(size_t)i];
            float ms = 0.f;
            HIP_TRY(hipEventElapsedTime(&ms, ev.e[0], ev.e[1]));
            kernel_ms += ms;
            for (int i = 0; i < n; ++i) {
                if (done[(size_t)i]) continue;
                const uint32_t *f = hf.data() + (size_t)i * ring;
                for (int k = 1; k <= pl->sync; ++k) {
                    const int64_t t = t0 + k;
                    if (f[t % ring] == 0u) {
                        done[(size_t)i] = 1;
                        absorbed[(size_t)i] = 1;
                        steps_run[(size_t)i] = t;
                        break;
                    }
                    if (t == jb[(size_t)i].K) {
                        done[(size_t)i] = 1;
                        steps_run[(size_t)i] = t;
                        break;
                    }
                }
                if (tail_on[(size_t)i])
                    tail_steps[(size_t)i] += (done[(size_t)i] ? steps_run[(size_t)i] : t0 + pl->sync) - t0;
                if (done[(size_t)i]) --remaining;
            }
            t0 += pl->sync;
        }
        for (int i = 0; i < n; ++i) {
            const fsg_job &j = pl->jobs[(size_t)i];
            int rc = finalize_job(jb[(size_t)i], steps_run[(size_t)i], j.final_states,
                                  j.infected_counts, st);
            if (rc) return rc;
            if (infos) {
                infos[i].steps_run = steps_run[(size_t)i];
                infos[i].absorbed = absorbed[(size_t)i];
                infos[i].tail_steps = (int32_t)std::min<int64_t>(tail_steps[(size_t)i], INT32_MAX);
                infos[i].step_kernel_ms = 0.0;
                infos[i].step_launches = 0;
                infos[i].setup_ms = 0.0;
                infos[i].finalize_ms = 0.0;
                infos[i].philox_calls = 0;
            }
        }
        if (total_ms) *total_ms = kernel_ms;
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

}  // extern "C"

// --------------------------------------------------------------- autotuner

namespace {

std::vector<fsg_schedule> candidates(const fsg_graph *g, const fsg_params *prm, int64_t B,
                                     bool batch_only)
{
    std::vector<fsg_schedule> out;
    const int64_t W = (B + 63) / 64;
    const int gmax = (int)std::min<int64_t>(next_pow2(W), 64);
    auto add = [&](int lanes, int block, int tile, int heavy, int variant) {
        fsg_schedule s;
        memset(&s, 0, sizeof(s));
        s.row_lanes = lanes;
        s.block_threads = block;
        s.tile_edges = tile;
        s.heavy_threshold = heavy;
        s.steps_per_sync = 16;
        s.kernel_variant = variant;
        out.push_back(s);
    };
    if (!batch_only && prm->model == FSG_IC && W == 1) {
        if (g->has_out) add(16, 512, 16384, 32768, 3);
        for (int block : {256, 512, 1024})
            for (int tile : {8192, 16384, 32768})
                for (int heavy : {8192, 32768}) add(16, block, tile, heavy, 2);
    }
    std::vector<int> lanes;
    for (int l = gmax; l <= 64; l *= 2) lanes.push_back(l);
    if (gmax < 16 && std::find(lanes.begin(), lanes.end(), 16) == lanes.end()) lanes.push_back(16);
    for (int l : lanes)
        for (int block : batch_only ? std::vector<int>{kBatchBlock} : std::vector<int>{256, 512})
            for (int tile : {2048, 4096, 16384})
                for (int heavy : {512, 1024, 4096}) add(l, block, tile, heavy, 1);
    return out;
}

std::string tune_key(const fsg_graph *g, const fsg_params *prm, int64_t B, bool batch_only)
{
    std::ostringstream k;
    k << "n=" << g->n << ",nnz=" << g->nnz << ",dmax=" << g->max_indeg << ",model=" << prm->model
      << ",icp=" << prm->ic_prob << ",B=" << B << ",batch=" << (batch_only ? 1 : 0)
      << ",out=" << (g->has_out ? 1 : 0);
    return k.str();
}

bool cache_lookup(const char *path, const std::string &key, fsg_schedule *out, double *ms)
{
    if (!path) return false;
    std::ifstream f(path);
    std::string line;
    bool found = false;
    while (std::getline(f, line)) {
        std::istringstream is(line);
        std::string k;
        fsg_schedule s;
        memset(&s, 0, sizeof(s));
        double m = 0;
        if (!(is >> k >> s.row_lanes >> s.block_threads >> s.tile_edges >> s.heavy_threshold >>
              s.steps_per_sync >> s.kernel_variant >> m))
            continue;
        if (k == key) {  // the last entry for a key wins
            *out = s;
            *ms = m;
            found = true;
        }
    }
    return found;
}

void cache_store(const char *path, const std::string &key, const fsg_schedule &s, double ms)
{
    if (!path) return;
    std::ofstream f(path, std::ios::app);
    f << key << " " << s.row_lanes << " " << s.block_threads << " " << s.tile_edges << " "
      << s.heavy_threshold << " " << s.steps_per_sync << " " << s.kernel_variant << " " << ms
      << "\n";
}

}  // namespace

extern "C" {

int fsg_autotune_workspace_size(const fsg_graph *g_, const fsg_params *prm, int64_t B,
                                int32_t batch_only, size_t *bytes)
{
    try {
        if (!bytes) return fail(FSG_EINVAL, "bytes is NULL");
        int rc = check_params(g_, prm, B);
        if (rc) return rc;
        size_t best = 0;
        fsg_schedule d;
        default_sched(g_, prm, B, &d);
        std::vector<fsg_schedule> cs = candidates(g_, prm, B, batch_only != 0);
        cs.push_back(d);
        for (fsg_schedule s : cs) {
            s.steps_per_sync = 64;  // the longest poll interval fsg_autotune uses
            size_t b = 0;
            rc = fsg_sim_workspace_size(g_, prm, B, &s, &b);
            if (rc) return rc;
            best = std::max(best, b);
        }
        *bytes = best;
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

int fsg_autotune(const fsg_graph *g, const fsg_params *prm, const int32_t *seeds, int64_t n_seeds,
                 int64_t B, uint64_t rng_key, int32_t tune_steps, int32_t batch_only,
                 const char *cache_path, void *dev_ws, size_t ws_bytes, fsg_schedule *best,
                 double *best_ms, double *default_ms, void *stream)
{
    try {
        if (!best) return fail(FSG_EINVAL, "best is NULL");
        if (tune_steps < 1) return fail(FSG_EINVAL, "tune_steps must be >= 1");
        int rc = check_params(g, prm, B);
        if (rc) return rc;
        const std::string key = tune_key(g, prm, B, batch_only != 0);
        double cached_ms = 0;
        if (cache_lookup(cache_path, key, best, &cached_ms)) {
            if (best_ms) *best_ms = cached_ms;
            if (default_ms) *default_ms = -1.0;
            return FSG_OK;
        }
        // Objective: device time of whole steps (pull step, heavy-row merge
        // and frontier clear), from runs of K and 2K steps timed with HIP
        // events on the stream; their difference leaves out the set-up.
        hipStream_t st = (hipStream_t)stream;
        EventPool ev;
        HIP_TRY(ev.init(2));
        auto run_for = [&](const fsg_schedule &s, int64_t k, double *ms, int64_t *steps) -> int {
            fsg_params tp = *prm;
            tp.max_steps = prm->max_steps < 0 ? k : std::min<int64_t>(prm->max_steps, k);
            fsg_run_info info;
            HIP_TRY(hipEventRecord(ev.e[0], st));
            int r = fsg_simulate(g, &tp, seeds, n_seeds, B, 0, rng_key, &s, dev_ws, ws_bytes,
                                 nullptr, nullptr, &info, stream);
            if (r) return r;
            HIP_TRY(hipEventRecord(ev.e[1], st));
            HIP_TRY(hipEventSynchronize(ev.e[1]));
            float f = 0.f;
            HIP_TRY(hipEventElapsedTime(&f, ev.e[0], ev.e[1]));
            *ms = f;
            *steps = info.steps_run;
            return FSG_OK;
        };
        auto time_one = [&](const fsg_schedule &s0, double *ms) -> int {
            fsg_schedule s = s0;
            s.time_kernels = 0;
            s.steps_per_sync = std::max(1, std::min(tune_steps, 64));
            double t1 = 0, t2 = 0;
            int64_t s1 = 0, s2 = 0;
            int r = run_for(s, tune_steps, &t1, &s1);
            if (r) return r;
            r = run_for(s, 2 * (int64_t)tune_steps, &t2, &s2);
            if (r) return r;
            *ms = s2 > s1 ? std::max(0.0, t2 - t1) / (double)(s2 - s1)
                          : (s2 > 0 ? t2 / (double)s2 : 1e30);
            return FSG_OK;
        };
        fsg_schedule d;
        default_sched(g, prm, B, &d);
        if (batch_only) {
            d.kernel_variant = 1;
            d.block_threads = kBatchBlock;
        }
        double dms = 0;
        rc = time_one(d, &dms);  // also a warm-up of the code objects
        if (rc) return rc;
        rc = time_one(d, &dms);
        if (rc) return rc;
        fsg_schedule win = d;
        double wms = dms;
        for (const fsg_schedule &s : candidates(g, prm, B, batch_only != 0)) {
            double ms = 0;
            rc = time_one(s, &ms);
            if (rc) return rc;
            if (ms < wms) {
                wms = ms;
                win = s;
            }
        }
        win.time_kernels = 0;
        *best = win;
        if (best_ms) *best_ms = wms;
        if (default_ms) *default_ms = dms;
        cache_store(cache_path, key, win, wms);
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

}  // extern "C"

// ------------------------------------------------------ batch autotuner ----
// The batch is tuned as a batch: every trial plans and runs the whole batch
// (all jobs to absorption or their caps) and is scored by its device time,
// so a schedule that helps one job alone but costs the batch is not taken.
namespace {

struct BatchTrial {
    std::vector<fsg_schedule> sched;  // per job
    int sync = 16, blocks_per_cu = 4;
};

// Knob values tried per model class (0 keeps the library default).
const int kTryLanes[] = {0, 16, 32, 64};
const int kTryTile[] = {0, 4096, 16384};
const int kTryHeavy[] = {0, 512, 1024};
const int kTrySync[] = {16, 8, 32, 64};

int model_class(int model)
{
    const int k = model_kind(model);
    return k == kKindIC ? 0 : (k == kKindLT ? 2 : 1);
}

}  // namespace

extern "C" {

int fsg_batch_autotune_workspace_size(const fsg_job *jobs, int32_t n_jobs, size_t *bytes)
{
    try {
        if (!jobs || !bytes || n_jobs < 1 || n_jobs > kMaxBatchJobs)
            return fail(FSG_EINVAL, "bad arguments");
        // The tuner mixes schedules over the model classes, so every job gets
        // the room of its own largest layout: over the lanes and heavy cuts
        // tried and its own, with the smallest tiles any of them means (larger
        // tiles are fewer, but for those that the wide rows and kMaxTileRows
        // split off).
        const int longest = *std::max_element(std::begin(kTrySync), std::end(kTrySync));
        const Fill fill = batch_fill(jobs, n_jobs);
        size_t best = 0, items = 0;
        for (int32_t i = 0; i < n_jobs; ++i) {
            fsg_job j = jobs[i];
            fsg_graph *g = const_cast<fsg_graph *>(j.g);
            int rc = validate_run(g, &j.prm, j.seeds, j.n_seeds, j.B, j.replicate_offset);
            if (rc) return fail(rc, "job " + std::to_string(i) + ": " + g_err);
            const fsg_schedule own = j.sched;
            std::vector<int> lanes(std::begin(kTryLanes), std::end(kTryLanes)),
                tiles(std::begin(kTryTile), std::end(kTryTile)),
                heavy(std::begin(kTryHeavy), std::end(kTryHeavy));
            lanes.push_back(own.row_lanes);
            tiles.push_back(own.tile_edges);
            heavy.push_back(own.heavy_threshold);
            int64_t small = INT64_MAX;
            for (int l : lanes)
                for (int t : tiles) {
                    j.sched = own;
                    j.sched.row_lanes = l;
                    j.sched.tile_edges = t;
                    j.sched.heavy_threshold = 0;
                    Sched s;
                    if (resolve_batch_sched(j, fill, &s) == FSG_OK)
                        small = std::min<int64_t>(small, s.tile_edges);
                }
            size_t job = 0, job_items = 0;
            for (int l : lanes)
                for (int h : heavy) {
                    j.sched = own;
                    j.sched.row_lanes = l;
                    j.sched.tile_edges = (int32_t)std::min<int64_t>(small, INT32_MAX);
                    j.sched.heavy_threshold = h;
                    Sched s;
                    rc = resolve_batch_sched(j, fill, &s);
                    if (rc) {  // (a schedule of the job's own that no trial can run)
                        if (l != own.row_lanes && h != own.heavy_threshold)
                            return fail(rc, "job " + std::to_string(i) + ": " + g_err);
                        continue;
                    }
                    s.sync = longest;
                    const Plan &p = get_plan(g, s.heavy, s.tile_edges, s.light, s.narrow);
                    Layout L;
                    layout(g, &j.prm, j.B, s, p, &L);
                    const size_t split =
                        (size_t)(fill_of(g).load / s.tile_edges + g->n / kMaxTileRows + 2);
                    job = std::max(job, align256(L.total + 8 * split));
                    job_items = std::max(job_items, (size_t)batch_items(p) + split);
                }
            best = align256(best + job);
            items += job_items;
        }
        best = align256(best + ctl_layout((size_t)n_jobs, (size_t)longest + 1, items).total);
        *bytes = best;
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

int fsg_batch_autotune(const fsg_job *jobs, int32_t n_jobs, int32_t max_trials, void *dev_ws,
                       size_t ws_bytes, fsg_job *tuned, int32_t *steps_per_sync,
                       int32_t *blocks_per_cu, double *best_ms, double *default_ms,
                       int32_t *trials_run, void *stream)
{
    try {
        if (!jobs || !tuned || !steps_per_sync || !blocks_per_cu || n_jobs < 1 ||
            n_jobs > kMaxBatchJobs)
            return fail(FSG_EINVAL, "bad arguments");
        if (max_trials < 1) return fail(FSG_EINVAL, "max_trials must be >= 1");
        const std::vector<fsg_job> base(jobs, jobs + n_jobs);
        int trials = 0;
        auto run = [&](const BatchTrial &t, double *ms) -> int {
            std::vector<fsg_job> js = base;
            for (int i = 0; i < n_jobs; ++i) js[(size_t)i].sched = t.sched[(size_t)i];
            fsg_plan *pl = nullptr;
            size_t need = 0;
            int rc = fsg_batch_plan(js.data(), n_jobs, t.sync, &pl, &need);
            if (rc) return rc;
            std::unique_ptr<fsg_plan, int (*)(fsg_plan *)> guard(pl, fsg_plan_destroy);
            if (need > ws_bytes) return fail(FSG_EWORKSPACE, "batch autotune workspace too small");
            pl->blocks_per_cu = t.blocks_per_cu;
            double total = 0;
            rc = fsg_batch_run(pl, dev_ws, ws_bytes, nullptr, &total, stream);
            if (rc) return rc;
            *ms = total;
            ++trials;
            return FSG_OK;
        };
        BatchTrial cur;
        for (const auto &j : base) {
            fsg_schedule s = j.sched;
            s.time_kernels = 0;
            cur.sched.push_back(s);
        }
        double cms = 0;
        int rc = run(cur, &cms);  // warm-up
        if (rc) return rc;
        rc = run(cur, &cms);
        if (rc) return rc;
        const double dms = cms;
        auto consider = [&](const BatchTrial &t) -> int {
            if (trials >= max_trials) return FSG_OK;
            double ms = 0;
            int r = run(t, &ms);
            if (r) return r;
            if (ms < cms) {
                cms = ms;
                cur = t;
            }
            return FSG_OK;
        };
        // steps per sync, then per model class lanes, tiles, heavy cut
        for (int v : kTrySync) {
            if (v == cur.sync) continue;
            BatchTrial t = cur;
            t.sync = v;
            rc = consider(t);
            if (rc) return rc;
        }
        for (int cls = 0; cls < 3; ++cls) {
            bool present = false;
            for (const auto &j : base) present |= model_class(j.prm.model) == cls;
            if (!present) continue;
            for (int knob = 0; knob < 3; ++knob) {
                const int *vals = knob == 0 ? kTryLanes : (knob == 1 ? kTryTile : kTryHeavy);
                const int nv = knob == 0 ? 4 : 3;
                const BatchTrial start = cur;
                for (int k = 0; k < nv; ++k) {
                    BatchTrial t = start;
                    bool changed = false;
                    for (int i = 0; i < n_jobs; ++i) {
                        if (model_class(base[(size_t)i].prm.model) != cls) continue;
                        fsg_schedule &sc = t.sched[(size_t)i];
                        int32_t &field = knob == 0 ? sc.row_lanes
                                                   : (knob == 1 ? sc.tile_edges : sc.heavy_threshold);
                        if (field != vals[k]) {
                            field = vals[k];
                            changed = true;
                        }
                    }
                    if (!changed) continue;
                    rc = consider(t);
                    if (rc) return rc;
                }
            }
        }
        for (int i = 0; i < n_jobs; ++i) {
            tuned[i] = base[(size_t)i];
            tuned[i].sched = cur.sched[(size_t)i];
        }
        *steps_per_sync = cur.sync;
        *blocks_per_cu = cur.blocks_per_cu;
        if (best_ms) *best_ms = cms;
        if (default_ms) *default_ms = dms;
        if (trials_run) *trials_run = trials;
        return FSG_OK;
    } catch (const std::bad_alloc &) {
        return fail(FSG_ENOMEM, "host allocation failed");
    }
}

}  // extern "C"
