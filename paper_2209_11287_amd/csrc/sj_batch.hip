// Batched form: many independent self-joins (uneven n and d) refined by one
// persistent work-queue kernel whose items are ordered longest first, with
// the count pipeline (queue reset, persistent count kernel, per-problem
// prefix sums) captured once into a HIP graph and replayed; an optional
// autotuner picks the number of indexed dimensions per d by timing.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "sj_internal.h"

namespace sj {

namespace {

// Last problem p with base[p] <= x.
__device__ __forceinline__ int problem_of(const int64_t *__restrict__ base, int B, int64_t x) {
    int lo = 0, hi = B;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (base[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ unsigned long long cost_key(int form, unsigned long long c) {
    const unsigned long long cap = 0xffffffffull;
    return ((unsigned long long)form << 32) | (cap - (c < cap ? c : cap));
}

// Sort key of each work item of the batch, all problems in one launch (a
// launch each took 1.5 ms for 256 problems): its problem's tile form in the high
// bits (form[p]: the problems the hit-list count takes after the others, then
// d), then descending cost (candidate tiles x K-steps); value = global item
// index.
__global__ void k_item_cost(const BProb *__restrict__ probs, const int64_t *__restrict__ item_base,
                            const int32_t *__restrict__ form, int B, int64_t total, bool sym,
                            unsigned long long *__restrict__ key, int32_t *__restrict__ val) {
    const int64_t gi = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gi >= total) return;
    const int p = problem_of(item_base, B, gi);
    DevGrid G = probs[p].G;
    G.ranges = global_ptr(G.ranges);
    G.items = global_ptr(G.items);
    G.blocks = global_ptr(G.blocks);
    const int64_t it = gi - item_base[p];
    // half stencil: the ranges as the count cuts them (from the first query on)
    const int32_t cut = sym ? G.items[it].qbegin : INT32_MIN;
    unsigned long long c = 0;
    for (int o = 0; o < G.nranges; ++o) {
        const Range r = G.ranges[it * G.nranges + o];
        const int32_t b = max(r.begin, cut);
        c += (unsigned long long)(r.end > b ? (r.end - b + 15) / 16 : 0);
    }
    key[gi] = cost_key(form[p], c * (unsigned long long)(G.da >> 2));
    val[gi] = (int32_t)gi;
}

// Sort key of each block item of the problems counted with LDS-shared tiles
// (FP64 MFMA, d = 5 .. 16): d in the high bits, then descending cost (its
// list's tiles x K-steps x items; half stencil: the list cut at the block's
// first query); value = global block index.
__global__ void k_block_cost(const BProb *__restrict__ probs, const int64_t *__restrict__ block_base, int B,
                             int64_t total, bool sym, unsigned long long *__restrict__ key,
                             int32_t *__restrict__ val) {
    const int64_t gb = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gb >= total) return;
    const int p = problem_of(block_base, B, gb);
    DevGrid G = probs[p].G;
    G.ranges = global_ptr(G.ranges);
    G.items = global_ptr(G.items);
    G.blocks = global_ptr(G.blocks);
    const int b = (int)(gb - block_base[p]);
    const int64_t it0 = G.blocks[b] - G.item_base;
    const int ni = G.blocks[b + 1] - G.blocks[b];
    const int32_t cut = sym ? G.items[it0].qbegin : INT32_MIN;
    unsigned long long c = 0;
    for (int o = 0; o < G.nranges; ++o) {
        const Range r = G.ranges[it0 * G.nranges + o];
        const int32_t rb = max(r.begin, cut);
        c += (unsigned long long)(r.end > rb ? r.end - rb : 0);
    }
    key[gb] = cost_key(G.d, (c + 15) / 16 * (unsigned long long)(G.da >> 2) * (unsigned long long)ni);
    val[gb] = (int32_t)gb;
}

// One problem's offsets from those of many: out[i] = off[i] - off[0].
__global__ void k_copy_offsets(const int64_t *__restrict__ off, int64_t n, int64_t *__restrict__ out) {
    const int64_t base = off[0];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = off[i] - base;
}

// Tuned choices, per path, d and size class: index_dims and the
// short-circuit setting (sj_opts.short_circuit).
struct TuneCache {
    std::mutex mu;
    std::map<std::string, int> v;
};
TuneCache g_tune;

std::string tune_key(int path, int d, int64_t n) {
    int lg = 0;
    while ((int64_t(1) << (lg + 1)) <= std::max<int64_t>(1, n)) ++lg;
    return std::to_string(path) + "/" + std::to_string(d) + "/" + std::to_string(lg);
}

void tune_load(const char *path) {
    if (!path) return;
    FILE *f = std::fopen(path, "r");
    if (!f) return;
    char key[128];
    int v;
    // one "key value" pair per line
    while (std::fscanf(f, "%127s %d", key, &v) == 2) g_tune.v[key] = v;
    std::fclose(f);
}

void tune_save(const char *path) {
    if (!path) return;
    FILE *f = std::fopen(path, "w");
    if (!f) return;
    for (auto &kv : g_tune.v) std::fprintf(f, "%s %d\n", kv.first.c_str(), kv.second);
    std::fclose(f);
}

// Device time of the FP64 MFMA count kernel on one problem built with
// (index_dims, short_circuit); the second of two runs.
float time_count(const double *pts, int64_t n, int d, double eps, int k, int sc, hipStream_t s) {
    Grid g;
    g.sc = sc;
    float ms = 0.f;
    try {
        build_grid(g, pts, n, d, eps, k, s);
        int32_t *cnt = dev_alloc_n<int32_t>((size_t)n + 1, s);
        RefineOut ro;
        ro.timed = true;
        ro.hits = hits_usable(g, SJ_FP64_MFMA, HitUse::PAIRS) && hits_prepare(g, s);
        ro.ctr = dev_alloc_n<DevCounters>(1, s);
        refine_count(g, SJ_FP64_MFMA, cnt, ro, s);  // warm
        ro.kt.ms();
        refine_count(g, SJ_FP64_MFMA, cnt, ro, s);
        ms = ro.kt.ms();
        dev_free(cnt, s);
        dev_free(ro.ctr, s);
    } catch (...) {
        free_grid(g, s);
        throw;
    }
    free_grid(g, s);
    return ms;
}

// The tile choices of one d, timed on one problem (result-neutral): first
// index_dims = 1 .. min(d, 4) (cell geometry, so which candidates share a
// tile), then, for d > 4, the short-circuit on (the library's schedule) or
// off.
void tune_problem(const double *pts, int64_t n, int d, double eps, hipStream_t s, int *k_out, int *sc_out) {
    int best_k = std::min(d, kMaxIndexDims);
    float best = 1e30f;
    for (int k = 1; k <= std::min(d, kMaxIndexDims); ++k) {
        const float ms = time_count(pts, n, d, eps, k, 0, s);
        if (ms < best) {
            best = ms;
            best_k = k;
        }
    }
    int best_sc = 0;
    if (d > 4 && time_count(pts, n, d, eps, best_k, -1, s) < best) best_sc = -1;
    *k_out = best_k;
    *sc_out = best_sc;
}

}  // namespace

struct Batch {
    int B = 0;
    std::vector<Grid *> grids;
    std::vector<int> kdims, scs;
    int64_t total_items = 0;
    std::vector<int64_t> item_base;       // B + 1
    int64_t *item_base_dev = nullptr;     // B + 1
    int32_t *queue = nullptr;             // global item indices: by d, longest first
    int32_t *bqueue = nullptr;            // global block item indices (LDS-shared FP64 MFMA count), same order
    int64_t *block_base_dev = nullptr;    // B + 1: first global block item of each problem
    std::vector<BatchForm> forms;         // one per distinct d
    int sched = 0;                        // 0 = persistent grids, 1 = one wave per item
    bool tune_sched = false;              // choose sched on the first count (timed, or from the cache)
    std::string sched_key, tune_cache;    // the choice's cache key (batch shape) and file
    DevCounters *ctr = nullptr;
    BProb *probs_dev = nullptr;
    std::vector<BProb> probs;
    int64_t *totals_dev = nullptr;
    std::vector<int64_t> totals;
    unsigned long long *masks = nullptr;  // in-masks (or null: pairs re-run the tiles)
    int64_t mask_tiles = 0;               // their tile slots
    std::vector<int64_t> tile_base;       // first tile slot of each problem, all problems together (segmented
                                          // builds: tile_off counts from there), else 0
    HitBatch hb;                          // the hit-list count of the problems it takes (FP64 MFMA)
    std::vector<char> in_hb;              // those problems
    bool hits_counted = false;            // the last count ran it
    int32_t *rest = nullptr;              // the other problems' indices
    int nrest = 0;
    int64_t rest_items = 0;               // their items (the first of the queue)
    int32_t *cnt_all = nullptr;           // per-query counts and offsets of every problem
    int64_t *off_all = nullptr;
    bool segmented = false;               // grids from one segmented build (their arrays in `owned`)
    std::vector<void *> owned;
    bool masks_valid = false;
    bool counted = false;
    bool sym = false;                     // half-stencil count (sj_opts.symmetric): no in-masks
    int64_t max_n = 0;                    // largest problem
    int64_t sym_cand[2] = {-1, -1};       // candidate pairs the half-stencil tiles evaluate (on first use): of all
                                          // problems, of those without the hit list
    double ms_build = 0;                  // wall time of the grid builds and the queue
    // graphs per path: the count pipeline, and the pairs launch (per output buffer)
    hipGraphExec_t exec[2] = {nullptr, nullptr};
    hipStream_t graph_stream[2] = {nullptr, nullptr};
    int graph_sched[2] = {-1, -1};
    hipGraphExec_t pexec[2] = {nullptr, nullptr};
    hipStream_t pgraph_stream[2] = {nullptr, nullptr};
    int32_t *pgraph_pairs[2] = {nullptr, nullptr};
    int pgraph_mode[2] = {-1, -1};
};

constexpr int64_t kBatchMaskBudget = int64_t(64) << 30;  // largest in-mask buffer of a batch (bytes)

void batch_free(Batch &b, hipStream_t s) {
    for (int i = 0; i < 2; ++i) {
        if (b.exec[i]) (void)hipGraphExecDestroy(b.exec[i]);
        if (b.pexec[i]) (void)hipGraphExecDestroy(b.pexec[i]);
        b.exec[i] = b.pexec[i] = nullptr;
    }
    for (Grid *g : b.grids) {
        if (!g) continue;
        g->cnt = nullptr;  // slices of cnt_all, off_all
        g->off = nullptr;
        free_grid(*g, s);
        delete g;
    }
    b.grids.clear();
    for (void *p : b.owned) dev_free(p, s);
    b.owned.clear();
    hit_batch_free(b.hb, s);
    void *bufs[] = {b.item_base_dev, b.queue,  b.ctr,            b.probs_dev, b.totals_dev, b.masks,
                    b.bqueue,        b.block_base_dev, b.rest, b.cnt_all,   b.off_all};
    for (void *p : bufs)
        if (p) dev_free(p, s);
    b.bqueue = nullptr;
    b.block_base_dev = nullptr;
    b.item_base_dev = nullptr;
    b.queue = nullptr;
    b.ctr = nullptr;
    b.probs_dev = nullptr;
    b.totals_dev = nullptr;
    b.masks = nullptr;
    b.rest = nullptr;
    b.cnt_all = nullptr;
    b.off_all = nullptr;
}

void batch_build(Batch &b, int B, const double *const *points, const int64_t *n, const int32_t *d, const double *eps,
                 const sj_opts *opts, hipStream_t s) {
    const auto t0 = std::chrono::steady_clock::now();
    b.B = B;
    b.sym = opts && opts->symmetric;
    b.grids.assign(B, nullptr);
    b.kdims.assign(B, 0);
    b.scs.assign(B, 0);
    const bool tune = opts && opts->tune;
    if (tune) {
        std::lock_guard<std::mutex> lk(g_tune.mu);
        tune_load(opts->tune_cache);
        // one representative (largest n) per d
        std::map<int, int> rep;
        for (int i = 0; i < B; ++i)
            if (n[i] > 0 && (!rep.count(d[i]) || n[i] > n[rep[d[i]]])) rep[d[i]] = i;
        for (auto &kv : rep) {
            const int i = kv.second;
            const std::string key = tune_key(SJ_FP64_MFMA, d[i], n[i]);
            if (!g_tune.v.count(key + "/k") || !g_tune.v.count(key + "/sc")) {
                int k = 0, sc = 0;
                tune_problem(points[i], n[i], d[i], eps[i], s, &k, &sc);
                g_tune.v[key + "/k"] = k;
                g_tune.v[key + "/sc"] = sc;
            }
        }
        tune_save(opts->tune_cache);
        for (int i = 0; i < B; ++i) {
            const std::string key = tune_key(SJ_FP64_MFMA, d[i], n[rep.count(d[i]) ? rep[d[i]] : i]);
            auto ik = g_tune.v.find(key + "/k");
            auto is = g_tune.v.find(key + "/sc");
            b.kdims[i] = ik != g_tune.v.end() ? ik->second : 0;
            b.scs[i] = is != g_tune.v.end() ? is->second : 0;
        }
        b.tune_sched = true;
        if (opts->tune_cache) b.tune_cache = opts->tune_cache;
    } else if (opts) {
        for (int i = 0; i < B; ++i) {
            b.kdims[i] = opts->index_dims;
            b.scs[i] = opts->short_circuit;
        }
    }
    b.item_base.assign(B + 1, 0);
    int64_t rows = 0;
    int64_t mask_tiles = 0;
    b.tile_base.assign(B + 1, 0);
    // every problem's grid in one segmented build (tile slots counted over
    // all problems together), else one build per problem
    std::vector<SegInput> sin(B);
    for (int i = 0; i < B; ++i)
        sin[i] = SegInput{points[i], n[i], d[i], eps[i], b.kdims[i], b.scs[i], opts ? opts->dim_order : 0};
    std::vector<Grid *> gs;
    b.segmented = build_grids_segmented(sin, gs, b.owned, s);
    for (int i = 0; i < B; ++i) {
        if (b.segmented) {
            b.grids[i] = gs[i];
        } else {
            b.grids[i] = new Grid();
            b.grids[i]->sc = b.scs[i];
            if (opts) b.grids[i]->dim_order = opts->dim_order;
            build_grid(*b.grids[i], points[i], n[i], d[i], eps[i], b.kdims[i], s);
        }
        Grid &g = *b.grids[i];
        rows += g.n + 1;
        b.item_base[i + 1] = b.item_base[i] + g.items;
        b.max_n = std::max(b.max_n, g.n);
        b.tile_base[i] = b.segmented ? mask_tiles : 0;
        mask_tiles += g.tiles;
    }
    b.cnt_all = dev_alloc_n<int32_t>((size_t)std::max<int64_t>(rows, 1), s);
    b.off_all = dev_alloc_n<int64_t>((size_t)std::max<int64_t>(rows, 1), s);
    for (int64_t i = 0, at = 0; i < B; ++i) {
        b.grids[i]->cnt = b.cnt_all + at;
        b.grids[i]->off = b.off_all + at;
        at += b.grids[i]->n + 1;
    }
    hit_batch_build(b.hb, b.grids, b.sym, s);
    b.in_hb.assign(B, 0);
    for (int i : b.hb.probs) b.in_hb[i] = 1;
    std::vector<int32_t> rest;
    for (int i = 0; i < B; ++i)
        if (!b.in_hb[i]) {
            rest.push_back(i);
            b.rest_items += b.grids[i]->items;
        }
    b.nrest = (int)rest.size();
    b.ctr = dev_alloc_n<DevCounters>(1, s);
    b.totals_dev = dev_alloc_n<int64_t>(B, s);
    b.probs.resize(B);
    for (int i = 0; i < B; ++i) {
        const Grid &g = *b.grids[i];
        BProb &p = b.probs[i];
        p.G = make_dev_grid(g);
        p.delta = fp64_mfma_delta(g);
        p.cnt = g.cnt;
        p.off = g.off;
        p.pout = 0;
        p.masks = nullptr;
    }
    b.probs_dev = dev_alloc_n<BProb>(B, s);
    SJ_HIP(hipMemcpyAsync(b.probs_dev, b.probs.data(), B * sizeof(BProb), hipMemcpyHostToDevice, s));
    b.total_items = b.item_base[B];
    if (b.total_items >= (int64_t(1) << 31)) throw std::string("too many work items in one batch");
    b.sched_key = "sched/" + std::to_string(B) + "/" + std::to_string(b.total_items);
    b.item_base_dev = dev_alloc_n<int64_t>(B + 1, s);
    SJ_HIP(hipMemcpyAsync(b.item_base_dev, b.item_base.data(), (B + 1) * sizeof(int64_t), hipMemcpyHostToDevice, s));
    // the queue: items grouped by d, longest first within a group
    const int64_t T = std::max<int64_t>(1, b.total_items);
    unsigned long long *ka = dev_alloc_n<unsigned long long>(T, s), *kb = dev_alloc_n<unsigned long long>(T, s);
    int32_t *va = dev_alloc_n<int32_t>(T, s), *vb = dev_alloc_n<int32_t>(T, s);
    // tile forms: d, the hit-list count's problems after the others
    int maxd = 1;
    for (int i = 0; i < B; ++i) maxd = std::max(maxd, b.grids[i]->d);
    std::map<int, int64_t> per_form;
    std::vector<int32_t> ids(2 * (size_t)B);  // form of each problem, then the other problems' indices
    for (int i = 0; i < B; ++i) {
        ids[i] = b.grids[i]->d + (b.in_hb[i] ? maxd + 1 : 0);
        if (b.grids[i]->items > 0) per_form[ids[i]] += b.grids[i]->items;
    }
    std::copy(rest.begin(), rest.end(), ids.begin() + B);
    b.rest = dev_alloc_n<int32_t>(2 * (size_t)B, s);
    SJ_HIP(hipMemcpyAsync(b.rest, ids.data(), ids.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
    SJ_HIP(hipStreamSynchronize(s));
    if (b.total_items > 0) {
        hipLaunchKernelGGL(k_item_cost, dim3((unsigned)((b.total_items + 255) / 256)), dim3(256), 0, s, b.probs_dev,
                           b.item_base_dev, b.rest, B, b.total_items, b.sym, ka, va);
        SJ_HIP(hipGetLastError());
    }
    int dbits = 0;
    while ((1 << dbits) <= 2 * maxd + 1) ++dbits;
    unsigned long long *k_sorted = ka;
    int32_t *v_sorted = va;
    radix_sort_pairs(&k_sorted, &v_sorted, k_sorted == ka ? kb : ka, v_sorted == va ? vb : va, b.total_items,
                     32 + dbits, s);
    b.queue = v_sorted;
    dev_free(v_sorted == va ? vb : va, s);
    dev_free(ka, s);
    dev_free(kb, s);
    // block queue: the block items of the problems whose FP64 MFMA count
    // stages tiles in LDS (2 to 4 K-steps, united lists), by d, longest first
    std::vector<int64_t> bbase(B + 1, 0);
    std::map<int, int64_t> per_d_blocks;
    auto lds_form = [](const Grid &g) {
        const int ks = g.da >> 2;
        return g.united && g.blocks && g.nblocks > 0 && ks >= 2 && ks <= 4;
    };
    for (int i = 0; i < B; ++i) {
        const Grid &g = *b.grids[i];
        const int64_t nb = lds_form(g) && !b.in_hb[i] ? g.nblocks : 0;
        bbase[i + 1] = bbase[i] + nb;
        if (nb) per_d_blocks[g.d] += nb;
    }
    if (bbase[B] > 0) {
        const int64_t NB = bbase[B];
        unsigned long long *bka = dev_alloc_n<unsigned long long>(NB, s), *bkb = dev_alloc_n<unsigned long long>(NB, s);
        int32_t *bva = dev_alloc_n<int32_t>(NB, s), *bvb = dev_alloc_n<int32_t>(NB, s);
        b.block_base_dev = dev_alloc_n<int64_t>(B + 1, s);
        SJ_HIP(hipMemcpyAsync(b.block_base_dev, bbase.data(), (B + 1) * sizeof(int64_t), hipMemcpyHostToDevice, s));
        hipLaunchKernelGGL(k_block_cost, dim3((unsigned)((NB + 255) / 256)), dim3(256), 0, s, b.probs_dev,
                           b.block_base_dev, B, NB, b.sym, bka, bva);
        SJ_HIP(hipGetLastError());
        unsigned long long *bks = bka;
        int32_t *bvs = bva;
        radix_sort_pairs(&bks, &bvs, bks == bka ? bkb : bka, bvs == bva ? bvb : bva, NB, 32 + dbits, s);
        b.bqueue = bvs;
        dev_free(bvs == bva ? bvb : bva, s);
        dev_free(bka, s);
        dev_free(bkb, s);
    }
    b.forms.clear();
    int64_t pos = 0, bpos = 0;
    for (auto &kv : per_form) {  // ascending, the key order
        BatchForm f;
        f.hits = kv.first > maxd;
        f.d = f.hits ? kv.first - maxd - 1 : kv.first;
        f.lo = (int32_t)pos;
        f.hi = (int32_t)(pos + kv.second);
        f.sched = 0;
        const int64_t nb = !f.hits && per_d_blocks.count(f.d) ? per_d_blocks[f.d] : 0;
        f.blo = (int32_t)bpos;
        f.bhi = (int32_t)(bpos + nb);
        bpos += nb;
        b.forms.push_back(f);
        pos += kv.second;
    }
    SJ_HIP(hipStreamSynchronize(s));
    b.totals.assign(B, 0);
    b.ms_build = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
}

// Captures `enqueue` (kernel nodes only: no memset or copy nodes) on the
// stream s (a private stream for the legacy null stream, which cannot be
// captured) into an executable graph.
template <typename F>
hipGraphExec_t capture(hipStream_t s, F enqueue) {
    hipStream_t cs = s;
    bool own = false;
    if (!cs) {
        SJ_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
        own = true;
    }
    hipGraph_t graph;
    hipGraphExec_t exec = nullptr;
    SJ_HIP(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    try {
        enqueue(cs);
    } catch (...) {
        (void)hipStreamEndCapture(cs, &graph);
        if (own) (void)hipStreamDestroy(cs);
        throw;
    }
    SJ_HIP(hipStreamEndCapture(cs, &graph));
    const hipError_t e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (own) SJ_HIP(hipStreamDestroy(cs));
    SJ_HIP(e);
    return exec;
}

void set_sched(Batch &b, int sched) {
    for (BatchForm &f : b.forms) f.sched = sched;
    b.sched = sched;
}

// In-masks of the problems that the count's tile kernels take (32 bytes per
// tile slot): the pairs pass then expands them instead of re-running the tiles (a
// half-stencil count records none). `all`: every problem, else those without
// the hit list.
void batch_masks(Batch &b, bool all, hipStream_t s) {
    int64_t tiles = 0;
    for (int i = 0; i < b.B; ++i)
        if (all || !b.in_hb[i]) tiles += b.grids[i]->tiles;
    if (b.sym || tiles * 32 > kBatchMaskBudget) tiles = 0;
    if (tiles > b.mask_tiles) {
        if (b.masks) dev_free(b.masks, s);
        b.masks = nullptr;
        b.mask_tiles = 0;
        try {
            b.masks = dev_alloc_n<unsigned long long>((size_t)tiles * 4, s);
            b.mask_tiles = tiles;
        } catch (const OomError &) {
            tiles = 0;
        }
    }
    int64_t at = 0;
    bool changed = false;
    for (int i = 0; i < b.B; ++i) {
        unsigned long long *m = nullptr;
        if (tiles > 0 && (all || !b.in_hb[i])) {
            // the problem's slots begin at `at`; its tile_off values at tile_base
            m = b.masks + 4 * (at - b.tile_base[i]);
            at += b.grids[i]->tiles;
        }
        changed = changed || m != b.probs[i].masks;
        b.probs[i].masks = m;
    }
    b.masks_valid = tiles > 0;
    if (changed) {
        SJ_HIP(hipMemcpyAsync(b.probs_dev, b.probs.data(), b.B * sizeof(BProb), hipMemcpyHostToDevice, s));
        SJ_HIP(hipStreamSynchronize(s));
    }
}

// Count pipeline: counter reset (and, for the half stencil, the per-point
// counts), one kernel per tile form (recording the in-masks when the batch
// holds them), per-problem prefix sums; captured on first use per (path,
// stream, schedule) and replayed.
float batch_count_graph(Batch &b, sj_path path, hipStream_t s) {
    const int pi = path == SJ_FP64_MFMA ? 1 : 0;
    if (!b.exec[pi] || b.graph_stream[pi] != s || b.graph_sched[pi] != b.sched) {
        if (b.exec[pi]) (void)hipGraphExecDestroy(b.exec[pi]);
        b.exec[pi] = nullptr;
        b.exec[pi] = capture(s, [&](hipStream_t cs) {
            batch_reset(b.ctr, cs);
            if (b.sym) launch_batch_zero_counts(b.probs_dev, b.B, b.max_n, cs);
            const bool hits = pi == 1 && !b.hb.probs.empty();
            for (const BatchForm &f : b.forms)
                if (!(hits && f.hits))
                    launch_batch_form(false, b.sym, f, path, b.probs_dev, b.item_base_dev, b.B, b.queue, nullptr, b.ctr,
                                      cs, b.block_base_dev, b.bqueue);
            launch_seg_scan(b.probs_dev, hits ? b.rest + b.B : nullptr, hits ? b.nrest : b.B, b.totals_dev, cs);
        });
        b.graph_stream[pi] = s;
        b.graph_sched[pi] = b.sched;
    }
    hipEvent_t e0, e1;
    SJ_HIP(hipEventCreate(&e0));
    SJ_HIP(hipEventCreate(&e1));
    SJ_HIP(hipEventRecord(e0, s));
    SJ_HIP(hipGraphLaunch(b.exec[pi], s));
    if (pi == 1 && !b.hb.probs.empty()) hit_batch_count(b.hb, !b.sym, b.ctr, b.totals.data(), s);
    SJ_HIP(hipEventRecord(e1, s));
    SJ_HIP(hipEventSynchronize(e1));
    float ms = 0;
    SJ_HIP(hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return ms;
}

float batch_count(Batch &b, sj_path path, hipStream_t s, HostCounters *hc) {
    b.counted = false;  // until this pass is through
    b.hits_counted = path == SJ_FP64_MFMA && !b.hb.probs.empty();
    batch_masks(b, !b.hits_counted, s);
    if (b.tune_sched) {
        // the schedule (persistent grids or one wave per item): both timed
        // once after a warm run, the faster kept (and cached by batch shape)
        b.tune_sched = false;
        std::lock_guard<std::mutex> lk(g_tune.mu);
        const std::string key = b.sched_key + "/" + std::to_string((int)path) + (b.sym ? "/sym" : "");
        auto it = g_tune.v.find(key);
        if (it != g_tune.v.end()) {
            set_sched(b, it->second);
        } else {
            float best = 1e30f;
            int best_s = 0;
            for (int sc = 0; sc < 2; ++sc) {
                set_sched(b, sc);
                batch_count_graph(b, path, s);
                const float ms = batch_count_graph(b, path, s);
                if (ms < best) {
                    best = ms;
                    best_s = sc;
                }
            }
            set_sched(b, best_s);
            g_tune.v[key] = best_s;
            tune_save(b.tune_cache.empty() ? nullptr : b.tune_cache.c_str());
        }
    }
    const float ms = batch_count_graph(b, path, s);
    DevCounters hb{};
    std::vector<int64_t> ht(b.B);
    SJ_HIP(hipMemcpyAsync(ht.data(), b.totals_dev, b.B * sizeof(int64_t), hipMemcpyDeviceToHost, s));
    SJ_HIP(hipMemcpyAsync(&hb, b.ctr, sizeof hb, hipMemcpyDeviceToHost, s));
    SJ_HIP(hipStreamSynchronize(s));
    *hc = read_counters(hb);
    for (int i = 0; i < b.B; ++i) {
        if (!(b.hits_counted && b.in_hb[i])) b.totals[i] = ht[i];
        b.grids[i]->total = b.totals[i];
        b.grids[i]->have_counts = true;
    }
    b.counted = true;
    return ms;
}

// The hit-list count's offsets into its problems' own arrays, for an emission
// that runs their tiles again.
void batch_offsets(Batch &b, hipStream_t s) {
    int64_t row0 = 0;
    for (int i : b.hb.probs) {
        Grid &g = *b.grids[i];
        hipLaunchKernelGGL(k_copy_offsets, dim3((unsigned)std::min<int64_t>((g.n + 256) / 256, 1024)), dim3(256), 0, s,
                           b.hb.off + row0, g.n + 1, g.off);
        SJ_HIP(hipGetLastError());
        row0 += g.n;
    }
}

// Emission of every problem's pairs into one buffer: problem i's rows at
// [offsets[i], offsets[i + 1]). The hit-list count's problems from its list; the
// others from the recorded in-masks when the batch holds them (one launch over
// all items), else their tiles re-run in emission form (one launch per tile
// form); captured per (path, stream, buffer).
float batch_pairs(Batch &b, sj_path path, int32_t *pairs, hipStream_t s) {
    std::vector<int64_t> pout(b.B);
    int64_t off = 0;
    for (int i = 0; i < b.B; ++i) {
        b.probs[i].pout = pout[i] = off;
        off += b.totals[i];
    }
    SJ_HIP(hipMemcpyAsync(b.probs_dev, b.probs.data(), b.B * sizeof(BProb), hipMemcpyHostToDevice, s));
    const int pi = path == SJ_FP64_MFMA ? 1 : 0;
    const bool use_masks = b.masks_valid;
    hipEvent_t e0, e1;
    SJ_HIP(hipEventCreate(&e0));
    SJ_HIP(hipEventCreate(&e1));
    SJ_HIP(hipEventRecord(e0, s));
    // the list: kept by the count, or (half-stencil option, a list that outgrew
    // its first guess) made again; without room for it those tiles run again too
    const bool hits = b.hits_counted && (b.hb.valid || hit_batch_ensure(b.hb, b.ctr, b.totals, s)) &&
                      hit_batch_bins(b.hb, s);
    if (b.hits_counted && !hits) batch_offsets(b, s);
    const int mode = (use_masks ? 1 : 0) | (b.hits_counted ? 2 : 0) | (hits ? 4 : 0);
    const bool tiles = !hits || b.rest_items > 0;  // something for the graph to launch
    if (tiles && (!b.pexec[pi] || b.pgraph_stream[pi] != s || b.pgraph_pairs[pi] != pairs || b.pgraph_mode[pi] != mode)) {
        if (b.pexec[pi]) (void)hipGraphExecDestroy(b.pexec[pi]);
        b.pexec[pi] = nullptr;
        b.pexec[pi] = capture(s, [&](hipStream_t cs) {
            if (use_masks)
                launch_batch_emit(b.probs_dev, b.item_base_dev, b.B, b.queue,
                                  (int)(b.hits_counted ? b.rest_items : b.total_items), 1, pairs, cs);
            for (const BatchForm &f : b.forms)
                if (f.hits && b.hits_counted ? !hits : !use_masks)
                    launch_batch_form(true, false, f, path, b.probs_dev, b.item_base_dev, b.B, b.queue, pairs, b.ctr, cs);
        });
        b.pgraph_stream[pi] = s;
        b.pgraph_pairs[pi] = pairs;
        b.pgraph_mode[pi] = mode;
    }
    if (tiles) SJ_HIP(hipGraphLaunch(b.pexec[pi], s));
    if (hits) hit_batch_pairs(b.hb, pout, pairs, s);
    SJ_HIP(hipEventRecord(e1, s));
    SJ_HIP(hipEventSynchronize(e1));
    float ms = 0;
    SJ_HIP(hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return ms;
}

}  // namespace sj

struct sj_batch {
    sj::Batch b;
};

using namespace sj;

#define SJB_TRY try {
#define SJB_CATCH                                                                      \
    }                                                                                  \
    catch (const HipError &e) {                                                        \
        set_error(e.where + ": " + hipGetErrorString(e.code));                         \
        return SJ_ERR_HIP;                                                             \
    }                                                                                  \
    catch (const OomError &e) {                                                        \
        set_error("device allocation of " + std::to_string(e.bytes) + " bytes failed"); \
        return SJ_ERR_OOM;                                                             \
    }                                                                                  \
    catch (const Unsupported &u) {                                                     \
        set_error(u.what);                                                             \
        return SJ_ERR_UNSUPPORTED;                                                     \
    }                                                                                  \
    catch (const std::string &msg) {                                                   \
        set_error(msg);                                                                \
        return SJ_ERR_INVALID;                                                         \
    }                                                                                  \
    catch (...) {                                                                      \
        set_error("unexpected exception");                                             \
        return SJ_ERR_HIP;                                                             \
    }

extern "C" {

sj_status selfjoin_batch_build(int32_t B, const double *const *points, const int64_t *n, const int32_t *d,
                               const double *eps, const sj_opts *opts, void *stream, sj_batch **out) {
    set_error("");
    if (!out || B < 0 || (B > 0 && (!points || !n || !d || !eps))) {
        set_error("invalid batch arguments");
        return SJ_ERR_INVALID;
    }
    for (int i = 0; i < B; ++i) {
        if (n[i] < 0 || n[i] > kMaxPoints || d[i] < 1 || d[i] > kMaxDims || !(eps[i] > 0.0) ||
            !std::isfinite(eps[i]) || (n[i] > 0 && !points[i])) {
            set_error("invalid arguments for batch problem " + std::to_string(i));
            return SJ_ERR_INVALID;
        }
    }
    if (opts && (opts->index_dims < 0 || opts->index_dims > kMaxIndexDims)) {
        set_error("index_dims must be in [0, 4]");
        return SJ_ERR_INVALID;
    }
    if (opts && (opts->short_circuit < -1 || opts->short_circuit > 64 || opts->dim_order < 0 || opts->dim_order > 1)) {
        set_error("short_circuit must be in [-1, 64] and dim_order 0 or 1");
        return SJ_ERR_INVALID;
    }
    if (opts && (opts->symmetric < 0 || opts->symmetric > 1)) {
        set_error("symmetric must be 0 or 1");
        return SJ_ERR_INVALID;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    sj_batch *h = new sj_batch();
    SJB_TRY
    try {
        batch_build(h->b, B, points, n, d, eps, opts, s);
    } catch (...) {
        batch_free(h->b, s);
        delete h;
        throw;
    }
    *out = h;
    return SJ_OK;
    SJB_CATCH
}

sj_status selfjoin_batch_count(sj_batch *bh, sj_path path, int64_t *totals, sj_stats *stats, void *stream) {
    set_error("");
    if (!bh || !totals) {
        set_error("NULL argument");
        return SJ_ERR_INVALID;
    }
    if (path != SJ_FP64_MFMA && path != SJ_FP64_VALU) {
        set_error("the batched form runs the FP64 paths");
        return SJ_ERR_UNSUPPORTED;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    SJB_TRY
    Batch &b = bh->b;
    HostCounters hc;
    const float ms = batch_count(b, path, s, &hc);
    int64_t sum = 0, cev = hc.met;  // (the hit list's problems)
    for (int i = 0; i < b.B; ++i) {
        totals[i] = b.totals[i];
        sum += b.totals[i];
    }
    if (stats && b.sym) {
        int64_t &cand = b.sym_cand[b.hits_counted ? 1 : 0];
        if (cand < 0) {  // ranges cut at each item's first query (once per batch)
            DevBuf<unsigned long long> acc(1, s);
            unsigned long long h = 0;
            fill_zero(acc.p, sizeof h, s);
            for (int i = 0; i < b.B; ++i)
                if (!(b.hits_counted && b.in_hb[i])) launch_sym_cand(*b.grids[i], acc.p, s);
            SJ_HIP(hipMemcpyAsync(&h, acc.p, sizeof h, hipMemcpyDeviceToHost, s));
            SJ_HIP(hipStreamSynchronize(s));
            cand = (int64_t)h;
        }
        cev += cand;
    } else {
        for (int i = 0; i < b.B; ++i)
            if (!(b.hits_counted && b.in_hb[i])) cev += b.grids[i]->cand_items;
    }
    if (stats) {
        std::memset(stats, 0, sizeof *stats);
        stats->cand_ref = -1;
        stats->cand_eval = cev;
        stats->pairs = sum;
        stats->rechecked = hc.rechecked;
        stats->rechecked_in = hc.rechecked_in;
        stats->ms = ms;
        stats->ms_build = b.ms_build;
        stats->ms_refine = ms;
        stats->tiles_pruned = hc.pruned;
        stats->path_run = (int32_t)path;
    }
    return SJ_OK;
    SJB_CATCH
}

sj_status selfjoin_batch_pairs(sj_batch *bh, sj_path path, int32_t *pairs, int64_t capacity, int64_t *offsets,
                               sj_stats *stats, void *stream) {
    set_error("");
    if (!bh || !offsets) {
        set_error("NULL argument");
        return SJ_ERR_INVALID;
    }
    if (path != SJ_FP64_MFMA && path != SJ_FP64_VALU) {
        set_error("the batched form runs the FP64 paths");
        return SJ_ERR_UNSUPPORTED;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    SJB_TRY
    Batch &b = bh->b;
    if (!b.counted) {
        HostCounters hc;
        batch_count(b, path, s, &hc);
    }
    int64_t sum = 0;
    for (int i = 0; i < b.B; ++i) sum += b.totals[i];
    if (sum > capacity) {
        offsets[b.B] = sum;
        set_error("capacity too small for the batch's pairs");
        return SJ_ERR_CAPACITY;
    }
    if (sum > 0 && !pairs) {
        set_error("pairs is NULL");
        return SJ_ERR_INVALID;
    }
    const float ms = batch_pairs(b, path, pairs, s);
    int64_t off = 0;
    for (int i = 0; i < b.B; ++i) {
        offsets[i] = off;
        off += b.totals[i];
    }
    offsets[b.B] = off;
    if (stats) {
        std::memset(stats, 0, sizeof *stats);
        stats->cand_ref = -1;
        stats->pairs = sum;
        stats->ms = ms;
        stats->ms_emit = ms;
        stats->path_run = (int32_t)path;
    }
    return SJ_OK;
    SJB_CATCH
}

sj_status selfjoin_batch_info(const sj_batch *bh, int32_t i, int32_t *index_dims, int64_t *items) {
    if (!bh || i < 0 || i >= bh->b.B) {
        set_error("invalid batch index");
        return SJ_ERR_INVALID;
    }
    if (index_dims) *index_dims = bh->b.grids[i]->k;
    if (items) *items = bh->b.grids[i]->items;
    return SJ_OK;
}

void selfjoin_batch_free(sj_batch *bh, void *stream) {
    if (!bh) return;
    try {
        batch_free(bh->b, static_cast<hipStream_t>(stream));
    } catch (...) {
    }
    delete bh;
}

}  // extern "C"
