// Hit-list count for d = 5 .. 64 (FP64, FP32 and split-BF16 MFMA tiles).
//
// At higher d a point has few neighbours among many candidates (the grid
// indexes at most four dimensions), so nearly every 16 x 16 tile is empty and
// the time goes into the tiles themselves. This count evaluates about half of
// them, drops those that cannot hold a pair before their rows are read, and
// records the few pairs it finds instead of a mask bit per candidate:
//
//  - Half of the tiles. Each unordered pair of block items (up to 64
//    consecutive rows of one grid line) meets in one place only: block a takes
//    block b > a when a + b is even, b < a when a + b is odd (so every block
//    takes about half of its neighbours, wherever it lies in the order), and
//    of its own rows the pairs (q, c > q). A pair within eps is a candidate of
//    both of its points, so either side may evaluate it.
//  - Box filter. Every work item (up to 16 consecutive rows) has a bounding
//    box over all d dimensions; an item has no pair with a query tile whose box
//    is more than eps from its own, and runs only against the others. In clustered data the grid's candidates
//    are mostly other clusters: on a 1M-point mixture of 100 clusters in 64
//    dimensions the lists hold 77k candidates a point, its cluster 10k.
//  - Hit list. A pair within eps is appended to a list (i, c) of sorted
//    indices and counted for both points; the pairs call sorts the list by
//    point. The lists of a 1M-point set with 50 neighbours a point take 0.2
//    GB, where a bit per candidate takes 10 GB.
//
// Measured, count + pairs of one join (MI355X): Gaussian mixture of 1M points
// and 50 neighbours, d = 16: count kernel 9.3 -> 4.2 ms, pairs 0.95 -> 1.6 ms;
// d = 64: count 144 -> 16.2 ms (10.7 ms of it FP64 MFMA). Index-free count of
// 65536 points, d = 16: 4.29 -> 1.46 ms (0.88 ms of MFMA). Uniform, 2M points,
// d = 5: 8.7 -> 3.9 ms.
//
// The box test is safe in FP32: boxes hold the centred coordinates times a
// power of two that puts eps in [1, 2), rounded outward and widened by one more
// step (which covers the rounding of the centring), a gap is one subtraction,
// and the threshold carries a relative margin of 1e-4 against at most
// 3 (d + 2) 2^-24 of the sum.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <climits>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <type_traits>

#include "sj_internal.h"
#include "sj_lowp.h"

namespace sj {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kRound = kThreads;    // candidate items tested per round
constexpr int kSurv = 2 * kRound;   // surviving items held for the tile loop
constexpr int kHitChunk = 256;      // list entries a wave reserves at a time
constexpr int kWaveBin = 1024;      // neighbours of a point that one wave orders in LDS
constexpr int kBigBits = 1 << 18;   // list positions per bitmap window of the larger ones

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef short short8_t __attribute__((ext_vector_type(8)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

struct HitGrid {
    const double *xs, *xa, *nrm;
    const int32_t *perm;
    const Item *items;
    const Range *ranges;
    const int32_t *blocks;       // first item of each block item, plus item_base
    const int32_t *item_block;   // block of each item
    const int2 *span;            // per block and range: candidate items [x, y)
    const float *blo, *bhi;      // boxes: [dimension][item], dimensions padded to a multiple of 4
    int64_t bstride;             // items per dimension of blo / bhi
    int32_t d, dp, da, nranges, nitems, nblocks, item_base;
    int32_t boxes;               // 0: no box test (short_circuit = -1)
    double sc, eps_s, eps2_s;    // low precision: the tiles' power-of-two scale, scaled eps and eps^2
    float thr;                   // box test: squared gap sum that drops an item (scaled units)
    double eps2;
};

struct HitOut {
    int32_t *cnt;                // per-point counts (sorted order), zeroed before the launch
    DevCounters *ctr;
    int2 *hits;                  // kHitRegions regions of `cap` entries, or null: count only
    unsigned long long *cursor;  // entries reserved in each region, kHitCursorStride apart
    unsigned long long *tally;   // kHitTally pairs (candidate pairs met, tiles dropped), kHitCursorStride apart
    unsigned long long cap;
    int32_t row0;                // list entries are rows plus this (batched form: the problem's first row)
};

// One problem of a batch's hit-list count. Its rows are [row0, row0 + n) of
// the batch's counts, offsets and list.
struct HitProb {
    HitGrid G;
    double delta;
    int32_t row0;
    int32_t nbox;      // index launch: blocks that make boxes (the others: candidate items)
    double sc;
    int64_t pout;      // first output row of this problem's pairs
};

__device__ __forceinline__ HitGrid hit_grid(const HitProb &P) {
    HitGrid G = P.G;
    G.xs = global_ptr(G.xs);
    G.xa = global_ptr(G.xa);
    G.nrm = global_ptr(G.nrm);
    G.perm = global_ptr(G.perm);
    G.items = global_ptr(G.items);
    G.ranges = global_ptr(G.ranges);
    G.blocks = global_ptr(G.blocks);
    G.item_block = global_ptr(G.item_block);
    G.span = global_ptr(G.span);
    G.blo = global_ptr(G.blo);
    G.bhi = global_ptr(G.bhi);
    return G;
}

__device__ __forceinline__ int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The oracle's chain: ascending dimensions from +0.0, fl(a - b) then fma.
__device__ __forceinline__ double exact_d2(const double *__restrict__ a, const double *__restrict__ b, int d) {
    double acc = 0.0;
    for (int t = 0; t < d; ++t) {
        const double delta = __dsub_rn(a[t], b[t]);
        acc = __fma_rn(delta, delta, acc);
    }
    return acc;
}

// Chunks of 16 consecutive blocks (which share candidates) dealt round-robin
// to the 8 XCDs; hardware block b runs on XCD b % 8.
__device__ __forceinline__ int xcd_block(int b, int nb) {
    constexpr int kChunk = 16;
    const int full = nb / (8 * kChunk) * (8 * kChunk);
    if (b >= full) return b;
    const int x = b & 7, k = b >> 3;
    return ((k / kChunk) * 8 + x) * kChunk + (k % kChunk);
}

__device__ __forceinline__ unsigned lane_rank(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

__device__ __forceinline__ int64_t readlane_i64(int64_t v, int lane) {
    const int lo = __builtin_amdgcn_readlane((int)(v & 0xffffffff), lane);
    const int hi = __builtin_amdgcn_readlane((int)(v >> 32), lane);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// ------------------------------------------------------------------ index --
__device__ __forceinline__ float below(float v) { return nextafterf(v, -INFINITY); }
__device__ __forceinline__ float above(float v) { return nextafterf(v, INFINITY); }

// First item in [a, b) whose end (END) or begin lies past x.
template <bool END>
__device__ __forceinline__ int first_item(const Item *__restrict__ items, int a, int b, int x) {
    while (a < b) {
        const int m = a + (b - a) / 2;
        if ((END ? items[m].qend : items[m].qbegin + 1) > x) b = m;
        else a = m + 1;
    }
    return a;
}

// The index of the count, in one launch. Blocks [0, nbox): boxes of 16 work
// items each, one wave per item at a time, lane t the column t of its rows
// (whole rows read), then whole runs of 16 items stored per dimension. The
// blocks after them: the candidate items of each block item and range (the
// items that hold a row of the range; an item lies in one line, so no item
// appears twice), and the block of each item.
__device__ __forceinline__ void hit_index_block(const HitGrid &G, double sc, unsigned block, unsigned nbox) {
    __shared__ float lo[kHitMaxD][17], hi[kHitMaxD][17];
    float *__restrict__ blo = const_cast<float *>(G.blo), *__restrict__ bhi = const_cast<float *>(G.bhi);
    int2 *__restrict__ span = const_cast<int2 *>(G.span);
    int32_t *__restrict__ item_block = const_cast<int32_t *>(G.item_block);
    if (block >= nbox) {  // whole block
        const int64_t t = (int64_t)(block - nbox) * kThreads + threadIdx.x;
        if (t >= (int64_t)G.nblocks * G.nranges) return;
        const int b = (int)(t / G.nranges), o = (int)(t - (int64_t)b * G.nranges);
        const int ib = G.blocks[b] - G.item_base, ie = G.blocks[b + 1] - G.item_base;
        if (o == 0)
            for (int i = ib; i < ie; ++i) item_block[i] = b;
        const Range r = G.ranges[(int64_t)ib * G.nranges + o];
        int2 s = make_int2(0, 0);
        if (r.end > r.begin) {
            s.x = first_item<true>(G.items, 0, G.nitems, r.begin);
            s.y = first_item<false>(G.items, s.x, G.nitems, r.end);
        }
        span[t] = s;
        return;
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int i0 = block * 16;
    for (int u = wv; u < 16; u += kWaves) {
        float l = -FLT_MAX, h = INFINITY;  // a padded dimension bounds nothing
        if (i0 + u < G.nitems && lane < G.d) {
            const Item I = G.items[i0 + u];
            double mn = INFINITY, mx = -INFINITY;
#pragma unroll 4
            for (int r = I.qbegin; r < I.qend; ++r) {
                const double v = G.xa[(int64_t)r * G.da + lane];
                mn = fmin(mn, v);
                mx = fmax(mx, v);
            }
            l = below(__double2float_rd(mn * sc));
            h = above(__double2float_ru(mx * sc));
        }
        lo[lane][u] = l;
        hi[lane][u] = h;
    }
    __syncthreads();
    const int dims = (G.d + 3) & ~3;
    for (int e = threadIdx.x; e < 16 * dims; e += kThreads) {
        const int t = e >> 4, u = e & 15;
        if (i0 + u < G.nitems) {
            blo[(int64_t)t * G.bstride + i0 + u] = lo[t][u];
            bhi[(int64_t)t * G.bstride + i0 + u] = hi[t][u];
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_hit_index(HitGrid G, double sc, unsigned nbox) {
    hit_index_block(G, sc, blockIdx.x, nbox);
}

// Last problem p with base[p] <= x.
template <typename T>
__device__ __forceinline__ int problem_of(const T *__restrict__ base, int B, T x) {
    int lo = 0, hi = B;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (base[mid] <= x) lo = mid;
        else hi = mid;
    }
    return uniform_i32(lo);
}

__global__ __launch_bounds__(kThreads) void k_hit_index_batch(const HitProb *__restrict__ P,
                                                              const int64_t *__restrict__ first, int B) {
    const int p = problem_of<int64_t>(first, B, blockIdx.x);
    const HitGrid G = hit_grid(P[p]);
    hit_index_block(G, P[p].sc, blockIdx.x - (unsigned)first[p], P[p].nbox);
}

// ------------------------------------------------------------- tile parts --
// What the tile loop of a block shares, whatever the tile's precision.
struct BlockShared {
    int2 surv[kSurv];     // surviving items: first row, rows | own block << 8 | query tiles near it << 16
    int pre[28], first[28];
    int wcount[kWaves];
    unsigned wmet[kWaves];
    int cntq[64];         // pairs of the block's rows as query
    float4_t alo[kHitMaxD], ahi[kHitMaxD];  // the four query tiles' boxes
};

// Walks a block's candidate items, kRound at a time, and keeps those of the
// block's half whose boxes are near enough. State is block-uniform except, per
// thread, the rows of its half's items and the tiles that their boxes dropped.
struct Walk {
    int total, pos, step;
    unsigned met, dropped;
};

__device__ __forceinline__ Walk walk_init(const HitGrid &G, BlockShared &S, int bi, int ib, int ie, int seg, int nseg) {
    const int tid = threadIdx.x;
    Walk W;
    if (tid < 64) {
        int2 s = make_int2(0, 0);
        if (tid < G.nranges) s = G.span[(int64_t)bi * G.nranges + tid];
        const int len = s.y - s.x;
        int incl = len;
        for (int o = 1; o < 32; o <<= 1) {
            const int y = __shfl_up(incl, o);
            if (tid >= o) incl += y;
        }
        if (tid < 28) {
            S.pre[tid] = tid < G.nranges ? incl - len : INT_MAX;
            S.first[tid] = s.x - (incl - len);
        }
        if (tid == 31) S.wcount[0] = incl;  // lanes past the ranges add nothing
    }
    if (tid < 64) S.cntq[tid] = 0;
    const int dims = (G.d + 3) & ~3;
    for (int e = tid; e < 4 * dims; e += kThreads) {
        const int t = e >> 2, i = min(ib + (e & 3), ie - 1);
        reinterpret_cast<float *>(S.alo)[e] = G.blo[(int64_t)t * G.bstride + i];
        reinterpret_cast<float *>(S.ahi)[e] = G.bhi[(int64_t)t * G.bstride + i];
    }
    __syncthreads();
    W.total = S.wcount[0];
    W.pos = seg * kRound;
    W.step = nseg * kRound;
    W.met = W.dropped = 0;
    __syncthreads();
    return W;
}

// Refills the survivor list (at least kRound entries unless the walk ends);
// returns their number. Every thread of the block calls it. An item is tested
// against the box of each of the block's query tiles, and the tiles that it is
// near go with it. Against one box around the whole block: Gaussian mixture, 1M
// points, d = 16, count and pairs 6.22 -> 6.11 ms; 200k points, d = 64 1.82 -> 1.75
// ms; uniform 2M points, d = 5 8.21 -> 8.10 ms.
__device__ __forceinline__ int walk_fill(const HitGrid &G, BlockShared &S, Walk &W, int bi, int nt) {
    const int tid = threadIdx.x, wv = tid >> 6;
    int have = 0;
    while (W.pos < W.total && have < kRound) {
        const int p = W.pos + tid;
        bool ok = false;
        int2 ent = make_int2(0, 0);
        if (p < W.total) {
            int o = 0;
#pragma unroll
            for (int st = 16; st > 0; st >>= 1)
                if (o + st < 28 && S.pre[o + st] <= p) o += st;
            const int it = S.first[o] + p;
            const int b = G.item_block[it];
            ok = b == bi || ((bi < b) == (((bi + b) & 1) == 0));
            if (ok) {
                const Item I = G.items[it];
                W.met += (unsigned)(I.qend - I.qbegin);
                unsigned near = (1u << nt) - 1u;  // query tiles
                if (G.boxes && b != bi) {
                    float s[4] = {0.f, 0.f, 0.f, 0.f};
                    for (int t = 0; t < G.d; t += 4) {
                        float l[4], h[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            l[u] = G.blo[(int64_t)(t + u) * G.bstride + it];
                            h[u] = G.bhi[(int64_t)(t + u) * G.bstride + it];
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const float4_t al = S.alo[t + u], ah = S.ahi[t + u];
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const float g = fmaxf(fmaxf(l[u] - ah[v], al[v] - h[u]), 0.f);
                                s[v] = fmaf(g, g, s[v]);
                            }
                        }
                        if (fminf(fminf(s[0], s[1]), fminf(s[2], s[3])) > G.thr) break;
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) near &= s[v] > G.thr ? ~(1u << v) : ~0u;
                    W.dropped += nt - __popc(near);
                    ok = near != 0u;
                }
                ent = make_int2(I.qbegin, (I.qend - I.qbegin) | (b == bi ? 256 : 0) | (int)(near << 16));
            }
        }
        const unsigned long long m = __ballot(ok);
        if ((tid & 63) == 0) S.wcount[wv] = __popcll(m);
        __syncthreads();
        int base = have;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            if (w < wv) base += S.wcount[w];
            have += S.wcount[w];
        }
        if (ok) S.surv[base + lane_rank(m)] = ent;
        __syncthreads();
        W.pos += W.step;
    }
    return have;
}

// A wave's run of reserved list entries.
struct HitRun {
    unsigned long long at;  // next entry (index into the region)
    int left;               // entries left
};

__device__ __forceinline__ void hit_pad(const HitOut &R, HitRun &H, int region, int lane) {
    for (int e = lane; e < H.left; e += 64)
        if (H.at + e < R.cap) R.hits[region * R.cap + H.at + e] = make_int2(-1, -1);
}

// Appends (q, c) for the lanes of m. Past the region's capacity the entries
// are only counted by the cursor (the list is then not valid).
__device__ __forceinline__ void hit_push(const HitOut &R, HitRun &H, int region, unsigned long long m, bool mine,
                                         int q, int c, int lane) {
    const int k = __popcll(m);
    if (k > H.left) {
        hit_pad(R, H, region, lane);
        unsigned long long a = 0;
        if (lane == 0) a = atomicAdd(R.cursor + region * kHitCursorStride, (unsigned long long)kHitChunk);
        H.at = ((unsigned long long)(unsigned)uniform_i32((int)(a >> 32)) << 32) | (unsigned)uniform_i32((int)a);
        H.left = kHitChunk;
    }
    if (mine) {
        const unsigned long long e = H.at + lane_rank(m);
        if (e < R.cap) R.hits[region * R.cap + e] = make_int2(R.row0 + q, R.row0 + c);
    }
    H.at += k;
    H.left -= k;
}

// A wave's share of the counters and of the list.
struct HitCtx {
    HitRun run;
    int region;
    unsigned long long band, band_in;  // wave-uniform
    int2 *wait;   // low precision: the wave's band pairs (row of the block, candidate), in LDS
    int waiting;  // their number (below kBandRun before a tile)
};
constexpr int kBandRun = 64;

// The chain of exact_d2 on padded rows (zero from d to dp, a multiple of 4:
// those steps add +0.0), 16 dimensions' loads in flight at a time.
__device__ __forceinline__ double exact_d2_rows(const double *__restrict__ a, const double *__restrict__ b, int dp) {
    double acc = 0.0;
    for (int t0 = 0; t0 < dp; t0 += 16) {
        double2 x[8], y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int t = min(t0 + 2 * u, dp - 2);
            x[u] = *reinterpret_cast<const double2 *>(a + t);
            y[u] = *reinterpret_cast<const double2 *>(b + t);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (t0 + 2 * u >= dp) break;
            const double d0 = __dsub_rn(x[u].x, y[u].x), d1 = __dsub_rn(x[u].y, y[u].y);
            acc = __fma_rn(d0, d0, acc);
            acc = __fma_rn(d1, d1, acc);
        }
    }
    return acc;
}

// Decides the first min(waiting, 64) of the wave's band pairs, one to a lane.
__device__ __forceinline__ void band_flush(const HitGrid &G, const HitOut &R, BlockShared &S, HitCtx &C, int q0,
                                           int lane) {
    const int n = min(C.waiting, 64);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int2 p = C.wait[min(lane, n - 1)];
    const int2 more = C.wait[64 + lane];
    const bool hit = lane < n && exact_d2_rows(G.xs + (int64_t)(q0 + p.x) * G.dp, G.xs + (int64_t)p.y * G.dp, G.dp) <=
                                     G.eps2;
    const unsigned long long w = __ballot(hit);
    C.band += (unsigned long long)n;
    C.band_in += (unsigned long long)__popcll(w);
    if (w) {
        if (hit) {
            atomicAdd(&S.cntq[p.x], 1);
            atomicAdd(R.cnt + p.y, 1);
        }
        if (R.hits) hit_push(R, C.run, C.region, w, hit, q0 + p.x, p.y, lane);
    }
    C.wait[lane] = more;  // those past the first 64 move up
    C.waiting -= n;
}

// The pairs of one tile: bit l of w[r] = the value of lane l's register r, row
// row0 + RS r of the block against candidate c, may be within eps; of in[r] =
// it is (the band between them is decided by the exact chain on the original
// coordinates: at once where the band is all but empty, else (DEFER) 64 pairs at
// a time, a pair to a lane, since the chain is a serial one over whole rows).
// own: a tile of the block's own rows, each pair once.
template <int RS, bool DEFER>
__device__ __forceinline__ void hit_record(const HitGrid &G, const HitOut &R, BlockShared &S, HitCtx &C,
                                           const unsigned long long wm[4], const unsigned long long in[4], int q0,
                                           int row0, int c, bool own, int lane) {
    int mine = 0;  // pairs of the lane's candidate in this tile
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        unsigned long long w = wm[r];
        const int q = q0 + row0 + RS * r;
        if (own) w &= __ballot(c > q);
        if (w == 0ull) continue;
        const unsigned long long bm = w & ~in[r];
        if (DEFER && bm != 0ull) {
            if (__builtin_amdgcn_inverse_ballot_w64(bm)) C.wait[C.waiting + lane_rank(bm)] = make_int2(row0 + RS * r, c);
            C.waiting += __popcll(bm);
            if (C.waiting >= kBandRun) band_flush(G, R, S, C, q0, lane);
            w &= ~bm;
            if (w == 0ull) continue;
        } else if (__builtin_expect(bm != 0ull, 0)) {
            bool ok = false;
            if (__builtin_amdgcn_inverse_ballot_w64(bm))
                ok = exact_d2(G.xs + (int64_t)q * G.dp, G.xs + (int64_t)c * G.dp, G.d) <= G.eps2;
            const unsigned long long okm = __ballot(ok);
            C.band += (unsigned long long)__popcll(bm);
            C.band_in += (unsigned long long)__popcll(okm);
            w = (w & ~bm) | okm;
            if (w == 0ull) continue;
        }
        const bool hit = __builtin_amdgcn_inverse_ballot_w64(w);
        if (hit) {
            ++mine;
            atomicAdd(&S.cntq[row0 + RS * r], 1);
        }
        if (R.hits) hit_push(R, C.run, C.region, w, hit, q, c, lane);
    }
    if (mine) atomicAdd(R.cnt + c, mine);
}

// The end of a block: the list's last entries, the rows' counts as query (and
// the point itself, once per row), the counters.
template <bool DROPPED>
__device__ __forceinline__ void hit_finish(const HitOut &R, BlockShared &S, HitCtx &C, const Walk &W, int q0, int nrows,
                                           int seg) {
    const int tid = threadIdx.x, lane = tid & 63;
    if (R.hits) hit_pad(R, C.run, C.region, lane);
    __syncthreads();
    if (tid < nrows) {
        const int v = S.cntq[tid] + (seg == 0 ? 1 : 0);
        if (v) atomicAdd(R.cnt + q0 + tid, v);
    }
    unsigned dr = DROPPED ? W.dropped : 0, met = W.met;
    for (int sh = 32; sh > 0; sh >>= 1) {
        if (DROPPED) dr += __shfl_xor(dr, sh);
        met += __shfl_xor(met, sh);
    }
    if (lane == 0) {
        if (DROPPED) S.wcount[tid >> 6] = (int)dr;
        S.wmet[tid >> 6] = met;
        if (C.band) {
            atomicAdd(&R.ctr->rechecked, C.band);
            atomicAdd(&R.ctr->rechecked_in, C.band_in);
        }
    }
    __syncthreads();
    if (tid == 0) {
        unsigned long long d = 0, m = 0;
        for (int w = 0; w < kWaves; ++w) {
            if (DROPPED) d += (unsigned)S.wcount[w];
            m += S.wmet[w];
        }
        // (on one address the blocks' atomics would queue up, 13 ns each: 2.25 -> 2.63 ms for 2.4M points)
        unsigned long long *T = R.tally + (blockIdx.x & (kHitTally - 1)) * kHitCursorStride;
        if (m) atomicAdd(T, m * (unsigned long long)nrows);
        if (DROPPED && d) atomicAdd(T + 1, d);
    }
}

// ------------------------------------------------------------------- FP64 --
// One wave runs the block's (up to) four 16-row query tiles against one
// candidate item at a time: its B operand is loaded straight into registers
// (one item ahead), the A operand (-2 q, zero past d) of all four tiles sits in
// LDS, so a candidate row is read once per 64 queries, nothing in the loop
// waits on another wave, and the four tiles' chains are independent. Bound by
// the FP64 matrix unit: KS MFMAs of 64 cycles per tile and about 16 vector
// instructions, which the counters show on top of them rather than beside them
// (256 problems, d = 16: 112M cycles per SIMD of MFMA and 27M of vector issue in
// 151M). K order: two K-steps share one 16-byte load of the row (lane g
// holds dimensions 8p + 2g and 8p + 2g + 1 of K-step pair p), a last single
// K-step dimension 4 (KS - 1) + g.
// The accumulator starts at |q|^2 (+inf for absent rows), so D = |q|^2 - 2 q.c
// and a value is in iff D <= eps^2 - |c|^2; the band of +-Delta around it goes
// to the exact chain (the sum of the same terms as in k_m64, in another order,
// which its Delta covers).
template <int KS>
struct HitTile {
    double b[KS];
    double nc;
    int c, n;  // the lane's column: its row; the item's survivor word
};

template <int KS>
__device__ __forceinline__ void hit_load(HitTile<KS> &T, int2 e, const HitGrid &G, int g, int j) {
    const int n = e.y & 255;
    T.n = e.y;
    T.c = e.x + min(j, n - 1);
    const double *__restrict__ row = G.xa + (int64_t)T.c * G.da;
#pragma unroll
    for (int p = 0; p < KS / 2; ++p) {
        const double2 v = *reinterpret_cast<const double2 *>(row + 8 * p + 2 * g);
        T.b[2 * p] = v.x;
        T.b[2 * p + 1] = v.y;
    }
    if (KS & 1) T.b[KS - 1] = row[4 * (KS - 1) + g];
    T.nc = G.nrm[T.c];
}

// The high word of a double as a float: the same order (sign, exponent,
// leading mantissa bits), so x <= y implies high(x) <= high(y); infinities
// become NaN, below nothing. FP64 compares would contend with the MFMAs for
// the FP64 pipe; this test only has to let every candidate value through.
__device__ __forceinline__ float high(double v) { return __int_as_float(__double2hiint(v)); }
__device__ __forceinline__ float low4(const double4_t &v) {
    return fminf(fminf(high(v[0]), high(v[1])), fminf(high(v[2]), high(v[3])));
}

template <int KS>
constexpr int hit_k(int s, int g) {
    return (s == KS - 1 && (KS & 1)) ? 4 * s + g : 8 * (s >> 1) + 2 * g + (s & 1);
}

template <int KS>
__device__ __forceinline__ void hit_f64_block(const HitGrid &G, const HitOut &R, double delta, int bi, int seg,
                                              int nseg) {
    __shared__ double A[4 * KS * 64];
    __shared__ double4_t qn[4 * 4];  // [tile][row group g]: |q|^2 of rows g + 4r
    __shared__ BlockShared S;
    const int tid = threadIdx.x, lane = tid & 63, wv = uniform_i32(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int ib = uniform_i32(G.blocks[bi] - G.item_base), ie = uniform_i32(G.blocks[bi + 1] - G.item_base);
    const int nt = ie - ib;
    // the block's rows are consecutive: only the last item can be short
    const int q0 = uniform_i32(G.items[ib].qbegin);
    const int nrows = uniform_i32(G.items[ie - 1].qend) - q0;
    for (int e = tid; e < nt * KS * 64; e += kThreads) {
        const int ln = e & 63, s = (e >> 6) % KS, t = (e >> 6) / KS;
        const int row = 16 * t + (ln & 15), k = hit_k<KS>(s, ln >> 4);
        A[e] = (row < nrows && k < G.d) ? -2.0 * G.xa[(int64_t)(q0 + row) * G.da + k] : 0.0;
    }
    if (tid < 64) {
        const int t = tid >> 4, gg = (tid >> 2) & 3, r = tid & 3, row = 16 * t + gg + 4 * r;
        reinterpret_cast<double *>(qn)[tid] = row < nrows ? G.nrm[q0 + row] : INFINITY;
    }
    Walk W = walk_init(G, S, bi, ib, ie, seg, nseg);
    HitCtx C{{0, 0}, (int)((blockIdx.x ^ (blockIdx.x >> 4)) & (kHitRegions - 1)), 0, 0, nullptr, 0};
    const double clo = G.eps2 - delta, chi = G.eps2 + delta;
    auto record = [&](const HitTile<KS> &T, const double4_t &acc, int t, bool valid, bool own) {
        const double hi = valid ? chi - T.nc : -INFINITY, lo = valid ? clo - T.nc : -INFINITY;
        unsigned long long w[4], in[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            w[r] = __ballot(acc[r] <= hi);
            in[r] = __ballot(acc[r] <= lo);
        }
        hit_record<4, false>(G, R, S, C, w, in, q0, 16 * t + g, T.c, own, lane);
    };
    auto run = [&](const HitTile<KS> &T) {
        const int tn = uniform_i32(T.n);
        const bool own = (tn & 256) != 0, valid = j < (tn & 255);
        const float thr = high(valid ? chi - T.nc : -INFINITY);
        const double *a = A + lane;
        for (int near = tn >> 16; near; near &= near - 1) {
            const int t = __builtin_ctz(near);
            double4_t acc = qn[4 * t + g];
#pragma unroll
            for (int s = 0; s < KS; ++s)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[(t * KS + s) * 64], T.b[s], acc, 0, 0, 0);
            if (__ballot(low4(acc) <= thr)) record(T, acc, t, valid, own);
        }
    };
    for (;;) {
        const int ns = walk_fill(G, S, W, bi, nt);
        if (ns == 0) break;
        HitTile<KS> T0, T1;
        if (wv < ns) hit_load<KS>(T0, S.surv[wv], G, g, j);
        for (int e = wv; e < ns; e += 2 * kWaves) {
            // past the end the loads repeat the last item (the same count on every path)
            hit_load<KS>(T1, S.surv[min(e + kWaves, ns - 1)], G, g, j);
            run(T0);
            if (e + kWaves >= ns) break;
            hit_load<KS>(T0, S.surv[min(e + 2 * kWaves, ns - 1)], G, g, j);
            run(T1);
        }
        __syncthreads();
    }
    hit_finish<true>(R, S, C, W, q0, nrows, seg);
}

template <int KS>
__global__ __launch_bounds__(kThreads, KS <= 8 ? 4 : 3) void k_hit_f64(HitGrid G, HitOut R, double delta, int nseg) {
    const int lb = xcd_block(blockIdx.x, gridDim.x);
    const int bi = lb / nseg;
    hit_f64_block<KS>(G, R, delta, bi, lb - bi * nseg, nseg);
}

// The block items of many problems (queue: global block indices, longest
// first; block_base: the problems' first).
template <int KS>
__global__ __launch_bounds__(kThreads, KS <= 8 ? 4 : 3) void k_hit_f64_batch(const HitProb *__restrict__ P,
                                                                              const int64_t *__restrict__ block_base,
                                                                              int B, const int32_t *__restrict__ queue,
                                                                              HitOut R, int nseg) {
    const int pos = blockIdx.x / nseg;
    const int gb = uniform_i32(queue[pos]);
    const int p = problem_of<int64_t>(block_base, B, gb);
    const HitGrid G = hit_grid(P[p]);
    R.row0 = P[p].row0;
    R.cnt += R.row0;
    hit_f64_block<KS>(G, R, P[p].delta, gb - (int)block_base[p], blockIdx.x - pos * nseg, nseg);
}

// ---------------------------------------------------------- low precision --
// FP32 and split-BF16 tiles (rounding, band and test of k_lowp, sj_lowp.hip):
// rows centred on the block's first query, scaled and rounded; D = |c'|^2 -
// 2 q'.c' with the candidate norm (FP64, rounded once) in the accumulator and a
// threshold pair per row. A wave rounds a candidate item in its own registers,
// straight from the FP64 rows, and runs the block's four query tiles against
// it: five FP64 and a few FP32 operations per coordinate for 64 queries, and no
// staging of tiles through LDS, which bounded the block kernels (two barriers
// per 64 candidates, every rounded value written and read back). FP32 is then
// bound by its MFMAs (32 cycles per K-step of 4 and tile), split BF16 by the
// rounding (about 700 cycles per item at d = 64 against 384 of MFMA). Gaussian
// mixture, 1M points: FP32, d = 32 21.7 -> 5.5 ms; split BF16, d = 64 86 -> 9.2 ms
// (33 ms with the band pairs rechecked one by one where they were met).
// K order: FP32 as in the FP64 tiles; split BF16 lane g holds dimensions
// 32 s + 8 g .. + 7.
template <int PREC, int KS>
struct LpTile {
    static constexpr int NB = PREC == PREC_F32 ? KS : 8 * KS;  // coordinates per lane
    double b[NB];
    int c, n;
};

// Dimension of the lane's coordinate u.
template <int PREC, int KS>
__device__ __forceinline__ int lp_k(int u, int g) {
    if (PREC == PREC_F32) return hit_k<KS>(u, g);
    return 32 * (u >> 3) + 8 * g + (u & 7);
}

template <int PREC, int KS>
__device__ __forceinline__ void lp_load(LpTile<PREC, KS> &T, int2 e, const HitGrid &G, int g, int j) {
    T.n = e.y;
    T.c = e.x + min(j, (e.y & 255) - 1);
    const double *__restrict__ row = G.xs + (int64_t)T.c * G.dp;
#pragma unroll
    for (int u = 0; u + 1 < LpTile<PREC, KS>::NB; u += 2) {
        const int k = lp_k<PREC, KS>(u, g);
        // rows are zero from d to dp (a multiple of 4); past dp nothing is read
        double2 v = make_double2(0.0, 0.0);
        if (PREC == PREC_F32 || k < G.dp) v = *reinterpret_cast<const double2 *>(row + k);
        T.b[u] = v.x;
        T.b[u + 1] = v.y;
    }
    if (PREC == PREC_F32 && (KS & 1)) T.b[KS - 1] = row[4 * (KS - 1) + g];
}

// Two values to BF16 (round to nearest even), the first in the low half.
__device__ __forceinline__ unsigned bf16_pair(float a, float b) {
    const bf16x2_t v = __builtin_convertvector((float2_t){a, b}, bf16x2_t);
    return __builtin_bit_cast(unsigned, v);
}

template <int PREC, int KS>
__global__ __launch_bounds__(kThreads, PREC == PREC_F32 ? (KS <= 10 ? 4 : 3) : (KS == 1 ? 4 : 3)) void k_hit_lp(
    HitGrid G, HitOut R, int nseg) {
    using Tile = LpTile<PREC, KS>;
    constexpr int NB = Tile::NB;
    constexpr int NP = PREC == PREC_F32 ? 1 : 2;  // parts of an operand (hi, lo)
    // A operand of lane l: FP32 one float per K-step, split BF16 eight halves (hi parts, then lo parts)
    __shared__ uint4 Abuf[PREC == PREC_F32 ? KS * 64 : NP * 4 * KS * 64];
    __shared__ double xr[64];
    __shared__ int2 wait[kWaves][2 * kBandRun];
    __shared__ float4_t thi[16], tlo[16];  // [tile][row group g]: thresholds of rows 4g + r
    __shared__ BlockShared S;
    const int tid = threadIdx.x, lane = tid & 63, wv = uniform_i32(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int lb = xcd_block(blockIdx.x, gridDim.x);
    const int bi = lb / nseg, seg = lb - bi * nseg;
    const int ib = uniform_i32(G.blocks[bi] - G.item_base), ie = uniform_i32(G.blocks[bi + 1] - G.item_base);
    const int nt = ie - ib;
    const int q0 = uniform_i32(G.items[ib].qbegin);
    const int nrows = uniform_i32(G.items[ie - 1].qend) - q0;
    if (tid < 64) xr[tid] = tid < G.dp ? G.xs[(int64_t)q0 * G.dp + tid] : 0.0;
    __syncthreads();
    // wave t rounds query tile t (rows 16 t + j) as the tile loop rounds candidates
    {
        const int row = 16 * wv + j;
        double nn = 0.0;
        const double *__restrict__ q = G.xs + (int64_t)(q0 + min(row, nrows - 1)) * G.dp;
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int k = lp_k<PREC, KS>(u, g);
            unsigned bits = 0;
            double y = 0.0;
            if (row < nrows && k < G.d) y = round_in<PREC>(__dsub_rn(q[k], xr[k]) * G.sc, bits);
            nn = __fma_rn(y, y, nn);
            if constexpr (PREC == PREC_F32) {
                reinterpret_cast<float *>(Abuf)[(wv * KS + u) * 64 + lane] = -2.0f * __uint_as_float(bits);
            } else {  // -2 hi and -2 lo are exact
                unsigned short *h = reinterpret_cast<unsigned short *>(Abuf + (wv * KS + (u >> 3)) * 64 + lane);
                unsigned short *l = reinterpret_cast<unsigned short *>(Abuf + ((4 + wv) * KS + (u >> 3)) * 64 + lane);
                h[u & 7] = f32_to_bf16(-2.0f * bf16_to_f32((unsigned short)(bits & 0xffffu)));
                l[u & 7] = f32_to_bf16(-2.0f * bf16_to_f32((unsigned short)(bits >> 16)));
            }
        }
        nn += __shfl_xor(nn, 16);
        nn += __shfl_xor(nn, 32);  // |q'|^2 of row j in every lane of its column
        double dl = 0.0;
        if (g == 0) {
            const int K = PREC == PREC_F32 ? 4 * KS : 32 * KS;
            dl = lp_delta<PREC>(nn, G.eps_s, G.eps2_s, G.d, K);
            const double thr = G.eps2_s - nn;
            const bool ok = row < nrows;
            reinterpret_cast<float *>(thi)[16 * wv + j] = ok ? (float)(thr + dl) : -INFINITY;
            reinterpret_cast<float *>(tlo)[16 * wv + j] = ok ? (float)(thr - dl) : -INFINITY;
            if (!ok) dl = 0.0;
        }
        for (int sh = 8; sh > 0; sh >>= 1) dl = fmax(dl, __shfl_xor(dl, sh));
        if (lane == 0 && seg == 0) atomicMax(&R.ctr->max_delta, (unsigned long long)__double_as_longlong(dl));
    }
    Walk W = walk_init(G, S, bi, ib, ie, seg, nseg);
    HitCtx C{{0, 0}, (int)((blockIdx.x ^ (blockIdx.x >> 4)) & (kHitRegions - 1)), 0, 0, wait[wv], 0};

    auto run = [&](const Tile &T) {
        const int tn = uniform_i32(T.n);
        const bool own = (tn & 256) != 0, valid = j < (tn & 255);
        // round the candidate: y = (x - r) sc in FP64, then as round_in
        float f[NB];
        double np = 0.0;
#pragma unroll
        for (int u = 0; u < NB; ++u) f[u] = (float)(__dsub_rn(T.b[u], xr[lp_k<PREC, KS>(u, g)]) * G.sc);
        short8_t bh[PREC == PREC_F32 ? 1 : KS], bl[PREC == PREC_F32 ? 1 : KS];
        if constexpr (PREC == PREC_F32) {
#pragma unroll
            for (int u = 0; u < NB; ++u) np = __fma_rn((double)f[u], (double)f[u], np);
        } else {
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                uint4 h, l;
                unsigned *hw = reinterpret_cast<unsigned *>(&h), *lw = reinterpret_cast<unsigned *>(&l);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float f0 = f[8 * s + 2 * e], f1 = f[8 * s + 2 * e + 1];
                    const unsigned hp = bf16_pair(f0, f1);
                    const float h0 = __uint_as_float(hp << 16), h1 = __uint_as_float(hp & 0xffff0000u);
                    const unsigned lp = bf16_pair(f0 - h0, f1 - h1);  // differences exact
                    // hi + lo is a multiple of f's last place not above it by more than one: exact in FP32
                    const double v0 = (double)(h0 + __uint_as_float(lp << 16));
                    const double v1 = (double)(h1 + __uint_as_float(lp & 0xffff0000u));
                    np = __fma_rn(v0, v0, np);
                    np = __fma_rn(v1, v1, np);
                    hw[e] = hp;
                    lw[e] = lp;
                }
                bh[s] = __builtin_bit_cast(short8_t, h);
                bl[s] = __builtin_bit_cast(short8_t, l);
            }
        }
        np += __shfl_xor(np, 16);
        np += __shfl_xor(np, 32);
        const float nc = valid ? (float)np : INFINITY;
        for (int near = tn >> 16; near; near &= near - 1) {
            const int t = __builtin_ctz(near);
            float4_t acc = (float4_t){nc, nc, nc, nc};
            const float4_t hi = thi[4 * t + g];
            if constexpr (PREC == PREC_F32) {
                const float *a = reinterpret_cast<const float *>(Abuf) + t * KS * 64 + lane;
#pragma unroll
                for (int s = 0; s < KS; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s * 64], f[s], acc, 0, 0, 0);
            } else {
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const short8_t ah = __builtin_bit_cast(short8_t, Abuf[(t * KS + s) * 64 + lane]);
                    const short8_t al = __builtin_bit_cast(short8_t, Abuf[((4 + t) * KS + s) * 64 + lane]);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh[s], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl[s], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[s], acc, 0, 0, 0);
                }
            }
            unsigned long long w[4], in[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) w[r] = __ballot(acc[r] <= hi[r]);
            if ((w[0] | w[1] | w[2] | w[3]) == 0ull) continue;
            const float4_t lo = tlo[4 * t + g];
#pragma unroll
            for (int r = 0; r < 4; ++r) in[r] = __ballot(acc[r] <= lo[r]);
            hit_record<1, true>(G, R, S, C, w, in, q0, 16 * t + 4 * g, T.c, own, lane);
        }
    };
    for (;;) {
        const int ns = walk_fill(G, S, W, bi, nt);
        if (ns == 0) break;
        Tile T0, T1;
        if (wv < ns) lp_load(T0, S.surv[wv], G, g, j);
        for (int e = wv; e < ns; e += 2 * kWaves) {
            lp_load(T1, S.surv[min(e + kWaves, ns - 1)], G, g, j);
            run(T0);
            if (e + kWaves >= ns) break;
            lp_load(T0, S.surv[min(e + 2 * kWaves, ns - 1)], G, g, j);
            run(T1);
        }
        __syncthreads();
    }
    if (C.waiting) band_flush(G, R, S, C, q0, lane);
    hit_finish<false>(R, S, C, W, q0, nrows, seg);  // tiles_pruned is 0 on these paths
}

// --------------------------------------------------------------- hit list --
// From the list to the bins. Point i's bin holds its other neighbours,
// [off[i], off[i + 1] - 1), in any order. Both points of a pair are anywhere in
// the set, so placing the pairs one by one costs two returning atomics and two
// scattered stores a pair (1.6 ms for 25M pairs of a 1M-point set). Instead the
// points are cut into buckets of 2^sh consecutive ones (at most kBuckets; a
// bucket's share of the bins is known from off): k_hit_part deals the pairs to
// the buckets, a slab of the list at a time with one reservation per slab and
// bucket, and k_hit_place then orders each bucket by point with LDS counters,
// its stores staying inside the bucket's own stretch of the bins.
constexpr int kBuckets = 4096;
constexpr int kPartThreads = 512;
constexpr int kPartItems = 16;
constexpr int kSlab = kPartThreads * kPartItems;

__global__ __launch_bounds__(kPartThreads) void k_hit_part(const int2 *__restrict__ hits,
                                                           const unsigned long long *__restrict__ cursor,
                                                           unsigned long long cap, const int64_t *__restrict__ off,
                                                           int sh, int nbuckets, unsigned *__restrict__ fill,
                                                           uint2 *__restrict__ part) {
    __shared__ unsigned slot[kBuckets];
    const int2 *h = hits + blockIdx.y * cap;
    const int64_t n = (int64_t)min(cursor[blockIdx.y * kHitCursorStride], cap);
    const int tid = threadIdx.x;
    for (int64_t s0 = (int64_t)blockIdx.x * kSlab; s0 < n; s0 += (int64_t)gridDim.x * kSlab) {
        for (int b = tid; b < nbuckets; b += kPartThreads) slot[b] = 0;
        __syncthreads();
        int2 p[kPartItems];
        unsigned rank[kPartItems];  // ranks within the slab's share of the two buckets (each below 2^14 + 1)
#pragma unroll
        for (int k = 0; k < kPartItems; ++k) {
            const int64_t e = s0 + k * kPartThreads + tid;
            p[k] = e < n ? h[e] : make_int2(-1, -1);
        }
#pragma unroll
        for (int k = 0; k < kPartItems; ++k)
            if (p[k].x >= 0) {
                const unsigned r = atomicAdd(&slot[p[k].x >> sh], 1u);
                rank[k] = r | (atomicAdd(&slot[p[k].y >> sh], 1u) << 16);
            }
        __syncthreads();
        for (int b = tid; b < nbuckets; b += kPartThreads) {
            const unsigned c = slot[b];
            const int64_t first = (int64_t)b << sh;
            if (c) slot[b] = (unsigned)(off[first] - first) + atomicAdd(fill + b, c);
        }
        __syncthreads();
        const unsigned mask = (1u << sh) - 1u;
#pragma unroll
        for (int k = 0; k < kPartItems; ++k)
            if (p[k].x >= 0) {
                part[slot[p[k].x >> sh] + (rank[k] & 0xffffu)] = make_uint2((unsigned)p[k].x & mask, (unsigned)p[k].y);
                part[slot[p[k].y >> sh] + (rank[k] >> 16)] = make_uint2((unsigned)p[k].y & mask, (unsigned)p[k].x);
            }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kThreads) void k_hit_place(const uint2 *__restrict__ part,
                                                        const int64_t *__restrict__ off, int64_t n, int sh,
                                                        int32_t *__restrict__ bin) {
    extern __shared__ unsigned at[];  // next free place of each point, from the bucket's first
    const int64_t p0 = (int64_t)blockIdx.x << sh, p1 = min(n, p0 + (int64_t(1) << sh));
    const int64_t o0 = off[p0];
    for (int64_t i = p0 + threadIdx.x; i < p1; i += kThreads) at[i - p0] = (unsigned)(off[i] - o0);
    __syncthreads();
    const int64_t m = off[p1] - o0 - (p1 - p0);
    const uint2 *src = part + (o0 - p0);
    int32_t *dst = bin + o0;
#pragma unroll 4
    for (int64_t e = threadIdx.x; e < m; e += kThreads) {
        const uint2 v = src[e];
        dst[atomicAdd(&at[v.x], 1u)] = (int32_t)v.y;
    }
}

// The pairs placed one by one, for lists too long for 32-bit bucket places.
__global__ __launch_bounds__(kThreads) void k_hit_bin(const int2 *__restrict__ hits,
                                                      const unsigned long long *__restrict__ cursor,
                                                      unsigned long long cap, const int64_t *__restrict__ off,
                                                      int32_t *__restrict__ fill, int32_t *__restrict__ bin) {
    const int2 *h = hits + blockIdx.y * cap;
    const int64_t n = (int64_t)min(cursor[blockIdx.y * kHitCursorStride], cap);
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int2 p = h[e];
        if (p.x < 0) continue;
        bin[off[p.x] + atomicAdd(fill + p.x, 1)] = p.y;
        bin[off[p.y] + atomicAdd(fill + p.y, 1)] = p.x;
    }
}

// Position of a candidate row in an item's list (its ranges in order): the
// ranges sorted by row are the ranges in the order of their line keys (the
// base-3 digits of the range index reversed), so a binary search over them
// finds the row's range. sb / sd: per sorted slot u < 27 the begin of the last
// non-empty range up to u, and its list position minus its begin.
struct ListMap {
    int sb[32], sd[32];
};

// Returns the list's length.
__device__ __forceinline__ int list_map(const HitGrid &G, int it, int lane, ListMap &M) {
    int rb = 0, len = 0;
    if (lane < G.nranges) {
        const Range r = G.ranges[(int64_t)it * G.nranges + lane];
        rb = r.begin;
        len = max(0, r.end - r.begin);
    }
    int incl = len;
    for (int o = 1; o < 32; o <<= 1) {
        const int y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    const int dl = incl - len - rb;
    // slot u holds range o(u): the base-3 digits reversed
    int u = lane, o = 0;
    for (int m = G.nranges; m > 1; m /= 3) {
        o = o * 3 + u % 3;
        u /= 3;
    }
    int src = lane < G.nranges ? o : 0;
    const int rbs = __shfl(rb, src), dls = __shfl(dl, src), lens = __shfl(len, src);
    int x = (lane < G.nranges && lens > 0) ? lane : -1;  // last non-empty slot so far
    for (int s = 1; s < 32; s <<= 1) {
        const int y = __shfl_up(x, s);
        if (lane >= s) x = max(x, y);
    }
    const int fb = __shfl(rbs, max(x, 0)), fd = __shfl(dls, max(x, 0));
    if (lane < 32) {
        M.sb[lane] = lane >= G.nranges ? INT_MAX : (x >= 0 ? fb : INT_MIN);
        M.sd[lane] = fd;
    }
    return __builtin_amdgcn_readlane(incl, 31);
}

__device__ __forceinline__ int list_pos(const ListMap &M, int c) {
    int o = 0;
#pragma unroll
    for (int st = 16; st > 0; st >>= 1)
        if (M.sb[o + st] <= c) o += st;
    return c + M.sd[o];
}

// Pairs of the points [qlo, qhi), one wave per work item (or a part of one): a
// point's bin and the point itself, ordered by list position (the candidate
// order). A neighbour's rank is found in one of two ways, whichever takes fewer
// instructions: the number of smaller positions, compared against all of them
// from LDS, four to a read (few neighbours in a long list); or a bitmap of the
// list positions in LDS, kWinBits of them at a time, with the number of bits
// before each word (many neighbours: 21M pairs of a skewed set of 216408 points
// in 5 dimensions took 1.21 ms by comparison alone, the dense points having
// hundreds of neighbours). Points with more than kWaveBin neighbours go to
// k_hit_emit_big.
constexpr int kWinBits = 32768;

struct EmitOut {
    const int64_t *off;
    const int32_t *bin;
    int64_t base;
    int32_t qlo, qhi, item_lo, item_hi;
    int2 *pairs;
    double *d2;
    int32_t *big;  // [0]: number, then (point, item) of the larger ones
    int32_t per;   // queries of an item that one wave takes (a power of two up to 16)
    int32_t row0;  // the bins hold rows plus this
};

// What a launch emits: one grid's items, or (P) the items of many problems,
// item_base their first.
struct EmitSrc {
    HitGrid G;
    EmitOut E;
    const HitProb *P;
    const int64_t *item_base;
    int B;
};

// The problem of global item `it`: its grid and outputs; returns the item's
// index in it.
__device__ __forceinline__ int emit_problem(const EmitSrc &S, int it, HitGrid &G, EmitOut &E) {
    const int p = problem_of<int64_t>(S.item_base, S.B, it);
    G = hit_grid(S.P[p]);
    E.row0 = S.P[p].row0;
    E.off += E.row0;
    E.base = E.off[0] - S.P[p].pout;
    E.qlo = 0;
    E.qhi = INT_MAX;
    return it - (int)S.item_base[p];
}

template <bool BATCH>
__global__ __launch_bounds__(kThreads) void k_hit_emit(EmitSrc Src) {
    __shared__ ListMap maps[kWaves];
    __shared__ uint4 keys[kWaves][kWaveBin / 4 + 1];  // positions, or the bitmap
    __shared__ unsigned short before[kWaves][kWinBits / 32];
    const int lane = threadIdx.x & 63, wv = uniform_i32(threadIdx.x >> 6);
    const int64_t w = (int64_t)blockIdx.x * kWaves + wv;
    const int parts = kTileQ / Src.E.per;
    const int item = uniform_i32((int)(Src.E.item_lo + w / parts)), part = uniform_i32((int)(w % parts));
    if (item >= Src.E.item_hi) return;
    HitGrid G = Src.G;
    EmitOut E = Src.E;
    int it = item;
    if (BATCH) it = emit_problem(Src, item, G, E);
    ListMap &M = maps[wv];
    const Item I = G.items[it];
    const int qb = max(I.qbegin + part * E.per, E.qlo), nq = min(min(I.qend, I.qbegin + (part + 1) * E.per), E.qhi) - qb;
    if (nq <= 0) return;
    // lane i: offset and input index of query qb + i; the offset of the end
    // in the lane after the last
    const int64_t offs = E.off[qb + min(lane, nq)];
    const int32_t pqs = G.perm[qb + min(lane, nq - 1)];
    const int64_t o_first = readlane_i64(offs, 0);
    int nxt = E.bin[o_first + min((int64_t)lane, readlane_i64(offs, 1) - o_first - 1)] - E.row0;
    const int total = list_map(G, it, lane, M);
    unsigned *ks = reinterpret_cast<unsigned *>(keys[wv]);
    auto settle = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    settle();
    auto rank_of = [&](unsigned k, int m) {
        int rank = 0;
#pragma unroll 4
        for (int f = 0; f < (m + 3) >> 2; ++f) {
            const uint4 o = keys[wv][f];
            rank += (o.x < k) + (o.y < k) + (o.z < k) + (o.w < k);
        }
        return rank;
    };
    auto put = [&](int64_t at, int32_t pq, int q, int c, int32_t pc) {
        E.pairs[at] = make_int2(pq, pc);
        if (E.d2) E.d2[at] = exact_d2_rows(G.xs + (int64_t)q * G.dp, G.xs + (int64_t)c * G.dp, G.dp);
    };
    // pairs of one query by bitmap; neighbour e of m is cur (m <= 64) or from the bin
    const int nwin = (total + kWinBits - 1) / kWinBits;
    auto by_bitmap = [&](int64_t o0, int m, int q, int32_t pq, int cur) {
        int at = 0;  // pairs of the windows before
        for (int w = 0; w < nwin; ++w) {
            const int w0 = w * kWinBits, words = (min(total - w0, kWinBits) + 31) >> 5;
            const int per = (words + 63) >> 6;  // words per lane, consecutive
            for (int u = 0; u < per; ++u) ks[u * 64 + lane] = 0;
            settle();
            for (int e = lane; e < m; e += 64) {
                const int p = list_pos(M, e == m - 1 ? q : m <= 64 ? cur : E.bin[o0 + e] - E.row0) - w0;
                if (p >= 0 && p < kWinBits) atomicOr(ks + (p >> 5), 1u << (p & 31));
            }
            settle();
            int sum = 0;
            for (int u = 0; u < per; ++u) {
                before[wv][lane * per + u] = (unsigned short)sum;
                sum += __popc(ks[lane * per + u]);
            }
            int incl = sum;
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (lane >= o) incl += y;
            }
            const int excl = incl - sum;
            for (int u = 0; u < per; ++u) before[wv][lane * per + u] += (unsigned short)excl;
            settle();
            for (int e = lane; e < m; e += 64) {
                const int c = e == m - 1 ? q : m <= 64 ? cur : E.bin[o0 + e] - E.row0;
                const int p = list_pos(M, c) - w0;
                if (p >= 0 && p < kWinBits) {
                    const int rank = before[wv][p >> 5] + __popc(ks[p >> 5] & ((1u << (p & 31)) - 1u));
                    put(o0 - E.base + at + rank, pq, q, c, G.perm[c]);
                }
            }
            at += __builtin_amdgcn_readlane(incl, 63);
            settle();
        }
    };
    for (int i = 0; i < nq; ++i) {
        const int q = qb + i;
        const int64_t o0 = readlane_i64(offs, i), m64 = readlane_i64(offs, i + 1) - o0;  // the point itself included
        const int cur = nxt;
        if (i + 1 < nq) {  // the next query's neighbours, in flight during this one
            const int64_t o1 = o0 + m64;
            nxt = E.bin[o1 + min((int64_t)lane, readlane_i64(offs, i + 2) - o1 - 1)] - E.row0;
        }
        const int32_t pq = __builtin_amdgcn_readlane(pqs, i);
        if (m64 > kWaveBin) {
            if (lane == 0) {
                const int s = atomicAdd(E.big, 1);
                E.big[2 + 2 * s] = q;
                E.big[3 + 2 * s] = item;
            }
            continue;
        }
        const int m = (int)m64;
        settle();
        // instructions of the two ways, about: 9 per read of four positions
        // and 64 neighbours; per window 70, 10 per word of a lane and 40 per 64
        // neighbours
        const int chunks = (m + 63) >> 6;
        const int by_rank = 9 * ((m + 3) >> 2) * chunks;
        const int by_bits = nwin * (70 + 40 * chunks) + 10 * ((total + 2047) >> 11);
        if (by_bits < by_rank) {
            by_bitmap(o0, m, q, pq, cur);
        } else if (m <= 64) {
            const int c = lane < m - 1 ? cur : q;
            const int32_t pc = G.perm[c];
            const unsigned k = (unsigned)list_pos(M, c);
            ks[lane] = lane < m ? k : 0xffffffffu;
            settle();
            const int rank = rank_of(k, m);
            if (lane < m) put(o0 - E.base + rank, pq, q, c, pc);
        } else {
            for (int e = lane; e < ((m + 3) & ~3); e += 64) {
                unsigned k = 0xffffffffu;
                if (e < m) k = (unsigned)list_pos(M, e < m - 1 ? E.bin[o0 + e] - E.row0 : q);
                ks[e] = k;
            }
            settle();
            for (int e = lane; e < m; e += 64) {
                const int c = e < m - 1 ? E.bin[o0 + e] - E.row0 : q;
                put(o0 - E.base + rank_of(ks[e], m), pq, q, c, G.perm[c]);
            }
        }
    }
}

// Points with many neighbours: one block per point, the list positions of
// the neighbours as bits of an LDS window, which then leave in order.
template <bool BATCH>
__global__ __launch_bounds__(kThreads) void k_hit_emit_big(EmitSrc Src) {
    __shared__ ListMap M;
    __shared__ unsigned bits[kBigBits / 32];
    __shared__ int wsum[kWaves];
    __shared__ int total_pos;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int nbig = Src.E.big[0];
    for (int s = blockIdx.x; s < nbig; s += gridDim.x) {
        HitGrid G = Src.G;
        EmitOut E = Src.E;
        const int q = E.big[2 + 2 * s];
        int it = E.big[3 + 2 * s];
        if (BATCH) it = emit_problem(Src, it, G, E);
        __syncthreads();
        if (tid < 64) list_map(G, it, lane, M);
        if (tid == 0) {
            int t = 0;
            for (int o = 0; o < G.nranges; ++o) {
                const Range r = G.ranges[(int64_t)it * G.nranges + o];
                t += max(0, r.end - r.begin);
            }
            total_pos = t;
        }
        __syncthreads();
        const int64_t o0 = E.off[q], m = E.off[q + 1] - o0;
        const int32_t pq = G.perm[q];
        int64_t at = o0 - E.base;
        for (int64_t w0 = 0; w0 < total_pos; w0 += kBigBits) {
            for (int e = tid; e < kBigBits / 32; e += kThreads) bits[e] = 0;
            __syncthreads();
            for (int64_t e = tid; e < m; e += kThreads) {
                const int c = e < m - 1 ? E.bin[o0 + e] - E.row0 : q;
                const int64_t p = (int64_t)list_pos(M, c) - w0;
                if (p >= 0 && p < kBigBits) atomicOr(&bits[p >> 5], 1u << (p & 31));
            }
            __syncthreads();
            for (int b0 = 0; b0 < kBigBits / 32; b0 += kThreads) {
                unsigned v = bits[b0 + tid];
                const int c0 = __popc(v);
                int incl = c0;
                for (int o = 1; o < 64; o <<= 1) {
                    const int y = __shfl_up(incl, o);
                    if (lane >= o) incl += y;
                }
                if (lane == 63) wsum[wv] = incl;
                __syncthreads();
                int pre = incl - c0, all = 0;
                for (int w = 0; w < kWaves; ++w) {
                    if (w < wv) pre += wsum[w];
                    all += wsum[w];
                }
                int64_t o = at + pre;
                while (v) {
                    const int bit = __builtin_ctz(v);
                    v &= v - 1;
                    const int64_t p = w0 + 32 * (int64_t)(b0 + tid) + bit;
                    // back to the row: the range holding list position p
                    int64_t left = p;
                    int c = 0;
                    for (int r = 0; r < G.nranges; ++r) {
                        const Range x = G.ranges[(int64_t)it * G.nranges + r];
                        const int len = max(0, x.end - x.begin);
                        if (left < len) {
                            c = x.begin + (int)left;
                            break;
                        }
                        left -= len;
                    }
                    E.pairs[o] = make_int2(pq, G.perm[c]);
                    if (E.d2) E.d2[o] = exact_d2(G.xs + (int64_t)q * G.dp, G.xs + (int64_t)c * G.dp, G.d);
                    ++o;
                }
                at += all;
                __syncthreads();
            }
        }
    }
}

// Sort key of each block item of a batch: its K-step count above, then
// descending cost (its list's length; the blocks of one form have the same
// number of K-steps); value = global block index.
__global__ __launch_bounds__(kThreads) void k_hit_cost(const HitProb *__restrict__ P,
                                                       const int64_t *__restrict__ block_base, int B, int64_t nb,
                                                       unsigned long long *__restrict__ key, int32_t *__restrict__ val) {
    const int64_t gb = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (gb >= nb) return;
    int lo = 0, hi = B;  // the problem (not wave-uniform here)
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (block_base[mid] <= gb) lo = mid;
        else hi = mid;
    }
    const HitGrid G = hit_grid(P[lo]);
    const int b = (int)(gb - block_base[lo]);
    const int64_t it = G.blocks[b] - G.item_base;
    unsigned long long c = 0;
    for (int o = 0; o < G.nranges; ++o) {
        const Range r = G.ranges[it * G.nranges + o];
        c += (unsigned long long)max(0, r.end - r.begin);
    }
    c = (c + 63) / 64;
    const unsigned long long cap = (1ull << 27) - 1;
    key[gb] = ((unsigned long long)(G.da >> 2) << 27) | (cap - (c < cap ? c : cap));
    val[gb] = (int32_t)gb;
}

// The tally of a count, added to its counters.
__device__ __forceinline__ void hit_fold(const unsigned long long *__restrict__ tally, DevCounters *ctr) {
    unsigned long long met = 0, pruned = 0;
#pragma unroll 16
    for (int r = 0; r < kHitTally; ++r) {
        met += tally[r * kHitCursorStride];
        pruned += tally[r * kHitCursorStride + 1];
    }
    ctr->met += met;
    ctr->pruned += pruned;
}

__global__ void k_hit_fold(const unsigned long long *__restrict__ tally, DevCounters *ctr) { hit_fold(tally, ctr); }

// Totals of a batch's problems, then the entries reserved in the fullest region.
__global__ __launch_bounds__(kThreads) void k_hit_totals(const HitProb *__restrict__ P, const int64_t *__restrict__ off,
                                                         int64_t rows, int B,
                                                         const unsigned long long *__restrict__ cursor,
                                                         const unsigned long long *__restrict__ tally, DevCounters *ctr,
                                                         int64_t *__restrict__ out) {
    const int k = blockIdx.x * kThreads + threadIdx.x;
    if (k < B) out[k] = off[k + 1 < B ? P[k + 1].row0 : rows] - off[P[k].row0];
    if (k == B) {
        unsigned long long m = 0;
        for (int r = 0; r < kHitRegions; ++r) m = max(m, cursor[r * kHitCursorStride]);
        out[B] = (int64_t)m;
        hit_fold(tally, ctr);
    }
}

// Calls f with the compile-time K-step count `ks` (LO .. HI).
template <int LO, int HI, typename F>
void by_k_steps(int ks, F f) {
    if constexpr (LO > HI) {
        throw Unsupported{"hit-list count: d out of range"};
    } else {
        if (ks == LO) f(std::integral_constant<int, LO>{});
        else by_k_steps<LO + 1, HI>(ks, f);
    }
}

double hit_scale(const Grid &g) { return std::ldexp(1.0, -std::ilogb(g.eps)); }

HitGrid hit_grid(const Grid &g) {
    HitGrid G{};
    G.xs = g.xs;
    G.xa = g.xa;
    G.nrm = g.nrm;
    G.perm = g.perm;
    G.items = g.item;
    G.ranges = g.ranges;
    G.blocks = g.blocks;
    G.item_block = g.hit_item_block;
    G.span = g.hit_span;
    G.blo = g.hit_blo;
    G.bhi = g.hit_bhi;
    G.bstride = g.items;
    G.d = g.d;
    G.dp = g.dp;
    G.da = g.da;
    G.nranges = g.nranges;
    G.nitems = (int32_t)g.items;
    G.nblocks = (int32_t)g.nblocks;
    G.item_base = g.item_base;
    G.boxes = g.sc != -1;
    const double sc = hit_scale(g);
    G.sc = sc;
    G.eps_s = g.eps * sc;
    G.eps2_s = g.eps2 * sc * sc;
    G.thr = (float)(G.eps2_s * (1.0 + 1e-4));
    G.eps2 = g.eps2;
    return G;
}

size_t align_up(size_t b) { return (b + 255) & ~size_t(255); }

constexpr size_t kTallyBytes = kHitTally * kHitCursorStride * sizeof(unsigned long long);

// Bytes of the index that hits_prepare adds to a grid, the count's tally last.
size_t hit_index_bytes(int64_t items, int64_t nblocks, int nranges, int d) {
    const size_t dims = (size_t)((d + 3) & ~3);
    return 2 * align_up(dims * items * sizeof(float)) + align_up(items * sizeof(int32_t)) +
           align_up((size_t)nblocks * nranges * sizeof(int2)) + kTallyBytes;
}

}  // namespace

// Blocks per block item: its walk is dealt to them, a round of kRound items each
// in turn. Few block items: so many that the chip is filled, whatever their
// length. Otherwise up to 2^15 blocks in all, each with four rounds at least:
// about 1280 blocks run at once, and with 2922 of equal length a third of the
// last turn stays empty. Uniform points, 187k: d = 16 (40 rounds) 10.45 ms with one
// block per block item, 9.85 so; d = 8 (7 rounds) 1.87 and 1.74. With one round at
// least, d = 8 takes 1.70 ms, but Gaussian mixtures, 200k points, d = 64 (2 rounds),
// lose the start of each block: 1.89 ms against 1.75.
static int hit_segments(const Grid &g) {
    const int64_t rounds = (int64_t)((double)g.cand_items / ((double)g.n * kTileQ * kRound));
    const int64_t fill = std::min<int64_t>(16, 4096 / g.nblocks);
    const int64_t even = std::min<int64_t>(32768 / g.nblocks, rounds / 4);
    return (int)std::max<int64_t>(1, std::max(fill, std::min<int64_t>(even, 64)));
}

thread_local int32_t tl_hits_always = 0;
thread_local unsigned long long tl_hits_first = 0;

// The grids and paths this count takes: block items with one candidate list
// (d > 4), d <= 64 (whole rows in a wave's lanes; more dimensions stay on the
// per-wave tiles), work items at least half full (an item is a tile here, and
// lines with few points leave most of its columns empty: the packed lists of
// k_m64 / k_lowp then have fewer tiles), enough tile work (candidate pairs x
// K-steps) to pay for the index and for ordering the list, some 60 us of
// launches (n = 5000, d = 16, 1.8e6: join 411 us without, 440 with; index-free
// n = 2048, d = 8, 8.4e6: 315 and 333; n = 5000, d = 6, 2.3e7: 530 and 493;
// n = 30000, d = 5, 1.3e8: 559 and 514; n = 9001, d = 23 index-free, 4.9e8: 1169
// and 502), eps far enough from the ends of the range for the boxes'
// power-of-two scale, few enough pairs (hits_pay), and a block for each block
// item within one launch (below 2^32 threads).
constexpr int64_t kHitMaxBlocks = ((int64_t(1) << 32) - 1) / kThreads;

static bool hits_fit(const Grid &g) {
    return g.united && g.blocks && g.items > 0 && g.d > 4 && g.d <= kHitMaxD && g.n >= 8 * g.items &&
           g.nblocks <= kHitMaxBlocks && g.eps >= 0x1p-500 && g.eps <= 0x1p500;
}
static double hits_work(const Grid &g) { return (double)g.cand_items * (g.da >> 2); }
constexpr double kHitWork = 0x1p24;

// The upper end: a pair costs this count more than a candidate's mask bit costs
// the tiles of all candidates, so a set with many pairs a point, or with few
// candidates, stays on those. Which takes less is estimated from C candidates
// and s pairs a point (s from the build's sample), KS K-steps of 4 dimensions and
// the fill f of the work items (points over 16 times the items: an item is a
// tile here, the other tiles pack their candidates):
//   tiles ms = n (C (c + ck KS) + p s) 1e-9 + C (w + wk KS) 1e-6 + t
//   list  ms = n (C / f (c + ck KS) + s (p + q min(3, max(0, s / 300 - 1)))) 1e-9 + w C 1e-6 + t
// (w, wk: one wave's walk over its candidates, which few items leave bare; q: the
// ordering of long bins, by the mean s or point by point as the sample has it,
// whichever is more: 1000 points at one place among 200k, ten times, d = 5, 1.06 ms
// by tiles and 1.62 by list). Least squares over 461 joins (count and pairs; 5000 to
// 1M points, uniform, exponential and mixture, d = 5 .. 64, s = 8 .. 800), each
// mostly within 30 %; taking the smaller estimate costs 1.5 % over the faster of
// the two in FP64 with up to 4 K-steps (tiles shared through LDS; the forms
// meet there: mixture of 200k points, d = 16, C = 2325, s = 50 0.82 ms by tiles,
// 0.61 by list, s = 99 0.85 and 0.90; uniform, d = 5, C = 9730, s = 198 1.76 and 1.59,
// s = 398 2.58 and 2.76; mixture of 400k, d = 5, half-filled items, C = 696, s = 8
// 0.71 and 1.18) and less than 0.2 % elsewhere (mixture of 30k, d = 29, C = 895, s = 87
// 0.76 and 0.28; split BF16, d = 16, s = 197 2.4 and 1.8). Against the half-stencil tiles
// (148 counts): 0.6 % there, the list always for more K-steps. A count without
// list or in-masks only bears its pairs' atomics, and loses (by up to 10 %) only
// in FP64 where 30 pairs outweigh the candidates (mixture of 200k, d = 8, C = 2112,
// s = 389 0.84 and 0.91).
struct TilesCost { double c, ck, p, w, wk, t; };
struct ListCost { double c, ck, p, q, w, t; };

struct Costs {
    double tiles, list;
};

// Near the line the list is taken for up to 100 pairs a point: its count alone,
// which is all that some callers ask for, is the cheaper one there (mixture of 91k
// points, d = 13, s = 28: 0.16 and 0.27 ms). Where the same call emits distances, which
// the in-masks' rows gather points for, the forms meet later (hits_pay; mixture of
// 200k, d = 16, 10 neighbours, s = 150 3.0 ms by the list, 3.6 by in-masks, s = 220 4.2
// and 4.7, where pairs alone take 1.57 and 1.14, 1.95 and 1.26; d = 8, s = 150 2.27 and 2.11).
static double list_favour(const Grid &g) { return g.sample.pairs <= 100ull * (unsigned long long)g.n ? 1.15 : 1.0; }

// alone: the launches and the walk are this grid's alone (not a batch's).
static Costs hits_costs(const Grid &g, sj_path path, HitUse use, bool alone) {
    static const TilesCost tiles[5] = {{0.458, 0.096, 3.95, 35.5, 0.0, 0.147},    // FP64, up to 4 K-steps
                                       {3.11, 0.0356, 0.0, 60.8, 0.403, 0.196},   // FP64, more
                                       {0.726, 0.143, 9.41, 0.0, 7.13, 0.330},    // FP32
                                       {0.360, 0.210, 24.3, 0.0, 5.46, 0.416},    // split BF16
                                       {0.0584, 0.098, 1.23, 28.0, 0.0063, 0.108}};  // half stencil, up to 4
    static const ListCost list[5] = {{0.107, 0.0479, 27.0, 20.8, 5.56, 0.203},
                                     {0.329, 0.0038, 25.3, 17.9, 14.1, 0.193},
                                     {0.215, 0.0079, 33.9, 12.0, 1.60, 0.225},
                                     {0.241, 0.0044, 39.7, 9.19, 0.0, 0.236},
                                     {0.136, 0.0369, 4.45, 1.0, 1.40, 0.119}};
    const double ks = path == SJ_FP64_MFMA ? g.da >> 2 : g.dp >> 2;
    const int k = use == HitUse::HALF ? 4 : path == SJ_FP32_MFMA ? 2 : path == SJ_BF16X3_MFMA ? 3 : ks <= 4 ? 0 : 1;
    const double n = (double)g.n, s = (double)g.sample.pairs / n, c = (double)g.cand_items / n;
    const double fill = n / (16.0 * (double)g.items);
    const TilesCost &T = tiles[k];
    const ListCost &L = list[k];
    Costs r;
    r.tiles = 1e-9 * n * (c * (T.c + T.ck * ks) + T.p * s);
    const double even = s * std::min(3.0, std::max(0.0, s / 300.0 - 1.0));
    r.list = 1e-9 * n * (c / fill * (L.c + L.ck * ks) + s * L.p + L.q * std::max(even, (double)g.sample.dense / n));
    if (alone) {
        r.tiles += 1e-6 * c * (T.w + T.wk * ks) + T.t;
        r.list += 1e-6 * c * L.w + L.t;
    }
    return r;
}

static bool hits_pay(const Grid &g, sj_path path, HitUse use) {
    if (tl_hits_always) return tl_hits_always > 0;
    const int ks = path == SJ_FP64_MFMA ? g.da >> 2 : g.dp >> 2;
    const bool few = path == SJ_FP64_MFMA && ks <= 4;
    if (use == HitUse::COUNT) return !few || (double)g.cand_items * (2 * ks + 1) >= 30.0 * (double)g.sample.pairs;
    if (use == HitUse::HALF && !few) return true;
    const Costs r = hits_costs(g, path, use, true);
    return r.list < std::max(list_favour(g), few && use == HitUse::DISTANCES ? 1.6 : 0.0) * r.tiles;
}

// Pairs of the result that the list is laid out for: the sample's, and what
// its spread may hide.
static double pairs_up(const Grid &g) {
    const double pairs = (double)g.sample.pairs, hits = (double)g.sample.hits, cand = (double)g.cand_items;
    const double each = std::max(cand / (double)std::max<int64_t>(g.samples, 1), hits > 0 ? pairs / hits : 0.0);
    return std::min(cand, 1.15 * pairs + 3.0 * std::sqrt(hits + 1.0) * each);
}

// Entries of a list of `listed` pairs that `waves` waves write: each may leave
// the rest of its last run unused.
static double list_entries(double listed, double waves) {
    return listed + (double)kHitChunk * std::min(waves, listed + 1.0);
}

// Entries per region to begin with: twice the pairs that are expected (the
// regions fill unevenly). Past the budget the budget: the cursors count on, so
// that a count that overflows still tells the need.
static unsigned long long region_first(double listed, double waves, int64_t budget) {
    if (tl_hits_first) return tl_hits_first;
    const double most = list_entries(2.0 * listed, waves) / kHitRegions + 16 * kHitChunk;
    const unsigned long long lim = (unsigned long long)budget / (kHitRegions * sizeof(int2)) / kHitChunk;
    return std::min((unsigned long long)(most / kHitChunk) + 1, lim) * kHitChunk;
}

// Entries per region for `most` of them in the fullest, 0 past the budget.
static unsigned long long region_cap(unsigned long long most, int64_t budget) {
    most = (most + kHitChunk - 1) / kHitChunk * kHitChunk;
    return most * kHitRegions * sizeof(int2) <= (unsigned long long)budget ? most : 0;
}

static double listed_up(const Grid &g) { return std::max(0.0, 0.5 * (pairs_up(g) - (double)g.n)); }

bool hits_usable(const Grid &g, sj_path path, HitUse use) {
    if (path != SJ_FP64_MFMA && path != SJ_FP32_MFMA && path != SJ_BF16X3_MFMA) return false;
    if (!hits_fit(g) || hits_work(g) < kHitWork || !hits_pay(g, path, use)) return false;
    if (use != HitUse::PAIRS && use != HitUse::DISTANCES) return true;
    // a join whose list would not fit keeps in-masks, if they do
    const double waves = (double)g.nblocks * hit_segments(g) * kWaves;
    return list_entries(listed_up(g), waves) * sizeof(int2) <= (double)kMaskBudget;
}

size_t hits_lean_bytes(int64_t n, int32_t d) {
    if (d <= 4 || d > kHitMaxD || n == 0) return 0;
    const int64_t items = n / 8;  // hits_usable
    return hit_index_bytes(items, items, 27, d) + 8 * 256;
}

// Lays the grid's index out at p.
static void hit_layout(Grid &g, char *p) {
    const size_t dims = (size_t)((g.d + 3) & ~3);
    g.hit_blo = reinterpret_cast<float *>(p);
    p += align_up(dims * g.items * sizeof(float));
    g.hit_bhi = reinterpret_cast<float *>(p);
    p += align_up(dims * g.items * sizeof(float));
    g.hit_item_block = reinterpret_cast<int32_t *>(p);
    p += align_up(g.items * sizeof(int32_t));
    g.hit_span = reinterpret_cast<int2 *>(p);
    p += align_up((size_t)g.nblocks * g.nranges * sizeof(int2));
    g.hit_tally = reinterpret_cast<unsigned long long *>(p);
}

static unsigned box_blocks(const Grid &g) { return (unsigned)((g.items + 15) / 16); }
static unsigned span_blocks(const Grid &g) { return (unsigned)((g.nblocks * g.nranges + kThreads - 1) / kThreads); }

// Makes the grid's index on the first such count; false when there is no
// memory for it (the count then runs the tiles of all candidates).
bool hits_prepare(Grid &g, hipStream_t s) {
    if (g.hit_index) return true;
    try {
        g.hit_index = dev_alloc(hit_index_bytes(g.items, g.nblocks, g.nranges, g.d), s);
    } catch (const OomError &) {
        return false;
    }
    hit_layout(g, static_cast<char *>(g.hit_index));
    const unsigned nbox = box_blocks(g);
    hipLaunchKernelGGL(k_hit_index, dim3(nbox + span_blocks(g)), dim3(kThreads), 0, s, hit_grid(g), hit_scale(g), nbox);
    SJ_HIP(hipGetLastError());
    return true;
}

void hits_free_list(Grid &g, hipStream_t s) {
    if (g.hits) dev_free(g.hits, s);
    if (g.hit_cursor) dev_free(g.hit_cursor, s);
    if (g.hit_bin) dev_free(g.hit_bin, s);
    g.hits = nullptr;
    g.hit_cursor = nullptr;
    g.hit_bin = nullptr;
    g.hit_cap = 0;
    g.hits_valid = false;
}

// Enqueues the count (hits_prepare has made the index): counts into cnt (n + 1
// entries, zeroed here), pairs into the grid's list when `record` and there is
// memory for it; ro.ctr and the grid's tally zeroed here.
// most: entries per region that a former run of this count reserved (0: not
// known).
void hits_count(Grid &g, sj_path path, int32_t *cnt, bool record, unsigned long long most, RefineOut &ro,
                hipStream_t s) {
    const int nseg = hit_segments(g);
    g.hits_valid = false;
    HitOut R{};
    R.cnt = cnt;
    R.ctr = ro.ctr;
    R.tally = g.hit_tally;
    if (record) {  // (a former list is dropped)
        const unsigned long long cap =
            most ? region_cap(most, kMaskBudget)
                 : region_first(listed_up(g), (double)g.nblocks * nseg * kWaves, kMaskBudget);
        if (g.hit_bin) dev_free(g.hit_bin, s);
        g.hit_bin = nullptr;
        if (cap > g.hit_cap) {
            hits_free_list(g, s);
            try {
                DevBuf<unsigned long long> cursor(kHitRegions * kHitCursorStride, s);
                g.hits = dev_alloc_n<int2>((size_t)(cap * kHitRegions), s);
                g.hit_cursor = cursor.release();
                g.hit_cap = cap;
            } catch (const OomError &) {  // the count goes on without a list
            }
        }
        if (g.hits) {
            R.hits = g.hits;
            R.cursor = g.hit_cursor;
            R.cap = g.hit_cap;
        }
    }
    fill_zero_many({{cnt, ((size_t)g.n + 1) * sizeof(int32_t)},
                    {R.cursor, R.cursor ? kHitRegions * kHitCursorStride * sizeof(unsigned long long) : 0},
                    {g.hit_tally, kTallyBytes},
                    {ro.ctr, sizeof(DevCounters)}},
                   s);
    const HitGrid G = hit_grid(g);
    const dim3 grid((unsigned)(g.nblocks * nseg));
    ro.kt.start(ro.timed, s);
    if (path == SJ_FP64_MFMA) {
        const double delta = fp64_mfma_delta(g);
        ro.band_rel = g.eps2 > 0 ? delta / g.eps2 : 0.0;
        by_k_steps<2, 16>(g.da >> 2, [&](auto ks) {
            hipLaunchKernelGGL(k_hit_f64<decltype(ks)::value>, grid, dim3(kThreads), 0, s, G, R, delta, nseg);
        });
    } else if (path == SJ_FP32_MFMA) {
        by_k_steps<2, 16>(g.dp >> 2, [&](auto ks) {
            hipLaunchKernelGGL((k_hit_lp<PREC_F32, decltype(ks)::value>), grid, dim3(kThreads), 0, s, G, R, nseg);
        });
    } else {
        by_k_steps<1, 2>((g.d + 31) / 32, [&](auto ks) {
            hipLaunchKernelGGL((k_hit_lp<PREC_BF16X3, decltype(ks)::value>), grid, dim3(kThreads), 0, s, G, R, nseg);
        });
    }
    SJ_HIP(hipGetLastError());
    ro.kt.stop(s);
}

// A list for a pairs call whose count kept none (half-stencil option, a count
// on another path, or a list that outgrew its first guess): the count run
// again, its counts dropped. False when the list would exceed the budget or
// there is no memory for it; ro.ctr may then hold this count's counters.
bool hits_ensure(Grid &g, sj_path path, RefineOut &ro, hipStream_t s) {
    if (!hits_prepare(g, s)) return false;
    unsigned long long most = g.hit_most;
    for (int tries = 0; tries < 2; ++tries) {
        if (most && !region_cap(most, kMaskBudget)) return false;
        RefineOut again;
        again.ctr = ro.ctr;
        try {
            DevBuf<int32_t> cnt((size_t)g.n + 1, s);
            hits_count(g, path, cnt.p, true, most, again, s);
        } catch (const OomError &) {
            return false;
        }
        if (!g.hits) return false;
        hipLaunchKernelGGL(k_hit_fold, dim3(1), dim3(1), 0, s, g.hit_tally, ro.ctr);
        SJ_HIP(hipGetLastError());
        unsigned long long cur[kHitRegions * kHitCursorStride];
        SJ_HIP(hipMemcpyAsync(cur, g.hit_cursor, sizeof cur, hipMemcpyDeviceToHost, s));
        SJ_HIP(hipStreamSynchronize(s));
        ro.band_rel = again.band_rel;
        most = 0;
        for (int r = 0; r < kHitRegions; ++r) most = std::max(most, cur[r * kHitCursorStride]);
        g.hit_most = most;
        if (most <= g.hit_cap) {
            g.hits_valid = true;
            g.hits_lowp = is_lowp(path);
            return true;
        }
    }
    return false;
}

// How the list is ordered by point (see k_hit_part): the buckets, or (too
// many points or pairs for them) the pairs one by one.
struct BinPlan {
    int sh, nbuckets;
    bool parts;
    int64_t entries;  // each listed pair twice
    size_t nfill;     // counters, zeroed by the caller
};
static BinPlan bin_plan(int64_t rows, int64_t total) {
    BinPlan b;
    b.sh = 6;
    while ((rows >> b.sh) >= kBuckets) ++b.sh;
    b.nbuckets = (int)std::min<int64_t>((rows + (int64_t(1) << b.sh) - 1) >> b.sh, INT_MAX);
    b.entries = total - rows;
    b.parts = b.sh <= 13 && b.entries * (int64_t)sizeof(uint2) <= kMaskBudget;
    b.nfill = b.parts ? (size_t)b.nbuckets : (size_t)rows;
    return b;
}
static void make_bins(const BinPlan &b, const int2 *hits, const unsigned long long *cursor, unsigned long long cap,
                      unsigned long long most, const int64_t *off, int64_t rows, int32_t *fill, int32_t *bin,
                      hipStream_t s) {
    if (!b.parts) {
        hipLaunchKernelGGL(k_hit_bin, dim3(256, kHitRegions), dim3(kThreads), 0, s, hits, cursor, cap, off, fill, bin);
        SJ_HIP(hipGetLastError());
        return;
    }
    DevBuf<uint2> part((size_t)std::max<int64_t>(b.entries, 1), s);
    const int64_t slabs = (int64_t)(most + kSlab - 1) / kSlab;
    hipLaunchKernelGGL(k_hit_part, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(slabs, 128)), kHitRegions),
                       dim3(kPartThreads), 0, s, hits, cursor, cap, off, b.sh, b.nbuckets,
                       reinterpret_cast<unsigned *>(fill), part.p);
    SJ_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_hit_place, dim3((unsigned)b.nbuckets), dim3(kThreads), sizeof(unsigned) << b.sh, s, part.p, off,
                       rows, b.sh, bin);
    SJ_HIP(hipGetLastError());
}

// Pairs of the chunk from the list (valid): the bins are made on the first
// call and kept for the chunks that follow. False (and nothing written) when
// there is no memory for them.
bool hits_pairs(Grid &g, const ChunkPlan &p, int64_t qlo, int32_t *pairs, double *d2, RefineOut &ro, hipStream_t s) {
    // more than kWaveBin neighbours: at most written / kWaveBin points
    const size_t nbig = (size_t)(p.written / kWaveBin) + 1;
    const BinPlan bp = bin_plan(g.n, g.total);
    const size_t nfill = g.hit_bin ? 0 : bp.nfill;
    std::unique_ptr<DevBuf<int32_t>> work;
    try {
        work.reset(new DevBuf<int32_t>(2 + 2 * nbig + nfill, s));
        int32_t *fill = work->p + 2 + 2 * nbig;
        ro.kt.start(ro.timed, s);
        fill_zero_many({{work->p, sizeof(int32_t)}, {fill, nfill * sizeof(int32_t)}}, s);
        if (!g.hit_bin) {  // the grid's once they are made: a call that fails on the way leaves none
            DevBuf<int32_t> bin((size_t)std::max<int64_t>(g.total, 1), s);
            make_bins(bp, g.hits, g.hit_cursor, g.hit_cap, g.hit_most, g.off, g.n, fill, bin.p, s);
            g.hit_bin = bin.release();
        }
    } catch (const OomError &) {
        return false;
    }
    const int nitems = (int)(p.item_hi - p.item_lo);
    if (nitems > 0) {
        EmitOut E{};
        E.off = g.off;
        E.bin = g.hit_bin;
        E.base = p.base;
        E.qlo = (int32_t)qlo;
        E.qhi = (int32_t)p.next;
        E.item_lo = (int32_t)p.item_lo;
        E.item_hi = (int32_t)p.item_hi;
        E.pairs = reinterpret_cast<int2 *>(pairs);
        E.d2 = d2;
        E.big = work->p;
        const HitGrid G = hit_grid(g);
        // a wave's queries run one after the other: few items are spread over more waves
        E.per = kTileQ;
        while (E.per > 1 && (int64_t)nitems * (kTileQ / E.per) < 16384) E.per /= 2;
        const int64_t waves = (int64_t)nitems * (kTileQ / E.per);
        EmitSrc src{G, E, nullptr, nullptr, 0};
        hipLaunchKernelGGL(k_hit_emit<false>, dim3((unsigned)((waves + kWaves - 1) / kWaves)), dim3(kThreads), 0, s, src);
        SJ_HIP(hipGetLastError());
        if (p.written > kWaveBin) {
            hipLaunchKernelGGL(k_hit_emit_big<false>, dim3((unsigned)std::min<size_t>(nbig, 1024)), dim3(kThreads), 0, s,
                               src);
            SJ_HIP(hipGetLastError());
        }
    }
    ro.kt.stop(s);
    return true;
}

// ------------------------------------------------------------------ batch --
// The hit-list count of a batch's problems: those whose grids it takes, if
// together they have the work. One index launch, one count launch per K-step
// count over their block items (longest first), one list, and one ordering and
// emission for all of them (256 problems of 1e3 to 2e5 uniform points, d = 2, 3,
// 4, 8, 16: count at d = 8 and 16 218 -> 74 ms, the whole call 243 -> 86 ms); their
// rows follow each other in the counts,
// offsets and list (entries are rows of all these problems together).
static int hit_batch_segments(int64_t blocks) { return (int)std::max<int64_t>(1, std::min<int64_t>(16, 4096 / blocks)); }

static void hit_batch_make(HitBatch &hb, const std::vector<Grid *> &grids, bool sym, hipStream_t s) {
    double work = 0;
    std::map<int, int64_t> blocks;  // by K-step count
    hb.listed_up = 0;
    // a problem takes the form that it is clearly cheaper in; the others one
    // form together, since each form has its launches (ms: 64 problems of 1600
    // points, d = 5, s = 16 0.45 by tiles and 0.38 by list, 0.05 and 0.06 of it work)
    constexpr double kBatchForm = 0.05;
    const HitUse use = sym ? HitUse::HALF : HitUse::PAIRS;
    double tiles = 0, list = 0;
    std::vector<Costs> costs(grids.size(), Costs{0, 0});
    for (size_t i = 0; i < grids.size(); ++i) {
        const Grid &g = *grids[i];
        if (!hits_fit(g) || !m64_in_range(g)) continue;
        costs[i] = hits_costs(g, SJ_FP64_MFMA, use, false);
        if (sym && (g.da >> 2) > 4) costs[i].list = 0;
        if (tl_hits_always) costs[i] = tl_hits_always > 0 ? Costs{1, 0} : Costs{0, 1};
        tiles += list_favour(g) * costs[i].tiles;
        list += costs[i].list;
    }
    for (size_t i = 0; i < grids.size(); ++i) {
        const Grid &g = *grids[i];
        const Costs &c = costs[i];
        if (c.tiles == 0 && c.list == 0) continue;
        if (!(c.list < 0.5 * c.tiles || (c.list < 2.0 * c.tiles && list < tiles + kBatchForm))) continue;
        hb.probs.push_back((int)i);
        work += hits_work(g);
        blocks[g.da >> 2] += g.nblocks;
        hb.listed_up += listed_up(g);
    }
    hb.waves = 0;
    for (const auto &kv : blocks) {
        hb.waves += (double)kv.second * hit_batch_segments(kv.second) * kWaves;
        if (kv.second > kHitMaxBlocks) work = 0;
    }
    if (work < kHitWork) hb.probs.clear();
    // (a list that would not fit: in-masks, if they do)
    if (!sym && list_entries(hb.listed_up, hb.waves) * sizeof(int2) > (double)kHitBatchBudget) hb.probs.clear();
    if (hb.probs.empty()) return;
    const int P = (int)hb.probs.size();
    // K-step counts grouped: the block queue is made form by form, in this order
    std::stable_sort(hb.probs.begin(), hb.probs.end(), [&](int a, int b) { return grids[a]->da < grids[b]->da; });
    size_t bytes = 0;
    for (int i : hb.probs) bytes += hit_index_bytes(grids[i]->items, grids[i]->nblocks, grids[i]->nranges, grids[i]->d);
    hb.index = dev_alloc(bytes, s);
    std::vector<HitProb> hp(P);
    std::vector<int64_t> bbase(P + 1, 0), ibase(P + 1, 0), first(P + 1, 0);
    char *at = static_cast<char *>(hb.index);
    hb.rows = 0;
    for (int k = 0; k < P; ++k) {
        Grid &g = *grids[hb.probs[k]];
        hit_layout(g, at);
        at += hit_index_bytes(g.items, g.nblocks, g.nranges, g.d);
        HitProb &x = hp[k];
        x.G = hit_grid(g);
        x.delta = fp64_mfma_delta(g);
        x.row0 = (int32_t)hb.rows;
        x.nbox = (int32_t)box_blocks(g);
        x.sc = hit_scale(g);
        x.pout = 0;
        hb.rows += g.n;
        bbase[k + 1] = bbase[k] + g.nblocks;
        ibase[k + 1] = ibase[k] + g.items;
        first[k + 1] = first[k] + box_blocks(g) + span_blocks(g);
        if (hb.forms.empty() || hb.forms.back().ks != g.da >> 2) hb.forms.push_back({g.da >> 2, (int32_t)bbase[k], 0});
        hb.forms.back().hi = (int32_t)bbase[k + 1];
    }
    hb.blocks = bbase[P];
    hb.items = ibase[P];
    // one upload: the problems, then the three prefix arrays
    const size_t pb = align_up(P * sizeof(HitProb)), nb = align_up((P + 1) * sizeof(int64_t));
    std::vector<char> host(pb + 3 * nb);
    std::memcpy(host.data(), hp.data(), P * sizeof(HitProb));
    std::memcpy(host.data() + pb, bbase.data(), (P + 1) * sizeof(int64_t));
    std::memcpy(host.data() + pb + nb, ibase.data(), (P + 1) * sizeof(int64_t));
    std::memcpy(host.data() + pb + 2 * nb, first.data(), (P + 1) * sizeof(int64_t));
    hb.dev = dev_alloc(host.size(), s);
    SJ_HIP(hipMemcpyAsync(hb.dev, host.data(), host.size(), hipMemcpyHostToDevice, s));
    SJ_HIP(hipStreamSynchronize(s));
    hb.host_probs.assign(host.begin(), host.begin() + pb);
    char *d = static_cast<char *>(hb.dev);
    hb.block_base = reinterpret_cast<int64_t *>(d + pb);
    hb.item_base = reinterpret_cast<int64_t *>(d + pb + nb);
    const HitProb *dp = reinterpret_cast<const HitProb *>(d);
    hipLaunchKernelGGL(k_hit_index_batch, dim3((unsigned)first[P]), dim3(kThreads), 0, s, dp,
                       reinterpret_cast<const int64_t *>(d + pb + 2 * nb), P);
    SJ_HIP(hipGetLastError());
    // the queue: block items of each form by descending cost
    DevBuf<unsigned long long> ka(hb.blocks, s), kb(hb.blocks, s);
    DevBuf<int32_t> va(hb.blocks, s), vb(hb.blocks, s);
    hipLaunchKernelGGL(k_hit_cost, dim3((unsigned)((hb.blocks + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, dp,
                       hb.block_base, P, hb.blocks, ka.p, va.p);
    SJ_HIP(hipGetLastError());
    unsigned long long *ks = ka.p;
    int32_t *vs = va.p;
    radix_sort_pairs(&ks, &vs, kb.p, vb.p, hb.blocks, 32, s);  // cost below the K-step count
    hb.queue = vs == va.p ? va.release() : vb.release();
    hb.cnt = dev_alloc_n<int32_t>((size_t)hb.rows + 1, s);
    hb.off = dev_alloc_n<int64_t>((size_t)hb.rows + 1, s);
    hb.cursor = dev_alloc_n<unsigned long long>((kHitRegions + kHitTally) * kHitCursorStride, s);
    hb.tally = hb.cursor + kHitRegions * kHitCursorStride;
}

void hit_batch_free(HitBatch &hb, hipStream_t s) {
    void *bufs[] = {hb.index, hb.dev, hb.queue, hb.cnt, hb.off, hb.cursor, hb.hits, hb.bin};
    for (void *p : bufs)
        if (p) dev_free(p, s);
    hb = HitBatch{};
}

// Without memory for the index no problem takes the hit list.
void hit_batch_build(HitBatch &hb, const std::vector<Grid *> &grids, bool sym, hipStream_t s) {
    try {
        hit_batch_make(hb, grids, sym, s);
    } catch (const OomError &) {
        hit_batch_free(hb, s);
    }
}

// Counts, offsets and totals (totals[i] for problem i of the batch) of these
// problems, and with `record` the list; counters are added to ctr.
void hit_batch_count(HitBatch &hb, bool record, DevCounters *ctr, int64_t *totals, hipStream_t s) {
    hb.valid = false;
    if (hb.bin) dev_free(hb.bin, s);
    hb.bin = nullptr;
    if (record) {
        const unsigned long long cap = hb.most ? region_cap(hb.most, kHitBatchBudget)
                                               : region_first(hb.listed_up, hb.waves, kHitBatchBudget);
        if (cap > hb.cap) {
            if (hb.hits) dev_free(hb.hits, s);
            hb.hits = nullptr;
            hb.cap = 0;
            try {
                hb.hits = dev_alloc_n<int2>((size_t)(cap * kHitRegions), s);
                hb.cap = cap;
            } catch (const OomError &) {  // the pairs call evaluates its tiles again
            }
        }
    }
    HitOut R{};
    R.cnt = hb.cnt;
    R.ctr = ctr;
    R.tally = hb.tally;
    if (record && hb.hits) {
        R.hits = static_cast<int2 *>(hb.hits);
        R.cursor = hb.cursor;
        R.cap = hb.cap;
    }
    fill_zero_many({{hb.cnt, ((size_t)hb.rows + 1) * sizeof(int32_t)},
                    {hb.cursor, (kHitRegions + kHitTally) * kHitCursorStride * sizeof(unsigned long long)}},
                   s);
    const HitProb *dp = static_cast<const HitProb *>(hb.dev);
    const int P = (int)hb.probs.size();
    for (const HitBatch::Form &f : hb.forms) {
        const int nb = f.hi - f.lo;
        const int nseg = hit_batch_segments(nb);
        by_k_steps<2, 16>(f.ks, [&](auto ks) {
            hipLaunchKernelGGL(k_hit_f64_batch<decltype(ks)::value>, dim3((unsigned)(nb * nseg)), dim3(kThreads), 0, s,
                               dp, hb.block_base, P, hb.queue + f.lo, R, nseg);
        });
        SJ_HIP(hipGetLastError());
    }
    exclusive_scan_i32_to_i64(hb.cnt, hb.off, hb.rows + 1, s);
    hb.listed = R.hits != nullptr;
    // totals and the fullest region: one copy
    int64_t *out = dev_alloc_n<int64_t>(P + 1, s);
    hipLaunchKernelGGL(k_hit_totals, dim3((unsigned)((P + 1 + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, dp,
                       hb.off, hb.rows, P, hb.cursor, hb.tally, ctr, out);
    SJ_HIP(hipGetLastError());
    std::vector<int64_t> h(P + 1);
    SJ_HIP(hipMemcpyAsync(h.data(), out, (P + 1) * sizeof(int64_t), hipMemcpyDeviceToHost, s));
    SJ_HIP(hipStreamSynchronize(s));
    dev_free(out, s);
    hb.total = 0;
    for (int k = 0; k < P; ++k) {
        totals[hb.probs[k]] = h[k];
        hb.total += h[k];
    }
    if (hb.listed) {
        hb.most = (unsigned long long)h[P];
        hb.valid = hb.most <= hb.cap;
    }
}

// A valid list for the pairs call, the count run again where it kept none.
bool hit_batch_ensure(HitBatch &hb, DevCounters *ctr, std::vector<int64_t> &totals, hipStream_t s) {
    for (int tries = 0; tries < 2 && !hb.valid; ++tries) {
        if (hb.most && !region_cap(hb.most, kHitBatchBudget)) return false;
        hit_batch_count(hb, true, ctr, totals.data(), s);
        if (!hb.listed) return false;
    }
    return hb.valid;
}

// The list's bins (valid list); false when there is no memory for them.
bool hit_batch_bins(HitBatch &hb, hipStream_t s) {
    if (hb.bin) return true;
    const BinPlan bp = bin_plan(hb.rows, hb.total);
    try {
        DevBuf<int32_t> fill(bp.nfill, s);
        DevBuf<int32_t> bin((size_t)std::max<int64_t>(hb.total, 1), s);
        fill_zero_many({{fill.p, bp.nfill * sizeof(int32_t)}}, s);
        make_bins(bp, static_cast<const int2 *>(hb.hits), hb.cursor, hb.cap, hb.most, hb.off, hb.rows, fill.p, bin.p, s);
        hb.bin = bin.release();
    } catch (const OomError &) {
        return false;
    }
    return true;
}

// Pairs of these problems from the bins, problem i's at pout[i].
void hit_batch_pairs(HitBatch &hb, const std::vector<int64_t> &pout, int32_t *pairs, hipStream_t s) {
    const int P = (int)hb.probs.size();
    HitProb *hp = reinterpret_cast<HitProb *>(hb.host_probs.data());
    for (int k = 0; k < P; ++k) hp[k].pout = pout[hb.probs[k]];
    SJ_HIP(hipMemcpyAsync(hb.dev, hp, P * sizeof(HitProb), hipMemcpyHostToDevice, s));
    const size_t nbig = (size_t)(hb.total / kWaveBin) + 1;
    DevBuf<int32_t> work(2 + 2 * nbig, s);
    fill_zero(work.p, sizeof(int32_t), s);
    EmitSrc src{};
    src.P = static_cast<const HitProb *>(hb.dev);
    src.item_base = hb.item_base;
    src.B = P;
    src.E.off = hb.off;
    src.E.bin = hb.bin;
    src.E.item_hi = (int32_t)hb.items;
    src.E.pairs = reinterpret_cast<int2 *>(pairs);
    src.E.big = work.p;
    src.E.per = kTileQ;
    while (src.E.per > 1 && hb.items * (kTileQ / src.E.per) < 16384) src.E.per /= 2;
    const int64_t waves = hb.items * (kTileQ / src.E.per);
    hipLaunchKernelGGL(k_hit_emit<true>, dim3((unsigned)((waves + kWaves - 1) / kWaves)), dim3(kThreads), 0, s, src);
    SJ_HIP(hipGetLastError());
    if (hb.total > kWaveBin) {
        hipLaunchKernelGGL(k_hit_emit_big<true>, dim3((unsigned)std::min<size_t>(nbig, 1024)), dim3(kThreads), 0, s, src);
        SJ_HIP(hipGetLastError());
    }
}

}  // namespace sj

extern "C" void sj_test_hits(int32_t always, unsigned long long first) {
    sj::tl_hits_always = always;
    sj::tl_hits_first = first;
}
