// Level-of-detail cut on the GPU.
//
// Top-down, level-synchronous traversal of the hierarchy for all views at
// once (NavGSim Sec. III-B: LOD rendering selects Gaussians from different
// levels of the tree).  The frontier holds (node, view) entries of one level,
// a node's views mostly next to each other (see k_level_emit).  Per level:
//   count : each block decides its contiguous chunk (in the learned cut the
//           network settles the candidates right there), stores the
//           decisions and reduces (emitted, children) counts, which are also
//           added to the bin of its 64 neighbours;
//   emit  : each block adds the bins and blocks before it, reads its chunk's
//           decisions back, scans within the block and writes emitted ids
//           and child ids in order; block 0 advances the cut size and sets
//           the next frontier size (capacity checks here).
// A level's grid is sized to its frontier's bound (nodes of the level times
// views), at most kCutBlocks workgroups.  The leading levels of at most
// kTopEntries entries run in one launch of one workgroup (k_cut_top).
// A launch of a small level costs 3 to 6 us whatever it does: a level was
// three launches with a one-block scan of the counts between the two.
// Ids come out ascending per view because ids are level-major, children
// of a node are contiguous and ordered like their parents, and each view's
// entries keep their order through the emission.
//
// The node test is exact: FP64 with +, -, * only, in a fixed order, with FMA
// contraction disabled, so every IEEE FP64 implementation selects the same
// node set.
#include "device_util.h"
#include "internal.h"
#include "lod_mlp.h"

namespace hgs {

namespace {

constexpr int kNT = 256;
constexpr int kNW = kNT / kWave;
static_assert(kCutBins * kWave == kCutBlocks, "a bin per 64 blocks");

// Leading levels of at most this many entries (nodes x views) run in the one
// workgroup of k_cut_top, an entry per thread.
constexpr int kTopEntries = 1024;

enum : uint32_t { kDrop = 0, kEmit = 1, kExpand = 2, kCandidate = 4 };

// Decide a node for a view: dropped (sphere outside the frustum), emitted,
// or expanded into its children.  kCandidate is or-ed into kExpand when the
// threshold rule refines the node and its projected size is at most s_hi
// pixels: the band in which the learned rule may keep the node instead (the
// count pass lets the network make that choice).
__device__ __forceinline__ uint32_t node_decision(const ViewDev& V, int k, float4 b, int nchild, double s_hi) {
#pragma clang fp contract(off)
    NodeGeom g;
    node_geometry(V, b, &g);
    if (g.pz + g.r < V.znear) return kDrop;
    const double rr = g.r * g.r;
    const double eL = V.fx * g.px + V.cx * g.pz;
    if (eL < 0.0 && eL * eL > rr * V.nl) return kDrop;
    const double eR = V.fx * g.px + (V.cx - V.W) * g.pz;
    if (eR > 0.0 && eR * eR > rr * V.nr) return kDrop;
    const double eT = V.fy * g.py + V.cy * g.pz;
    if (eT < 0.0 && eT * eT > rr * V.nt) return kDrop;
    const double eB = V.fy * g.py + (V.cy - V.H) * g.pz;
    if (eB > 0.0 && eB * eB > rr * V.nb) return kDrop;
    if (nchild == 0) return kEmit;
    const double a = V.f2 * g.r;
    const double lhs = a * a;
    const double rhs = V.tau2 * g.d2;
    if (!(lhs > rhs)) return kEmit;
    if (k == V.keep_node) return kEmit;
    const bool cand = lhs <= (s_hi * s_hi) * g.d2;
    return kExpand | (cand ? kCandidate : 0u);
}

struct LevelCtx {
    const float4* bound;
    const int2* child;
    const ViewDev* views;
    int n_views;
    const uint2* in;
    uint2* out;
    uint32_t in_cap;
    uint32_t out_cap;
    uint2* cut;
    uint32_t cut_cap;
    uint4* fine;              // [G] block counts
    uint4* bins;              // [kCutBins] sums of 64 blocks' counts, zero before the level
    uint4* lvl;               // per level: (frontier entries, cut entries and candidates before it)
    uint8_t* dec;             // per frontier entry: decision of the count pass
    bool defer;               // learned cut: the count pass lets the network settle candidates
    const float* w32;         // learned cut: FP32 weights (uniform: read through the scalar cache)
    Counters* ctr;
    int mode;
    const void* mlp;
    double s_hi;
    uint2* cand;
    uint32_t cand_cap;
    int level;
    bool leaves;              // the last level: every node is a leaf (no child ranges to read)
    bool group;               // children laid out child-major per group of a node's views
    uint32_t* zero;           // words to clear at the start
    uint32_t n_zero;
};

__device__ __forceinline__ void chunk_of(uint32_t n, int G, int b, uint32_t* lo, uint32_t* hi) {
    uint32_t chunk = ceil_div(n, (uint32_t)G);
    if (chunk < (uint32_t)kNT) chunk = kNT;
    chunk = ceil_div(chunk, (uint32_t)kNT) * kNT;
    uint64_t s = (uint64_t)b * chunk, e = s + chunk;
    *lo = (uint32_t)(s < n ? s : n);
    *hi = (uint32_t)(e < n ? e : n);
}

// (emitted, children, candidate) counts of a decision
__device__ __forceinline__ uint4 counts_of(const LevelCtx& c, uint32_t d, int nchild) {
    const uint32_t kind = d & 3u;
    return make_uint4(kind == kEmit ? 1u : 0u, kind == kExpand ? (uint32_t)nchild : 0u,
                      (c.cand != nullptr && (d & kCandidate)) ? 1u : 0u, 0u);
}

// Count pass: decide every entry of the block's chunk once, remember the
// decision for the emit pass, reduce the counts.  In the learned cut
// (DEFER) the candidates of each 256 entries are settled right here: their
// features are computed one lane per candidate and the matrix cores
// evaluate the network over the group (64 entries per wave; the network's
// work is negligible, so the group is not compacted).  The network keeps a
// candidate (emits it) unless its probability reaches p*.
//
// With node-grouped frontiers, views are staged in LDS: a wave's entries span
// several views (a node's views are next to each other), and LDS serves a
// lane's own view without a gather.  A window of kLdsViews views holds them
// all in most passes; with more, it starts at the view group of the step's
// first entry and moves with the frontier, whose groups follow one another
// (the entries of a step that lie outside it read their view from memory).
// Without the window the leaf level of a 96-view batch took 648 us, with it 290.
// Staged are the leading words through the side-plane normals and keep_node,
// all that the node test and the features read.
constexpr uint32_t kLdsViews = 2 * kCutViewGroup;
constexpr int kCutViewWords = (int)((offsetof(ViewDev, nb) + sizeof(double)) / 8);
static_assert(offsetof(ViewDev, o) == 0 && offsetof(ViewDev, nb) % 8 == 0, "views start with their FP64 words");

template <bool DEFER, int NT>
struct CountShared {
    float x[DEFER ? NT * kMlpXStride : 1];
    float w[DEFER ? kMlpParams : 1];               // the network's FP32 weights
    uint64_t view[kLdsViews * kCutViewWords];
    int32_t keep[kLdsViews];
};

// The window of views from v0 on (view-major frontiers keep a wave on one
// view: scalar loads serve it).
template <bool DEFER, int NT>
__device__ __forceinline__ void stage_views(const LevelCtx& c, CountShared<DEFER, NT>& S, uint32_t v0) {
    if (c.group) {
        const uint32_t n = min((uint32_t)c.n_views - v0, kLdsViews);
        const uint64_t* src = reinterpret_cast<const uint64_t*>(c.views + v0);
        for (uint32_t k = threadIdx.x; k < n * kCutViewWords; k += NT) {
            const uint32_t v = k / kCutViewWords, q = k - v * kCutViewWords;
            S.view[k] = src[(size_t)v * (sizeof(ViewDev) / 8) + q];
        }
        for (uint32_t v = threadIdx.x; v < n; v += NT) S.keep[v] = c.views[v0 + v].keep_node;
    }
    __syncthreads();
}

template <bool DEFER, int NT>
__device__ __forceinline__ void stage_weights(const LevelCtx& c, CountShared<DEFER, NT>& S) {
    if (DEFER)
        for (int k = threadIdx.x; k < kMlpParams; k += NT) S.w[k] = c.w32[k];
}

// f applied to view v, the staged window starting at v0 (the staged words;
// the others, which neither the node test nor the features read, stay zero).
template <bool DEFER, int NT, class F>
__device__ __forceinline__ auto with_view(const LevelCtx& c, const CountShared<DEFER, NT>& S, uint32_t v0, uint32_t v,
                                          F&& f) {
    if (c.group && v - v0 < kLdsViews) {
        const uint32_t at = v - v0;
        uint64_t wd[sizeof(ViewDev) / 8];
#pragma unroll
        for (int q = 0; q < (int)(sizeof(ViewDev) / 8); ++q)
            wd[q] = q < kCutViewWords ? S.view[at * kCutViewWords + q] : 0ull;
        ViewDev V;
        __builtin_memcpy(&V, wd, sizeof V);
        V.keep_node = S.keep[at];
        return f(V);
    }
    return on_view(c.views, v, f);
}

template <bool DEFER, int NT>
__device__ __forceinline__ uint32_t decide(const LevelCtx& c, const CountShared<DEFER, NT>& S, uint32_t v0, bool valid,
                                           uint2 e, float4 b, int nchild) {
    if (!valid) return kDrop;
    return with_view(c, S, v0, e.y, [&](const ViewDev& V) { return node_decision(V, (int)e.x, b, nchild, c.s_hi); });
}

// The network's say on the candidates among one entry per thread (every
// thread of the workgroup takes part).
template <int NT>
__device__ __forceinline__ uint32_t settle(const LevelCtx& c, CountShared<true, NT>& S, uint32_t v0, uint32_t d, uint2 e,
                                           float4 b) {
    const bool cand = (d & kCandidate) != 0;
    if (!__syncthreads_or(cand)) return d;         // also orders S.x's reuse and publishes S.w
    const LodMlpDev& m = *(const LodMlpDev*)c.mlp;
    float f[kMlpIn];
#pragma unroll
    for (int k = 0; k < kMlpIn; ++k) f[k] = 0.f;
    if (cand) {
        with_view(c, S, v0, e.y, [&](const ViewDev& V) {
            NodeGeom g;
            node_geometry(V, b, &g);
            lod_features(m, V, (int)e.x, b, g, c.level, f);
        });
#pragma unroll
        for (int k = 0; k < kMlpIn; ++k) f[k] = (f[k] - m.mean[k]) * m.inv_std[k];
    }
#pragma unroll
    for (int k = 0; k < kMlpIn; ++k) S.x[threadIdx.x * kMlpXStride + k] = f[k];
    __syncthreads();
    const float z = lod_mlp_logit_mfma(S.w, S.x + threadIdx.x / kWave * kWave * kMlpXStride);
    return (cand && !(1.f / (1.f + __expf(-z)) >= m.p_star)) ? (uint32_t)kEmit : d;
}

// Decide entries [lo, hi), the weights staged in S; returns this thread's
// share of the counts.
template <bool DEFER>
__device__ __forceinline__ uint4 count_chunk(const LevelCtx& c, uint32_t lo, uint32_t hi, CountShared<DEFER, kNT>& S) {
    uint4 acc = make_uint4(0, 0, 0, 0);
    auto count = [&](uint32_t i, bool valid, uint32_t d, int2 ch) {
        if (!valid) return;
        c.dec[i] = (uint8_t)d;
        const uint4 r = counts_of(c, d, ch.y);
        acc.x += r.x;
        acc.y += r.y;
        acc.z += r.z;
    };
    // two entries per lane and step: their gathers are in flight together
    uint32_t win = ~0u;                            // first staged view
    for (uint32_t s = lo; s < hi; s += 2 * kNT) {
        const uint32_t v0w = c.n_views <= (int)kLdsViews ? 0u : c.in[s].y / kCutViewGroup * kCutViewGroup;
        if (v0w != win) {
            if (win != ~0u) __syncthreads();
            stage_views(c, S, v0w);
            win = v0w;
        }
        const uint32_t i0 = s + threadIdx.x, i1 = i0 + kNT;
        const bool v0 = i0 < hi, v1 = i1 < hi;
        const uint2 e0 = v0 ? c.in[i0] : make_uint2(0, 0);
        const uint2 e1 = v1 ? c.in[i1] : make_uint2(0, 0);
        const float4 b0 = c.bound[e0.x], b1 = c.bound[e1.x];
        const int2 ch0 = c.leaves ? make_int2(0, 0) : c.child[e0.x];
        const int2 ch1 = c.leaves ? make_int2(0, 0) : c.child[e1.x];
        uint32_t d0 = decide(c, S, win, v0, e0, b0, ch0.y);
        uint32_t d1 = decide(c, S, win, v1, e1, b1, ch1.y);
        if constexpr (DEFER) {
            d0 = settle(c, S, win, d0, e0, b0);
            d1 = settle(c, S, win, d1, e1, b1);
        }
        count(i0, v0, d0, ch0);
        count(i1, v1, d1, ch1);
    }
    return acc;
}

// Sum of (x, y, z) over a wave, in every lane.
__device__ __forceinline__ uint4 wave_sum3(uint4 v) {
    return make_uint4(wave_sum(v.x), wave_sum(v.y), wave_sum(v.z), 0u);
}

template <bool DEFER>
__global__ __launch_bounds__(kNT) void k_level_count(LevelCtx c) {
    __shared__ CountShared<DEFER, kNT> S;
    __shared__ uint4 s_tot[kNW];
    const uint32_t n = c.lvl[c.level].x;
    uint32_t lo, hi;
    chunk_of(n, gridDim.x, blockIdx.x, &lo, &hi);
    if (lo >= hi) return;                          // no block at or after this one is read
    stage_weights(c, S);
    const uint4 acc = wave_sum3(count_chunk<DEFER>(c, lo, hi, S));
    if (lane_id() == 0) s_tot[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint4 t = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int w = 0; w < kNW; ++w) {
            t.x += s_tot[w].x;
            t.y += s_tot[w].y;
            t.z += s_tot[w].z;
        }
        c.fine[blockIdx.x] = t;
        uint4* bin = c.bins + blockIdx.x / kWave;
        if (t.x) atomicAdd(&bin->x, t.x);
        if (t.y) atomicAdd(&bin->y, t.y);
        if (t.z) atomicAdd(&bin->z, t.z);
    }
}

// End of a level of n_in entries with totals tot (one thread): capacity
// checks, the cut size, and the next level's line of the table (returned).
__device__ __forceinline__ uint4 finish_level(const LevelCtx& c, uint32_t n_in, uint4 at, uint4 tot) {
    Counters* k = c.ctr;
    k->visited += n_in;
    uint4 next;
    const uint64_t want_cand = (uint64_t)at.z + tot.z;
    next.z = at.z;
    if (c.cand != nullptr) {
        if (want_cand > c.cand_cap) {
            k->overflow |= kOvCand;
            if (want_cand > k->need_cand) k->need_cand = (uint32_t)(want_cand < 0xffffffffull ? want_cand : 0xffffffffull);
        }
        next.z = (uint32_t)(want_cand < c.cand_cap ? want_cand : c.cand_cap);
        k->cand = next.z;
    }
    const uint64_t want_cut = (uint64_t)at.y + tot.x;
    if (want_cut > c.cut_cap) {
        k->overflow |= kOvCut;
        if (want_cut > k->need_cut) k->need_cut = (uint32_t)(want_cut < 0xffffffffull ? want_cut : 0xffffffffull);
    }
    next.y = (uint32_t)(want_cut < c.cut_cap ? want_cut : c.cut_cap);
    k->cut = next.y;
    if (tot.y > c.out_cap) {
        k->overflow |= kOvFrontier;
        if (tot.y > k->need_frontier) k->need_frontier = tot.y;
    }
    next.x = tot.y < c.out_cap ? tot.y : c.out_cap;
    next.w = 0;
    c.lvl[c.level + 1] = next;
    return next;
}

// Each thread takes kEmitPer consecutive entries of the chunk, so that one
// workgroup scan places 1,024 entries.  The children an iteration appends
// to the next frontier form one run; it is assembled in LDS (up to
// kEmitStage entries, the rest stored directly) and written out coalesced.
// Within the run, the children of one group (consecutive entries of the
// same node, one per view) are laid out child-major: (c0, v1), (c0, v2),
// ..., (c1, v1), ...  A node's views thus stay next to each other at every
// level, so that the passes reading a node's data per entry (this cut's
// node tests, the projection's Gaussian and SH reads) find it in cache for
// the second and later views.  Each view's entries keep their order.
constexpr int kEmitPer = 4;
constexpr uint32_t kEmitStage = 4096;
__global__ __launch_bounds__(kNT) void k_level_emit(LevelCtx c) {
    __shared__ uint4 sh[kNT / kWave + 1];
    __shared__ uint4 s_off[2];
    __shared__ uint2 s_out[kEmitStage];
    __shared__ uint2 s_last[kNT];                       // (node, view group) of each thread's last entry
    __shared__ uint32_t s_gbase[kEmitPer * kNT + 1];    // children before each group, then the total
    const uint32_t blk = blockIdx.x, l = lane_id();
    // what the blocks before this one emitted: whole bins (first wave), then
    // the blocks before it in its bin (second wave)
    static_assert(kCutBins == kWave, "one bin per lane");
    const uint4 zero = make_uint4(0, 0, 0, 0);
    uint4 cnt = zero;
    if (threadIdx.x < kWave) cnt = c.bins[l];
    else if (threadIdx.x < 2 * kWave) cnt = c.fine[blk - blk % kWave + l];
    const uint4 at = c.lvl[c.level];
    const uint32_t n = at.x;
    uint32_t lo, hi;
    chunk_of(n, gridDim.x, blk, &lo, &hi);
    if (threadIdx.x < kWave && blk == 0) {
        const uint4 tot = wave_sum3(cnt);
        if (l == 0) finish_level(c, n, at, tot);
    }
    if (lo >= hi) return;
    if (threadIdx.x < 2 * kWave) {
        const uint4 before = wave_sum3(l < (threadIdx.x < kWave ? blk / kWave : blk % kWave) ? cnt : zero);
        if (l == 0) s_off[threadIdx.x / kWave] = before;
    }
    __syncthreads();
    uint4 off = make_uint4(s_off[0].x + s_off[1].x, s_off[0].y + s_off[1].y, s_off[0].z + s_off[1].z, 0u);
    const uint32_t base = at.y, cbase = at.z;
    for (uint32_t s = lo; s < hi; s += kEmitPer * kNT) {
        // chunks start at multiples of kNT, so i0 is a multiple of kEmitPer
        const uint32_t i0 = s + kEmitPer * threadIdx.x;
        uint2 e[kEmitPer];
        uint32_t d[kEmitPer];
        if (i0 + kEmitPer <= hi) {
            const uint4 q0 = *reinterpret_cast<const uint4*>(c.in + i0);
            const uint4 q1 = *reinterpret_cast<const uint4*>(c.in + i0 + 2);
            e[0] = make_uint2(q0.x, q0.y);
            e[1] = make_uint2(q0.z, q0.w);
            e[2] = make_uint2(q1.x, q1.y);
            e[3] = make_uint2(q1.z, q1.w);
            const uint32_t dd = *reinterpret_cast<const uint32_t*>(c.dec + i0);
#pragma unroll
            for (int j = 0; j < kEmitPer; ++j) d[j] = (dd >> (8 * j)) & 0xffu;
        } else {
#pragma unroll
            for (int j = 0; j < kEmitPer; ++j) {
                const bool v = i0 + j < hi;
                e[j] = v ? c.in[i0 + j] : make_uint2(0, 0);
                d[j] = v ? c.dec[i0 + j] : (uint32_t)kDrop;
            }
        }
        uint4 r[kEmitPer];
        int first[kEmitPer];
        bool head[kEmitPer];
        uint4 mine = make_uint4(0, 0, 0, 0);
        const bool grouped = c.group && !c.leaves;
        if (grouped) {
            s_last[threadIdx.x] = make_uint2(e[kEmitPer - 1].x, e[kEmitPer - 1].y / kCutViewGroup);
            __syncthreads();
        }
        uint2 prev = (grouped && threadIdx.x > 0) ? s_last[threadIdx.x - 1] : make_uint2(~0u, ~0u);
#pragma unroll
        for (int j = 0; j < kEmitPer; ++j) {
            const bool expand = (d[j] & 3u) == kExpand;
            const int2 ch = (expand && !c.leaves) ? c.child[e[j].x] : make_int2(0, 0);
            first[j] = ch.x;
            r[j] = counts_of(c, d[j], ch.y);
            // a group starts where the node or the view group changes (node
            // ids are below 2^31)
            const uint32_t vg = e[j].y / kCutViewGroup;
            head[j] = e[j].x != prev.x || vg != prev.y;
            prev = make_uint2(e[j].x, vg);
            mine.x += r[j].x;
            mine.y += r[j].y;
            mine.z += r[j].z;
            mine.w += head[j] ? 1u : 0u;
        }
        uint4 tot;
        uint4 ex = block_excl_scan4<kNT>(mine, sh, &tot);
        uint32_t grp[kEmitPer], ey[kEmitPer];
        {
            uint4 run = ex;
#pragma unroll
            for (int j = 0; j < kEmitPer; ++j) {
                run.w += head[j] ? 1u : 0u;
                grp[j] = run.w - 1u;                    // this entry's group within the iteration
                ey[j] = run.y;
                if (grouped && head[j]) s_gbase[grp[j]] = run.y;
                run.y += r[j].y;
            }
        }
        if (grouped) {
            if (threadIdx.x == 0) s_gbase[tot.w] = tot.y;
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < kEmitPer; ++j) {
            if (r[j].x) {
                const uint64_t pos = (uint64_t)base + off.x + ex.x;
                if (pos < c.cut_cap) c.cut[pos] = e[j];
            }
            if (r[j].z) {
                const uint64_t pos = (uint64_t)cbase + off.z + ex.z;
                if (pos < c.cand_cap) c.cand[pos] = e[j];
            }
            const uint32_t m = r[j].y;
            if (m) {
                // every expanding entry of the group has this node's m
                // children: the group's children are m * n_exp, this entry
                // is the rank-th expanding one (ungrouped: its children in
                // order at ey)
                uint32_t gb = ey[j], n_exp = 1, rank = 0;
                if (grouped) {
                    gb = s_gbase[grp[j]];
                    n_exp = (s_gbase[grp[j] + 1] - gb) / m;
                    rank = (ey[j] - gb) / m;
                }
                for (uint32_t q = 0; q < m; ++q) {
                    const uint32_t L = gb + q * n_exp + rank;
                    const uint2 child = make_uint2((uint32_t)(first[j] + (int)q), e[j].y);
                    if (L < kEmitStage) {
                        s_out[L] = child;
                    } else {
                        const uint64_t pos = (uint64_t)off.y + L;
                        if (pos < c.out_cap) c.out[pos] = child;
                    }
                }
            }
            ex.x += r[j].x;
            ex.z += r[j].z;
        }
        if (!c.leaves) {
            __syncthreads();
            const uint32_t staged = tot.y < kEmitStage ? tot.y : kEmitStage;
            for (uint32_t q = threadIdx.x; q < staged; q += kNT) {
                const uint64_t pos = (uint64_t)off.y + q;
                if (pos < c.out_cap) c.out[pos] = s_out[q];
            }
            __syncthreads();
        }
        off.x += tot.x;
        off.y += tot.y;
        off.z += tot.z;
    }
}

// Entry i of the frontier of every view's roots (nodes [0, n_roots)):
// grouped, view groups in order and node-major within a group; otherwise
// view-major.
__device__ __forceinline__ uint2 root_entry(uint32_t i, uint32_t n_roots, uint32_t n_views, bool grouped) {
    if (!grouped) return make_uint2(i % n_roots, i / n_roots);
    const uint32_t per = n_roots * kCutViewGroup;          // entries of a full group
    const uint32_t vb = i / per, loc = i - vb * per;
    const uint32_t nb = min(kCutViewGroup, n_views - vb * kCutViewGroup);
    return make_uint2(loc / nb, vb * kCutViewGroup + loc % nb);
}

// Counters of a new render, with the roots' frontier size checked.
__device__ __forceinline__ void start_counters(Counters* ctr, uint64_t roots, uint32_t cap) {
    Counters z = {};
    if (roots > cap) {
        z.overflow = kOvFrontier;
        z.need_frontier = (uint32_t)(roots < 0xffffffffull ? roots : 0xffffffffull);
    }
    *ctr = z;
}

// Start of a cut: counters, the counts of binned entries and the levels' bins,
// the roots' frontier.
__global__ __launch_bounds__(kNT) void k_cut_init(LevelCtx c, uint2* out, uint32_t n_roots, uint4* clear, int n_clear) {
    const uint32_t total = n_roots * (uint32_t)c.n_views;
    const uint32_t i0 = blockIdx.x * kNT + threadIdx.x, step = gridDim.x * kNT;
    for (uint32_t i = i0; i < total && i < c.in_cap; i += step) out[i] = root_entry(i, n_roots, c.n_views, c.group);
    for (uint32_t i = i0; i < (uint32_t)n_clear; i += step) clear[i] = make_uint4(0, 0, 0, 0);
    for (uint32_t i = i0; i < c.n_zero; i += step) c.zero[i] = 0;
    if (i0 == 0) {
        start_counters(c.ctr, total, c.in_cap);
        c.lvl[0] = make_uint4(total < c.in_cap ? total : c.in_cap, 0, 0, 0);
    }
}

// The same start, then the first `levels` levels, by one workgroup with an
// entry per thread (every one of these levels holds at most kTopEntries
// entries): an entry is decided, counted, placed and its children written to
// the next frontier, in LDS, without a trip through memory in between; the
// children of the last of these levels go to out.  The same cut order as
// k_level_emit's: children child-major within a node's views.  One view's
// four leading levels of a 2M-leaf tree: 15.0 us here, 54 as a reset, a
// roots' launch and three launches a level.
template <bool DEFER>
__global__ __launch_bounds__(kTopEntries) void k_cut_top(LevelCtx c, uint2* out, uint32_t n_roots, int levels,
                                                         int n_levels, uint4* clear, int n_clear) {
    constexpr int NT = kTopEntries;
    __shared__ CountShared<DEFER, NT> S;
    __shared__ uint2 s_f[2][NT];
    __shared__ uint4 s_scan[NT / kWave + 1];
    __shared__ uint32_t s_gbase[NT + 1];
    __shared__ uint4 s_next;
    const uint32_t t = threadIdx.x;
    const uint32_t total = n_roots * (uint32_t)c.n_views;
    uint4 at = make_uint4(total < c.in_cap ? total : c.in_cap, 0, 0, 0);
    if (t < total) s_f[0][t] = root_entry(t, n_roots, c.n_views, c.group);
    for (int i = t; i < n_clear; i += NT) clear[i] = make_uint4(0, 0, 0, 0);
    for (uint32_t i = t; i < c.n_zero; i += NT) c.zero[i] = 0;
    if (t == 0) start_counters(c.ctr, total, c.in_cap);
    stage_weights(c, S);
    stage_views(c, S, 0);                          // (also orders the roots' entries)
    for (int L = 0; L < levels; ++L) {
        c.level = L;
        const bool leaves = L == n_levels - 1, last = L == levels - 1;
        const bool valid = t < at.x;
        const uint2 e = valid ? s_f[L & 1][t] : make_uint2(0, 0);
        const uint2 prev = valid && t > 0 ? s_f[L & 1][t - 1] : make_uint2(~0u, ~0u);
        const float4 b = c.bound[e.x];
        const int2 ch = leaves ? make_int2(0, 0) : c.child[e.x];
        uint32_t d = decide(c, S, 0u, valid, e, b, ch.y);
        if constexpr (DEFER) d = settle(c, S, 0u, d, e, b);
        uint4 r = counts_of(c, d, ch.y);
        // a group starts where the node or the view group changes; ungrouped,
        // every entry is one
        r.w = !c.group || e.x != prev.x || e.y / kCutViewGroup != prev.y / kCutViewGroup || t == 0 ? 1u : 0u;
        uint4 tot;
        const uint4 ex = block_excl_scan4<NT>(r, s_scan, &tot);
        const uint32_t grp = ex.w + r.w - 1u;
        if (r.w) s_gbase[grp] = ex.y;
        if (t == 0) {
            s_gbase[tot.w] = tot.y;
            s_next = finish_level(c, at.x, at, tot);
        }
        __syncthreads();
        if (r.x) {
            const uint64_t pos = (uint64_t)at.y + ex.x;
            if (pos < c.cut_cap) c.cut[pos] = e;
        }
        if (r.z) {
            const uint64_t pos = (uint64_t)at.z + ex.z;
            if (pos < c.cand_cap) c.cand[pos] = e;
        }
        if (r.y) {
            const uint32_t m = r.y, gb = s_gbase[grp];
            const uint32_t n_exp = (s_gbase[grp + 1] - gb) / m, rank = (ex.y - gb) / m;
            for (uint32_t q = 0; q < m; ++q) {
                const uint32_t pos = gb + q * n_exp + rank;
                const uint2 child = make_uint2((uint32_t)ch.x + q, e.y);
                if (last) {
                    if (pos < c.out_cap) out[pos] = child;
                } else if (pos < (uint32_t)NT) {
                    s_f[(L & 1) ^ 1][pos] = child;
                }
            }
        }
        __syncthreads();
        at = s_next;
    }
}

// Every listed id (or 0..n-1 when ids is null) for every view, view-major.
__global__ void k_emit_all(uint2* cut, const int32_t* ids, uint32_t n, uint32_t n_views, uint32_t cap, Counters* ctr,
                           uint32_t* zero, uint32_t n_zero, uint4* seen) {
    const uint64_t total = (uint64_t)n * n_views;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < total && i < cap;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t k = (uint32_t)(i % n);
        cut[i] = make_uint2(ids ? (uint32_t)ids[k] : k, (uint32_t)(i / n));
    }
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n_zero; i += gridDim.x * blockDim.x) zero[i] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        Counters z = {};
        if (total > cap) {
            z.overflow = kOvCut;
            z.need_cut = (uint32_t)(total < 0xffffffffull ? total : 0xffffffffull);
        }
        z.cut = (uint32_t)(total < cap ? total : cap);
        *ctr = z;
    }
    if (blockIdx.x == 0 && threadIdx.x < kSeenSlots / 4) seen[threadIdx.x] = make_uint4(0, 0, 0, 0);
}

// Features and screen footprint of each collected candidate.  The level of
// a node is recovered from the geometry record (mlp_geom.level_offset).
__global__ void k_lod_features(const uint2* cand, const uint32_t* count, const ViewDev* views, LodMlpDev m,
                               float* feats, int4* rects) {
    const uint32_t n = *count;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const uint2 e = cand[i];
        const ViewDev& V = views[e.y];
        const float4 b = m.bound[e.x];
        NodeGeom g;
        node_geometry(V, b, &g);
        int level = 0;
        while (level + 1 < m.n_levels && (int64_t)e.x >= m.level_offset[level + 1]) ++level;
        float f[kMlpIn];
        lod_features(m, V, (int)e.x, b, g, level, f);
#pragma unroll
        for (int k = 0; k < kMlpIn; ++k) feats[(size_t)i * kMlpIn + k] = f[k];
        // footprint: projection of the bounding sphere (centre +- f r / z),
        // the whole image when the sphere reaches the near plane; clamped to
        // the image and never empty
        int x0 = 0, y0 = 0, x1 = (int)V.W - 1, y1 = (int)V.H - 1;
        if (g.pz - g.r > V.znear) {
            const double u = V.fx * g.px / g.pz + V.cx, v = V.fy * g.py / g.pz + V.cy;
            const double ru = V.fx * g.r / (g.pz - g.r) + 1.0, rv = V.fy * g.r / (g.pz - g.r) + 1.0;
            const double lox = fmin(fmax(floor(u - ru), 0.0), V.W - 1.0), hix = fmin(fmax(ceil(u + ru), 0.0), V.W - 1.0);
            const double loy = fmin(fmax(floor(v - rv), 0.0), V.H - 1.0), hiy = fmin(fmax(ceil(v + rv), 0.0), V.H - 1.0);
            x0 = (int)lox; x1 = (int)hix; y0 = (int)loy; y1 = (int)hiy;
        }
        rects[i] = make_int4(x0, y0, x1, y1);
    }
}

}  // namespace

void launch_lod_features(const uint2* cand, const uint32_t* count, const ViewDev* views, const void* mlp_geom,
                         float* feats, int4* rects, hipStream_t s) {
    k_lod_features<<<1024, 256, 0, s>>>(cand, count, views, *(const LodMlpDev*)mlp_geom, feats, rects);
}

void launch_cut(const CutArgs& a, hipStream_t s) {
    if (a.flat || a.mode == HGS_LOD_ALL_LEAVES) {
        const uint32_t n = a.flat ? (uint32_t)a.n_nodes : (uint32_t)a.n_leaves;
        const int32_t* ids = a.flat ? nullptr : a.leaf_ids;
        k_emit_all<<<2048, 256, 0, s>>>(a.cut, ids, n, (uint32_t)a.n_views, a.cut_cap, a.ctr, a.zero, a.n_zero,
                                      a.scan_tmp + kSeenAt);
        return;
    }
    const uint32_t n_roots = (uint32_t)a.level_offset_host[1];
    // scratch: block counts, the level table, the bins of every level
    uint4* lvl = a.scan_tmp + kCutBlocks;
    uint4* seen = a.scan_tmp + kSeenAt;             // (cleared with the bins behind them)
    uint4* bins = seen + kSeenSlots / 4;
    const int n_clear = kSeenSlots / 4 + a.n_levels * kCutBins;
    LevelCtx c;
    c.bound = a.bound;
    c.child = a.child;
    c.views = a.views;
    c.n_views = a.n_views;
    c.in_cap = c.out_cap = a.frontier_cap;
    c.cut = a.cut;
    c.cut_cap = a.cut_cap;
    c.fine = a.scan_tmp;
    c.lvl = lvl;
    c.dec = a.dec;
    // p* = 0 refines every candidate: nothing for the network to decide
    c.defer = a.mode == HGS_LOD_LEARNED && a.mlp != nullptr && a.p_star > 0.f;
    c.w32 = a.mlp_w32;
    c.ctr = a.ctr;
    c.mode = a.mode;
    c.mlp = a.mlp;
    c.s_hi = a.s_hi;
    c.cand = a.cand;
    c.cand_cap = a.cand_cap;
    c.group = a.group_children;
    c.zero = a.zero;
    c.n_zero = a.n_zero;
    // a level's frontier holds at most (nodes of the level) x views entries
    auto bound_of = [&](int L) {
        return (uint64_t)(a.level_offset_host[L + 1] - a.level_offset_host[L]) * (uint64_t)a.n_views;
    };
    int top = 0;
    while (top < a.n_levels && bound_of(top) <= (uint64_t)kTopEntries) ++top;
    auto set_level = [&](int L) {
        c.in = a.frontier[L & 1];
        c.out = a.frontier[(L & 1) ^ 1];
        c.bins = bins + (size_t)L * kCutBins;
        c.level = L;
        c.leaves = L == a.n_levels - 1;
    };
    set_level(0);
    if (top == 0)
        k_cut_init<<<64, kNT, 0, s>>>(c, a.frontier[0], n_roots, seen, n_clear);
    else if (c.defer)
        k_cut_top<true><<<1, kTopEntries, 0, s>>>(c, a.frontier[top & 1], n_roots, top, a.n_levels, seen, n_clear);
    else
        k_cut_top<false><<<1, kTopEntries, 0, s>>>(c, a.frontier[top & 1], n_roots, top, a.n_levels, seen, n_clear);
    for (int L = top; L < a.n_levels; ++L) {
        set_level(L);
        // small levels get a grid of their bound's size (the chunking keeps
        // the entries' order, so the cut does not depend on the grid)
        const int GL = (int)std::min<uint64_t>((uint64_t)kCutBlocks, std::max<uint64_t>(1, (bound_of(L) + kNT - 1) / kNT));
        // a leaf is never refined, so the last level has no candidates
        if (c.defer && !c.leaves)
            k_level_count<true><<<GL, kNT, 0, s>>>(c);
        else
            k_level_count<false><<<GL, kNT, 0, s>>>(c);
        k_level_emit<<<GL, kNT, 0, s>>>(c);
    }
}

}  // namespace hgs
