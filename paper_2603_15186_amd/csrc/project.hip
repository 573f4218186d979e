// EWA projection of the cut's Gaussians with spherical-harmonic colour, and
// pair emission in depth order.
//
// Per cut entry (node, view): Sigma = R S S^T R^T (Supplementary Material of
// NavGSim), camera-space mean t = W (mu - o), first-order perspective
// Jacobian J at the mean (x/z and y/z clamped to the image's range widened
// by 15 % of its size per side), Sigma' = J W Sigma W^T J^T + 0.3 I, 2D mean
// (fx tx/tz + cx, fy ty/tz + cy), colour clamp(sum_k f_k Y_k(d) + 0.5, 0, 1).
//
// The geometry runs in FP64 (which keeps the conic of edge-on sheets
// accurate).  The pass is bound by its instructions, then by the 76 bytes an
// entry writes: with IEEE divisions and square roots and divisions by the
// tile sides 1,000 instructions an entry, 1,480 us for 38 M of them (writes
// 470 at the rate of a copy); with rcp64, rsqrt64 and shifts 1,340, and
// 370 -> 313 us for the 8 M entries of a 50-view batch.  Sigma' is formed as
// T T^T with T = J W R S (2x3), which is symmetric positive semidefinite by
// construction.  The depth key is the single-precision value of the FP64
// camera depth, whose three-term sum is evaluated in a fixed order with
// contraction disabled, so the depth order is an exact, reproducible result.
#include "device_util.h"
#include "internal.h"

namespace hgs {

namespace {

constexpr int kNT = 256;
// Binning covers q <= 9 (1 + kBinSlack): a superset of every pixel the
// compositor can take, whatever the rounding of its single-precision q.
constexpr double kBinSlack = 1e-3;
constexpr double kBinQ = 9.0 * (1.0 + kBinSlack);
constexpr double kBinReach = 3.0014996251273827;     // sqrt(kBinQ)

// Tile sides are powers of two.
__device__ __forceinline__ int log2_of(int side) { return 31 - __builtin_clz((uint32_t)side); }

// Entries of more tile rows than kTallRows (pairs than kBigPairs) may be
// counted (emitted) by their whole wave.
constexpr int kTallRows = 8;
constexpr uint32_t kBigPairs = 64;

// Rectangles of at most kMaskTiles tiles, in at most kTallRows rows, which their
// own lane counts, keep the tiles that the ellipse reaches as a bit mask (row
// by row) in their record, and the emission reads neither their projection
// nor solves for the rows again: k_emit of 41 M pairs 321 -> 278 us, of 77 M in
// two per entry 880 -> 811.
constexpr uint32_t kMaskTiles = 16;
__device__ __forceinline__ bool small_rect(ushort4 rc) {
    return rc.w - rc.y < kTallRows && (uint32_t)(rc.z - rc.x + 1) * (uint32_t)(rc.w - rc.y + 1) <= kMaskTiles;
}

// Entries per workgroup of a pass over m cut entries: 256, fewer when there
// are few, so that they spread over `blocks` workgroups.  A small view's pass
// lasts as long as its slowest workgroup, and a Gaussian close to the camera
// covers hundreds of tiles (a 1600 x 900 view of 80 of them, 89,000 pairs,
// rendered by one workgroup: 693 us; spread, and the large ones by whole
// waves: 194).  1,024 workgroups where each starts at once, 256 where each
// first clears the tiles' counts in LDS.  Wave w of a workgroup takes entries
// [w per / 4, (w + 1) per / 4), a lane each.
__device__ __forceinline__ uint32_t entries_per_block(uint32_t m, uint32_t blocks) {
    const uint32_t per = (ceil_div(m, blocks) + 3u) & ~3u;
    return per < (uint32_t)kNT ? (per > 4u ? per : 4u) : (uint32_t)kNT;
}

// Sums of 2^20 entries' pairs, enough for every entry index.
constexpr int kTopSums = 1 << (kNtShift - 20);
static_assert(kTopSums <= kNT && kTopSums / 2 <= kCutBlocks, "a thread per sum; they fit the cut's block counts");

__device__ __forceinline__ void clear_bins(const SortBins& b) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < b.n; i += gridDim.x * blockDim.x) b.words[i] = 0;
}

// This thread's entry among the block's `per` (per or more: none).
__device__ __forceinline__ uint32_t entry_slot(uint32_t per) {
    const uint32_t l = lane_id(), q = per / (kNT / kWave);
    return l < q ? threadIdx.x / kWave * q + l : per;
}

// Real spherical-harmonic basis (Condon-Shortley phase) up to degree 3 as
// Cartesian polynomials of the unit direction; index l*l + l + m.
// Constants: sqrt((2l+1)/(4 pi) (l-m)!/(l+m)!) times the polynomial's
// normalising factor, e.g. 0.5 sqrt(1/pi), sqrt(3/(4 pi)), 0.5 sqrt(15/pi),
// 0.25 sqrt(5/pi), 0.25 sqrt(15/pi), 0.25 sqrt(35/(2 pi)), 0.5 sqrt(105/pi),
// 0.25 sqrt(21/(2 pi)), 0.25 sqrt(7/pi), 0.25 sqrt(105/pi).
// With Blend, coefficient f of node g becomes f_p + t (f_g - f_p) with f_p
// that of node pg (pg < 0: no blending).  The coefficients of a Gaussian are
// one contiguous run of 3 K floats ([k][c]), read with 16-byte loads when
// 3 K is a multiple of four.
template <int DEG>
__device__ __forceinline__ void load_sh(const float* __restrict__ sh, int64_t g, float f[3 * (DEG + 1) * (DEG + 1)]) {
    constexpr int NF = 3 * (DEG + 1) * (DEG + 1);
    const float* src = sh + g * NF;
    if constexpr (NF % 4 == 0) {
#pragma unroll
        for (int q = 0; q < NF / 4; ++q) {
            const float4 v = reinterpret_cast<const float4*>(src)[q];
            f[4 * q] = v.x;
            f[4 * q + 1] = v.y;
            f[4 * q + 2] = v.z;
            f[4 * q + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int q = 0; q < NF; ++q) f[q] = src[q];
    }
}

template <bool Blend, int DEG>
__device__ __forceinline__ void sh_colour(const float* __restrict__ sh, int64_t g, int64_t pg, float t, float x,
                                          float y, float z, float rgb[3]) {
    constexpr int K = (DEG + 1) * (DEG + 1);
    constexpr float k00 = 0.28209479177387814f;
    constexpr float k1 = 0.48860251190291992f;
    constexpr float k2a = 1.0925484305920792f, k2b = 0.31539156525252005f, k2c = 0.54627421529603959f;
    constexpr float k3a = 0.59004358992664352f, k3b = 2.8906114426405538f, k3c = 0.45704579946446572f,
                    k3d = 0.3731763325901154f, k3e = 1.4453057213202769f;
    float Y[16];
    Y[0] = k00;
    if constexpr (DEG >= 1) {
        Y[1] = -k1 * y;
        Y[2] = k1 * z;
        Y[3] = -k1 * x;
    }
    if constexpr (DEG >= 2) {
        const float xx = x * x, yy = y * y, zz = z * z;
        Y[4] = k2a * x * y;
        Y[5] = -k2a * y * z;
        Y[6] = k2b * (3.f * zz - 1.f);
        Y[7] = -k2a * x * z;
        Y[8] = k2c * (xx - yy);
        if constexpr (DEG >= 3) {
            Y[9] = -k3a * y * (3.f * xx - yy);
            Y[10] = k3b * x * y * z;
            Y[11] = -k3c * y * (5.f * zz - 1.f);
            Y[12] = k3d * z * (5.f * zz - 3.f);
            Y[13] = -k3c * x * (5.f * zz - 1.f);
            Y[14] = k3e * z * (xx - yy);
            Y[15] = -k3a * x * (xx - 3.f * yy);
        }
    }
    float f[3 * K];
    load_sh<DEG>(sh, g, f);
    if (Blend && pg >= 0) {
        float fp[3 * K];
        load_sh<DEG>(sh, pg, fp);
#pragma unroll
        for (int q = 0; q < 3 * K; ++q) f[q] = fp[q] + t * (f[q] - fp[q]);
    }
    float acc[3] = {0.5f, 0.5f, 0.5f};
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[c] = fmaf(f[3 * k + c], Y[k], acc[c]);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) rgb[c] = fminf(fmaxf(acc[c], 0.f), 1.f);
}

// Tiles of one tile row that the ellipse q(d) <= Q reaches.  The ellipse
// meets the row's band of pixel-centre heights [yb0, yb1] (relative to the
// mean) in a convex set whose x-extent [xa, xb] is found in closed form: with
// q = (p dx + r dy)^2 + (s dy)^2, for a height dy the ellipse spans dx =
// (-r dy +- sqrt(Q - (s dy)^2)) / p, a concave right end and convex left end
// whose extremes over the band sit at the clamped heights of the ellipse's
// rightmost and leftmost points, -/+ r sqrt(Q) / (s sqrt(r^2 + s^2)).  A
// tile is reached iff its pixel-centre x-range overlaps [xa, xb]; the
// result is an interval of tiles (empty: lo > hi).  The factors are the
// stored single-precision ones (the same in the counting and the emitting
// pass).
struct RowSpan {
    double ip, r, s, ey, ymax_at_x;          // 1 / p; ymax_at_x: height of the rightmost point
};

// These functions are compiled into every place that counts an entry's tiles
// or lists them, by its own lane or by its wave, and all of them must find the
// same tiles, else a pair lands outside its run: the sums' roundings are
// written out, none is left to the compiler.
__device__ __forceinline__ RowSpan row_span_init(const Proj& p) {
#pragma clang fp contract(off)
    RowSpan r;
    r.ip = rcp64(p.p);
    r.r = p.r;
    r.s = p.s;
    r.ey = kBinReach * rcp64(r.s);
    r.ymax_at_x = -r.r * r.ey * rsqrt64(fma(r.r, r.r, r.s * r.s));
    return r;
}

// x-extent [xa, xb] (absolute pixels) of the ellipse within the band of
// pixel-centre heights [ya, yb] (absolute); false if they do not meet.
__device__ __forceinline__ bool band_span(const RowSpan& r, double u, double v, double ya, double yb, double* xa,
                                          double* xb) {
#pragma clang fp contract(off)
    double y0 = fmax(ya - v, -r.ey);
    double y1 = fmin(yb - v, r.ey);
    if (y0 > y1) return false;
    const double yr = fmin(fmax(r.ymax_at_x, y0), y1);
    const double yl = fmin(fmax(-r.ymax_at_x, y0), y1);
    const double tr = r.s * yr, tl = r.s * yl;
    const double sr = fmax(fma(-tr, tr, kBinQ), 1e-30), sl = fmax(fma(-tl, tl, kBinQ), 1e-30);
    *xb = fma(fma(-r.r, yr, sr * rsqrt64(sr)), r.ip, u) + 1e-7;
    *xa = fma(-fma(r.r, yl, sl * rsqrt64(sl)), r.ip, u) - 1e-7;
    return true;
}

// Tiles [lo, hi] of tile row ty (tiles of tw x th pixels) that the ellipse
// reaches, within [tx_lo, tx_hi]; lo > hi when none.
__device__ __forceinline__ void row_tiles(const RowSpan& r, double u, double v, int ty, int tw, int th, int H,
                                          int tx_lo, int tx_hi, int* lo, int* hi) {
#pragma clang fp contract(off)
    double xa, xb;
    const double ya = ty * th + 0.5, yb = fmin((double)(ty * th + th - 1), (double)(H - 1)) + 0.5;
    if (!band_span(r, u, v, ya, yb, &xa, &xb)) {
        *lo = 1;
        *hi = 0;
        return;
    }
    // tile tx covers pixel centres [tw tx + 0.5, tw tx + tw - 0.5]
    const double itw = __builtin_ldexp(1.0, -log2_of(tw));
    const int a = (int)ceil((xa - (tw - 0.5)) * itw);
    const int b = (int)floor((xb - 0.5) * itw);
    *lo = a > tx_lo ? a : tx_lo;
    *hi = b < tx_hi ? b : tx_hi;
}

// Tiles [lo, hi] of every tile row of rect `rc` that the ellipse reaches (all
// of the rect's when exact is false), handed to row(ty, lo, hi).
template <class F>
__device__ __forceinline__ void rect_rows(const Proj& p, ushort4 rc, int tw, int th, int H, bool exact, F row) {
    if (!exact || (rc.x == rc.z && rc.y == rc.w)) {
        for (int ty = rc.y; ty <= rc.w; ++ty) row(ty, (int)rc.x, (int)rc.z);
        return;
    }
    const RowSpan r = row_span_init(p);
    for (int ty = rc.y; ty <= rc.w; ++ty) {
        int lo, hi;
        row_tiles(r, p.u, p.v, ty, tw, th, H, rc.x, rc.z, &lo, &hi);
        row(ty, lo, hi);
    }
}

__device__ __forceinline__ float lane_f(float x, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
__device__ __forceinline__ double lane_d(double x, int l) {
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, l), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), l);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// Whether the wave's large entries are better taken by the whole wave, one
// after the other (about 200 instructions each and 18 per tile row), than by
// their own lanes side by side, where the longest sets the time (about 150
// per exact row, 8 per pair).  Uniform over the wave.
__device__ __forceinline__ bool wave_is_better(bool large, uint32_t rows, uint32_t pairs, bool exact) {
    if (__ballot(large) == 0) return false;
    const uint32_t together = wave_sum(large ? 200u + 18u * rows : 0u);
    uint32_t alone = large ? 8u * pairs + (exact ? 150u : 8u) * rows : 0u;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) alone = max(alone, (uint32_t)__shfl_xor(alone, d, kWave));
    return together < alone;
}

// The same rows by a whole wave, for the lanes with `big` set one after the
// other, a lane per row: rows(src, ty0, n, lo, hi) for up to 64 tile rows
// ty0 .. ty0 + n - 1 of lane src's entry, lane l holding the interval of row
// ty0 + l (empty: lo > hi; also the lanes past the n rows).  Every lane of
// the wave takes part.
template <class F>
__device__ __forceinline__ void wave_rect_rows(bool big, const Proj& p, ushort4 rc, int tw, int th, int H, bool exact,
                                               F rows) {
    uint64_t todo = __ballot(big);
    while (todo) {
        const int src = __builtin_ctzll(todo);
        todo &= todo - 1;
        Proj q = {};
        q.u = lane_d(p.u, src);
        q.v = lane_d(p.v, src);
        q.p = lane_f(p.p, src);
        q.r = lane_f(p.r, src);
        q.s = lane_f(p.s, src);
        const uint32_t xy0 = __builtin_amdgcn_readlane((uint32_t)rc.x | (uint32_t)rc.y << 16, src);
        const uint32_t xy1 = __builtin_amdgcn_readlane((uint32_t)rc.z | (uint32_t)rc.w << 16, src);
        const int x0 = (int)(xy0 & 0xffffu), y0 = (int)(xy0 >> 16), x1 = (int)(xy1 & 0xffffu), y1 = (int)(xy1 >> 16);
        const int h = __builtin_amdgcn_readlane(H, src);
        const RowSpan r = row_span_init(q);
        for (int ty0 = y0; ty0 <= y1; ty0 += kWave) {
            const int ty = ty0 + lane_id();
            int lo = 1, hi = 0;
            if (ty <= y1) {
                if (exact) {
                    row_tiles(r, q.u, q.v, ty, tw, th, h, x0, x1, &lo, &hi);
                } else {
                    lo = x0;
                    hi = x1;
                }
            }
            rows(src, ty0, min(kWave, y1 - ty0 + 1), lo, hi);
        }
    }
}

// Rows of T = M R diag(s) for the Gaussian with quaternion (w, x, y, z) =
// q and scales sc, and the entries of T T^T.
__device__ __forceinline__ void proj_cov(const double M0[3], const double M1[3], float4 q, float4 sc, double* a00,
                                         double* a01, double* a11) {
    double qw = q.x, qx = q.y, qy = q.z, qz = q.w;
    const double qi = rsqrt64(qw * qw + qx * qx + qy * qy + qz * qz);
    qw *= qi; qx *= qi; qy *= qi; qz *= qi;
    const double Rq[9] = {1.0 - 2.0 * (qy * qy + qz * qz), 2.0 * (qx * qy - qw * qz), 2.0 * (qx * qz + qw * qy),
                          2.0 * (qx * qy + qw * qz), 1.0 - 2.0 * (qx * qx + qz * qz), 2.0 * (qy * qz - qw * qx),
                          2.0 * (qx * qz - qw * qy), 2.0 * (qy * qz + qw * qx), 1.0 - 2.0 * (qx * qx + qy * qy)};
    const double s[3] = {sc.x, sc.y, sc.z};
    double T0[3], T1[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        T0[k] = (M0[0] * Rq[k] + M0[1] * Rq[3 + k] + M0[2] * Rq[6 + k]) * s[k];
        T1[k] = (M1[0] * Rq[k] + M1[1] * Rq[3 + k] + M1[2] * Rq[6 + k]) * s[k];
    }
    *a00 = T0[0] * T0[0] + T0[1] * T0[1] + T0[2] * T0[2];
    *a01 = T0[0] * T1[0] + T0[1] * T1[1] + T0[2] * T1[2];
    *a11 = T1[0] * T1[0] + T1[1] * T1[1] + T1[2] * T1[2];
}

// Projected bounding-sphere size 2 max(fx, fy) r / |c - o| in pixels, FP64
// in the cut's order of operations.
__device__ __forceinline__ double sphere_size(const ViewDev& V, float4 b) {
#pragma clang fp contract(off)
    const double bx = (double)b.x - V.o[0], by = (double)b.y - V.o[1], bz = (double)b.z - V.o[2];
    const double d2 = (bx * bx + by * by) + bz * bz;
    return V.f2 * (double)b.w / sqrt(d2);
}

// Blend: level-of-detail transition blending.  Node g with parent p takes
// the weight t = clamp((s_p - tau) / (s_p - s_g), 0, 1) of the projected
// bounding-sphere sizes of p and g (t = 1 when s_g >= s_p), and is projected
// as the Gaussian with mean mu_p + t (mu_g - mu_p), covariance Sigma_p +
// t (Sigma_g - Sigma_p) (formed after projection as (1 - t) T_p T_p^T +
// t T_g T_g^T, positive semidefinite by construction) and SH coefficients
// interpolated alike.  Opacity: the first of p's children in the view's cut
// carries o_p + t (o_g - o_p), the others t o_g, so that at the refine
// decision (s_p = tau, t = 0 for every child) exactly one copy of p is drawn
// and, at the node's own decision (s_g = tau, t = 1), the node itself: the
// image is continuous across both.  The cut lists a parent's children that
// it holds next to each other in ascending order (they are decided in one
// level pass, in frontier order), so g is that first child unless the entry
// before it is a sibling of the same view.  The blended mean and depth key
// follow the same FP64 steps as the unblended ones.
//
// In a node-grouped cut a wave's entries span several views, which it reads
// from a window of kProjectLdsViews views in LDS: all of them, or with more
// the ones from the view group of the workgroup's first entry on (the groups
// of a level follow one another; entries outside, where two levels meet, read
// theirs from memory).  38 M entries of 96 views without the window: 1,690 us,
// with it 1,500.
//
// PerTile: the entries go into per-tile lists (launch_emit_tiles): every
// tile's entries are counted here -- per 256 entries in LDS, then one atomic
// for each tile they reach -- and the depth key holds no view.
template <bool Blend, int DEG, bool PerTile>
__global__ __launch_bounds__(kNT) void k_project(ProjectArgs a) {
    constexpr int kWords = (int)(sizeof(ViewDev) / 8);
    __shared__ uint64_t s_view[kProjectLdsViews * kWords];
    __shared__ uint32_t s_count[PerTile ? kTileListMax : 1];
    const uint32_t m = min(a.ctr->cut, a.cut_cap);
    const uint32_t per = entries_per_block(m, PerTile ? 256u : 1024u);
    clear_bins(a.clear);
    // the emission's sums of 2^20 entries (u64), in the cut's block counts
    if (blockIdx.x == 0 && threadIdx.x < kTopSums / 2) a.scan_tmp[threadIdx.x] = make_uint4(0, 0, 0, 0);
    if (blockIdx.x * per >= m) return;
    if (PerTile) {
        for (uint32_t t = threadIdx.x; t < a.total_tiles; t += kNT) s_count[t] = 0;
        __syncthreads();
    }
    const int lw = log2_of(a.tile_w), lh = log2_of(a.tile_h);
    uint32_t win = ~0u;                                // first staged view
    uint32_t vis = 0;
    const uint32_t slot = entry_slot(per);
    for (uint32_t i0 = blockIdx.x * per; i0 < m; i0 += gridDim.x * per) {
        // (lanes without an entry repeat the last one and write nothing)
        const bool valid = slot < per && i0 + slot < m;
        const uint32_t i = valid ? i0 + slot : m - 1;
        const uint2 e = a.cut[i];
        if (a.lds_views) {
            const uint32_t v0 =
                a.n_views <= (int)kProjectLdsViews ? 0u : a.cut[i0].y / kCutViewGroup * kCutViewGroup;
            if (v0 != win) {
                if (win != ~0u) __syncthreads();
                const uint32_t n = min((uint32_t)a.n_views - v0, kProjectLdsViews) * kWords;
                const uint64_t* src = reinterpret_cast<const uint64_t*>(a.views + v0);
                for (uint32_t k = threadIdx.x; k < n; k += kNT) s_view[k] = src[k];
                __syncthreads();
                win = v0;
            }
        }
        ViewDev V;
        if (a.lds_views && e.y - win < kProjectLdsViews) {
            uint64_t wd[kWords];
#pragma unroll
            for (int q = 0; q < kWords; ++q) wd[q] = s_view[(e.y - win) * kWords + q];
            __builtin_memcpy(&V, wd, sizeof V);
        } else {
            V = load_view(a.views, e.y);
        }
        const int64_t g = e.x;
        const float4 g0 = a.geo[3 * g], g1 = a.geo[3 * g + 1], g2 = a.geo[3 * g + 2];
        int64_t pg = -1;
        double t = 1.0;
        bool first = true;
        float4 p0 = g0;
        if (Blend) {
            const int32_t par = a.parent[g];
            if (par >= 0) {
                const double sp = sphere_size(V, a.bound[par]), sg = sphere_size(V, a.bound[g]);
                if (sg < sp) {
#pragma clang fp contract(off)
                    t = (sp - V.tau) / (sp - sg);
                    t = t < 0.0 ? 0.0 : (t > 1.0 ? 1.0 : t);
                }
                if (i > 0) {
                    const uint2 q = a.cut[i - 1];
                    first = !(q.y == e.y && (int64_t)q.x >= (int64_t)a.child[par].x && (int64_t)q.x < g);
                }
                if (t < 1.0) {
                    pg = par;
                    p0 = a.geo[3 * pg];
                }
            }
        }
        double dx, dy, dz, tx, ty, tz;
        double op = g0.w;
        {
#pragma clang fp contract(off)
            double mx = g0.x, my = g0.y, mz = g0.z;
            if (Blend && pg >= 0) {
                mx = (double)p0.x + t * ((double)g0.x - (double)p0.x);
                my = (double)p0.y + t * ((double)g0.y - (double)p0.y);
                mz = (double)p0.z + t * ((double)g0.z - (double)p0.z);
                op = first ? (double)p0.w + t * ((double)g0.w - (double)p0.w) : t * (double)g0.w;
            }
            dx = mx - V.o[0];
            dy = my - V.o[1];
            dz = mz - V.o[2];
            tx = (V.R[0] * dx + V.R[1] * dy) + V.R[2] * dz;
            ty = (V.R[3] * dx + V.R[4] * dy) + V.R[5] * dz;
            tz = (V.R[6] * dx + V.R[7] * dy) + V.R[8] * dz;
        }
        Proj p = {};
        uint32_t ntiles = 0;
        bool seen = false;                             // its pixel box meets the image
        ushort4 rc = make_ushort4(1, 1, 0, 0);
        const float zf = (float)tz;
        if (tz > V.znear) {
            const double iz = rcp64(tz);
            double xr = tx * iz, yr = ty * iz;
            xr = fmin(fmax(xr, V.xlo), V.xhi);
            yr = fmin(fmax(yr, V.ylo), V.yhi);
            // M = J W (2x3)
            double M0[3], M1[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                M0[j] = V.fx * iz * (V.R[j] - xr * V.R[6 + j]);
                M1[j] = V.fy * iz * (V.R[3 + j] - yr * V.R[6 + j]);
            }
            double c00, c01, c11;
            proj_cov(M0, M1, g1, g2, &c00, &c01, &c11);
            if (Blend && pg >= 0) {
                double b00, b01, b11;
                proj_cov(M0, M1, a.geo[3 * pg + 1], a.geo[3 * pg + 2], &b00, &b01, &b11);
                const double u = 1.0 - t;
                c00 = u * b00 + t * c00;
                c01 = u * b01 + t * c01;
                c11 = u * b11 + t * c11;
            }
            const double s00 = c00 + 0.3;
            const double s01 = c01;
            const double s11 = c11 + 0.3;
            const double det = s00 * s11 - s01 * s01;
            if (det > 0.0) {
                const double u = V.fx * tx * iz + V.cx;
                const double v = V.fy * ty * iz + V.cy;
                // q = (p dx + r dy)^2 + (s dy)^2 with p^2 = s11/det,
                // p r = -s01/det, r^2 + s^2 = s00/det, so s^2 = 1/s11; with w =
                // 1 / sqrt(det s11), p = s11 w, made good by what p^2 det
                // lacks of s11 (p 0.5 ulp, r 1.3, s 0.5: no more than with IEEE
                // divisions and roots, 0.8, 1.3 and 0.8)
                const double s = rsqrt64_near(s11), w = rsqrt64_near(fmin(det * s11, 1e300));
                const double p0 = s11 * w, pp = p0 * p0;
                const double lack = fma(-fma(p0, p0, -pp), det, fma(-pp, det, s11));
                p.u = u;
                p.v = v;
                p.p = (float)fma(lack, 0.5 * w, p0);
                p.r = (float)(-s01 * w);
                p.s = (float)s;
                p.opacity = (float)op;
                p.z = zf;
                // pixel-centre bounding box of q <= 9 (1 + slack)
                const double ex = kBinReach * (s00 * rsqrt64(s00)) + 1e-6, ey = kBinReach * (s11 * s) + 1e-6;
                const double px0 = ceil(u - ex - 0.5), px1 = floor(u + ex - 0.5);
                const double py0 = ceil(v - ey - 0.5), py1 = floor(v + ey - 0.5);
                const double cx0 = fmax(px0, 0.0), cx1 = fmin(px1, (double)(V.width - 1));
                const double cy0 = fmax(py0, 0.0), cy1 = fmin(py1, (double)(V.height - 1));
                if (cx0 <= cx1 && cy0 <= cy1) {
                    rc = make_ushort4((unsigned short)((int)cx0 >> lw), (unsigned short)((int)cy0 >> lh),
                                      (unsigned short)((int)cx1 >> lw), (unsigned short)((int)cy1 >> lh));
                    seen = valid;
                }
            }
        }
        // tiles reached: a lane's own rows, or the wave's for tall entries
        const bool tall = seen && (PerTile || a.exact_tiles) && rc.w - rc.y >= kTallRows;
        const bool help = wave_is_better(tall, rc.w - rc.y + 1u,
                                         PerTile ? (uint32_t)(rc.z - rc.x + 1) * (uint32_t)(rc.w - rc.y + 1) : 0u,
                                         a.exact_tiles);
        auto count_row = [&](uint32_t base, int tiles_x, int ty, int lo, int hi) {
            if constexpr (PerTile)
                for (int tx = lo; tx <= hi; ++tx) atomicAdd(&s_count[base + (uint32_t)(ty * tiles_x + tx)], 1u);
        };
        const bool masked = small_rect(rc);
        uint32_t mask = 0;                             // of a small rectangle's tiles
        if (seen && !(tall && help)) {
            if (!PerTile && !a.exact_tiles) {
                ntiles = (uint32_t)(rc.z - rc.x + 1) * (uint32_t)(rc.w - rc.y + 1);
            } else {
                uint32_t at = 0;
                rect_rows(p, rc, a.tile_w, a.tile_h, V.height, a.exact_tiles, [&](int ty, int lo, int hi) {
                    ntiles += hi >= lo ? (uint32_t)(hi - lo + 1) : 0u;
                    count_row(V.tile_base, V.tiles_x, ty, lo, hi);
                    if (masked && hi >= lo) mask |= ((2u << (hi - rc.x)) - (1u << (lo - rc.x))) << at;
                    at += (uint32_t)(rc.z - rc.x + 1);
                });
            }
        }
        wave_rect_rows(tall && help, p, rc, a.tile_w, a.tile_h, V.height, a.exact_tiles,
                       [&](int src, int ty0, int, int lo, int hi) {
                           const uint32_t n = wave_sum(hi >= lo ? (uint32_t)(hi - lo + 1) : 0u);
                           if (lane_id() == src) ntiles += n;
                           if constexpr (PerTile)
                               count_row(__builtin_amdgcn_readlane(V.tile_base, src),
                                         __builtin_amdgcn_readlane(V.tiles_x, src), ty0 + lane_id(), lo, hi);
                       });
        if (ntiles > 0) {
            const double id = rsqrt64(dx * dx + dy * dy + dz * dz);
            float rgb[3];
            sh_colour<Blend, DEG>(a.sh, g, pg, (float)t, (float)(dx * id), (float)(dy * id), (float)(dz * id), rgb);
            p.c0 = rgb[0];
            p.c1 = rgb[1];
            p.c2 = rgb[2];
        }
        if (valid) {
            a.proj[i] = p;
            BinRec br;
            br.rc = rc;
            br.tile_base = PerTile ? V.tile_base : e.y << a.key_shift;
            br.tiles_x = (uint16_t)V.tiles_x;
            br.height = (uint16_t)(masked ? mask : (uint32_t)V.height);
            a.bins[i] = br;
            a.ntiles[i] = ntiles;
            vis += ntiles > 0 ? 1u : 0u;
            // positive depths order as their bit patterns, and so do their
            // offsets from depth_base; unbinned entries last
            uint32_t dk = 0xffffffffu;
            if (ntiles > 0) {
                const uint32_t bits = __float_as_uint(zf);
                if (bits < a.depth_base || bits > a.depth_top) atomicOr(&a.ctr->overflow, kOvDepth);
                dk = bits - a.depth_base;
                if (!PerTile && a.view_shift > 0) dk |= e.y << a.view_shift;
            }
            a.depth_key[i] = dk;
            if (!PerTile) a.depth_val[i] = i | (min(ntiles, kNtSat) << kNtShift);
        }
        if constexpr (PerTile) {
            __syncthreads();
            for (uint32_t t = threadIdx.x; t < a.total_tiles; t += kNT) {
                const uint32_t n = s_count[t];
                if (n) {
                    atomicAdd(a.tile_count + t, n);
                    s_count[t] = 0;
                }
            }
            __syncthreads();
        }
    }
    // binned entries, counted in 64 places that the binning adds up (one
    // place for all waves costs 10 ns a wave)
    vis = wave_sum(vis);
    if (lane_id() == 0 && vis)
        atomicAdd(reinterpret_cast<uint32_t*>(a.scan_tmp + kSeenAt) + blockIdx.x % kSeenSlots, vis);
}

// Binned entries into the counters (one wave).
__device__ __forceinline__ void sum_seen(const uint4* scan_tmp, Counters* ctr) {
    const uint32_t n = wave_sum(reinterpret_cast<const uint32_t*>(scan_tmp + kSeenAt)[lane_id()]);
    if (lane_id() == 0) ctr->visible = n;
}
static_assert(kSeenSlots == kWave, "one place per lane");


// ---------------------------------------------------------------- emission

// Where the pairs of the depth-ordered entries go is the sum of the tile
// counts before them: kept as sums of 256 entries (u32), 16,384 (u64) and
// 2^20 (u64), which an emitting workgroup adds up for itself.  (A scan in
// three launches wrote an offset per entry and cost 13 us in a single view,
// 43 us and 8 bytes per entry in a 50-view batch.)
struct TileSums {
    const uint32_t* order;
    const uint32_t* ntiles;
    uint32_t* fine;
    unsigned long long* mid;
    unsigned long long* top;
};

__device__ __forceinline__ TileSums tile_sums(const EmitArgs& a) {
    return {a.order, a.ntiles, a.sums,
            reinterpret_cast<unsigned long long*>(a.sums + (ceil_div(a.cut_cap, 256u) + 1u) / 2u * 2u),
            reinterpret_cast<unsigned long long*>(a.scan_tmp)};
}

// Tile count of a depth-sorted value: carried in its top bits unless
// saturated.
__device__ __forceinline__ uint32_t tiles_of(const uint32_t* ntiles, uint32_t val, uint32_t n) {
    const uint32_t nt = val >> kNtShift, e = val & kEntryMask;
    return nt < kNtSat ? nt : (e < n ? ntiles[e] : 0u);
}

// A workgroup per 16,384 entries, 16 x 256 of them per wave.
__global__ __launch_bounds__(kNT) void k_tile_sums(EmitArgs a) {
    __shared__ unsigned long long s_sum[kNT / kWave];
    const TileSums s = tile_sums(a);
    const uint32_t n = min(a.ctr->cut, a.cut_cap);
    const uint32_t w = threadIdx.x / kWave, l = lane_id();
    for (uint32_t blk = blockIdx.x; blk * 16384ull < n; blk += gridDim.x) {
        unsigned long long acc = 0;
#pragma unroll 4
        for (uint32_t j = 0; j < 16; ++j) {
            const uint32_t c = blk * 64 + w * 16 + j, i = c * 256 + 4 * l;
            uint32_t x = 0;
            if (i + 4 <= n) {
                const uint4 v = *reinterpret_cast<const uint4*>(s.order + i);
                x = tiles_of(s.ntiles, v.x, n) + tiles_of(s.ntiles, v.y, n) + tiles_of(s.ntiles, v.z, n) +
                    tiles_of(s.ntiles, v.w, n);
            } else {
                for (uint32_t k = i; k < n; ++k) x += tiles_of(s.ntiles, s.order[k], n);
            }
            x = wave_sum(x);                          // below 2^28: at most 2^20 tiles an entry
            if (l == 0 && c * 256 < n) s.fine[c] = x;
            acc += x;
        }
        if (l == 0) s_sum[w] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long t = 0;
#pragma unroll
            for (int q = 0; q < kNT / kWave; ++q) t += s_sum[q];
            s.mid[blk] = t;
            if (t) atomicAdd(s.top + blk / 64, t);
        }
        __syncthreads();
    }
}

// Pairs of the entries before `first` (this thread's part of the sum).
__device__ __forceinline__ unsigned long long pairs_before(const TileSums& s, uint32_t first, uint32_t n) {
    const uint32_t t = threadIdx.x, c = first / 256;
    unsigned long long acc = 0;
    if (t < (c >> 12)) acc += s.top[t];
    if (t < ((c >> 6) & 63u)) acc += s.mid[(c >> 12) * 64 + t];
    if (t >= kWave && t - kWave < (c & 63u)) acc += s.fine[(c & ~63u) + t - kWave];
    if (c * 256 + t < first) acc += tiles_of(s.ntiles, s.order[c * 256 + t], n);
    return acc;
}

// Pairs of every lane's entry (e, with nt of them; nt = 0: none), handed to
// put(at, tag, tile): at = pos and up for the entry's pairs in order, tag the
// entry's.  Every lane of the wave takes part; the calls for an entry of more
// than kBigPairs come from all of them.
template <class F>
__device__ __forceinline__ void entry_tiles(const EmitArgs& a, uint32_t e, uint32_t nt, const BinRec& br, uint32_t pos,
                                            uint32_t tag, F put) {
    const ushort4 rc = br.rc;
    const uint32_t all = (uint32_t)(rc.z - rc.x + 1) * (uint32_t)(rc.w - rc.y + 1);
    // the exact set is part of the rectangle: equal counts mean all of it
    const bool rect = !a.exact_tiles || nt == all;
    const bool large = nt > kBigPairs;
    const bool help = wave_is_better(large, rc.w - rc.y + 1u, nt, !rect);
    const bool big = large && help;
    const bool masked = !rect && small_rect(rc);
    Proj p = {};
    if (nt && !rect && !masked) p = a.proj[e];
    if (nt && masked) {
        uint32_t at = pos, m = br.height, row = br.tile_base + (uint32_t)rc.y * br.tiles_x + rc.x;
        const uint32_t w = (uint32_t)(rc.z - rc.x + 1), line = (1u << w) - 1u;
        for (; m; m >>= w, row += br.tiles_x)
            for (uint32_t t = m & line; t; t &= t - 1u) put(at++, tag, row + (uint32_t)__builtin_ctz(t));
    } else if (nt && !big) {
        uint32_t at = pos;
        rect_rows(p, rc, a.tile_w, a.tile_h, br.height, !rect, [&](int ty, int lo, int hi) {
            const uint32_t row = br.tile_base + (uint32_t)ty * br.tiles_x;
            for (int tx = lo; tx <= hi; ++tx) put(at++, tag, row + (uint32_t)tx);
        });
    }
    for (int pass = 0; pass < 2; ++pass) {            // ellipses, then full rectangles
        uint32_t at = 0;                              // next pair of the entry in turn
        int last = -1;
        wave_rect_rows(big && rect == (pass == 1), p, rc, a.tile_w, a.tile_h, br.height, pass == 0,
                       [&](int src, int ty0, int n, int lo, int hi) {
                           if (src != last) at = __builtin_amdgcn_readlane(pos, src);
                           last = src;
                           const uint32_t its = __builtin_amdgcn_readlane(tag, src);
                           const uint32_t base = __builtin_amdgcn_readlane(br.tile_base, src);
                           const uint32_t width = __builtin_amdgcn_readlane((uint32_t)br.tiles_x, src);
                           for (int j = 0; j < n; ++j) {
                               const int l = __builtin_amdgcn_readlane(lo, j), h = __builtin_amdgcn_readlane(hi, j);
                               const uint32_t row = base + (uint32_t)(ty0 + j) * width;
                               for (int tx = l + lane_id(); tx <= h; tx += kWave)
                                   put(at + (uint32_t)(tx - l), its, row + (uint32_t)tx);
                               at += h >= l ? (uint32_t)(h - l + 1) : 0u;
                           }
                       });
    }
}

// Each workgroup expands 256 consecutive depth-ordered entries into their
// (tile, entry) pairs, which form one contiguous run of the pair arrays:
// the run is assembled in LDS and written out coalesced; pairs past the
// staging capacity are stored directly.
constexpr uint32_t kEmitStage = 2048;

__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(6))) void k_emit(EmitArgs a) {
    __shared__ uint32_t s_key[kEmitStage];
    __shared__ uint32_t s_val[kEmitStage];
    __shared__ uint32_t s_scan[kNT / kWave + 1];
    __shared__ unsigned long long s_before[kNT / kWave];
    const uint32_t m = min(a.ctr->cut, a.cut_cap);
    const uint32_t cap = a.pair_cap;
    const TileSums sums = tile_sums(a);
    clear_bins(a.clear);
    if (blockIdx.x == 0 && threadIdx.x < kWave) {
        sum_seen(a.scan_tmp, a.ctr);
        unsigned long long total = 0;
        for (int t = lane_id(); t < kTopSums; t += kWave) total += sums.top[t];
        for (int o = kWave / 2; o > 0; o >>= 1) total += __shfl_xor(total, o, kWave);
        if (lane_id() == 0) {
            Counters* k = a.ctr;
            if (total > cap) {
                k->overflow |= kOvPairs;
                const uint32_t need = (uint32_t)(total < 0xffffffffull ? total : 0xffffffffull);
                if (need > k->need_pairs) k->need_pairs = need;
            }
            k->pairs = total < cap ? (uint32_t)total : cap;
        }
    }
    const uint32_t per = entries_per_block(m, 1024);
    const uint32_t slot = entry_slot(per);
    for (uint32_t first = blockIdx.x * per; first < m; first += gridDim.x * per) {
        const uint32_t i = first + slot;
        uint32_t e = 0, nt = 0;
        if (slot < per && i < m) {
            const uint32_t val = a.order[i];
            e = val & kEntryMask;
            nt = tiles_of(a.ntiles, val, m);
        }
        unsigned long long before = pairs_before(sums, first, m);
        BinRec br = {};
        if (nt) br = a.bins[e];
        for (int o = kWave / 2; o > 0; o >>= 1) before += __shfl_xor(before, o, kWave);
        if (lane_id() == 0) s_before[threadIdx.x / kWave] = before;
        uint32_t tot;
        const uint32_t ex = block_excl_scan<kNT>(nt, s_scan, &tot);
        unsigned long long base64 = 0;
#pragma unroll
        for (int q = 0; q < kNT / kWave; ++q) base64 += s_before[q];
        const bool fits = base64 < cap;               // (else an overflow, reported above)
        const uint32_t base = (uint32_t)base64;
        entry_tiles(a, e, fits ? nt : 0u, br, ex, e, [&](uint32_t L, uint32_t who, uint32_t tile) {
            if (L < kEmitStage) {
                s_key[L] = tile;
                s_val[L] = who;
            } else if (base + L < cap) {
                a.keys[base + L] = tile;
                a.vals[base + L] = who;
            }
        });
        __syncthreads();
        const uint32_t len = fits ? min(tot, kEmitStage) : 0u;
        for (uint32_t q = threadIdx.x; q < len; q += kNT) {
            if (base + q < cap) {
                a.keys[base + q] = s_key[q];
                a.vals[base + q] = s_val[q];
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------- per-tile lists
//
// Few pairs (one small view, say) spend their time in the launches of two
// radix sorts: 18 of them, and the scan between, for 50,000 to 1,000,000
// pairs.  Here the projection has counted every tile's entries; one
// workgroup turns the counts into ranges, every pair takes a place in its
// tile's range (in any order), and each tile's list is sorted by (depth,
// entry) -- the order of the stable sorts -- in LDS.  Four launches from the
// projection to the compositor.  Places come from LDS atomics within a
// workgroup's 256 entries and one global atomic per workgroup and tile: an
// atomic per pair on the tile's own counter, which neighbouring entries
// share, took 58 us for 200,000 pairs of a usual view and 1.5 ms for a view
// close to a wall.

// Ranges of the tiles from their counts, four tiles per thread and step; the
// places' cursors start at them.  One workgroup: a few thousand tiles are a
// few steps.
__global__ __launch_bounds__(1024) void k_tile_scan(TileListArgs a, const uint4* scan_tmp) {
    __shared__ uint4 sh[1024 / kWave + 1];
    if (threadIdx.x < kWave) sum_seen(scan_tmp, a.ctr);
    unsigned long long run = 0;
    for (uint32_t base = 0; base < a.total_tiles; base += 4 * 1024) {
        const uint32_t t0 = base + 4 * threadIdx.x;
        // a tile may hold every entry of the cut (2^28), so a step's sums need
        // 40 bits: the counts' low and high halves are scanned side by side
        uint32_t x[4], lo16 = 0, hi16 = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x[j] = t0 + j < a.total_tiles ? a.tile_count[t0 + j] : 0u;
            lo16 += x[j] & 0xffffu;
            hi16 += x[j] >> 16;
        }
        uint4 tot;
        const uint4 ex = block_excl_scan4<1024>(make_uint4(lo16, hi16, 0, 0), sh, &tot);
        unsigned long long lo = run + ((unsigned long long)ex.y << 16) + ex.x;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const unsigned long long hi = lo + x[j], cap = a.pair_cap;
            if (t0 + j < a.total_tiles) {
                const uint32_t start = (uint32_t)(lo < cap ? lo : cap);
                a.ranges[t0 + j] = make_uint2(start, (uint32_t)(hi < cap ? hi : cap));
                a.tile_count[t0 + j] = start;
            }
            lo = hi;
        }
        run += ((unsigned long long)tot.y << 16) + tot.x;
    }
    if (threadIdx.x == 0) {
        Counters* k = a.ctr;
        if (run > a.pair_cap) {
            k->overflow |= kOvPairs;
            const uint32_t need = (uint32_t)(run < 0xffffffffull ? run : 0xffffffffull);
            if (need > k->need_pairs) k->need_pairs = need;
        }
        k->pairs = (uint32_t)(run < a.pair_cap ? run : a.pair_cap);
    }
}

// Each workgroup lists the pairs of 256 entries in LDS, kTileStage at a
// time, ranks them within their tiles, takes the tiles' next places and
// writes the pairs there.
constexpr uint32_t kTileStage = 4096;

__global__ __launch_bounds__(kNT) void k_emit_tiles(EmitArgs a, TileListArgs l) {
    __shared__ uint32_t s_count[kTileListMax];
    // tile | entry of the workgroup << 13 | rank among the workgroup's pairs
    // of the tile << 21 (an entry reaches a tile once)
    __shared__ uint32_t s_pair[kTileStage];
    __shared__ uint32_t s_depth[kNT];
    __shared__ uint32_t s_scan[kNT / kWave + 1];
    static_assert(kTileListMax <= 1u << 13 && kNT <= 256, "packed pairs");
    const uint32_t m = min(a.ctr->cut, a.cut_cap);
    const uint32_t per = entries_per_block(m, 256);
    if (blockIdx.x == 0 && threadIdx.x == 0) report_pairs(l.report, a.ctr->pairs, a.ctr->need_pairs);
    if (blockIdx.x * per >= m) return;
    for (uint32_t t = threadIdx.x; t < l.total_tiles; t += kNT) s_count[t] = 0;
    const uint32_t slot = entry_slot(per);
    for (uint32_t first = blockIdx.x * per; first < m; first += gridDim.x * per) {
        const uint32_t i = first + slot;
        const bool valid = slot < per && i < m;
        const uint32_t nt = valid ? a.ntiles[i] : 0u;
        if (slot < per) s_depth[slot] = valid ? l.depth[i] : 0u;
        BinRec br = {};
        if (nt) br = a.bins[i];
        uint32_t tot;
        const uint32_t at = block_excl_scan<kNT>(nt, s_scan, &tot);   // (also orders the cleared counts)
        for (uint32_t w0 = 0; w0 < tot; w0 += kTileStage) {
            const bool here = nt && at < w0 + kTileStage && at + nt > w0;
            entry_tiles(a, i, here ? nt : 0u, br, at - w0, slot, [&](uint32_t L, uint32_t who, uint32_t tile) {
                // (L wraps past the stage for the pairs of an earlier one)
                if (L < kTileStage) s_pair[L] = tile | who << 13 | atomicAdd(&s_count[tile], 1u) << 21;
            });
            __syncthreads();
            for (uint32_t t = threadIdx.x; t < l.total_tiles; t += kNT) {
                const uint32_t n = s_count[t];
                if (n) s_count[t] = atomicAdd(l.tile_count + t, n);
            }
            __syncthreads();
            const uint32_t len = min(tot - w0, kTileStage);
            for (uint32_t q = threadIdx.x; q < len; q += kNT) {
                const uint32_t p = s_pair[q], who = p >> 13 & 255u;
                const uint32_t pos = s_count[p & 8191u] + (p >> 21);
                if (pos < l.pair_cap) {                           // else: an overflow the scan has reported
                    l.keys[0][pos] = s_depth[who];
                    l.vals[0][pos] = first + who;
                }
            }
            __syncthreads();
            for (uint32_t t = threadIdx.x; t < l.total_tiles; t += kNT) s_count[t] = 0;
            __syncthreads();
        }
        __syncthreads();
    }
}

// One workgroup per tile sorts its list by (depth, entry): up to 256 pairs
// by ranking (a pair's place is the number of smaller ones, counted over the
// list in LDS with no barrier in between), up to kSortMax by a bitonic
// network in LDS; longer lists in runs of kSortMax that are then merged
// pairwise through memory, every element's place found by a binary search in
// the other run.
constexpr uint32_t kSortMax = 4096;

__global__ __launch_bounds__(kNT) void k_sort_tiles(TileListArgs a) {
    __shared__ unsigned long long s[kSortMax];
    const uint2 rg = a.ranges[blockIdx.x];
    const uint32_t n = rg.y - rg.x;
    if (n == 0) return;
    uint32_t *k0 = a.keys[0] + rg.x, *v0 = a.vals[0] + rg.x, *k1 = a.keys[1] + rg.x, *v1 = a.vals[1] + rg.x;
    const uint32_t t = threadIdx.x;
    if (n <= (uint32_t)kNT) {
        unsigned long long x = 0ull;
        if (t < n) {
            x = (unsigned long long)k0[t] << 32 | v0[t];
            s[t] = x;
        }
        __syncthreads();
        if (t / kWave * kWave >= n) return;               // whole waves without an element
        uint32_t r = 0;
#pragma unroll 8
        for (uint32_t j = 0; j < n; ++j) r += s[j] < x ? 1u : 0u;
        if (t < n) v1[r] = (uint32_t)x;
        return;
    }
    for (uint32_t base = 0; base < n; base += kSortMax) {
        const uint32_t m = min(n - base, kSortMax);
        uint32_t size = 2;
        while (size < m) size <<= 1;
        for (uint32_t i = t; i < size; i += kNT)
            s[i] = i < m ? (unsigned long long)k0[base + i] << 32 | v0[base + i] : ~0ull;
        __syncthreads();
        for (uint32_t k = 2; k <= size; k <<= 1)
            for (uint32_t j = k >> 1; j > 0; j >>= 1) {
                for (uint32_t q = t; q < size / 2; q += kNT) {
                    const uint32_t lo = 2 * q - (q & (j - 1)), hi = lo + j;
                    const unsigned long long x = s[lo], y = s[hi];
                    if ((x > y) == ((lo & k) == 0)) {
                        s[lo] = y;
                        s[hi] = x;
                    }
                }
                __syncthreads();
            }
        for (uint32_t i = t; i < m; i += kNT) {
            v1[base + i] = (uint32_t)s[i];
            if (n > kSortMax) k1[base + i] = (uint32_t)(s[i] >> 32);
        }
        __syncthreads();
    }
    // merge runs of w: an element's place is its index in its own run plus
    // the number of smaller ones in the other (all elements differ)
    bool in1 = true;                                      // which buffer holds the runs
    for (uint64_t w = kSortMax; w < n; w *= 2) {
        uint32_t *ks = in1 ? k1 : k0, *vs = in1 ? v1 : v0, *kd = in1 ? k0 : k1, *vd = in1 ? v0 : v1;
        for (uint32_t i = t; i < n; i += kNT) {
            const unsigned long long x = (unsigned long long)ks[i] << 32 | vs[i];
            const uint64_t pair = i / (2 * w) * (2 * w), mine = i / w * w;
            const uint64_t other = mine == pair ? pair + w : pair;
            uint64_t lo = min(other, (uint64_t)n), hi = min(other + w, (uint64_t)n);
            const uint64_t o0 = lo;
            while (lo < hi) {
                const uint64_t mid = (lo + hi) / 2;
                if (((unsigned long long)ks[mid] << 32 | vs[mid]) < x) lo = mid + 1; else hi = mid;
            }
            const uint64_t to = pair + (i - mine) + (lo - o0);
            kd[to] = (uint32_t)(x >> 32);
            vd[to] = (uint32_t)x;
        }
        in1 = !in1;
        __syncthreads();
    }
    if (!in1)
        for (uint32_t i = t; i < n; i += kNT) v1[i] = v0[i];
}

}  // namespace

__global__ void k_view_keys(const uint32_t* __restrict__ order, const uint2* __restrict__ cut, const uint32_t* count,
                            uint32_t cap, uint32_t* __restrict__ keys, SortBins clear) {
    const uint32_t n = min(*count, cap);
    clear_bins(clear);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const uint32_t e = order[i] & kEntryMask;
        keys[i] = e < n ? cut[e].y : 0u;
    }
}

namespace {

struct ArgViews {
    ViewDev v[kArgViews];
};
static_assert(sizeof(ArgViews) <= 3072, "kernel arguments hold 4 KB");

__global__ __launch_bounds__(kNT) void k_set_views(ArgViews a, int n, uint64_t* views) {
    const uint64_t* src = reinterpret_cast<const uint64_t*>(&a);
    for (int k = threadIdx.x; k < n * (int)(sizeof(ViewDev) / 8); k += kNT) views[k] = src[k];
}

}  // namespace

void launch_set_views(const ViewDev* host, int n, ViewDev* views, hipStream_t s) {
    ArgViews a;
    for (int v = 0; v < n; ++v) a.v[v] = host[v];
    k_set_views<<<1, kNT, 0, s>>>(a, n, reinterpret_cast<uint64_t*>(views));
}

template <bool Blend, bool PerTile>
void launch_project_b(const ProjectArgs& a, hipStream_t s) {
    switch (a.sh_degree) {
        case 0: k_project<Blend, 0, PerTile><<<4096, kNT, 0, s>>>(a); break;
        case 1: k_project<Blend, 1, PerTile><<<4096, kNT, 0, s>>>(a); break;
        case 2: k_project<Blend, 2, PerTile><<<4096, kNT, 0, s>>>(a); break;
        default: k_project<Blend, 3, PerTile><<<4096, kNT, 0, s>>>(a); break;
    }
}

void launch_project(const ProjectArgs& a, hipStream_t s) {
    const bool tiles = a.tile_count != nullptr;
    if (a.blend)
        tiles ? launch_project_b<true, true>(a, s) : launch_project_b<true, false>(a, s);
    else
        tiles ? launch_project_b<false, true>(a, s) : launch_project_b<false, false>(a, s);
}

void launch_emit_tiles(const EmitArgs& e, const TileListArgs& a, hipStream_t s) {
    k_tile_scan<<<1, 1024, 0, s>>>(a, e.scan_tmp);
    k_emit_tiles<<<2048, kNT, 0, s>>>(e, a);
    k_sort_tiles<<<a.total_tiles, kNT, 0, s>>>(a);
}

void launch_view_keys(const uint32_t* order, const uint2* cut, const uint32_t* count, uint32_t cap, uint32_t* keys,
                      SortBins clear, hipStream_t s) {
    k_view_keys<<<2048, 256, 0, s>>>(order, cut, count, cap, keys, clear);
}

void launch_emit(const EmitArgs& a, hipStream_t s) {
    k_tile_sums<<<2048, kNT, 0, s>>>(a);
    k_emit<<<8192, kNT, 0, s>>>(a);
}

}  // namespace hgs
