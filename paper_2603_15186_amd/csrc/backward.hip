// Backward pass of the renderer: gradients of a loss, given its gradients
// with respect to the output images (RGB, raw depth D = sum w z, alpha =
// 1 - T), with respect to the Gaussians' means, scales, rotations,
// opacities and SH coefficients (the optimisation behind the paper's scene
// reconstruction, Sec. III-B).
//
// Compositing (one 128-thread workgroup per 16x16 tile, two adjacent pixels
// per thread, 8 lanes per 4x4 block): the tile's depth-ordered entries are
// staged in LDS in batches and listed per block exactly as the forward stages
// and lists them.  Where each pixel stopped and its final transmittance T_N
// come from the forward compositor when the render kept them; else the pixel
// replays the forward recurrence over its block's list with the same
// single-precision operations.  It then walks the lists back to front,
// recovering T before entry i as T_{i+1} / (1 - alpha_i), with
//   dL/dalpha_i = T_i (g . c_i) - (B_i - gA T_N) / (1 - alpha_i)
// where g . c_i = sum_c gC_c c_ic + gD z_i and B_i = sum of g . c_j alpha_j
// T_j over the entries behind i plus T_N gC . bg: one number per pixel holds
// what lies behind.  Through alpha = o e^{-q/2} (no gradient where capped at
// 0.99) and q = t1^2 + t2^2, t1 = p dx + r dy, t2 = s dy, with h = alpha
// dL/dalpha, each pixel yields ten numbers per entry: h, h t1, h t1 dx,
// h t1 dy, h t2, h t2 dy and the four of colour and depth, from which the
// projection's backward forms the gradients of the 2D mean, the conic factors
// and the opacity.  The 8 lanes of a block, which walk the same entry, sum
// them (ten_sums), the blocks add them in LDS, and a tile adds its entries'
// sums to the per-entry buffer with consecutive lanes on consecutive words.
//
// What bounds it: vector issue, about 100 instructions per two pixels and
// entry, and before that the atomics: with one pixel per thread, ten full row
// sums per block and entry and ten scattered global atomics per tile and
// entry, four 640 x 480 views of a 700,000-leaf plan took 650 us here;
// 401 this way.
//
// Projection (FP64): the cut entries are sorted by Gaussian (the radix sort
// of the binning); one thread per entry in that order takes the chain rule
// from the 2D mean, the conic factors of Sigma' = T T^T + 0.3 I
// (T = J W R S), the camera depth and the colour back to the Gaussian's
// mean, scale, rotation and opacity, written as a per-entry record (in the
// sorted order) with the entry's colour gradient and view direction.  One
// thread per Gaussian then sums its run of records, forming the SH
// coefficients' gradients sum g_c Y_k(d) on the way: no scattered atomics on
// the parameter arrays.
#include <type_traits>

#include "blocks.h"
#include "device_util.h"
#include "internal.h"

namespace hgs {

namespace {

constexpr int kB = 128;                         // entries staged per batch
constexpr int kNT = kTilePx / 2;                // two pixels per thread
constexpr int kNW = kNT / kWave;
constexpr int kLanes = 8;                       // threads per block
constexpr int kNG = 10;                         // per-entry numbers
static_assert(kB <= kNT && kNG <= kEntryGrad, "an entry per staging thread");

// Staged records as the forward compositor's: factors scaled by kS, nlo =
// -log2(opacity).
struct alignas(16) BwdA { float p, r, c1, s; };
// The mean (u, v) is relative to the tile.
struct alignas(16) BwdB { float c2, nlo, u, v; };
struct alignas(16) BwdC { float col0, col1, col2, z; };

struct BwdShared {
    BwdA a[kB + 1];
    BwdB b[kB + 1];
    BwdC c[kB + 1];
    float acc[(kB + 1) * kEntryGrad];
    uint32_t entry[kB];
    alignas(16) uint16_t idx[kBlocks * kB];
    uint32_t wc[kNW * kBlocks];
    uint32_t n[kBlocks];
    uint32_t maxlast;
};

// This thread's entry of a batch, on its way from memory: loaded while the
// batch before it is walked, since a tile's time is its batches' and a batch
// starts with two dependent gathers.
struct Fetched {
    uint32_t e;
    Proj P;
};
__device__ __forceinline__ void fetch(const BwdArgs& a, uint32_t base, uint32_t cnt, Fetched* f) {
    if (threadIdx.x < cnt) {
        f->e = a.vals[base + threadIdx.x];
        f->P = a.proj[f->e < a.cut_cap ? f->e : 0u];
    }
}

// Stage a batch of cnt entries (f: this thread's) and build each 4x4
// block's list of staged offsets (16 B units, depth order), padded with the
// empty record up to a multiple of four of its wave's longest list, whose
// padded length is returned.
__device__ __forceinline__ uint32_t stage_lists(const Fetched& f, BwdShared& S, uint32_t cnt, double dx0, double dy0,
                                                int w, int lane, int blk, int k) {
    uint32_t m = 0;
    const int j = threadIdx.x;
    if (j < (int)cnt) {
        const uint32_t e = f.e;
        const Proj& P = f.P;
        const float nlo = -__log2f(P.opacity);
        const float u = (float)(P.u - dx0), v = (float)(P.v - dy0);
        const float c1 = -fmaf(P.p, u, P.r * v), c2 = -P.s * v;
        S.a[j] = BwdA{kS * P.p, kS * P.r, kS * c1, kS * P.s};
        S.b[j] = BwdB{kS * c2, nlo, u, v};
        S.c[j] = BwdC{P.c0, P.c1, P.c2, P.z};
        S.entry[j] = e;
        m = block_mask(u, v, P.p, P.r, P.s);
    }
    uint32_t pre[kBlocks];
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) {
        const uint64_t bal = __ballot((m >> b) & 1u);
        pre[b] = (uint32_t)__popcll(bal & lanemask_lt());
        if (lane == 0) S.wc[w * kBlocks + b] = (uint32_t)__popcll(bal);
    }
    __syncthreads();
    if (threadIdx.x < kBlocks) {
        uint32_t t = 0;
#pragma unroll
        for (int ww = 0; ww < kNW; ++ww) {
            const uint32_t c = S.wc[ww * kBlocks + threadIdx.x];
            S.wc[ww * kBlocks + threadIdx.x] = t;
            t += c;
        }
        S.n[threadIdx.x] = t;
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < kBlocks; ++b)
        if ((m >> b) & 1u) S.idx[b * kB + S.wc[w * kBlocks + b] + pre[b]] = (uint16_t)(j * 16);
    uint32_t n_wave = 0;
#pragma unroll
    for (int b = 0; b < kBlocks / kNW; ++b) n_wave = max(n_wave, S.n[w * (kBlocks / kNW) + b]);
    n_wave = __builtin_amdgcn_readfirstlane(n_wave);
    const uint32_t n_step = (n_wave + 3u) & ~3u;
    uint16_t* list = S.idx + blk * kB;
    for (uint32_t p = S.n[blk] + (uint32_t)k; p < n_step; p += kLanes) list[p] = (uint16_t)(kB * 16);
    __syncthreads();
    return n_step;
}

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}

// Sums of ten values over 8 consecutive lanes, spread over lanes 0-3 of the
// eight: lane k gets those of values k and 4 + k in *s0 and *s1, lanes 0 and
// 1 those of values 8 and 9 in *s2.  Each exchange keeps one of two values
// and sends the other, so the work halves from step to step: 25 instructions
// where ten separate sums take 30 and ten adds to LDS after them.
__device__ __forceinline__ void ten_sums(const float (&v)[kNG], bool odd1, bool odd2, float* s0, float* s1, float* s2) {
    float r[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const float keep = odd1 ? v[2 * i + 1] : v[2 * i], send = odd1 ? v[2 * i] : v[2 * i + 1];
        r[i] = keep + dpp_f<0xb1>(send);                  // quad_perm [1, 0, 3, 2]
    }
    float q[3];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float keep = odd2 ? r[2 * i + 1] : r[2 * i], send = odd2 ? r[2 * i] : r[2 * i + 1];
        q[i] = keep + dpp_f<0x4e>(send);                  // quad_perm [2, 3, 0, 1]
    }
    q[2] = r[4] + dpp_f<0x4e>(r[4]);
    *s0 = q[0] + dpp_f<0x104>(q[0]);                      // row_shl:4
    *s1 = q[1] + dpp_f<0x104>(q[1]);
    *s2 = q[2] + dpp_f<0x104>(q[2]);
}

// Batches of 128 entries and the 121 registers of four waves per SIMD: the
// reverse walk is a chain of LDS reads, exponentials and LDS adds, whose latency
// the other waves, the records read four at a time and the next batch fetched
// ahead hide (444 -> 401 us with these two at the size above).
template <bool KEPT>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(4))) void k_composite_bwd(BwdArgs a) {
    __shared__ BwdShared S;
    const uint32_t tile = blockIdx.x;
    const uint2 rg = a.ranges[tile];
    const uint32_t n = rg.y - rg.x;
    if (n == 0) return;                             // nothing drawn: no gradient
    const uint32_t view = a.tile_view[tile];
    const ViewDev& V = a.views[view];
    const ImgGrad G = a.dimg[view];
    const uint32_t local = tile - V.tile_base;
    const int tx = (int)(local % (uint32_t)V.tiles_x), ty = (int)(local / (uint32_t)V.tiles_x);
    const int x0 = tx * kTile, y0 = ty * kTile;
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int k = lane % kLanes, blk = w * (kBlocks / kNW) + lane / kLanes;
    const int lx0 = (blk % 4) * 4 + (k % 2) * 2, ly = (blk / 4) * 4 + k / 2;
    const int py = y0 + ly;
    const float fy = (float)ly + 0.5f;
    const double dx0 = (double)x0, dy0 = (double)y0;
    float fx[2], Tc[2];
    bool inside[2];
    uint32_t last[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        fx[q] = (float)(lx0 + q) + 0.5f;
        inside[q] = x0 + lx0 + q < V.width && py < V.height;
        Tc[q] = 1.f;
        last[q] = n;
    }
    if (threadIdx.x == 0) {
        S.a[kB] = BwdA{0.f, 0.f, 0.f, 0.f};
        S.b[kB] = BwdB{0.f, __builtin_inff(), 0.f, 0.f};    // Q = inf: above any bound
        S.c[kB] = BwdC{0.f, 0.f, 0.f, 0.f};
        S.maxlast = 0;
    }
    const char* ra = reinterpret_cast<const char*>(S.a);
    const char* rb = reinterpret_cast<const char*>(S.b);
    const char* rc = reinterpret_cast<const char*>(S.c);
    const uint2* list4 = reinterpret_cast<const uint2*>(S.idx + blk * kB);

    // 1. where the pixels stopped and their final transmittance: kept by the
    // forward compositor, else a forward replay over the block lists (the
    // forward's operations)
    if constexpr (KEPT) {
        // (the forward's thread of a pixel: blocks of 16 pixels, row-major)
        const uint2* st = a.state + (size_t)tile * kTilePx + blk * 16 + (k / 2) * 4 + (k % 2) * 2;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint2 x = st[q];
            last[q] = x.x;
            Tc[q] = __uint_as_float(x.y);
        }
        __syncthreads();                            // S.maxlast is set
    } else {
        bool live[2] = {inside[0], inside[1]};
        Fetched f;
        fetch(a, rg.x, min((uint32_t)kB, n), &f);
        for (uint32_t b0 = 0; b0 < n; b0 += kB) {
            const uint32_t n_step = stage_lists(f, S, min((uint32_t)kB, n - b0), dx0, dy0, w, lane, blk, k);
            if (b0 + kB < n) fetch(a, rg.x + b0 + kB, min((uint32_t)kB, n - b0 - kB), &f);
            for (uint32_t i = 0; i < n_step; i += 4) {
                const uint2 q4 = list4[i >> 2];
                const uint32_t id4[4] = {q4.x & 0xffffu, q4.x >> 16, q4.y & 0xffffu, q4.y >> 16};
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const BwdA A = *reinterpret_cast<const BwdA*>(ra + id4[u]);
                    const BwdB B = *reinterpret_cast<const BwdB*>(rb + id4[u]);
                    const float ry = fmaf(A.r, fy, A.c1), t2 = fmaf(A.s, fy, B.c2), t22 = fmaf(t2, t2, B.nlo);
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const float t1 = fmaf(A.p, fx[q], ry);
                        const float Q = fmaf(t1, t1, t22);
                        const float al = fminf(0.99f, __builtin_amdgcn_exp2f(-Q));
                        const float Tn = Tc[q] - al * Tc[q];
                        const bool add = live[q] && Q <= entry_qmax(B.nlo);
                        if (add && Tn < 1e-4f) {
                            live[q] = false;
                            last[q] = b0 + id4[u] / 16;
                        }
                        Tc[q] = add && live[q] ? Tn : Tc[q];
                    }
                }
                if (__ballot(live[0] || live[1]) == 0) break;
            }
            if (__syncthreads_count(live[0] || live[1] ? 1 : 0) == 0) break;
        }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) last[q] = inside[q] ? last[q] : 0u;
    atomicMax(&S.maxlast, max(last[0], last[1]));

    // 2. back to front over the same lists
    const size_t plane = (size_t)V.width * V.height;
    float gC0[2], gC1[2], gC2[2], gD[2], behind[2];
    bool bad = false;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const size_t pix = (size_t)py * V.width + (x0 + lx0 + q);
        const bool in = inside[q];
        gC0[q] = in && G.rgb ? G.rgb[pix] : 0.f;
        gC1[q] = in && G.rgb ? G.rgb[plane + pix] : 0.f;
        gC2[q] = in && G.rgb ? G.rgb[2 * plane + pix] : 0.f;
        gD[q] = in && G.depth ? G.depth[pix] : 0.f;
        const float gA = in && G.alpha ? G.alpha[pix] : 0.f;
        behind[q] = Tc[q] * (gC0[q] * V.bg[0] + gC1[q] * V.bg[1] + gC2[q] * V.bg[2] - gA);
        bad |= !(fabsf(gC0[q]) + fabsf(gC1[q]) + fabsf(gC2[q]) + fabsf(gD[q]) < __builtin_inff());
    }
    // An entry that a pixel does not take has al = wgt = 0 there, and h and
    // what lies behind are passed by; its colour and depth terms are zero by
    // the product, except with a gradient that is not finite: waves that hold
    // such a pixel select them too (eight selects, in a loop of their own).
    const bool bad_wave = __ballot(bad) != 0;
    for (int i = threadIdx.x; i < kB * kEntryGrad; i += kNT) S.acc[i] = 0.f;
    __syncthreads();
    const uint32_t maxlast = S.maxlast;
    const bool odd1 = k & 1, odd2 = k & 2;
    const int nb = (int)((maxlast + kB - 1) / kB);
    Fetched f;
    if (nb > 0) fetch(a, rg.x + (nb - 1) * kB, min((uint32_t)kB, n - (nb - 1) * kB), &f);
    for (int bi = nb - 1; bi >= 0; --bi) {
        const uint32_t b0 = (uint32_t)bi * kB;
        const uint32_t cnt = min((uint32_t)kB, n - b0);
        const uint32_t n_step = stage_lists(f, S, cnt, dx0, dy0, w, lane, blk, k);
        if (bi > 0) fetch(a, rg.x + b0 - kB, kB, &f);
        // offsets below lim are entries before the pixel's stop
        uint32_t lim[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) lim[q] = last[q] > b0 ? min(last[q] - b0, (uint32_t)kB) * 16u : 0u;
        auto walk = [&](auto bad_pixels) {
            using Bad = decltype(bad_pixels);
            for (int i = (int)n_step - 4; i >= 0; i -= 4) {
                const uint2 q4 = list4[i >> 2];
                const uint32_t id4[4] = {q4.x & 0xffffu, q4.x >> 16, q4.y & 0xffffu, q4.y >> 16};
                // the four records together, ahead of the sums' LDS adds
                BwdA A4[4];
                BwdB B4[4];
                BwdC C4[4];
#pragma unroll
                for (int u = 3; u >= 0; --u) {
                    A4[u] = *reinterpret_cast<const BwdA*>(ra + id4[u]);
                    B4[u] = *reinterpret_cast<const BwdB*>(rb + id4[u]);
                    C4[u] = *reinterpret_cast<const BwdC*>(rc + id4[u]);
                }
#pragma unroll
                for (int u = 3; u >= 0; --u) {
                    const uint32_t off = id4[u];
                    const BwdA A = A4[u];
                    const BwdB B = B4[u];
                    const BwdC C = C4[u];
                    const float qmax = entry_qmax(B.nlo);
                    const float ry = fmaf(A.r, fy, A.c1), t2 = fmaf(A.s, fy, B.c2), t22 = fmaf(t2, t2, B.nlo);
                    float v[kNG];
#pragma unroll
                    for (int t = 0; t < kNG; ++t) v[t] = 0.f;
                    bool has = false;
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const float t1 = fmaf(A.p, fx[q], ry);
                        const float Q = fmaf(t1, t1, t22);
                        const float al0 = fminf(0.99f, __builtin_amdgcn_exp2f(-Q));
                        const bool on = Q <= qmax && off < lim[q];
                        has = has || on;
                        const float al = on ? al0 : 0.f;
                        const float iom = __builtin_amdgcn_rcpf(1.f - al);
                        const float Ti = Tc[q] * iom;
                        const float wgt = al * Ti;
                        const float gc = fmaf(gC0[q], C.col0, fmaf(gC1[q], C.col1, fmaf(gC2[q], C.col2, gD[q] * C.z)));
                        const float dLda = fmaf(Ti, gc, -iom * behind[q]);
                        behind[q] = on ? fmaf(wgt, gc, behind[q]) : behind[q];
                        Tc[q] = on ? Ti : Tc[q];
                        const float h = on && al0 < 0.99f ? al * dLda : 0.f;
                        const float s1 = h * t1;
                        v[0] += h;
                        v[1] += s1;
                        v[2] = fmaf(s1, fx[q] - B.u, v[2]);
                        v[6] = !Bad::value || on ? fmaf(gC0[q], wgt, v[6]) : v[6];
                        v[7] = !Bad::value || on ? fmaf(gC1[q], wgt, v[7]) : v[7];
                        v[8] = !Bad::value || on ? fmaf(gC2[q], wgt, v[8]) : v[8];
                        v[9] = !Bad::value || on ? fmaf(gD[q], wgt, v[9]) : v[9];
                    }
                    if (__ballot(has) == 0) continue;
                    const float dy = fy - B.v;                  // shared by the thread's pixels, as t2
                    v[3] = v[1] * dy;
                    v[4] = v[0] * t2;
                    v[5] = v[4] * dy;
                    float s0, s1, s2;
                    ten_sums(v, odd1, odd2, &s0, &s1, &s2);
                    float* acc = S.acc + off / 16 * kEntryGrad;
                    if (k < 4) {
                        if (s0 != 0.f) atomicAdd(acc + k, s0);
                        if (s1 != 0.f) atomicAdd(acc + 4 + k, s1);
                        if (k < 2 && s2 != 0.f) atomicAdd(acc + 8 + k, s2);
                    }
                }
            }
        };
        if (bad_wave) walk(std::true_type{}); else walk(std::false_type{});
        __syncthreads();
        // the tile's sums: twelve consecutive words per entry
        for (uint32_t i = threadIdx.x; i < cnt * kEntryGrad; i += kNT) {
            const float x = S.acc[i];
            const uint32_t e = S.entry[i / kEntryGrad];
            if (x != 0.f && e < a.cut_cap) atomicAdd(a.egrad + (size_t)e * kEntryGrad + i % kEntryGrad, x);
            S.acc[i] = 0.f;
        }
        __syncthreads();
    }
}

// Zeros to the entries' sums; the image gradients of up to kArgViews views come
// along as arguments (with a copy and its event a 253 x 191 step took 222 us, so
// 214).
struct ArgGrads {
    ImgGrad g[kArgViews];
};
__global__ void k_zero_egrad(float* g, const Counters* ctr, uint32_t cap, ArgGrads few, int n_few, uint64_t* dimg) {
    const int words = n_few * (int)(sizeof(ImgGrad) / 8);
    const uint64_t* src = reinterpret_cast<const uint64_t*>(&few);
    if (blockIdx.x == 0 && (int)threadIdx.x < words) dimg[threadIdx.x] = src[threadIdx.x];
    const uint64_t n = (uint64_t)min(ctr->cut, cap) * kEntryGrad;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        g[i] = 0.f;
}

// Real SH basis (as in the projection) and its gradient with respect to the
// direction's components, FP64.
template <int DEG>
__device__ __forceinline__ void sh_basis_grad(double x, double y, double z, double Y[16], double dY[16][3]) {
    constexpr int deg = DEG;
    constexpr double k00 = 0.28209479177387814, k1 = 0.48860251190291992;
    constexpr double k2a = 1.0925484305920792, k2b = 0.31539156525252005, k2c = 0.54627421529603959;
    constexpr double k3a = 0.59004358992664352, k3b = 2.8906114426405538, k3c = 0.45704579946446572,
                     k3d = 0.3731763325901154, k3e = 1.4453057213202769;
    for (int k = 0; k < 16; ++k) Y[k] = dY[k][0] = dY[k][1] = dY[k][2] = 0.0;
    Y[0] = k00;
    if (deg >= 1) {
        Y[1] = -k1 * y; dY[1][1] = -k1;
        Y[2] = k1 * z; dY[2][2] = k1;
        Y[3] = -k1 * x; dY[3][0] = -k1;
    }
    if (deg >= 2) {
        Y[4] = k2a * x * y; dY[4][0] = k2a * y; dY[4][1] = k2a * x;
        Y[5] = -k2a * y * z; dY[5][1] = -k2a * z; dY[5][2] = -k2a * y;
        Y[6] = k2b * (3.0 * z * z - 1.0); dY[6][2] = 6.0 * k2b * z;
        Y[7] = -k2a * x * z; dY[7][0] = -k2a * z; dY[7][2] = -k2a * x;
        Y[8] = k2c * (x * x - y * y); dY[8][0] = 2.0 * k2c * x; dY[8][1] = -2.0 * k2c * y;
    }
    if (deg >= 3) {
        Y[9] = -k3a * y * (3.0 * x * x - y * y);
        dY[9][0] = -6.0 * k3a * x * y; dY[9][1] = -k3a * (3.0 * x * x - 3.0 * y * y);
        Y[10] = k3b * x * y * z;
        dY[10][0] = k3b * y * z; dY[10][1] = k3b * x * z; dY[10][2] = k3b * x * y;
        Y[11] = -k3c * y * (5.0 * z * z - 1.0);
        dY[11][1] = -k3c * (5.0 * z * z - 1.0); dY[11][2] = -10.0 * k3c * y * z;
        Y[12] = k3d * z * (5.0 * z * z - 3.0);
        dY[12][2] = k3d * (15.0 * z * z - 3.0);
        Y[13] = -k3c * x * (5.0 * z * z - 1.0);
        dY[13][0] = -k3c * (5.0 * z * z - 1.0); dY[13][2] = -10.0 * k3c * x * z;
        Y[14] = k3e * z * (x * x - y * y);
        dY[14][0] = 2.0 * k3e * x * z; dY[14][1] = -2.0 * k3e * y * z; dY[14][2] = k3e * (x * x - y * y);
        Y[15] = -k3a * x * (x * x - 3.0 * y * y);
        dY[15][0] = -k3a * (3.0 * x * x - 3.0 * y * y); dY[15][1] = 6.0 * k3a * x * y;
    }
}

template <int DEG>
__global__ __launch_bounds__(256) void k_project_bwd(ProjBwdArgs a) {
    const uint32_t m = min(a.ctr->cut, a.cut_cap);
    constexpr int K = (DEG + 1) * (DEG + 1);
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < m; p += gridDim.x * blockDim.x) {
        const uint32_t i = a.order[p];
        const float* eg = a.egrad + (size_t)i * kEntryGrad;
        double gin[kNG];
        bool any = false;
#pragma unroll
        for (int k = 0; k < kNG; ++k) {
            gin[k] = eg[k];
            any = any || gin[k] != 0.0;
        }
        float4* rec0 = reinterpret_cast<float4*>(a.rec + (size_t)p * kEntryRec);
        for (int t = 0; t < kEntryRec / 4; ++t) rec0[t] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (!any) continue;
        const uint2 e = a.cut[i];
        const ViewDev& V = a.views[e.y];
        const int64_t g = e.x;
        const float4 g0 = a.geo[3 * g], g1 = a.geo[3 * g + 1], g2 = a.geo[3 * g + 2];
        const double dx = (double)g0.x - V.o[0], dy = (double)g0.y - V.o[1], dz = (double)g0.z - V.o[2];
        const double tx = (V.R[0] * dx + V.R[1] * dy) + V.R[2] * dz;
        const double ty = (V.R[3] * dx + V.R[4] * dy) + V.R[5] * dz;
        const double tz = (V.R[6] * dx + V.R[7] * dy) + V.R[8] * dz;
        if (!(tz > V.znear)) continue;
        const double iz = 1.0 / tz;
        const double xr0 = tx * iz, yr0 = ty * iz;
        const bool xcl = xr0 < V.xlo || xr0 > V.xhi, ycl = yr0 < V.ylo || yr0 > V.yhi;
        const double xr = fmin(fmax(xr0, V.xlo), V.xhi), yr = fmin(fmax(yr0, V.ylo), V.yhi);
        double M[2][3];
        for (int j = 0; j < 3; ++j) {
            M[0][j] = V.fx * iz * (V.R[j] - xr * V.R[6 + j]);
            M[1][j] = V.fy * iz * (V.R[3 + j] - yr * V.R[6 + j]);
        }
        double qw = g1.x, qx = g1.y, qy = g1.z, qz = g1.w;
        const double qn = sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
        qw /= qn; qx /= qn; qy /= qn; qz /= qn;
        const double R[3][3] = {{1.0 - 2.0 * (qy * qy + qz * qz), 2.0 * (qx * qy - qw * qz), 2.0 * (qx * qz + qw * qy)},
                                {2.0 * (qx * qy + qw * qz), 1.0 - 2.0 * (qx * qx + qz * qz), 2.0 * (qy * qz - qw * qx)},
                                {2.0 * (qx * qz - qw * qy), 2.0 * (qy * qz + qw * qx), 1.0 - 2.0 * (qx * qx + qy * qy)}};
        const double sc[3] = {g2.x, g2.y, g2.z};
        double MR[2][3], Tm[2][3];
        for (int r = 0; r < 2; ++r)
            for (int k = 0; k < 3; ++k) {
                MR[r][k] = M[r][0] * R[0][k] + M[r][1] * R[1][k] + M[r][2] * R[2][k];
                Tm[r][k] = MR[r][k] * sc[k];
            }
        const double s00 = Tm[0][0] * Tm[0][0] + Tm[0][1] * Tm[0][1] + Tm[0][2] * Tm[0][2] + 0.3;
        const double s01 = Tm[0][0] * Tm[1][0] + Tm[0][1] * Tm[1][1] + Tm[0][2] * Tm[1][2];
        const double s11 = Tm[1][0] * Tm[1][0] + Tm[1][1] * Tm[1][1] + Tm[1][2] * Tm[1][2] + 0.3;
        const double det = s00 * s11 - s01 * s01;
        if (!(det > 0.0)) continue;
        // conic factors p = sqrt(s11 / det), r = -s01 / sqrt(det s11),
        // s = 1 / sqrt(s11) and their derivatives
        const double pp = sqrt(s11 / det), idet2 = 1.0 / (det * det);
        const double mm = det * s11, im12 = 1.0 / sqrt(mm), im32 = im12 / mm;
        // the entry's sums h, h t1, h t1 dx, h t1 dy, h t2, h t2 dy (t1 and t2
        // scaled by kS) to the gradients of the 2D mean and the factors:
        // dL/dq = -h / 2
        const double iks = 1.0 / (double)kS;
        const double st1 = gin[1] * iks, st2 = gin[4] * iks;
        const double rf = -s01 * im12, sf = 1.0 / sqrt(s11);
        const double gu = pp * st1, gv = rf * st1 + sf * st2;
        const double gp = -gin[2] * iks, gr = -gin[3] * iks, gs = -gin[5] * iks;
        const double h00 = gp * (0.5 / pp) * (-s11 * s11 * idet2) + gr * 0.5 * s01 * im32 * s11 * s11;
        const double h01 = gp * (0.5 / pp) * (2.0 * s11 * s01 * idet2) + gr * (-im12 - s01 * s01 * s11 * im32);
        const double h11 = gp * (0.5 / pp) * (-s01 * s01 * idet2) + gr * 0.5 * s01 * im32 * (det + s00 * s11) +
                           gs * (-0.5 / (s11 * sqrt(s11)));
        // Sigma' = T T^T: dL/dT
        double gT[2][3];
        for (int k = 0; k < 3; ++k) {
            gT[0][k] = 2.0 * h00 * Tm[0][k] + h01 * Tm[1][k];
            gT[1][k] = 2.0 * h11 * Tm[1][k] + h01 * Tm[0][k];
        }
        double gsc[3], gMR[2][3];
        for (int k = 0; k < 3; ++k) {
            gsc[k] = gT[0][k] * MR[0][k] + gT[1][k] * MR[1][k];
            gMR[0][k] = gT[0][k] * sc[k];
            gMR[1][k] = gT[1][k] * sc[k];
        }
        double gR[3][3], gM[2][3];
        for (int j = 0; j < 3; ++j)
            for (int k = 0; k < 3; ++k) gR[j][k] = M[0][j] * gMR[0][k] + M[1][j] * gMR[1][k];
        for (int r = 0; r < 2; ++r)
            for (int j = 0; j < 3; ++j) gM[r][j] = gMR[r][0] * R[j][0] + gMR[r][1] * R[j][1] + gMR[r][2] * R[j][2];
        // quaternion: dL/d(normalised q), then through the normalisation
        const double gw = 2.0 * (-qz * gR[0][1] + qy * gR[0][2] + qz * gR[1][0] - qx * gR[1][2] - qy * gR[2][0] +
                                 qx * gR[2][1]);
        const double gx = 2.0 * (qy * gR[0][1] + qz * gR[0][2] + qy * gR[1][0] - 2.0 * qx * gR[1][1] - qw * gR[1][2] +
                                 qz * gR[2][0] + qw * gR[2][1] - 2.0 * qx * gR[2][2]);
        const double gy = 2.0 * (-2.0 * qy * gR[0][0] + qx * gR[0][1] + qw * gR[0][2] + qx * gR[1][0] +
                                 qz * gR[1][2] - qw * gR[2][0] + qz * gR[2][1] - 2.0 * qy * gR[2][2]);
        const double gz = 2.0 * (-2.0 * qz * gR[0][0] - qw * gR[0][1] + qx * gR[0][2] + qw * gR[1][0] -
                                 2.0 * qz * gR[1][1] + qy * gR[1][2] + qx * gR[2][0] + qy * gR[2][1]);
        const double qd = qw * gw + qx * gx + qy * gy + qz * gz;
        // camera-space mean: 2D mean, depth, Jacobian
        double gt0 = gu * V.fx * iz, gt1 = gv * V.fy * iz;
        double gt2 = -(gu * V.fx * tx + gv * V.fy * ty) * iz * iz + gin[9];
        const double iz2 = iz * iz;
        for (int j = 0; j < 3; ++j) {
            const double w0 = V.R[j], w1 = V.R[3 + j], w2 = V.R[6 + j];
            if (!xcl) {
                gt0 += gM[0][j] * (-V.fx * iz2 * w2);
                gt2 += gM[0][j] * (-V.fx * iz2 * w0 + 2.0 * V.fx * xr * iz2 * w2);
            } else {
                gt2 += gM[0][j] * (-V.fx * iz2 * (w0 - xr * w2));
            }
            if (!ycl) {
                gt1 += gM[1][j] * (-V.fy * iz2 * w2);
                gt2 += gM[1][j] * (-V.fy * iz2 * w1 + 2.0 * V.fy * yr * iz2 * w2);
            } else {
                gt2 += gM[1][j] * (-V.fy * iz2 * (w1 - yr * w2));
            }
        }
        double gmu[3];
        for (int j = 0; j < 3; ++j) gmu[j] = V.R[j] * gt0 + V.R[3 + j] * gt1 + V.R[6 + j] * gt2;
        // colour: SH coefficients and the view direction
        const double dn = sqrt(dx * dx + dy * dy + dz * dz), idn = 1.0 / dn;
        const double ux = dx * idn, uy = dy * idn, uz = dz * idn;
        double Y[16], dY[16][3];
        sh_basis_grad<DEG>(ux, uy, uz, Y, dY);
        double gdir[3] = {0.0, 0.0, 0.0};
        double gcm[3] = {0.0, 0.0, 0.0};                              // colour gradient, 0 where clamped
        for (int c = 0; c < 3; ++c) {
            const double gc = gin[6 + c];
            if (gc == 0.0) continue;
            double val = 0.5, d0 = 0.0, d1 = 0.0, d2 = 0.0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const double f = a.sh[((int64_t)g * K + k) * 3 + c];
                val += f * Y[k];
                d0 += f * dY[k][0];
                d1 += f * dY[k][1];
                d2 += f * dY[k][2];
            }
            if (val < 0.0 || val > 1.0) continue;                       // clamped colour
            gcm[c] = gc;
            gdir[0] += gc * d0;
            gdir[1] += gc * d1;
            gdir[2] += gc * d2;
        }
        const double dd = ux * gdir[0] + uy * gdir[1] + uz * gdir[2];
        gmu[0] += (gdir[0] - ux * dd) * idn;
        gmu[1] += (gdir[1] - uy * dd) * idn;
        gmu[2] += (gdir[2] - uz * dd) * idn;
        float4* rec = reinterpret_cast<float4*>(a.rec + (size_t)p * kEntryRec);
        rec[0] = make_float4((float)gmu[0], (float)gmu[1], (float)gmu[2], (float)gsc[0]);
        rec[1] = make_float4((float)gsc[1], (float)gsc[2], (float)((gw - qw * qd) / qn), (float)((gx - qx * qd) / qn));
        rec[2] = make_float4((float)((gy - qy * qd) / qn), (float)((gz - qz * qd) / qn), (float)(gin[0] / (double)g0.w), (float)gcm[0]);
        rec[3] = make_float4((float)gcm[1], (float)gcm[2], (float)ux, (float)uy);
        rec[4] = make_float4((float)uz, 0.f, 0.f, 0.f);
    }
}

// Entry records in Gaussian order: thread p starts a run when its key
// differs from the previous one and sums the run's records; the SH
// coefficients' gradients are sum_entries g_c Y_k(d_entry).  One thread per
// Gaussian, so the outputs are updated without atomics.
template <int DEG>
__global__ __launch_bounds__(256) void k_gather_bwd(GatherArgs a) {
    const uint32_t m = min(a.ctr->cut, a.cap);
    constexpr int K = (DEG + 1) * (DEG + 1);
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < m; p += gridDim.x * blockDim.x) {
        const uint32_t key = a.keys[p];
        if (p > 0 && a.keys[p - 1] == key) continue;
        float acc[11];
#pragma unroll
        for (int t = 0; t < 11; ++t) acc[t] = 0.f;
        float sh[3 * K];
#pragma unroll
        for (int t = 0; t < 3 * K; ++t) sh[t] = 0.f;
        bool any = false;
        for (uint32_t q = p; q < m && a.keys[q] == key; ++q) {
            const float4* rec = reinterpret_cast<const float4*>(a.rec + (size_t)q * kEntryRec);
            const float4 r0 = rec[0], r1 = rec[1], r2 = rec[2], r3 = rec[3], r4 = rec[4];
            const float v[11] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w, r2.x, r2.y, r2.z};
#pragma unroll
            for (int t = 0; t < 11; ++t) {
                acc[t] += v[t];
                any = any || v[t] != 0.f;
            }
            const float gc[3] = {r2.w, r3.x, r3.y};
            if (gc[0] != 0.f || gc[1] != 0.f || gc[2] != 0.f) {
                any = true;
                double Y[16], dY[16][3];
                sh_basis_grad<DEG>(r3.z, r3.w, r4.x, Y, dY);
#pragma unroll
                for (int k = 0; k < K; ++k)
#pragma unroll
                    for (int c = 0; c < 3; ++c) sh[k * 3 + c] += (float)(gc[c] * Y[k]);
            }
        }
        if (!any) continue;
        const size_t g = key;
#pragma unroll
        for (int t = 0; t < 3; ++t) a.g_means[3 * g + t] += acc[t];
#pragma unroll
        for (int t = 0; t < 3; ++t) a.g_scales[3 * g + t] += acc[3 + t];
#pragma unroll
        for (int t = 0; t < 4; ++t) a.g_quats[4 * g + t] += acc[6 + t];
        a.g_opacity[g] += acc[10];
#pragma unroll
        for (int t = 0; t < 3 * K; ++t) a.g_sh[g * 3 * K + t] += sh[t];
    }
}

__global__ void k_entry_keys(const uint2* cut, const Counters* ctr, uint32_t cap, uint32_t* keys, uint32_t* vals,
                             SortBins clear) {
    const uint32_t m = min(ctr->cut, cap);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < clear.n; i += gridDim.x * blockDim.x) clear.words[i] = 0;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gridDim.x * blockDim.x) {
        keys[i] = cut[i].x;
        vals[i] = i;
    }
}

}  // namespace

void launch_backward_composite(const BwdArgs& b, const Counters* ctr, const ImgGrad* few, int n_few, hipStream_t s) {
    ArgGrads args{};
    for (int v = 0; v < n_few; ++v) args.g[v] = few[v];
    static_assert(sizeof(ArgGrads) / 8 <= 256, "a thread per word");
    k_zero_egrad<<<1024, 256, 0, s>>>(b.egrad, ctr, b.cut_cap, args, n_few,
                                      const_cast<uint64_t*>(reinterpret_cast<const uint64_t*>(b.dimg)));
    if (!b.total_tiles) return;
    if (b.state)
        k_composite_bwd<true><<<b.total_tiles, kNT, 0, s>>>(b);
    else
        k_composite_bwd<false><<<b.total_tiles, kNT, 0, s>>>(b);
}

void launch_backward_params(ProjBwdArgs p, SortArgs sa, GatherArgs ga, hipStream_t s) {
    // the entries in Gaussian order: the chain rule reads each Gaussian's
    // parameters for its views in a row and writes the records in that
    // order, which the sum then reads sequentially
    k_entry_keys<<<2048, 256, 0, s>>>(p.cut, p.ctr, p.cut_cap, sa.keys[0], sa.vals[0], sort_bins(sa));
    const int r = launch_sort(sa, s);
    p.order = sa.vals[r];
    ga.keys = sa.keys[r];
    switch (p.sh_degree) {
        case 0: k_project_bwd<0><<<2048, 256, 0, s>>>(p); break;
        case 1: k_project_bwd<1><<<2048, 256, 0, s>>>(p); break;
        case 2: k_project_bwd<2><<<2048, 256, 0, s>>>(p); break;
        default: k_project_bwd<3><<<2048, 256, 0, s>>>(p); break;
    }
    switch (ga.sh_degree) {
        case 0: k_gather_bwd<0><<<2048, 256, 0, s>>>(ga); break;
        case 1: k_gather_bwd<1><<<2048, 256, 0, s>>>(ga); break;
        case 2: k_gather_bwd<2><<<2048, 256, 0, s>>>(ga); break;
        default: k_gather_bwd<3><<<2048, 256, 0, s>>>(ga); break;
    }
}

}  // namespace hgs
