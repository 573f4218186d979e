// GS-slice occupancy: the scene's Gaussians cut by horizontal planes,
// rasterised into a 2D grid per plane and into their union (the collision
// map of Sec. III-C).
//
// Per Gaussian, in FP64: the inverse covariance C = R diag(1/s^2) R^T; the
// slice at height z is a 2D Gaussian with amplitude exp(-lambda (z-mu_z)^2/2),
// centre (mu_x, mu_y) - (z - mu_z)(alpha, beta) and inverse covariance the xy
// block of C, where (alpha, beta) solves the 2x2 system of that block with
// right-hand side (c_xz, c_yz) and lambda = c_zz - (alpha, beta) . (c_xz, c_yz)
// (Supplementary derivation; the printed second exponent's missing -1/2 is
// restored).  The Gaussian is solid where o a(z) exp(-q/2) >= rho_min, i.e.
// inside q <= 2 ln(o a(z) / rho_min); a cell (closed square) is marked when
// that ellipse meets it, found from the least value of q over the square:
// zero if the centre is inside, else the least over the four edges, each at
// the clamped stationary point of a 1D quadratic.
//
// One thread per Gaussian does its vertical test and, if it reaches a plane
// (floor and ceiling sheets and other floors do not), the FP64 slice algebra;
// the workgroup then shares out the (Gaussian, plane) pairs, of which a wave's
// Gaussians have few and unequal numbers, and a thread marks its pair's cells
// row by row.  Marks are byte stores of 1 (concurrent stores agree).  (A
// thread that walked its own Gaussian's planes and tested every cell of the
// bounding boxes, 20 per pair: 174 us for 2 M Gaussians and 15 planes; so 74.
// Their 96 MB take 16 at the rate of a copy, the algebra the rest.)
#include <algorithm>
#include <cmath>

#include "device_util.h"
#include "grid.h"
#include "internal.h"

namespace hgs {

namespace {

constexpr int kNT = 256;

// Zeros to two byte ranges, 16 bytes a thread between their ends.
__global__ __launch_bounds__(kNT) void k_fill_zero(uint8_t* p0, size_t n0, uint8_t* p1, size_t n1) {
    for (int r = 0; r < 2; ++r) {
        uint8_t* p = r ? p1 : p0;
        const size_t n = r ? n1 : n0, head = min(n, (size_t)(-reinterpret_cast<uintptr_t>(p) & 15u));
        const size_t n16 = (n - head) / 16, t = blockIdx.x * (size_t)kNT + threadIdx.x, stride = (size_t)gridDim.x * kNT;
        for (size_t i = t; i < n16; i += stride) reinterpret_cast<uint4*>(p + head)[i] = make_uint4(0, 0, 0, 0);
        if (t < head) p[t] = 0;
        const size_t tail = head + 16 * n16;
        if (t < n - tail) p[tail + t] = 0;
    }
}

// Least of q(d) = a dx^2 + 2 b dx dy + c dy^2 over the square
// [qx0, qx0 + w] x [qy0, qy0 + w], d = point - centre (m).
__device__ __forceinline__ double square_min(double a, double b, double c, double mx, double my, double qx0,
                                             double qy0, double w) {
    const double lx = qx0 - mx, hx = qx0 + w - mx;     // x-range of d
    const double ly = qy0 - my, hy = qy0 + w - my;
    if (lx <= 0.0 && hx >= 0.0 && ly <= 0.0 && hy >= 0.0) return 0.0;
    double best = 1e300;
    const double ex[2] = {lx, hx}, ey[2] = {ly, hy};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const double dx = ex[s];
        const double dy = fmin(fmax(-b * dx / c, ly), hy);
        best = fmin(best, (a * dx + 2.0 * b * dy) * dx + c * dy * dy);
        const double ey0 = ey[s];
        const double dx2 = fmin(fmax(-b * ey0 / a, lx), hx);
        best = fmin(best, (a * dx2 + 2.0 * b * ey0) * dx2 + c * ey0 * ey0);
    }
    return best;
}

// What a Gaussian's cells in a plane follow from, computed once by its thread
// and read by the threads that take its (Gaussian, plane) pairs.
struct SliceRec {
    double a, b, c;                        // xy block of the inverse covariance
    double al, be, lam, amp;               // amp = 2 ln(o / rho_min)
    // q = (p dx + r dy)^2 + (s dy)^2: 1 / p, r, s, 1 / s and the height of the
    // rightmost point of q <= 1; ip = 0: walk the bounding box instead
    double ip, r, s, is, yr;
    float4 g0;
};

// Planes whose pairs are listed at a time.
constexpr int kPlanes = 16;

// Every cell of the ellipse's bounding box by its least value of q: the
// definition, for the pairs whose outcome hangs on the last digits.
__device__ __forceinline__ void slice_cells(const SliceArgs& s, const SliceRec& G, int k) {
    const double dz = (double)s.heights[k] - (double)G.g0.z, o = G.g0.w;
    const double A = o * exp(-0.5 * G.lam * dz * dz);
    if (!(A >= s.rho_min)) return;
    const double r2 = 2.0 * log(A / s.rho_min);
    const double a = G.a, b = G.b, c = G.c, det = a * c - b * b;
    const double mx = (double)G.g0.x - G.al * dz, my = (double)G.g0.y - G.be * dz;
    // bounding box of the ellipse (half-extents r sqrt(c/det), r sqrt(a/det)), one cell wider
    const double hx = sqrt(r2 * c / det) + s.cell, hy = sqrt(r2 * a / det) + s.cell;
    const double fi0 = floor((mx - hx - s.x0) / s.cell), fi1 = floor((mx + hx - s.x0) / s.cell);
    const double fj0 = floor((my - hy - s.y0) / s.cell), fj1 = floor((my + hy - s.y0) / s.cell);
    // off the grid (or not finite): nothing to mark
    if (!(fi1 >= 0.0 && fi0 <= (double)(s.nx - 1) && fj1 >= 0.0 && fj0 <= (double)(s.ny - 1))) return;
    const int i0 = (int)fmax(fi0, 0.0), i1 = (int)fmin(fi1, (double)(s.nx - 1));
    const int j0 = (int)fmax(fj0, 0.0), j1 = (int)fmin(fj1, (double)(s.ny - 1));
    uint8_t* plane = s.occ ? s.occ + (size_t)k * s.nx * s.ny : nullptr;
    for (int j = j0; j <= j1; ++j) {
        const double qy0 = s.y0 + (double)j * s.cell;
        for (int i = i0; i <= i1; ++i) {
            const double qx0 = s.x0 + (double)i * s.cell;
            if (square_min(a, b, c, mx, my, qx0, qy0, s.cell) <= r2) {
                const size_t cidx = (size_t)j * s.nx + i;
                if (plane) plane[cidx] = 1;
                if (s.map) s.map[cidx] = 1;
            }
        }
    }
}

// The cells of a pair by rows: within the band of heights of a row of cells,
// the ellipse spans an interval of x, and the row's cells that meet it are
// marked.  False, before anything is marked, where a bound lies within kEdge
// of a cell's edge (or a sum is not finite): rounding may decide such a cell,
// and slice_cells does.
//
// The bounds' errors are held below kEdge too, else slice_cells decides.  To
// first order, in units of kUlp and with cond = a c / det, which the products
// of the inverse covariance lose to cancellation:
//   r2, and the q of a point on the ellipse as slice_cells forms it:
//     er = 4 cond r2 + lam dz^2 + amp + 8  (exp and log of that size);
//   positions, in cells: ec = coordinates + the ellipse's height;
//   the top and bottom: half of er / r2 and of cond times the height, and ec;
//   a row's ends, x = (sqrt(dr) - r y) / p with dr = r2 - (s y)^2:
//     (er + s reach ec cell) / (p sqrt(dr)) + (|r| ec cell + reach + |r| ey) / p + ec,
// where rows have dr > 1e-6 r2, and that is known: 16 er lie below it.
// Against sums in 60 digits, ends of ellipses of 100 to 3e7 cells and cond up
// to 1e5 were off by at most a fourteenth of this: 1e-13 cells at 100 cells and
// cond near 1, 3e-10 at cond 1e5, 2e-8 at 1e4 cells, 4e-6, past kEdge, at 1e6
// near the top.  (Once per pair for its worst row: 0.3 of 81 us for 2 M
// Gaussians and 15 planes; with each row's own 1.9.)
constexpr double kEdge = 1e-6;             // cells
constexpr double kUlp = 0x1p-51;           // four times the relative error of a rounding
__device__ __forceinline__ bool slice_rows(const SliceArgs& s, const SliceRec& G, int k, double icell) {
    const double dz = (double)s.heights[k] - (double)G.g0.z;
    const double drop = G.lam * dz * dz, r2 = fma(-G.lam * dz, dz, G.amp);
    if (r2 < -1e-8) return true;
    const double mx = (double)G.g0.x - G.al * dz, my = (double)G.g0.y - G.be * dz;
    if (!(r2 > 1e-8 && G.ip > 0.0)) return false;
    const double at = fabs(s.x0) + fabs(s.y0) + fabs(mx) + fabs(my);
    if (!(at * 1e-8 < s.cell)) return false;
    const double ir = rsqrt64(r2), reach = r2 * ir, ey = reach * G.is, ym = reach * G.yr;
    const double er = fma(4.0 * G.c * G.is * G.is, r2, fabs(drop) + (G.amp + 8.0)), ec = (at + ey) * icell;
    const double ends = fma(G.ip, fma(1e3 * G.s + fabs(G.r), ec, (er * (1e3 * ir) + reach + fabs(G.r) * ey) * icell), ec);
    const double tops = fma(er * ir, ir * ey * icell, ec);
    if (!(er < r2 * (1e-6 / 16.0 / kUlp) && ends < kEdge / kUlp && tops < kEdge / kUlp)) return false;
    const double u = (mx - s.x0) * icell, v = (my - s.y0) * icell;      // centre, in cells
    const double fj0 = floor(v - ey * icell - kEdge), fj1 = floor(v + ey * icell + kEdge);
    if (fj0 != floor(v - ey * icell + kEdge) || fj1 != floor(v + ey * icell - kEdge)) return false;
    if (!(fj1 >= 0.0 && fj0 <= (double)(s.ny - 1))) return true;
    const int j0 = (int)fmax(fj0, 0.0), j1 = (int)fmin(fj1, (double)(s.ny - 1));
    uint8_t* plane = s.occ ? s.occ + (size_t)k * s.nx * s.ny : nullptr;
    for (int pass = 0; pass < 2; ++pass) {             // all rows are sure before the first mark
        for (int j = j0; j <= j1; ++j) {
            const double y0 = fmax(((double)j - v) * s.cell, -ey), y1 = fmin(((double)(j + 1) - v) * s.cell, ey);
            const double yr = fmin(fmax(ym, y0), y1), yl = fmin(fmax(-ym, y0), y1);
            const double tr = G.s * yr, tl = G.s * yl;
            const double dr = fma(-tr, tr, r2), dl = fma(-tl, tl, r2);
            const double xr = u + (dr * rsqrt64(fmax(dr, 1e-30)) - G.r * yr) * G.ip * icell;
            const double xl = u - (dl * rsqrt64(fmax(dl, 1e-30)) + G.r * yl) * G.ip * icell;
            const double fi0 = floor(xl - kEdge), fi1 = floor(xr + kEdge);
            if (pass == 0) {
                // (near the ellipse's top and bottom its width is not known well)
                if (!(dr > 1e-6 * r2 && dl > 1e-6 * r2) || fi0 != floor(xl + kEdge) || fi1 != floor(xr - kEdge))
                    return false;
            } else if (fi1 >= 0.0 && fi0 <= (double)(s.nx - 1)) {
                const int i0 = (int)fmax(fi0, 0.0), i1 = (int)fmin(fi1, (double)(s.nx - 1));
                for (int i = i0; i <= i1; ++i) {
                    const size_t cidx = (size_t)j * s.nx + i;
                    if (plane) plane[cidx] = 1;
                    if (s.map) s.map[cidx] = 1;
                }
            }
        }
    }
    return true;
}

__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(4))) void k_slice(SliceArgs s) {
    __shared__ SliceRec S[kNT];
    __shared__ uint16_t s_pair[kNT * kPlanes];
    __shared__ uint32_t s_n;
    const double icell = 1.0 / s.cell;
    for (uint32_t t0 = blockIdx.x * kNT; t0 < s.n; t0 += gridDim.x * kNT) {
        const uint32_t t = t0 + threadIdx.x;
        double reach2 = -1.0;                          // no plane
        SliceRec G = {};
        if (t < s.n) {
            const int64_t g = s.ids ? (int64_t)s.ids[t] : (int64_t)t;
            const float4 g0 = s.geo[3 * g], g2 = s.geo[3 * g + 2];
            // No plane is within reach of the longest axis, whatever the
            // rotation: Sigma_zz <= the largest scale squared, o <= 1.  (15
            // planes of one floor of a 30 M-leaf building: 727 -> 470 us.)
            const double off = fmax(s.low - (double)g0.z, (double)g0.z - s.high);
            const double big = fmax(fmax(fabs((double)g2.x), fabs((double)g2.y)), fabs((double)g2.z));
            const bool far = g0.w <= 1.f && off > 0.0 && off * off > big * big * s.reach + 2e-12;
            if (!far) {
                const float4 g1 = s.geo[3 * g + 1];
                // rotation of the normalised quaternion (w, x, y, z); columns = axes
                double qw = g1.x, qx = g1.y, qy = g1.z, qz = g1.w;
                const double qi = 1.0 / sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
                qw *= qi; qx *= qi; qy *= qi; qz *= qi;
                const double R[3][3] = {{1.0 - 2.0 * (qy * qy + qz * qz), 2.0 * (qx * qy - qw * qz), 2.0 * (qx * qz + qw * qy)},
                                        {2.0 * (qx * qy + qw * qz), 1.0 - 2.0 * (qx * qx + qz * qz), 2.0 * (qy * qz - qw * qx)},
                                        {2.0 * (qx * qz - qw * qy), 2.0 * (qy * qz + qw * qx), 1.0 - 2.0 * (qx * qx + qy * qy)}};
                // vertical reach: o exp(-dz^2 / (2 Sigma_zz)) >= rho_min needs
                // dz^2 <= 2 Sigma_zz ln(o / rho_min) (lambda = 1 / Sigma_zz); planes
                // beyond it (with a relative margin) cannot be solid
                const double o = g0.w;
                bool any = false;
                if (o >= s.rho_min) {
                    const double szz = R[2][0] * R[2][0] * ((double)g2.x * g2.x) + R[2][1] * R[2][1] * ((double)g2.y * g2.y) +
                                       R[2][2] * R[2][2] * ((double)g2.z * g2.z);
                    G.amp = 2.0 * log(o / s.rho_min);
                    reach2 = szz * G.amp * (1.0 + 1e-6) + 1e-12;
                    for (int k = 0; k < s.n_planes; ++k) {
                        const double dz = (double)s.heights[k] - (double)g0.z;
                        any = any || dz * dz <= reach2;
                    }
                }
                if (any) {
                    const double iv[3] = {1.0 / ((double)g2.x * g2.x), 1.0 / ((double)g2.y * g2.y), 1.0 / ((double)g2.z * g2.z)};
                    double C[3][3];
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int j = 0; j < 3; ++j)
                            C[i][j] = R[i][0] * iv[0] * R[j][0] + R[i][1] * iv[1] * R[j][1] + R[i][2] * iv[2] * R[j][2];
                    G.a = C[0][0];
                    G.b = C[0][1];
                    G.c = C[1][1];
                    const double det = G.a * G.c - G.b * G.b;
                    G.al = (C[0][2] * G.c - C[1][2] * G.b) / det;
                    G.be = (C[1][2] * G.a - C[0][2] * G.b) / det;
                    G.lam = C[2][2] - G.al * C[0][2] - G.be * C[1][2];
                    G.g0 = g0;
                    // (a c / det: what det and the rows lose to cancellation)
                    G.ip = 0.0;
                    if (det > 1e-5 * (G.a * G.c) && G.a > 1e-30 && G.a < 1e30 && G.c > 1e-30 && G.c < 1e30) {
                        G.ip = rsqrt64(G.a);
                        G.r = G.b * G.ip;
                        G.s = det * rsqrt64(det) * G.ip;
                        G.is = rcp64(G.s);
                        G.yr = -G.r * G.is * rsqrt64(G.r * G.r + G.s * G.s);
                    }
                    S[threadIdx.x] = G;
                } else {
                    reach2 = -1.0;
                }
            }
        }
        if (!__syncthreads_or(reach2 >= 0.0)) continue;
        for (int k0 = 0; k0 < s.n_planes; k0 += kPlanes) {
            if (threadIdx.x == 0) s_n = 0;
            __syncthreads();
            const int k1 = min(k0 + kPlanes, s.n_planes);
            for (int k = k0; k < k1; ++k) {
                const double dz = (double)s.heights[k] - (double)G.g0.z;
                const bool hit = reach2 >= 0.0 && dz * dz <= reach2;
                const uint64_t bal = __ballot(hit);
                if (!bal) continue;
                uint32_t at = 0;
                if (lane_id() == 0) at = atomicAdd(&s_n, (uint32_t)__popcll(bal));
                at = __builtin_amdgcn_readfirstlane(at);
                if (hit) s_pair[at + __popcll(bal & lanemask_lt())] = (uint16_t)(threadIdx.x | (uint32_t)(k - k0) << 8);
            }
            __syncthreads();
            const uint32_t n = s_n;
            for (uint32_t i = threadIdx.x; i < n; i += kNT) {
                const uint32_t e = s_pair[i];
                const SliceRec& P = S[e & 0xffu];
                const int k = k0 + (int)(e >> 8);
                if (!slice_rows(s, P, k, icell)) slice_cells(s, P, k);
            }
            __syncthreads();
        }
    }
}

// Disc robots against a map: thread per query.
__global__ __launch_bounds__(kNT) void k_disc_collision(DiscArgs d) {
    for (int64_t q = blockIdx.x * (int64_t)kNT + threadIdx.x; q < d.n; q += (int64_t)gridDim.x * kNT)
        d.out[q] = disc_hits(d.map, d.x0, d.y0, d.cell, d.nx, d.ny, d.xy[2 * q], d.xy[2 * q + 1], d.radius) ? 1 : 0;
}

}  // namespace

void launch_disc_collision(const DiscArgs& d, hipStream_t st) {
    if (d.n == 0) return;
    const int64_t blocks = (d.n + kNT - 1) / kNT;
    k_disc_collision<<<(unsigned)(blocks < 4096 ? blocks : 4096), kNT, 0, st>>>(d);
}

void launch_slice(const SliceArgs& a, hipStream_t st) {
    const size_t plane = (size_t)a.nx * a.ny;
    SliceArgs b = a;
    b.low = *std::min_element(a.heights, a.heights + a.n_planes);
    b.high = *std::max_element(a.heights, a.heights + a.n_planes);
    b.reach = 2.0 * std::log(1.0 / a.rho_min) * (1.0 + 2e-6);
    k_fill_zero<<<1024, kNT, 0, st>>>(a.occ, a.occ ? a.n_planes * plane : 0, a.map, a.map ? plane : 0);
    if (a.n) k_slice<<<2048, kNT, 0, st>>>(b);
}

}  // namespace hgs
