// Image helpers for learned-LOD labels and PSNR: 2x2 box downsampling of a
// planar RGB image, and mean squared error of many image windows against
// crops of reference images.  FP64 sums in a fixed order.
#include "device_util.h"
#include "internal.h"

namespace hgs {

namespace {

// Streaming copy (the bandwidth probe): each workgroup copies contiguous
// chunks of 4 KiB per step -- four 16-byte nontemporal loads per thread in
// flight, then four nontemporal stores -- and the grid strides over the
// chunks.  (Measured on MI355X: 5.9 TB/s read + write; a grid-stride loop
// over single 16-byte words reached 4.2-4.8, a D2D hipMemcpy 5.1.)
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_stream_copy(const v4u* __restrict__ src, v4u* __restrict__ dst, size_t n16) {
    constexpr size_t kPer = 256 * 4;
    for (size_t base = blockIdx.x * kPer; base < n16; base += (size_t)gridDim.x * kPer) {
        v4u v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t i = base + u * 256 + threadIdx.x;
            if (i < n16) v[u] = __builtin_nontemporal_load(&src[i]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t i = base + u * 256 + threadIdx.x;
            if (i < n16) __builtin_nontemporal_store(v[u], &dst[i]);
        }
    }
}

__global__ void k_downsample2x(const float* __restrict__ src, int W, int H, float* __restrict__ dst) {
    const size_t plane = (size_t)W * H, splane = 4 * plane;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < 3 * plane; i += (size_t)gridDim.x * blockDim.x) {
        const size_t c = i / plane, r = i % plane;
        const int y = (int)(r / W), x = (int)(r % W);
        const float* s = src + c * splane + (size_t)(2 * y) * (2 * W) + 2 * x;
        dst[i] = 0.25f * ((s[0] + s[1]) + (s[2 * W] + s[2 * W + 1]));
    }
}

// Squared differences of a region are summed in chunks of whole image rows
// (RegionDev::rows of the 3 h channel rows each), one workgroup per chunk:
// the sum reads every pixel once, so it is bound by HBM, and one workgroup
// per region left the card idle on whole images (16 learned 1280 x 720
// renders with their errors: 8.62 ms, 6.94 of it here, with one workgroup
// per region and a 64-bit division per element; 1.61 ms in chunks).  Within
// a workgroup the lanes of a row sit next to each other, a power of two of
// them up to a wave, so that narrow windows still fill the workgroup and no
// index is divided.  Rows are read 16 bytes per lane where both images' rows
// allow it (RegionDev::vec).  FP64 sums in a fixed order.
__device__ __forceinline__ double sq_diff(float a, float b) {
    const double d = (double)a - (double)b;
    return d * d;
}

// Sum over channel rows [q0, q1) of r, in every thread (sh: 256 doubles).
__device__ double region_rows(const RegionDev& r, int64_t q0, int64_t q1, double* sh) {
    const size_t rplane = (size_t)r.ref_w * r.ref_h;
    const int units = r.vec ? r.w / 4 : r.w;                 // loads per row
    int lanes = 1;
    while (lanes < units && lanes < kWave) lanes <<= 1;
    const int per = 256 / lanes;                              // rows in flight
    const int x0 = (int)threadIdx.x & (lanes - 1);
    double acc = 0.0;
    for (int64_t q = q0 + (int)threadIdx.x / lanes; q < q1; q += per) {
        const int c = (q >= r.h ? 1 : 0) + (q >= 2 * (int64_t)r.h ? 1 : 0);
        const int64_t y = q - (int64_t)c * r.h;
        const float* a = r.img + (size_t)q * r.w;
        const float* b = r.ref + (size_t)c * rplane + (size_t)(r.y0 + y) * r.ref_w + r.x0;
        if (r.vec) {
            const float4* a4 = reinterpret_cast<const float4*>(a);
            const float4* b4 = reinterpret_cast<const float4*>(b);
#pragma unroll 4
            for (int x = x0; x < units; x += lanes) {
                const float4 u = a4[x], v = b4[x];
                acc += (sq_diff(u.x, v.x) + sq_diff(u.y, v.y)) + (sq_diff(u.z, v.z) + sq_diff(u.w, v.w));
            }
        } else {
#pragma unroll 4
            for (int x = x0; x < units; x += lanes) acc += sq_diff(a[x], b[x]);
        }
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    const double sum = sh[0];
    __syncthreads();
    return sum;
}

__device__ __forceinline__ float mse_of(const RegionDev& r, double sum) {
    return (float)(sum / (3.0 * ((double)r.w * (double)r.h)));
}

// Expand-vs-keep label from the errors of the window with the node refined
// (the threshold cut) and with its subtree collapsed to it, against the same
// reference crop: the window's PSNR drop from keeping the node, 10
// log10(MSE_kept / MSE_refined) with both MSEs floored at 1e-10, labels
// "refine" when it exceeds label_db.
__device__ __forceinline__ void put_label(uint32_t i, float refined, float kept, double label_db,
                                          float* __restrict__ labels, float* __restrict__ drop_db) {
    const double a = fmax((double)refined, 1e-10), b = fmax((double)kept, 1e-10);
    const double drop = 10.0 * log10(b / a);
    if (drop_db) drop_db[i] = (float)drop;
    labels[i] = drop > label_db ? 1.f : 0.f;
}

// Every region is one chunk: a workgroup per candidate (regions 2i, 2i + 1).
__global__ __launch_bounds__(256) void k_lod_labels(const RegionDev* __restrict__ reg, double label_db,
                                                    float* __restrict__ labels, float* __restrict__ drop_db) {
    __shared__ double sh[256];
    const RegionDev r = reg[2 * (size_t)blockIdx.x], k = reg[2 * (size_t)blockIdx.x + 1];
    const double sr = region_rows(r, 0, 3 * (int64_t)r.h, sh);
    const double sk = region_rows(k, 0, 3 * (int64_t)k.h, sh);
    if (threadIdx.x == 0) put_label(blockIdx.x, mse_of(r, sr), mse_of(k, sk), label_db, labels, drop_db);
}

// Every region is one chunk: a workgroup per region.
__global__ __launch_bounds__(256) void k_region_mse(const RegionDev* __restrict__ reg, float* __restrict__ out) {
    __shared__ double sh[256];
    const RegionDev r = reg[blockIdx.x];
    const double sum = region_rows(r, 0, 3 * (int64_t)r.h, sh);
    if (threadIdx.x == 0) out[blockIdx.x] = mse_of(r, sum);
}

// Workgroup b: chunk b - blk0 of the region whose chunks hold b.
__global__ __launch_bounds__(256) void k_region_chunks(const RegionDev* __restrict__ reg, int n,
                                                       double* __restrict__ part) {
    __shared__ double sh[256];
    int lo = 0, hi = n;                                       // reg[lo].blk0 <= b < reg[hi].blk0
    while (hi - lo > 1) {
        const int mid = lo + (hi - lo) / 2;
        if (reg[mid].blk0 <= blockIdx.x) lo = mid; else hi = mid;
    }
    const RegionDev r = reg[lo];
    const int64_t q0 = (int64_t)(blockIdx.x - r.blk0) * r.rows, q1 = min(q0 + r.rows, 3 * (int64_t)r.h);
    const double sum = region_rows(r, q0, q1, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = sum;
}

// A region's chunks summed by one wave: lane l takes chunks l, l + 64, ...
__device__ __forceinline__ float region_total(const RegionDev& r, const double* __restrict__ part) {
    const uint32_t chunks = (uint32_t)((3 * (int64_t)r.h + r.rows - 1) / r.rows);
    double s = 0.0;
    for (uint32_t k = lane_id(); k < chunks; k += kWave) s += part[r.blk0 + k];
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) s += __shfl_xor(s, d, kWave);
    return mse_of(r, s);
}

__global__ __launch_bounds__(kWave) void k_region_finish(const RegionDev* __restrict__ reg,
                                                         const double* __restrict__ part, float* __restrict__ out) {
    const float m = region_total(reg[blockIdx.x], part);
    if (threadIdx.x == 0) out[blockIdx.x] = m;
}

__global__ __launch_bounds__(kWave) void k_labels_finish(const RegionDev* __restrict__ reg,
                                                         const double* __restrict__ part, double label_db,
                                                         float* __restrict__ labels, float* __restrict__ drop_db) {
    const float refined = region_total(reg[2 * (size_t)blockIdx.x], part);
    const float kept = region_total(reg[2 * (size_t)blockIdx.x + 1], part);
    if (threadIdx.x == 0) put_label(blockIdx.x, refined, kept, label_db, labels, drop_db);
}

}  // namespace

void launch_stream_copy(const void* src, void* dst, size_t bytes, hipStream_t s) {
    k_stream_copy<<<256 * 32, 256, 0, s>>>(static_cast<const v4u*>(src), static_cast<v4u*>(dst), bytes / 16);
}

void launch_downsample2x(const float* src, int W, int H, float* dst, hipStream_t s) {
    const size_t n = 3 * (size_t)W * H;
    const int grid = (int)std::min<size_t>(4096, (n + 255) / 256);
    k_downsample2x<<<grid > 0 ? grid : 1, 256, 0, s>>>(src, W, H, dst);
}

// Elements of a region per chunk, about: 64 per thread, enough to cover the
// chunk's start-up, and a whole 720p image still makes 180 chunks.
constexpr int64_t kRegionChunk = 16384;

uint32_t plan_regions(RegionDev* reg, int64_t n) {
    // at most 256 chunks per region, fewer when the regions are so many that
    // the chunks would outnumber a grid
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>(256, (1ll << 30) / std::max<int64_t>(n, 1)));
    uint32_t blk = 0;
    for (int64_t i = 0; i < n; ++i) {
        RegionDev& r = reg[i];
        const int64_t rows = 3 * (int64_t)r.h;
        r.rows = std::max<int64_t>(std::max<int64_t>(1, kRegionChunk / r.w), (rows + most - 1) / most);
        r.blk0 = blk;
        // every row of both images starts on 16 bytes
        const uintptr_t at = reinterpret_cast<uintptr_t>(r.img) | reinterpret_cast<uintptr_t>(r.ref);
        r.vec = (r.w % 4 == 0 && r.ref_w % 4 == 0 && r.x0 % 4 == 0 && at % 16 == 0) ? 1u : 0u;
        blk += (uint32_t)((rows + r.rows - 1) / r.rows);
    }
    return blk;
}

void launch_region_mse(const RegionDev* reg, int n, uint32_t chunks, double* part, float* out, hipStream_t s) {
    if (n <= 0) return;
    if (chunks == (uint32_t)n) {
        k_region_mse<<<n, 256, 0, s>>>(reg, out);
        return;
    }
    k_region_chunks<<<chunks, 256, 0, s>>>(reg, n, part);
    k_region_finish<<<n, kWave, 0, s>>>(reg, part, out);
}

void launch_lod_labels(const RegionDev* reg, int n, uint32_t chunks, double* part, double label_db, float* labels,
                       float* drop_db, hipStream_t s) {
    if (n <= 0) return;
    if (chunks == 2u * (uint32_t)n) {
        k_lod_labels<<<n, 256, 0, s>>>(reg, label_db, labels, drop_db);
        return;
    }
    k_region_chunks<<<chunks, 256, 0, s>>>(reg, 2 * n, part);
    k_labels_finish<<<n, kWave, 0, s>>>(reg, part, label_db, labels, drop_db);
}

}  // namespace hgs
