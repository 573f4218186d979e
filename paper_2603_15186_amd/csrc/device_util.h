// Wave64 and workgroup primitives for gfx950: prefix sums over wavefronts
// and blocks.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace hgs {

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ uint64_t lanemask_lt() {
    const int l = lane_id();
    return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// x of the lane CTRL names, 0 where it names none or the row is masked out.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
}

// Prefix sums in the vector pipeline: shifts by 1, 2, 4 and 8 within the rows
// of 16 lanes, then lane 15 of a row onto the next row (rows 1 and 3) and
// lane 31 onto rows 2 and 3.  (Lane shifts through LDS cost some 60 cycles
// each of the six steps.)  Every lane of the wave takes part.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
    x += dpp_or_zero<0x111, 0xf>(x);       // row_shr:1
    x += dpp_or_zero<0x112, 0xf>(x);       // row_shr:2
    x += dpp_or_zero<0x114, 0xf>(x);       // row_shr:4
    x += dpp_or_zero<0x118, 0xf>(x);       // row_shr:8
    x += dpp_or_zero<0x142, 0xa>(x);       // row_bcast:15
    x += dpp_or_zero<0x143, 0xc>(x);       // row_bcast:31
    return x;
}

// Sum over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(x), kWave - 1);
}

// 1 / x and 1 / sqrt(x) in FP64 for positive normal x: the hardware's
// estimates (23 bits or more) and one step of Householder's third-order
// iteration, whose error is the cube of the estimate's; the last roundings
// remain: 0.50 ulp for 1 / x, 0.97 for 1 / sqrt(x) (the two IEEE operations:
// 1.44).  The IEEE sequences, which also serve every other x, are 12 to 20
// instructions, these 4 and 6.
__device__ __forceinline__ double rcp64(double x) {
    const double y = __builtin_amdgcn_rcp(x), e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}
__device__ __forceinline__ double rsqrt64(double x) {
    const double y = __builtin_amdgcn_rsq(x), e = fma(-(x * y), y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// The same with x y held in two parts: 0.50 ulp, two instructions more.
__device__ __forceinline__ double rsqrt64_near(double x) {
    const double y = __builtin_amdgcn_rsq(x), h = x * y;
    const double e = fma(-fma(x, y, -h), y, fma(-h, y, 1.0));
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// Exclusive scan over a block of NT threads; returns the thread's exclusive
// prefix and writes the block total to *total.  `sh` holds NT/64 + 1 words.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t* sh, uint32_t* total) {
    constexpr int NW = NT / kWave;
    const int w = threadIdx.x / kWave, l = lane_id();
    uint32_t inc = wave_incl_scan(x);
    if (l == kWave - 1) sh[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int i = 0; i < NW; ++i) { uint32_t t = sh[i]; sh[i] = run; run += t; }
        sh[NW] = run;
    }
    __syncthreads();
    uint32_t r = sh[w] + inc - x;
    *total = sh[NW];
    __syncthreads();
    return r;
}

template <int NT>
__device__ __forceinline__ uint4 block_excl_scan4(uint4 x, uint4* sh, uint4* total) {
    constexpr int NW = NT / kWave;
    const int w = threadIdx.x / kWave, l = lane_id();
    const uint4 inc = make_uint4(wave_incl_scan(x.x), wave_incl_scan(x.y), wave_incl_scan(x.z), wave_incl_scan(x.w));
    if (l == kWave - 1) sh[w] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint4 run = make_uint4(0, 0, 0, 0);
        for (int i = 0; i < NW; ++i) {
            const uint4 t = sh[i];
            sh[i] = run;
            run.x += t.x; run.y += t.y; run.z += t.z; run.w += t.w;
        }
        sh[NW] = run;
    }
    __syncthreads();
    const uint4 r = make_uint4(sh[w].x + inc.x - x.x, sh[w].y + inc.y - x.y, sh[w].z + inc.z - x.z,
                               sh[w].w + inc.w - x.w);
    *total = sh[NW];
    __syncthreads();
    return r;
}

// The pass's pairs to the host (one thread of a kernel that runs on): a store
// that the next kernels do not wait for, where a copy and its event would put
// off a render by 2 to 8 us.  (Not from the emission: under its traffic the
// store takes 10 us, which its workgroup waits for: 160 -> 173 us for 16 views.)
template <class Report>
__device__ __forceinline__ void report_pairs(const Report& r, uint32_t pairs, uint32_t need) {
    __hip_atomic_store(r.host, (unsigned long long)r.epoch << 32 | (pairs > need ? pairs : need), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

__host__ __device__ __forceinline__ uint32_t ceil_div(uint32_t a, uint32_t b) { return (a + b - 1) / b; }

}  // namespace hgs
