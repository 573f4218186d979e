// Stable LSD radix sort of 32-bit (key, value) pairs for wave64.
//
// A sort over `bits` key bits runs ceil(bits / D) passes with digits of
// ceil(bits / passes) bits, D the widest digit allowed (6..11: up to 2048
// buckets), so a 17-bit tile key takes two or three passes and a 32-bit depth
// key three to six.  The input is cut into groups (group_size); a workgroup
// takes groups b, b + G, b + 2G, ... so that the groups in flight at any moment
// form one contiguous window of the input and each digit's output advances as
// one front (writes of neighbouring groups land next to each other and fill
// whole cache lines).  Each pass is two launches with no inter-workgroup
// waiting:
//   upsweep   : the digit histogram of every group (LDS atomics into
//               per-wave histograms), also added to the sums of its 16 and
//               of its 256 neighbours;
//   downsweep : a group adds up what lies before it (whole 256s, then 16s,
//               then groups: some 25 reads per digit), then is ranked stably
//               sub-tile by sub-tile -- lanes with equal digits are found by
//               ballots over the digit bits, per-wave counters live in LDS --
//               and its keys and values are scattered.
// Element counts live in device memory so the launches can be captured in a
// graph.
#include "device_util.h"
#include "internal.h"

namespace hgs {

namespace {

constexpr int kNT = 256;
constexpr int kNW = kNT / kWave;
static_assert(kSortGroup % (kNT * 16) == 0, "a group holds whole sub-tiles of every width");

__device__ __forceinline__ uint32_t n_of(const uint32_t* count, uint32_t cap) {
    const uint32_t n = *count;
    return n < cap ? n : cap;
}

// Elements per histogram group of an n-element sort.  A pass over few
// elements is one sub-tile's latency (load, rank, place, store) per sub-tile
// that a workgroup takes, so sorts below 512 groups of kSortGroup get smaller
// groups of one sub-tile each, the smallest that keep their number at 512,
// two workgroups per compute unit; larger sorts take the smallest multiple of
// kSortGroup with at most kSortMaxGroups groups.  (A 20,000-element pass in
// three groups of 8,192: 17.4 us of downsweep; a blocking 256 x 256 render of
// a 20,000-Gaussian box 236 -> 165 us with groups of 1,024, a 700,000-entry
// backward step 1.49 -> 1.40 ms.)
constexpr uint32_t kSmallGroups = 512;
__device__ __forceinline__ uint32_t group_size(uint32_t n) {
    if (n <= kSmallGroups * 1024u) return 1024u;
    if (n <= kSmallGroups * 2048u) return 2048u;
    if (n <= kSmallGroups * 4096u) return 4096u;
    const uint32_t per = ceil_div(n, (uint32_t)kSortGroup * (uint32_t)kSortMaxGroups);
    return (per > 1u ? per : 1u) * (uint32_t)kSortGroup;
}
static_assert(kSortMaxGroups >= (int)kSmallGroups && kSortGroup >= 4096, "small sorts have at most kSmallGroups groups");

// Lanes of the wave (among `active`) whose DB-bit digit equals this lane's.
template <int DB>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, uint64_t active) {
    uint64_t m = active;
#pragma unroll
    for (int b = 0; b < DB; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bal = __ballot(bit);
        m &= bit ? bal : ~bal;
    }
    return m;
}

// Rows of NB counts: one per group, then (bins) one per 16 groups and one
// per 256 groups.  Two sets of bins take turns: a pass's upsweep clears the
// other set for the next pass, and the first pass finds its set cleared
// (sort_bins).
struct HistDev {
    uint32_t* group;
    uint32_t* b16;
    uint32_t* b256;
};

// Digit histogram of every group the block owns: per-wave LDS histograms
// take one atomic add per key (counts do not depend on order), four keys per
// thread and step with 16-byte loads (groups start at multiples of 1,024).
template <int DB>
__global__ __launch_bounds__(kNT) void k_upsweep(const uint32_t* __restrict__ keys, const uint32_t* count,
                                                 uint32_t cap, int shift, uint32_t MASK, HistDev H, SortBins next) {
    constexpr int NB = 1 << DB;
    __shared__ uint32_t h[kNW][NB];
    const int t = threadIdx.x;
    uint32_t* hw = h[t / kWave];
    const uint32_t n = n_of(count, cap);
    const uint32_t gs = group_size(n), ng = ceil_div(n, gs);
    for (uint32_t i = blockIdx.x * kNT + t; i < next.n; i += gridDim.x * kNT) next.words[i] = 0;
    for (uint32_t g = blockIdx.x; g < ng; g += gridDim.x) {
        for (int i = t; i < NB; i += kNT) {
#pragma unroll
            for (int w = 0; w < kNW; ++w) h[w][i] = 0;
        }
        __syncthreads();
        const uint32_t lo = g * gs;
        const uint32_t hi = min(lo + gs, n);
        uint32_t base = lo;
        for (; base + 4 * kNT <= hi; base += 4 * kNT) {
            const uint4 k4 = *reinterpret_cast<const uint4*>(keys + base + 4 * t);
            atomicAdd(&hw[(k4.x >> shift) & MASK], 1u);
            atomicAdd(&hw[(k4.y >> shift) & MASK], 1u);
            atomicAdd(&hw[(k4.z >> shift) & MASK], 1u);
            atomicAdd(&hw[(k4.w >> shift) & MASK], 1u);
        }
        for (uint32_t i = base + t; i < hi; i += kNT) atomicAdd(&hw[(keys[i] >> shift) & MASK], 1u);
        __syncthreads();
        for (int i = t; i < NB; i += kNT) {
            uint32_t c = 0;
#pragma unroll
            for (int w = 0; w < kNW; ++w) c += h[w][i];
            H.group[(size_t)g * NB + i] = c;
            if (c) {
                atomicAdd(H.b16 + (size_t)(g / 16) * NB + i, c);
                atomicAdd(H.b256 + (size_t)(g / 256) * NB + i, c);
            }
        }
        __syncthreads();
    }
}

// Keys of more than 32 bits, the ones above `low` in the cut: the first pass
// (digit bits [0, digit)) drops the bits it has sorted by and sets those of
// the value's entry above what is left.  (The values are still almost in
// entry order, so these reads hit: 38 M entries of 96 views add 130 us to the
// pass.  A pass of its own on the entries' views, gathered in depth order,
// cost 717 us for the gather; the digits are the same in number.)
struct TopBits {
    const uint2* src;
    int low, digit;
    __device__ __forceinline__ uint32_t at(uint32_t val, uint32_t n) const {
        const uint32_t e = val & kEntryMask;
        return e < n ? src[e].y : 0u;
    }
    __device__ __forceinline__ uint32_t key(uint32_t k, uint32_t t) const {
        return ((low < 32 ? k & ((1u << low) - 1u) : k) >> digit) | t << (low - digit);
    }
};

// Downsweep with a local reorder: each sub-tile of kItems * kNT elements is
// ranked (stable within the sub-tile), placed in LDS in digit order, then
// written out in that order so that consecutive lanes store consecutive
// addresses of one digit's run.
template <int DB, int ITEMS>
struct DownShared {
    static constexpr int NB = 1 << DB;
    uint32_t start[NB];                     // first output position of digit d
    uint32_t off[NB];                       // global position of the next element of digit d
    uint32_t loc[NB];                       // start of digit d inside the staged sub-tile
    uint32_t cnt[kNW][NB];
    uint32_t scan[kNW + 1];
    uint32_t key[kNT * ITEMS];
    uint32_t val[kNT * ITEMS];
};

// The groups of this workgroup in sub-tiles of ITEMS elements per thread.
template <int DB, int ITEMS, bool TOP, class SH>
__device__ __forceinline__ void downsweep_groups(SH& S, const uint32_t* __restrict__ kin,
                                                 const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
                                                 uint32_t* __restrict__ vout, uint32_t n, uint32_t gs, uint32_t ng,
                                                 int shift, uint32_t MASK, const HistDev& H, const TopBits& top) {
    constexpr int NB = 1 << DB;
    constexpr int PER = NB / kNT > 0 ? NB / kNT : 1;      // digits per thread
    constexpr uint32_t SUB = kNT * ITEMS;
    const int t = threadIdx.x;
    const int w = t / kWave, l = lane_id();
    for (uint32_t g = blockIdx.x; g < ng; g += gridDim.x) {
        __syncthreads();
        // elements of each digit in the groups before this one, the rows
        // dealt to kNT / NB slices of threads when the digits are fewer
        {
            const uint32_t q256 = g / 256, q16 = g / 16;
            constexpr int SL = NB < kNT ? kNT / NB : 1;
            static_assert(SL <= kNW, "a count row per slice");
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int d = NB < kNT ? t % NB : t + k * kNT;
                const uint32_t sl = NB < kNT ? t / NB : 0;
                uint32_t c = 0;
#pragma unroll 4
                for (uint32_t r = sl; r < q256; r += SL) c += H.b256[(size_t)r * NB + d];
#pragma unroll 4
                for (uint32_t r = 16 * q256 + sl; r < q16; r += SL) c += H.b16[(size_t)r * NB + d];
#pragma unroll 4
                for (uint32_t r = 16 * q16 + sl; r < g; r += SL) c += H.group[(size_t)r * NB + d];
                S.cnt[sl][d] = c;
            }
            __syncthreads();
            for (int d = t; d < NB; d += kNT) {
                uint32_t c = S.start[d];
#pragma unroll
                for (int q = 0; q < SL; ++q) c += S.cnt[q][d];
                S.off[d] = c;
            }
            __syncthreads();
        }
        const uint32_t lo = g * gs;
        const uint32_t hi = min(lo + gs, n);
        for (uint32_t base = lo; base < hi; base += SUB) {
            for (int i = t; i < NB; i += kNT) {
#pragma unroll
                for (int k = 0; k < kNW; ++k) S.cnt[k][i] = 0;
            }
            __syncthreads();
            uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
            const uint32_t seg = base + (uint32_t)w * (kWave * ITEMS);
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) {
                const uint32_t i = seg + r * kWave + l;
                const bool valid = i < hi;
                key[r] = valid ? kin[i] : 0u;
                val[r] = valid ? vin[i] : 0u;
            }
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) {
                const uint32_t i = seg + r * kWave + l;
                const bool valid = i < hi;
                const uint32_t d = (key[r] >> shift) & MASK;
                const uint64_t act = __ballot(valid);
                const uint64_t peers = match_digit<DB>(d, act);
                const uint64_t below = peers & lanemask_lt();
                uint32_t before = 0;
                if (valid) before = S.cnt[w][d];
                rank[r] = before + (uint32_t)__popcll(below);
                if (valid && below == 0) S.cnt[w][d] = before + (uint32_t)__popcll(peers);
            }
            __syncthreads();
            // per digit: local start of each wave's run inside the sub-tile
            {
                uint32_t mine[PER];
                uint32_t sum = 0;
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    const int d = t * PER + k;
                    uint32_t c = 0;
                    if (d < NB) {
#pragma unroll
                        for (int q = 0; q < kNW; ++q) c += S.cnt[q][d];
                    }
                    mine[k] = c;
                    sum += c;
                }
                uint32_t tot;
                uint32_t ex = block_excl_scan<kNT>(sum, S.scan, &tot);
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    const int d = t * PER + k;
                    if (d < NB) {
                        S.loc[d] = ex;
                        uint32_t run = ex;
#pragma unroll
                        for (int q = 0; q < kNW; ++q) {
                            const uint32_t c = S.cnt[q][d];
                            S.cnt[q][d] = run;
                            run += c;
                        }
                    }
                    ex += mine[k];
                }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) {
                const uint32_t i = seg + r * kWave + l;
                if (i < hi) {
                    const uint32_t d = (key[r] >> shift) & MASK;
                    const uint32_t p = S.cnt[w][d] + rank[r];
                    S.key[p] = key[r];
                    S.val[p] = val[r];
                }
            }
            __syncthreads();
            const uint32_t n_sub = (hi - base) < SUB ? (hi - base) : SUB;
            uint32_t over[TOP ? ITEMS : 1];       // (loaded together)
            if constexpr (TOP) {
#pragma unroll
                for (int r = 0; r < ITEMS; ++r) {
                    const uint32_t p = t + r * kNT;
                    over[r] = p < n_sub ? top.at(S.val[p], n) : 0u;
                }
            }
#pragma unroll (TOP ? ITEMS : 1)
            for (int r = 0; r < ITEMS; ++r) {
                const uint32_t p = t + r * kNT;
                if (p >= n_sub) break;
                const uint32_t k = S.key[p];
                const uint32_t d = (k >> shift) & MASK;
                const uint32_t pos = S.off[d] + (p - S.loc[d]);
                kout[pos] = TOP ? top.key(k, over[TOP ? r : 0]) : k;
                vout[pos] = S.val[p];
            }
            if (base + SUB >= hi) break;
            __syncthreads();
            // advance each digit's global position by its count in this sub-tile
            for (int d = t; d < NB; d += kNT) {
                const uint32_t next = (d + 1 < NB) ? S.loc[d + 1] : n_sub;
                S.off[d] += next - S.loc[d];
            }
            __syncthreads();
        }
    }
}

// (Four waves per SIMD, as many as the LDS of 8-bit digits allows: the
// registers are capped at that.)
template <int DB, int ITEMS, bool TOP>
__global__ __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(DB <= 8 ? 4 : 2)))
void k_downsweep(const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
                 uint32_t* __restrict__ vout, const uint32_t* count, uint32_t cap, int shift, uint32_t MASK, HistDev H,
                 TopBits top) {
    constexpr int NB = 1 << DB;
    constexpr int PER = NB / kNT > 0 ? NB / kNT : 1;      // digits per thread
    static_assert(kSortGroup % (kNT * ITEMS) == 0, "whole sub-tiles per group");
    __shared__ DownShared<DB, ITEMS> S;
    const int t = threadIdx.x;
    const uint32_t n = n_of(count, cap);
    const uint32_t gs = group_size(n), ng = ceil_div(n, gs);
    if (blockIdx.x >= ng) return;
    {
        uint32_t mine[PER];
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int d = t * PER + k;
            mine[k] = 0;
            if (d < NB) {
#pragma unroll 4
                for (uint32_t r = 0; r < ceil_div(ng, 256u); ++r) mine[k] += H.b256[(size_t)r * NB + d];
            }
            sum += mine[k];
        }
        uint32_t tot;
        uint32_t ex = block_excl_scan<kNT>(sum, S.scan, &tot);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int d = t * PER + k;
            if (d < NB) S.start[d] = ex;
            ex += mine[k];
        }
    }
    // small groups in one sub-tile of fewer elements per thread
    if (gs == 1024u)
        downsweep_groups<DB, 4, TOP>(S, kin, vin, kout, vout, n, gs, ng, shift, MASK, H, top);
    else if (ITEMS > 8 && gs == 2048u)
        downsweep_groups<DB, 8, TOP>(S, kin, vin, kout, vout, n, gs, ng, shift, MASK, H, top);
    else
        downsweep_groups<DB, ITEMS, TOP>(S, kin, vin, kout, vout, n, gs, ng, shift, MASK, H, top);
}

// Rows of bins for a sort of at most `cap` elements.
struct BinRows {
    uint32_t r16, r256;
};
BinRows bin_rows(uint32_t cap) {
    // groups: at most kSmallGroups up to kSmallGroups * kSortGroup elements
    const uint64_t g = std::min<uint64_t>(std::max<uint64_t>(kSmallGroups, ((uint64_t)cap + kSortGroup - 1) / kSortGroup),
                                          (uint64_t)kSortMaxGroups);
    return {(uint32_t)((g + 15) / 16), (uint32_t)((g + 255) / 256)};
}

// One pass over digit bits [shift, shift + nbits) (nbits <= DB), pass number
// p of the sort.
template <int DB>
void pass(const SortArgs& a, int cur, int shift, int nbits, int p, bool last, hipStream_t s) {
    const int G = kSortBlocks;
    constexpr uint32_t NB = 1u << DB;
    const BinRows rows = bin_rows(a.cap);
    const size_t set = sort_bin_words(a.hist_stride) / 2;
    uint32_t* bins = a.hist + (size_t)kSortBins * a.hist_stride;
    HistDev H;
    H.group = a.hist;
    H.b16 = bins + (p & 1) * set;
    H.b256 = H.b16 + (size_t)rows.r16 * NB;
    const SortBins next = {bins + ((p + 1) & 1) * set, last ? 0u : (rows.r16 + rows.r256) * NB};
    const uint32_t mask = nbits >= 32 ? 0xffffffffu : ((1u << nbits) - 1u);
    k_upsweep<DB><<<G, kNT, 0, s>>>(a.keys[cur], a.count, a.cap, shift, mask, H, next);
    constexpr int ITEMS = DB <= 8 ? 16 : 8;
    auto down = p == 0 && a.top ? k_downsweep<DB, ITEMS, true> : k_downsweep<DB, ITEMS, false>;
    down<<<G, kNT, 0, s>>>(a.keys[cur], a.vals[cur], a.keys[cur ^ 1], a.vals[cur ^ 1], a.count, a.cap, shift, mask, H,
                           TopBits{a.top, a.low_bits, nbits});
}

// Passes over key_bits bits and the digit width (at least 6) of each.
int plan_passes(const SortArgs& a, int* digit_bits) {
    const int maxdb = a.max_digit_bits < 6 ? 6 : (a.max_digit_bits > 11 ? 11 : a.max_digit_bits);
    const int passes = (a.key_bits + maxdb - 1) / maxdb;
    const int db = (a.key_bits + passes - 1) / passes;
    *digit_bits = db;
    return passes;
}

}  // namespace

SortBins sort_bins(const SortArgs& a) {
    int db;
    (void)plan_passes(a, &db);
    const BinRows rows = bin_rows(a.cap);
    return {a.hist + (size_t)kSortBins * a.hist_stride, (rows.r16 + rows.r256) << std::max(db, 6)};
}

bool wide_sort_fits(const SortArgs& a) {
    int db;
    return plan_passes(a, &db) > 1 && db < a.low_bits && a.key_bits - db <= 32;
}

int launch_sort(const SortArgs& a, hipStream_t s) {
    int db;
    const int passes = plan_passes(a, &db);
    int cur = 0, shift = 0;
    for (int p = 0; p < passes; ++p) {
        // the last pass may cover fewer bits: its mask drops key bits above key_bits
        const int nbits = std::min(a.key_bits - p * db, db);
        const bool last = p == passes - 1;
        switch (db) {
            case 1: case 2: case 3: case 4: case 5: case 6: pass<6>(a, cur, shift, nbits, p, last, s); break;
            case 7: pass<7>(a, cur, shift, nbits, p, last, s); break;
            case 8: pass<8>(a, cur, shift, nbits, p, last, s); break;
            case 9: pass<9>(a, cur, shift, nbits, p, last, s); break;
            case 10: pass<10>(a, cur, shift, nbits, p, last, s); break;
            default: pass<11>(a, cur, shift, nbits, p, last, s); break;
        }
        if (p > 0 || !a.top) shift += db;              // (top: the first pass drops its digit)
        cur ^= 1;
    }
    return cur;
}

}  // namespace hgs
