// The depth sort: every view's items ordered by their 32-bit depth key (the
// float bits of camera Z, which order like unsigned integers for positive
// values), equal depths by ascending point index (Sec. 3.2: points sorted by
// z-distance).
//
// A stable LSD radix sort of three passes.  The digits are of the distance of a
// key from the view's smallest, as wide as the view's depth range needs (the
// range's bits over three, at most 11): the depths of one view mostly span few
// octaves, so three 8- or 9-bit digits do where the full 32 bits took four.
// Dropped items (key 0xFFFFFFFF) count as one past the largest.
//
// Launches: k_sort_hist (the view's range, and the view's totals of all three
// digits, which no pass changes) and one k_sort_pass per digit.  A pass ranks a
// block of 8192 keys wave by wave in LDS, publishes the block's digit counts,
// and adds up those of the view's earlier blocks as they appear, so no separate
// histogram launch runs per pass.  A block takes its place in the view by a
// ticket and publishes before it waits, and it waits only for blocks with
// earlier tickets, which have therefore started: every wait ends.  A count and
// its "present" bit are one word, so no ordering between words is needed.
// Views of up to one block's keys are sorted in LDS by one launch in all.
//
// Bound by the ranking's serial rounds and by launches, not by memory: the 1.2M
// keys of four views of 300k points (29 MB a pass at most) take 62 us, the range
// and totals 9 and a pass 17 to 18; four passes of a histogram and a scatter
// launch took 96.  4096 keys in one launch take 28 us, against 50.
//
// Scratch: the view's part of the binning records, which are written after the
// sort (8 words per item): the depth range of each 64 points (written by the
// projection, which also clears the totals and tickets), the sort's parameters, and in views of more than one
// block the digit totals, tickets and published counts.
#include "dpr_internal.h"

namespace dpr {

constexpr int kSortWaves = kDepthSortThreads / 64;
constexpr int kSortItems = kDepthSortTile / kDepthSortThreads;       // keys per thread
constexpr uint32_t kPresent = 0x80000000u;
static_assert(kSortPasses == 3, "an odd number of passes ends in the other buffer");
static_assert(kDepthSortThreads == 1024 && kSortMaxBins == 2 * kDepthSortThreads, "at most two digits per thread");

struct SortParams {
    uint32_t kmin, top, bits;   // distance of a key: min(key - kmin, top); bits per digit
};

__device__ __forceinline__ SortParams sort_params(uint32_t lo, uint32_t hi) {
    SortParams p;
    p.kmin = lo;
    p.top = hi >= lo ? hi - lo + 1u : 1u;                 // no key at all: every item is a dropped one
    p.bits = (32u - (uint32_t)__clz(p.top) + kSortPasses - 1u) / kSortPasses;
    return p;
}

__device__ __forceinline__ uint32_t sort_digit(const SortParams &p, uint32_t key, int pass) {
    const uint32_t d = key == kDroppedKey ? p.top : key - p.kmin;
    return (d >> (pass * p.bits)) & ((1u << p.bits) - 1u);
}

struct SortLds {
    uint32_t keys[kDepthSortTile], vals[kDepthSortTile];
    uint16_t wcnt[kSortWaves][kSortMaxBins];                  // per wave: digit counts, then places in the block's digit
    uint32_t start[kSortMaxBins];                             // first place of a digit in the block
    uint32_t base[kSortMaxBins];                              // and in the output, less start
    uint32_t wave[kSortWaves], pre[kDepthSortThreads];
    uint32_t lb;
};

__device__ __forceinline__ void sort_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exclusive scan over the block's threads.
__device__ __forceinline__ uint32_t sort_scan(uint32_t v, uint32_t *s_wave) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d, 64);
        if (lane >= (uint32_t)d) incl += o;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t base = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
        const uint32_t c = s_wave[w];
        base += (uint32_t)w < wave ? c : 0u;
    }
    __syncthreads();
    return base + incl - v;
}

// Ranks the block's keys by their digit, stably: item r of a lane (in the order
// wave, r, lane) gets rank[r] among its wave's keys of its digit.  On return
// wcnt holds, per digit, each wave's first place among the block's keys of the
// digit, and cnt[] the block's counts of this thread's digits (per consecutive
// ones from per * thread on).
__device__ __forceinline__ void sort_rank(SortLds &s, const SortParams &p, int pass, const uint32_t (&k)[kSortItems],
                                          uint32_t valid, uint32_t per, uint32_t (&rank)[kSortItems],
                                          uint32_t (&cnt)[2]) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, bins = 1u << p.bits;
    const uint64_t below = (1ull << lane) - 1ull;
    uint16_t *const w = s.wcnt[wave];
    for (uint32_t i = lane; i < (bins + 1u) / 2u; i += 64u) reinterpret_cast<uint32_t *>(w)[i] = 0u;
    sort_wave_sync();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const bool ok = (valid >> r) & 1u;
        const uint32_t d = sort_digit(p, k[r], pass);
        uint64_t peers = __ballot(ok);
        for (uint32_t b = 0; b < p.bits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        // every lane of a digit reads the counter before its first lane adds the digit's count
        const uint32_t before = w[d];
        sort_wave_sync();
        const uint32_t lrank = (uint32_t)__popcll(peers & below);
        if (ok && lrank == 0) w[d] = (uint16_t)(before + (uint32_t)__popcll(peers));
        sort_wave_sync();
        rank[r] = before + lrank;
    }
    __syncthreads();
    cnt[0] = cnt[1] = 0u;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint32_t d = per * tid + (uint32_t)j;
        if ((uint32_t)j >= per || d >= bins) continue;
        uint32_t c = 0;
#pragma unroll
        for (int q = 0; q < kSortWaves; ++q) {
            const uint32_t x = s.wcnt[q][d];
            s.wcnt[q][d] = (uint16_t)c;
            c += x;
        }
        cnt[j] = c;
    }
}

// The places of the items in the block, from sort_rank's results; needs start[].
__device__ __forceinline__ void sort_to_lds(SortLds &s, const SortParams &p, int pass, const uint32_t (&k)[kSortItems],
                                            const uint32_t (&v)[kSortItems], uint32_t valid,
                                            const uint32_t (&rank)[kSortItems]) {
    const uint32_t wave = threadIdx.x >> 6;
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        if (!((valid >> r) & 1u)) continue;
        const uint32_t d = sort_digit(p, k[r], pass), at = s.start[d] + s.wcnt[wave][d] + rank[r];
        s.keys[at] = k[r];
        s.vals[at] = v[r];
    }
}

__device__ __forceinline__ void sort_range(uint32_t &lo, uint32_t &hi, uint32_t (*s_w)[2]) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, d, 64));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, 64));
    }
    if ((threadIdx.x & 63u) == 0) { s_w[threadIdx.x >> 6][0] = lo; s_w[threadIdx.x >> 6][1] = hi; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) { lo = min(lo, s_w[w][0]); hi = max(hi, s_w[w][1]); }
}

__global__ __launch_bounds__(kDepthSortThreads) void k_sort_hist(Tables tb, const uint32_t *keys, uint32_t *scratch) {
    __shared__ uint32_t s_h[kSortPasses * kSortMaxBins];
    __shared__ uint32_t s_w[kSortWaves][2];
    const int v = find_segment(tb.sort_block_start, tb.n_views, blockIdx.x);
    const ViewDesc &vd = tb.views[v];
    const uint32_t lb = blockIdx.x - vd.sort_block_off, tid = threadIdx.x;
    const SortScratch sc = sort_scratch(scratch, vd);
    const uint32_t nb = ((uint32_t)vd.n + 63u) / 64u;
    uint32_t k[kSortItems];                                // the block's keys, in flight with the ranges
    const uint32_t beg = vd.item_off + lb * (uint32_t)kDepthSortTile;
    const uint32_t end = min(beg + (uint32_t)kDepthSortTile, vd.item_off + (uint32_t)vd.n);
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const uint32_t i = beg + (uint32_t)r * kDepthSortThreads + tid;
        k[r] = vd.nsort_blocks > 1u && i < end ? keys[i] : 0u;
    }
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    for (uint32_t i = tid; i < nb; i += kDepthSortThreads) { lo = min(lo, sc.range[2 * i]); hi = max(hi, sc.range[2 * i + 1]); }
    sort_range(lo, hi, s_w);
    const SortParams p = sort_params(lo, hi);
    if (lb == 0 && tid == 0) { sc.par[0] = p.kmin; sc.par[1] = p.top; sc.par[2] = p.bits; }
    if (vd.nsort_blocks <= 1u) return;
    const uint32_t bins = 1u << p.bits;
    for (uint32_t i = tid; i < kSortPasses * bins; i += kDepthSortThreads) s_h[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r)
        if (beg + (uint32_t)r * kDepthSortThreads + tid < end) {
#pragma unroll
            for (int q = 0; q < kSortPasses; ++q) atomicAdd(&s_h[(uint32_t)q * bins + sort_digit(p, k[r], q)], 1u);
        }
    __syncthreads();
    for (uint32_t i = tid; i < kSortPasses * bins; i += kDepthSortThreads) {
        const uint32_t q = i >> p.bits, d = i & (bins - 1u);
        if (s_h[i]) atomicAdd(sc.total + q * kSortMaxBins + d, s_h[i]);
        sc.pub[((uint64_t)q * vd.nsort_blocks + lb) * kSortMaxBins + d] = 0u;
    }
}

// One pass over one block of keys.  FIRST: the values are the items' own numbers.
template <bool FIRST>
__global__ __launch_bounds__(kDepthSortThreads) void k_sort_pass(Tables tb, const uint32_t *kin, const uint32_t *vin,
                                                                 uint32_t *kout, uint32_t *vout, uint32_t *scratch,
                                                                 int pass) {
    __shared__ SortLds s;
    const int view = find_segment(tb.sort_block_start, tb.n_views, blockIdx.x);
    const ViewDesc &vd = tb.views[view];
    const SortScratch sc = sort_scratch(scratch, vd);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, nsb = vd.nsort_blocks;
    if (tid == 0) s.lb = nsb > 1u ? atomicAdd(sc.ticket + pass, 1u) : 0u;
    SortParams p;
    p.kmin = sc.par[0];
    p.top = sc.par[1];
    p.bits = sc.par[2];
    const uint32_t bins = 1u << p.bits, per = bins > (uint32_t)kDepthSortThreads ? 2u : 1u;
    // the view's totals of this thread's digits
    uint32_t tot[2] = {0u, 0u};
    if (nsb > 1u)
#pragma unroll
        for (uint32_t j = 0; j < 2u; ++j)
            if (j < per && per * tid + j < bins) tot[j] = sc.total[(uint32_t)pass * kSortMaxBins + per * tid + j];
    __syncthreads();
    const uint32_t lb = s.lb;
    const uint32_t beg = vd.item_off + lb * (uint32_t)kDepthSortTile;
    const uint32_t end = min(beg + (uint32_t)kDepthSortTile, vd.item_off + (uint32_t)vd.n);
    uint32_t k[kSortItems], v[kSortItems], rank[kSortItems], valid = 0, cnt[2];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const uint32_t i = beg + wave * (uint32_t)(kSortItems * 64) + (uint32_t)r * 64u + lane;
        const bool ok = i < end;
        k[r] = ok ? kin[i] : 0u;
        v[r] = FIRST ? i : ok ? vin[i] : 0u;
        valid |= ok ? 1u << r : 0u;
    }
    sort_rank(s, p, pass, k, valid, per, rank, cnt);
    uint32_t *const pub = sc.pub + (uint64_t)pass * nsb * kSortMaxBins;
    if (nsb > 1u)
#pragma unroll
        for (uint32_t j = 0; j < 2u; ++j)
            if (j < per && per * tid + j < bins)
                __hip_atomic_store(pub + (uint64_t)lb * kSortMaxBins + per * tid + j, cnt[j] | kPresent, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t start = sort_scan(cnt[0] + cnt[1], s.wave);
    if (per * tid < bins) {
        s.start[per * tid] = start;
        if (per == 2u) s.start[2u * tid + 1u] = start + cnt[0];
    }
    __syncthreads();
    sort_to_lds(s, p, pass, k, v, valid, rank);
    // the digits' first places in the view: smaller digits (of the whole view), and this digit in earlier blocks
    uint32_t below = start;
    if (nsb > 1u) {
        below = sort_scan(tot[0] + tot[1], s.wave);
        // group g of the block's threads takes the earlier blocks g, g + groups, ... of its digits
        const uint32_t groups = per == 2u ? 1u : (uint32_t)kDepthSortThreads / bins;
        for (uint32_t j = 0; j < per; ++j) {
            const uint32_t d = per == 2u ? 2u * tid + j : tid & (bins - 1u);
            uint32_t sum = 0;
            for (uint32_t b0 = per == 2u ? 0u : tid >> p.bits; b0 < lb; b0 += 8u * groups) {
                uint32_t x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t b = b0 + (uint32_t)u * groups;
                    x[u] = b < lb ? __hip_atomic_load(pub + (uint64_t)b * kSortMaxBins + d, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT)
                                  : kPresent;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    while (!(x[u] & kPresent)) {           // not published yet: that block is running
                        __builtin_amdgcn_s_sleep(1);
                        x[u] = __hip_atomic_load(pub + (uint64_t)(b0 + (uint32_t)u * groups) * kSortMaxBins + d,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    sum += x[u] & ~kPresent;
                }
            }
            if (per == 2u) s.base[d] = sum;
            else s.pre[tid] = sum;
        }
        __syncthreads();
        if (per == 1u && tid < bins) {
            uint32_t sum = 0;
            for (uint32_t g = 0; g < groups; ++g) sum += s.pre[g * bins + tid];
            s.base[tid] = sum;
        }
    } else if (per * tid < bins) {
        s.base[per * tid] = 0u;
        if (per == 2u) s.base[2u * tid + 1u] = 0u;
    }
    if (per * tid < bins) {
        s.base[per * tid] += vd.item_off + below - start;
        if (per == 2u) s.base[2u * tid + 1u] += vd.item_off + below + (nsb > 1u ? tot[0] : cnt[0]) - (start + cnt[0]);
    }
    __syncthreads();
    const uint32_t n = end - beg;
    for (uint32_t i = tid; i < n; i += kDepthSortThreads) {
        const uint32_t key = s.keys[i], at = s.base[sort_digit(p, key, pass)] + i;
        kout[at] = key;
        vout[at] = s.vals[i];
    }
}

// A view of at most one block's keys: all passes in LDS.
__global__ __launch_bounds__(kDepthSortThreads) void k_sort_small(Tables tb, const uint32_t *kin, uint32_t *kout,
                                                                  uint32_t *vout) {
    __shared__ SortLds s;
    __shared__ uint32_t s_w[kSortWaves][2];
    const ViewDesc &vd = tb.views[find_segment(tb.sort_block_start, tb.n_views, blockIdx.x)];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, n = (uint32_t)vd.n;
    uint32_t k[kSortItems], v[kSortItems], rank[kSortItems], valid = 0, cnt[2];
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const uint32_t i = wave * (uint32_t)(kSortItems * 64) + (uint32_t)r * 64u + lane;
        const bool ok = i < n;
        k[r] = ok ? kin[vd.item_off + i] : 0u;
        v[r] = vd.item_off + i;
        valid |= ok ? 1u << r : 0u;
        if (ok && k[r] != kDroppedKey) { lo = min(lo, k[r]); hi = max(hi, k[r]); }
    }
    sort_range(lo, hi, s_w);
    const SortParams p = sort_params(lo, hi);
    const uint32_t bins = 1u << p.bits, per = bins > (uint32_t)kDepthSortThreads ? 2u : 1u;
#pragma unroll 1
    for (int pass = 0; pass < kSortPasses; ++pass) {
        sort_rank(s, p, pass, k, valid, per, rank, cnt);
        const uint32_t start = sort_scan(cnt[0] + cnt[1], s.wave);
        if (per * tid < bins) {
            s.start[per * tid] = start;
            if (per == 2u) s.start[2u * tid + 1u] = start + cnt[0];
        }
        __syncthreads();
        sort_to_lds(s, p, pass, k, v, valid, rank);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
            const uint32_t i = wave * (uint32_t)(kSortItems * 64) + (uint32_t)r * 64u + lane;
            if (i < n) { k[r] = s.keys[i]; v[r] = s.vals[i]; }
        }
        __syncthreads();                                   // read before the next pass writes
    }
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const uint32_t i = wave * (uint32_t)(kSortItems * 64) + (uint32_t)r * 64u + lane;
        if (i < n) { kout[vd.item_off + i] = k[r]; vout[vd.item_off + i] = v[r]; }
    }
}

hipError_t launch_depth_sort(const Tables &tb, uint32_t sort_blocks, bool one_block_views, uint32_t *keys,
                             uint32_t *vals, uint32_t *keys_alt, uint32_t *vals_alt, uint32_t *scratch, hipStream_t st) {
    if (sort_blocks == 0) return hipSuccess;
    const dim3 grid(sort_blocks), block(kDepthSortThreads);
    if (one_block_views) {
        hipLaunchKernelGGL(k_sort_small, grid, block, 0, st, tb, keys_alt, keys, vals);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_sort_hist, grid, block, 0, st, tb, keys_alt, scratch);
    hipLaunchKernelGGL(k_sort_pass<true>, grid, block, 0, st, tb, keys_alt, vals_alt, keys, vals, scratch, 0);
    hipLaunchKernelGGL(k_sort_pass<false>, grid, block, 0, st, tb, keys, vals, keys_alt, vals_alt, scratch, 1);
    hipLaunchKernelGGL(k_sort_pass<false>, grid, block, 0, st, tb, keys_alt, vals_alt, keys, vals, scratch, 2);
    return hipGetLastError();
}

}  // namespace dpr
