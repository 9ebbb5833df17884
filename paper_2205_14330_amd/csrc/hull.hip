// Visual-hull initialisation and multi-view consistency filter (Sec. 3.1
// "Initialization"; the appendix's consistency check CC): a point is kept when
// its projection (Eq. 1) falls on a foreground pixel of every camera's mask.
//   sampling: candidates drawn uniformly in a box from a counter-based
//             generator (Philox4x32-10, Salmon et al. SC 2011: counter = the
//             candidate index, key = the seed), the consistent ones returned
//             in candidate order;
//   filter:   the consistent points of a cloud, every parameter, in order.
// The pixel decision is taken in float32 with the operations documented in
// include/dpr.h, each rounded once, so it is reproducible bit for bit.
//
// The masks are first packed to one bit per pixel in the workspace (sixteen
// 800x800 masks take 1.25 MB instead of 10 MB, so every XCD's L2 holds them
// all: the lookups of random candidates are L2 hits).
// Two passes over blocks of items: the first decides CC and writes one bit per
// item and one count per block; a scan of the counts gives each block its
// output offset; the second pass writes the kept items at offset + rank, which
// keeps the input order.  Camera and mask descriptors sit in one table in the
// workspace and are read through uniform (scalar) loads.
#include <vector>

#include "dpr_internal.h"

#pragma clang fp contract(off)

namespace dpr {

constexpr int kHullThreads = 256;
constexpr int kHullWaves = kHullThreads / 64;
constexpr int kHullPer = 8;                                  // items per lane of the compacting form
constexpr uint64_t kHullMany = 1u << 20;                     // candidates from which it is taken (below)
constexpr uint64_t kHullManyPoints = 1u << 22;               // points from which it is taken

// Items per thread of a block: one, or kHullPer from kHullMany items on.  Below,
// items packed kHullPer to a lane leave too few waves (a whole sampling call
// with 16 masks of 800x800, one per lane against kHullPer: 2^16 candidates 80
// us and 107, 2^19 91 and 99, 2^20 110 and 102, 2^22 205 and 154, 2^24 585 and
// 344).  Given points are mostly inside (a trained cloud is filtered once per
// epoch), so packing removes few of them, and they are read, not drawn: the
// predicate alone, 16 full masks, one per lane against kHullPer, 2^20 points 47
// us and 74, 2^21 82 and 88, 2^22 155 and 158 (with a fifth inside, 47 and 50,
// 69 and 60, 124 and 110).
__host__ __device__ constexpr int hull_per(uint64_t n, bool points) {
    return n < (points ? kHullManyPoints : kHullMany) ? 1 : kHullPer;
}

uint64_t hull_blocks(uint64_t n, bool points) {
    const uint64_t items = (uint64_t)kHullThreads * hull_per(n, points);
    return (n + items - 1) / items;
}

struct HullArgs {
    const HullCam *cams;
    int32_t n_cams;
    uint64_t n;
    // sampling (xyz == nullptr) or filter (xyz != nullptr)
    const float *xyz;
    uint32_t key0, key1;
    float lo[3], width[3];
    uint32_t *bits;        // [blocks][items of a block / 32]
    uint32_t *counts;      // [blocks]
    uint8_t *keep;         // [n] CC per item (optional)
};

// Ten rounds of Philox4x32 (multipliers and key increments of the SC 2011 paper).
// Both halves of a product come from one 64-bit multiply (a quarter-rate
// instruction either way): sampling 2^24 candidates 259 us, with a multiply for
// each half 262.
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint64_t m0 = (uint64_t)0xD2511F53u * c[0], m1 = (uint64_t)0xCD9E8D57u * c[2];
        c[0] = (uint32_t)(m1 >> 32) ^ c[1] ^ k0;
        c[1] = (uint32_t)m1;
        c[2] = (uint32_t)(m0 >> 32) ^ c[3] ^ k1;
        c[3] = (uint32_t)m0;
    }
}

// Candidate j: u = (r >> 8) 2^-24 of the first three words, lo + u (hi - lo) in one rounding.
__device__ __forceinline__ void candidate(const HullArgs &a, uint64_t j, float p[3]) {
    uint32_t c[4] = {(uint32_t)j, (uint32_t)(j >> 32), 0u, 0u};
    philox4x32_10(c, a.key0, a.key1);
#pragma unroll
    for (int d = 0; d < 3; ++d) p[d] = fmaf((float)(c[d] >> 8) * 0x1p-24f, a.width[d], a.lo[d]);
}

__device__ __forceinline__ void load_item(const HullArgs &a, uint64_t j, float p[3]) {
    if (a.xyz) {
        p[0] = a.xyz[3 * j];
        p[1] = a.xyz[3 * j + 1];
        p[2] = a.xyz[3 * j + 2];
    } else {
        candidate(a, j, p);
    }
}

// 1 if p falls on a foreground pixel of camera c (float32 decisions as documented).
__device__ __forceinline__ bool inside(const HullCam &c, const float p[3]) {
    float X[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) X[r] = fmaf(c.R[3 * r], p[0], fmaf(c.R[3 * r + 1], p[1], fmaf(c.R[3 * r + 2], p[2], c.t[r])));
    if (!(X[2] > 0.f)) return false;
    const float px = fmaf(c.fx, X[0] / X[2], c.cx);
    const float py = fmaf(c.fy, X[1] / X[2], c.cy);
    if (!(px >= 0.f && px < (float)c.width && py >= 0.f && py < (float)c.height)) return false;
    const uint64_t idx = (uint64_t)(int32_t)py * (uint32_t)c.width + (uint32_t)(int32_t)px;
    return (c.bits[idx >> 5] >> (idx & 31u)) & 1u;
}

// Packed word w of all cameras: bit b = 1 iff mask byte 32 w' + b != 0 (w' the
// word within its camera, bytes past the mask read as 0).  A whole word whose
// bytes are 16-byte aligned is read in two loads (sixteen 800x800 masks: 5.2
// us, byte by byte 22).
__global__ __launch_bounds__(kHullThreads) void k_pack_masks(const HullCam *cams, int32_t n_cams, uint64_t words,
                                                             uint32_t *packed) {
    const uint64_t w = (uint64_t)blockIdx.x * kHullThreads + threadIdx.x;
    if (w >= words) return;
    int32_t lo = 0, hi = n_cams - 1;                // last camera with word_off <= w
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (cams[mid].word_off <= w) lo = mid; else hi = mid - 1;
    }
    const HullCam &c = cams[lo];
    const uint64_t npix = (uint64_t)c.width * (uint32_t)c.height;
    const uint64_t p0 = (w - c.word_off) * 32;
    const uint8_t *m = c.mask + p0;
    uint32_t v = 0;
    if (p0 + 32 <= npix && ((uintptr_t)m & 15) == 0) {
        const uint4 q[2] = {reinterpret_cast<const uint4 *>(m)[0], reinterpret_cast<const uint4 *>(m)[1]};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t d[4] = {q[h].x, q[h].y, q[h].z, q[h].w};
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int b = 0; b < 4; ++b) v |= ((d[k] >> (8 * b)) & 0xFFu ? 1u : 0u) << (16 * h + 4 * k + b);
        }
    } else {
        for (uint32_t b = 0; b < 32 && p0 + b < npix; ++b) v |= (m[b] != 0 ? 1u : 0u) << b;
    }
    packed[w] = v;
}

// The predicate of few items: one per lane, so that the waves fill the chip,
// and four cameras at a time, so that four mask gathers are in flight; a wave
// leaves the loop once none of its items is still inside.  100k points, 16
// cameras: 14.6 us (four items per lane, one camera at a time: 37).
constexpr int kHullCamGroup = 4;

__global__ __launch_bounds__(kHullThreads) void k_hull_flags_few(HullArgs a) {
    __shared__ uint32_t s_cnt[kHullWaves];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t j = (uint64_t)blockIdx.x * kHullThreads + tid;
    float p[3] = {0.f, 0.f, 0.f};
    bool in = j < a.n;
    if (in) load_item(a, j, p);
    for (int32_t i = 0; i < a.n_cams; i += kHullCamGroup) {
        if (__ballot(in) == 0ull) break;
        if (in) {
            bool all = true;
#pragma unroll
            for (int q = 0; q < kHullCamGroup; ++q)
                if (i + q < a.n_cams) all = inside(a.cams[i + q], p) && all;
            in = all;
        }
    }
    const uint64_t m = __ballot(in);
    if (lane == 0) {
        uint32_t *w = a.bits + (uint64_t)blockIdx.x * (kHullThreads / 32) + 2 * wave;
        w[0] = (uint32_t)m;
        w[1] = (uint32_t)(m >> 32);
        s_cnt[wave] = (uint32_t)__popcll(m);
    }
    if (a.keep && j < a.n) a.keep[j] = in ? 1 : 0;
    __syncthreads();
    if (tid == 0) {
        uint32_t s = 0;
        for (int w = 0; w < kHullWaves; ++w) s += s_cnt[w];
        a.counts[blockIdx.x] = s;
    }
}

// The predicate of many items, bound by its arithmetic (some 60 instructions
// per item and camera).  Most candidates of a box fall outside the hull, and
// most of those leave in one of the first cameras; lanes whose item has left
// cost as much as the others, and a wave of 64 keeps an inside item nearly
// always.  So a wave owns 512 items: it takes all of them through the first
// two cameras, packs the ones still inside into LDS, and takes only these
// through the next two, packing again.  2^24 candidates, 16 cameras: 201 us
// (every camera for all items of a wave until none was inside: 414).
// Where more than kHullDense items are left after the first two, packing costs
// more than the lanes it saves: those are walked through the other cameras
// without it, four items to a lane, so that four lookups are in flight (a third
// of 2^24 candidates inside all 16 masks: predicate 0.44 ms, packed 0.57, the
// form before 0.53; with a twentieth inside, 257 us a call, always packed 260).
constexpr int kHullFirst = 2;
constexpr uint32_t kHullDense = 64 * kHullPer * 3 / 8;

__global__ __launch_bounds__(kHullThreads) void k_hull_flags_many(HullArgs a) {
    constexpr uint32_t kItems = 64 * kHullPer;                // of a wave
    constexpr int kHalf = kHullPer / 2;
    __shared__ float s_p[kHullWaves][3][kItems];
    __shared__ uint16_t s_j[kHullWaves][kItems];
    __shared__ uint32_t s_bits[kHullWaves][kItems / 32];
    __shared__ uint32_t s_cnt[kHullWaves];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t base = ((uint64_t)blockIdx.x * kHullWaves + wave) * kItems;
    const uint64_t below = (1ull << lane) - 1;
    auto sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    if (lane < kItems / 32) s_bits[wave][lane] = 0u;
    uint32_t n = 0, kept = 0;                                 // items still inside; and to the end
    for (int h = 0; h < kHullPer; h += kHalf) {
        float p[kHalf][3];
        bool in[kHalf];
#pragma unroll
        for (int k = 0; k < kHalf; ++k) {
            const uint64_t j = base + 64u * (uint32_t)(h + k) + lane;
            in[k] = j < a.n;
            if (in[k]) load_item(a, j, p[k]);
        }
        for (int32_t i = 0; i < kHullFirst && i < a.n_cams; ++i) {
            const HullCam &c = a.cams[i];
#pragma unroll
            for (int k = 0; k < kHalf; ++k)
                if (in[k]) in[k] = inside(c, p[k]);
        }
#pragma unroll
        for (int k = 0; k < kHalf; ++k) {
            const uint64_t m = __ballot(in[k]);
            if (in[k]) {
                const uint32_t at = n + (uint32_t)__popcll(m & below);
                s_p[wave][0][at] = p[k][0];
                s_p[wave][1][at] = p[k][1];
                s_p[wave][2][at] = p[k][2];
                s_j[wave][at] = (uint16_t)(64u * (uint32_t)(h + k) + lane);
            }
            n += (uint32_t)__popcll(m);
        }
    }
    sync();
    if (n > kHullDense) {
        // lanes keep kHalf items each; the ones that stay set their bits here
        uint32_t left = 0;
        for (uint32_t b = 0; b < n; b += 64u * kHalf) {
            float p[kHalf][3];
            bool in[kHalf];
#pragma unroll
            for (int k = 0; k < kHalf; ++k) {
                const uint32_t l = b + 64u * (uint32_t)k + lane;
                in[k] = l < n;
#pragma unroll
                for (int d = 0; d < 3; ++d) p[k][d] = in[k] ? s_p[wave][d][l] : 0.f;
            }
            for (int32_t i = kHullFirst; i < a.n_cams; ++i) {
                bool any = false;
#pragma unroll
                for (int k = 0; k < kHalf; ++k) any = any || in[k];
                if (__ballot(any) == 0ull) break;
                const HullCam &c = a.cams[i];
#pragma unroll
                for (int k = 0; k < kHalf; ++k)
                    if (in[k]) in[k] = inside(c, p[k]);
            }
#pragma unroll
            for (int k = 0; k < kHalf; ++k) {
                if (in[k]) {
                    const uint32_t j = s_j[wave][b + 64u * (uint32_t)k + lane];
                    atomicOr(&s_bits[wave][j >> 5], 1u << (j & 31));
                }
                left += (uint32_t)__popcll(__ballot(in[k]));
            }
        }
        kept = left;
        n = 0;
    }
    for (int32_t i = kHullFirst; i < a.n_cams && n > 0; i += 2) {
        uint32_t left = 0;
        for (uint32_t b = 0; b < n; b += 64) {
            bool in = b + lane < n;
            float p[3] = {0.f, 0.f, 0.f};
            uint16_t j = 0;
            if (in) {
                p[0] = s_p[wave][0][b + lane];
                p[1] = s_p[wave][1][b + lane];
                p[2] = s_p[wave][2][b + lane];
                j = s_j[wave][b + lane];
                bool both = inside(a.cams[i], p);
                if (i + 1 < a.n_cams) both = inside(a.cams[i + 1], p) && both;
                in = both;
            }
            const uint64_t m = __ballot(in);
            sync();                                           // the batch is read before its places are written
            if (in) {
                const uint32_t at = left + (uint32_t)__popcll(m & below);
                s_p[wave][0][at] = p[0];
                s_p[wave][1][at] = p[1];
                s_p[wave][2][at] = p[2];
                s_j[wave][at] = j;
            }
            left += (uint32_t)__popcll(m);
        }
        sync();
        n = left;
    }
    kept += n;
    for (uint32_t b = lane; b < n; b += 64) {
        const uint32_t j = s_j[wave][b];
        atomicOr(&s_bits[wave][j >> 5], 1u << (j & 31));
    }
    sync();
    if (lane < kItems / 32) a.bits[base / 32 + lane] = s_bits[wave][lane];
    if (a.keep) {
        for (int k = 0; k < kHullPer; ++k) {
            const uint32_t l = 64u * (uint32_t)k + lane;
            if (base + l < a.n) a.keep[base + l] = (uint8_t)((s_bits[wave][l >> 5] >> (l & 31)) & 1u);
        }
    }
    if (lane == 0) s_cnt[wave] = kept;
    __syncthreads();
    if (tid == 0) {
        uint32_t s = 0;
        for (int w = 0; w < kHullWaves; ++w) s += s_cnt[w];
        a.counts[blockIdx.x] = s;
    }
}

struct HullOut {
    const uint32_t *offsets;     // [blocks] exclusive scan of the counts
    uint64_t capacity;
    // sampling: positions; filter: every parameter (k3 floats of SH per point)
    float *xyz, *sh, *opacity, *radius;
    const float *in_sh, *in_opacity, *in_radius;
    int k3;
};

// The kept items of a block of 256 PER, in order.  Each thread expands 8 bits
// of the block's bitmask into a list in LDS; the list is then worked off in
// full waves (few candidates are kept, and each costs a draw of the generator)
// and the SH rows as one run of floats, so that reads and writes coalesce: 2^24
// candidates 8.5 us, 100k points of degree 2 13.9 (a thread per item, with a
// loop over its SH: 19.8 and 35.5).
template <int PER>
__global__ __launch_bounds__(kHullThreads) void k_hull_scatter(HullArgs a, HullOut o) {
    constexpr uint32_t kItems = kHullThreads * PER;
    __shared__ uint16_t s_list[kItems];
    __shared__ uint32_t s_sum[kHullWaves];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t bits = 0;
    if (tid < kItems / 8)
        bits = (a.bits[(uint64_t)blockIdx.x * (kItems / 32) + (tid >> 2)] >> (8 * (tid & 3))) & 0xFFu;
    const uint32_t c = (uint32_t)__popc(bits);
    uint32_t pre = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)pre, d, 64);
        if (lane >= (uint32_t)d) pre += v;
    }
    if (lane == 63) s_sum[wave] = pre;
    __syncthreads();
    uint32_t at = pre - c, kept = 0;
#pragma unroll
    for (uint32_t w = 0; w < (uint32_t)kHullWaves; ++w) {
        if (w < wave) at += s_sum[w];
        kept += s_sum[w];
    }
    for (uint32_t b = 0; b < 8; ++b)
        if ((bits >> b) & 1u) s_list[at++] = (uint16_t)(8 * tid + b);
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * kItems;
    const uint64_t off = o.offsets[blockIdx.x];
    if (off >= o.capacity) return;
    if (kept > o.capacity - off) kept = (uint32_t)(o.capacity - off);
    for (uint32_t i = tid; i < kept; i += kHullThreads) {
        const uint64_t j = base + s_list[i], rank = off + i;
        float p[3];
        load_item(a, j, p);
        o.xyz[3 * rank] = p[0];
        o.xyz[3 * rank + 1] = p[1];
        o.xyz[3 * rank + 2] = p[2];
        if (a.xyz) {
            o.opacity[rank] = o.in_opacity[j];
            o.radius[rank] = o.in_radius[j];
        }
    }
    if (a.xyz) {
        const uint32_t k3 = (uint32_t)o.k3, rows = kHullThreads / k3, rest = kHullThreads - rows * k3;
        uint32_t i = tid / k3, q = tid - i * k3;
        while (i < kept) {
            o.sh[k3 * (off + i) + q] = o.in_sh[k3 * (base + s_list[i]) + q];
            i += rows;
            q += rest;
            if (q >= k3) {
                q -= k3;
                ++i;
            }
        }
    }
}

HullLayout hull_layout(uint64_t n, int32_t n_cams, const HullCam *cams) {
    // sized for either form, so that a workspace for n items serves fewer
    const uint64_t nb = (n + kHullThreads - 1) / kHullThreads;
    HullLayout h;
    h.words = 0;
    for (int32_t i = 0; i < n_cams; ++i) h.words += ((uint64_t)cams[i].width * (uint32_t)cams[i].height + 31) / 32;
    uint64_t off = 0;
    auto add = [&](uint64_t bytes) {
        const uint64_t at = off;
        off += (bytes + 255) & ~255ull;
        return at;
    };
    h.cams = add(sizeof(HullCam) * (uint64_t)n_cams);
    h.packed = add(4 * h.words);
    h.bits = add(kHullThreads / 8 * (nb + kHullPer - 1));     // whole blocks of kHullPer items per thread
    h.counts = add(4 * (nb + 1));
    h.offsets = add(4 * (nb + 1));                 // the scan also writes the total after the last entry
    h.part = add(8 * (scan_partials(nb + 1) + 2));
    h.total = add(8);
    h.bytes = off;
    return h;
}

hipError_t launch_hull(const HullJob &job, uint8_t *ws, uint64_t *kept_host, hipStream_t st) {
    const HullLayout L = hull_layout(job.n, job.n_cams, job.cams);
    *kept_host = 0;
    // the table with each camera's packed words
    std::vector<HullCam> tab(job.cams, job.cams + job.n_cams);
    uint32_t *packed = reinterpret_cast<uint32_t *>(ws + L.packed);
    uint64_t woff = 0;
    for (HullCam &c : tab) {
        c.word_off = woff;
        c.bits = packed + woff;
        woff += ((uint64_t)c.width * (uint32_t)c.height + 31) / 32;
    }
    HullArgs a;
    a.cams = reinterpret_cast<const HullCam *>(ws + L.cams);
    a.n_cams = job.n_cams;
    a.n = job.n;
    a.xyz = job.xyz;
    a.key0 = (uint32_t)job.seed;
    a.key1 = (uint32_t)(job.seed >> 32);
    for (int d = 0; d < 3; ++d) {
        a.lo[d] = job.lo[d];
        a.width[d] = job.hi[d] - job.lo[d];
    }
    a.bits = reinterpret_cast<uint32_t *>(ws + L.bits);
    a.counts = reinterpret_cast<uint32_t *>(ws + L.counts);
    a.keep = job.keep;
    hipError_t e = upload_async(ws + L.cams, tab.data(), sizeof(HullCam) * (size_t)job.n_cams, st);
    if (e != hipSuccess || job.n == 0) return e;
    hipLaunchKernelGGL(k_pack_masks, dim3((uint32_t)((L.words + kHullThreads - 1) / kHullThreads)),
                       dim3(kHullThreads), 0, st, a.cams, job.n_cams, L.words, packed);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const bool points = job.xyz != nullptr;
    const uint64_t nb = hull_blocks(job.n, points);
    const bool many = hull_per(job.n, points) == kHullPer;
    if (many)
        hipLaunchKernelGGL(k_hull_flags_many, dim3((uint32_t)nb), dim3(kHullThreads), 0, st, a);
    else
        hipLaunchKernelGGL(k_hull_flags_few, dim3((uint32_t)nb), dim3(kHullThreads), 0, st, a);
    e = hipGetLastError();
    if (e != hipSuccess || (!job.out_xyz && !job.sync)) return e;     // the predicate alone needs no scan
    uint64_t *total = reinterpret_cast<uint64_t *>(ws + L.total);
    uint32_t *offsets = reinterpret_cast<uint32_t *>(ws + L.offsets);
    e = launch_scan(a.counts, offsets, nb, reinterpret_cast<uint64_t *>(ws + L.part), total, st);
    if (e != hipSuccess) return e;
    if (job.out_xyz && job.capacity > 0) {
        HullOut o;
        o.offsets = offsets;
        o.capacity = job.capacity;
        o.xyz = job.out_xyz;
        o.sh = job.out_sh;
        o.opacity = job.out_opacity;
        o.radius = job.out_radius;
        o.in_sh = job.sh;
        o.in_opacity = job.opacity;
        o.in_radius = job.radius;
        o.k3 = job.k3;
        if (many)
            hipLaunchKernelGGL(k_hull_scatter<kHullPer>, dim3((uint32_t)nb), dim3(kHullThreads), 0, st, a, o);
        else
            hipLaunchKernelGGL(k_hull_scatter<1>, dim3((uint32_t)nb), dim3(kHullThreads), 0, st, a, o);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (!job.sync) return hipSuccess;
    return read_count(total, kept_host, st);
}

}  // namespace dpr
