// Brute-force nearest neighbours over LDS tiles: a block takes 256 threads x 2
// queries against one range of up to 4096 points of the other cloud (so that a frame of
// some 10^4 points still fills the GPU), and folds its result into a 64-bit
// key per query with one atomic minimum: key = (d2 bits << 32) | index, which
// orders by (d2, index) because d2 >= 0 (ties go to the lower index, whatever
// the order in which the blocks finish).  Distances in float32 with each
// operation rounded: ((dx dx + dy dy) + dz dz).
#pragma once

#include "dpr_internal.h"

namespace dpr {

constexpr int kNnThreads = 256;
constexpr int kNnQueries = 2;                          // queries per thread
constexpr int kNnTile = 1024;                          // candidate points per LDS tile
constexpr uint32_t kNnRange = 4096;                    // candidate points per block, at most

__device__ __forceinline__ float nn_dist2(float ax, float ay, float az, float bx, float by, float bz) {
#pragma clang fp contract(off)
    const float a = ax - bx, b = ay - by, c = az - bz;
    float s = a * a;
    s = s + b * b;
    return s + c * c;
}

// One direction of a brute-force search: queries q, candidates c.
struct NnJob {
    const float *q;
    uint32_t nq;
    const float *c;
    uint32_t nc;
    unsigned long long *key;
    uint32_t qblocks, range, ranges;  // blocks of queries, candidates per block, their number
};

inline NnJob nn_job(const float *q, uint32_t nq, const float *c, uint32_t nc, unsigned long long *key) {
    const uint32_t qb = (nq + kNnThreads * kNnQueries - 1) / (kNnThreads * kNnQueries);
    // shorter ranges where the clouds are small, for about 1000 blocks
    uint32_t range = 256;
    while (range < kNnRange && (uint64_t)qb * (nc / range) > 1024u) range *= 2;
    return NnJob{q, nq, c, nc, key, qb, range, (nc + range - 1) / range};
}

// key[i] = min over candidate range `range` of (d2(q_i, c_j) bits << 32 | j),
// for the queries of block qblk; a range past the last does nothing.
__device__ __forceinline__ void nn_brute(const NnJob &j, uint32_t qblk, uint32_t range) {
    __shared__ float s_x[kNnTile], s_y[kNnTile], s_z[kNnTile];
    if (range >= j.ranges) return;
    const uint32_t q0 = qblk * (kNnThreads * kNnQueries) + threadIdx.x;
    const uint32_t cbeg = range * j.range, cend = min(cbeg + j.range, j.nc);
    float qx[kNnQueries], qy[kNnQueries], qz[kNnQueries], best[kNnQueries];
    uint32_t bj[kNnQueries];
#pragma unroll
    for (int k = 0; k < kNnQueries; ++k) {
        const uint32_t i = q0 + k * kNnThreads;
        const uint32_t ii = i < j.nq ? i : 0;
        qx[k] = j.q[3 * (size_t)ii]; qy[k] = j.q[3 * (size_t)ii + 1]; qz[k] = j.q[3 * (size_t)ii + 2];
        best[k] = INFINITY;
        bj[k] = 0xFFFFFFFFu;
    }
    for (uint32_t t0 = cbeg; t0 < cend; t0 += kNnTile) {
        const uint32_t tn = min((uint32_t)kNnTile, cend - t0);
        __syncthreads();
        for (uint32_t t = threadIdx.x; t < tn; t += kNnThreads) {
            s_x[t] = j.c[3 * (size_t)(t0 + t)];
            s_y[t] = j.c[3 * (size_t)(t0 + t) + 1];
            s_z[t] = j.c[3 * (size_t)(t0 + t) + 2];
        }
        __syncthreads();
        for (uint32_t t = 0; t < tn; ++t) {
            const float cx = s_x[t], cy = s_y[t], cz = s_z[t];
#pragma unroll
            for (int k = 0; k < kNnQueries; ++k) {
                const float d = nn_dist2(qx[k], qy[k], qz[k], cx, cy, cz);
                if (d < best[k]) {          // scanning in index order: the first minimum is the lowest index
                    best[k] = d;
                    bj[k] = t0 + t;
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kNnQueries; ++k) {
        const uint32_t i = q0 + k * kNnThreads;
        if (i < j.nq && bj[k] != 0xFFFFFFFFu)
            atomicMin(j.key + i, ((unsigned long long)__float_as_uint(best[k]) << 32) | bj[k]);
    }
}

// Key x into the K smallest so far (ascending); worst: the K-th of them.
template <int KMAX>
__device__ __forceinline__ void nn_insert(unsigned long long (&best)[KMAX], int K, unsigned long long x,
                                          unsigned long long &worst) {
    if (x >= worst) return;
    // keep the smaller key in each place, carry the larger one on
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        if (k < K) {
            const unsigned long long lo = best[k] < x ? best[k] : x;
            x = best[k] < x ? x : best[k];
            best[k] = lo;
        }
    }
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        if (k == K - 1) worst = best[k];
}

// The K smallest keys of each query by brute force: a group of kTopkLanes
// consecutive lanes per query y of S2, 32 queries per block.  Lane s of the
// group scans the candidates t = s mod kTopkLanes of every LDS tile of S1 and
// keeps the KM smallest keys (d2 bits << 32 | index, ascending) it met; the
// group's lists are then merged by exchanging them between partner lanes (xor
// 1, 2, 4).  The keys are distinct and totally ordered, so the K smallest are
// found exactly, whatever the split.  On return every lane of the group of
// query j = topk_query(blk) holds them.
constexpr int kTopkLanes = 8;
constexpr int kTopkBlock = 256;
constexpr uint32_t kTopkQueries = kTopkBlock / kTopkLanes;

__device__ __forceinline__ uint32_t topk_query(uint32_t blk) {
    return blk * kTopkQueries + threadIdx.x / (uint32_t)kTopkLanes;
}

__device__ __forceinline__ unsigned long long shfl_xor_u64(unsigned long long v, int m) {
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, m, 64);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), m, 64);
    return ((unsigned long long)hi << 32) | lo;
}

template <int KM>
__device__ __forceinline__ void topk_brute(const float *s1, uint32_t n1, const float *s2, uint32_t n2, int K,
                                           uint32_t blk, unsigned long long (&best)[KM]) {
    __shared__ float s_x[kNnTile], s_y[kNnTile], s_z[kNnTile];
    const uint32_t sub = threadIdx.x % (uint32_t)kTopkLanes, j = topk_query(blk);
    const uint32_t jj = j < n2 ? j : 0;
    const float qx = s2[3 * (size_t)jj], qy = s2[3 * (size_t)jj + 1], qz = s2[3 * (size_t)jj + 2];
#pragma unroll
    for (int k = 0; k < KM; ++k) best[k] = ~0ull;
    unsigned long long worst = ~0ull;
    for (uint32_t t0 = 0; t0 < n1; t0 += kNnTile) {
        const uint32_t tn = min((uint32_t)kNnTile, n1 - t0);
        __syncthreads();
        for (uint32_t t = threadIdx.x; t < tn; t += kTopkBlock) {
            s_x[t] = s1[3 * (size_t)(t0 + t)];
            s_y[t] = s1[3 * (size_t)(t0 + t) + 1];
            s_z[t] = s1[3 * (size_t)(t0 + t) + 2];
        }
        __syncthreads();
        for (uint32_t t = sub; t < tn; t += kTopkLanes) {
            const float d = nn_dist2(qx, qy, qz, s_x[t], s_y[t], s_z[t]);
            nn_insert(best, K, ((unsigned long long)__float_as_uint(d) << 32) | (t0 + t), worst);
        }
    }
    // after the exchange with lane ^ m every lane of a pair holds the K smallest of both (all lanes take part)
#pragma unroll
    for (int m = 1; m < kTopkLanes; m <<= 1) {
        unsigned long long other[KM];
#pragma unroll
        for (int k = 0; k < KM; ++k) other[k] = shfl_xor_u64(best[k], m);
#pragma unroll
        for (int k = 0; k < KM; ++k)
            if (k < K) nn_insert(best, K, other[k], worst);
    }
}

}  // namespace dpr
