// Video warm start (Sec. 3.4 "Video Synthesis"): the Chamfer distance of
// Eq. (9) between the learned cloud S1 of a frame and the initial cloud S2 of
// the next, its gradient with respect to the positions of S2, an Adam step on
// them, and the transfer to each S2 point of the mean SH coefficients of its
// k nearest S1 points.
//
// Nearest neighbours by brute force here (nn_brute.h); larger clouds are
// searched through a grid (chamfer_grid.hip) with the same results.  Four
// launches: both directions' keys cleared, searched, collected (Eq. (9)'s FP64
// block sums, and per S2 point the FP64 sum of the S1 points whose nearest it
// is), and the gradient with the final sum.  For 2000 points that is 25 us,
// where twelve launches and 4096-point ranges took 118.
// Top-k: one thread per query keeps its k best keys in registers (sorted)
// while all of S1 streams through LDS; SH means in FP64 in neighbour order.
#include <cmath>

#include "dpr_internal.h"
#include "nn_brute.h"

#pragma clang fp contract(off)

namespace dpr {

__global__ __launch_bounds__(kNnThreads) void k_nn(NnJob a, NnJob b) {
    if (blockIdx.x < a.qblocks) nn_brute(a, blockIdx.x, blockIdx.y);
    else nn_brute(b, blockIdx.x - a.qblocks, blockIdx.y);
}

// key12, key21 = ~0; acc, cnt = 0 (acc may be null)
__global__ void k_chamfer_clear(unsigned long long *key12, uint32_t n1, unsigned long long *key21, uint32_t n2,
                                double *acc, uint32_t *cnt) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n1) key12[i] = ~0ull;
    if (i >= n2) return;
    key21[i] = ~0ull;
    if (!acc) return;
#pragma unroll
    for (int a = 0; a < 3; ++a) acc[3 * (size_t)i + a] = 0.0;
    cnt[i] = 0u;
}

constexpr int kSumThreads = 256;

// Both directions' keys, blocks [0, blocks1) of S1 then those of S2:
//   nn = the nearest's index; part[b] = FP64 sum of the block's d2, in a fixed
//   order; per S2 point j: acc[j] = sum of the S1 points whose nearest is j
//   (FP64), cnt[j] their number.  Null outputs are skipped.
struct ChamferSums {
    const unsigned long long *key12, *key21;
    uint32_t n1, n2, blocks1;
    const float *s1;
    int32_t *nn12, *nn21;
    double *part1, *part2, *acc;
    uint32_t *cnt;
};

__global__ __launch_bounds__(kSumThreads) void k_collect(ChamferSums c) {
    __shared__ double s[kSumThreads];
    const bool first = blockIdx.x < c.blocks1;
    const uint32_t blk = first ? blockIdx.x : blockIdx.x - c.blocks1;
    const uint32_t i = blk * kSumThreads + threadIdx.x, n = first ? c.n1 : c.n2;
    const unsigned long long key = i < n ? (first ? c.key12 : c.key21)[i] : 0ull;
    if (i < n) {
        const uint32_t j = (uint32_t)(key & 0xFFFFFFFFull);
        int32_t *const nn = first ? c.nn12 : c.nn21;
        if (nn) nn[i] = (int32_t)j;
        if (first && c.acc && j < c.n2) {
#pragma unroll
            for (int a = 0; a < 3; ++a) atomicAdd(c.acc + 3 * (size_t)j + a, (double)c.s1[3 * (size_t)i + a]);
            atomicAdd(c.cnt + j, 1u);
        }
    }
    double *const part = first ? c.part1 : c.part2;
    if (!part) return;
    s[threadIdx.x] = i < n ? (double)__uint_as_float((uint32_t)(key >> 32)) : 0.0;
    __syncthreads();
    for (int w = kSumThreads / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blk] = s[0];
}

// The sum of n values by the whole block: thread t adds t, t + 256, ..., then a tree (a fixed order).
__device__ __forceinline__ double block_sum(const double *v, uint32_t n, double *s) {
    double a = 0.0;
    for (uint32_t k = threadIdx.x; k < n; k += kSumThreads) a += v[k];
    s[threadIdx.x] = a;
    __syncthreads();
    for (int w = kSumThreads / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    const double r = s[0];
    __syncthreads();
    return r;
}

// grad2[j] = 2/n2 (y_j - nn(y_j)) + 2/n1 (cnt_j y_j - acc_j), FP64 then rounded;
// the last block (if cd): cd = (sum part1) / n1 + (sum part2) / n2
__global__ __launch_bounds__(kSumThreads) void k_grad(ChamferSums c, const float *s2, float *grad2, double *cd) {
    __shared__ double s[kSumThreads];
    if (cd && blockIdx.x == gridDim.x - 1) {
        const double a = block_sum(c.part1, c.blocks1, s);
        const double b = block_sum(c.part2, (c.n2 + kSumThreads - 1) / kSumThreads, s);
        if (threadIdx.x == 0) *cd = a / (double)c.n1 + b / (double)c.n2;
        return;
    }
    const uint32_t j = blockIdx.x * kSumThreads + threadIdx.x;
    if (j >= c.n2) return;
    const uint32_t k = (uint32_t)(c.key21[j] & 0xFFFFFFFFull);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double y = (double)s2[3 * (size_t)j + a];
        const double x = k < c.n1 ? (double)c.s1[3 * (size_t)k + a] : (double)NAN;    // no neighbour: a NaN point
        const double g = 2.0 / (double)c.n2 * (y - x) +
                         2.0 / (double)c.n1 * ((double)c.cnt[j] * y - c.acc[3 * (size_t)j + a]);
        grad2[3 * (size_t)j + a] = (float)g;
    }
}

hipError_t launch_chamfer_finish(uint32_t n1, const float *s1, uint32_t n2, const float *s2, double *cd, float *grad2,
                                 int32_t *nn12, int32_t *nn21, uint8_t *ws, hipStream_t st) {
    const ChamferLayout L = chamfer_layout(n1, n2);
    const uint32_t nb1 = (n1 + kSumThreads - 1) / kSumThreads, nb2 = (n2 + kSumThreads - 1) / kSumThreads;
    ChamferSums c;
    c.key12 = reinterpret_cast<unsigned long long *>(ws + L.key12);
    c.key21 = reinterpret_cast<unsigned long long *>(ws + L.key21);
    c.n1 = n1;
    c.n2 = n2;
    c.blocks1 = nb1;
    c.s1 = s1;
    c.nn12 = nn12;
    c.nn21 = nn21;
    c.part1 = cd ? reinterpret_cast<double *>(ws + L.part1) : nullptr;
    c.part2 = cd ? reinterpret_cast<double *>(ws + L.part2) : nullptr;
    c.acc = grad2 ? reinterpret_cast<double *>(ws + L.acc) : nullptr;
    c.cnt = reinterpret_cast<uint32_t *>(ws + L.cnt);
    hipLaunchKernelGGL(k_collect, dim3(nb1 + nb2), dim3(kSumThreads), 0, st, c);
    const uint32_t gb = (grad2 ? nb2 : 0u) + (cd ? 1u : 0u);
    if (gb) hipLaunchKernelGGL(k_grad, dim3(gb), dim3(kSumThreads), 0, st, c, s2, grad2, cd);
    return hipGetLastError();
}

ChamferLayout chamfer_layout(uint64_t n1, uint64_t n2) {
    ChamferLayout L;
    uint64_t off = 0;
    auto add = [&](uint64_t bytes) {
        const uint64_t at = off;
        off += (bytes + 255) & ~255ull;
        return at;
    };
    L.key12 = add(8 * n1);
    L.key21 = add(8 * n2);
    L.acc = add(8 * 3 * n2);
    L.cnt = add(4 * n2);
    L.part1 = add(8 * ((n1 + kSumThreads - 1) / kSumThreads));
    L.part2 = add(8 * ((n2 + kSumThreads - 1) / kSumThreads));
    L.bytes = off;
    return L;
}

hipError_t launch_chamfer(uint32_t n1, const float *s1, uint32_t n2, const float *s2, double *cd, float *grad2,
                          int32_t *nn12, int32_t *nn21, uint8_t *ws, hipStream_t st) {
    const ChamferLayout L = chamfer_layout(n1, n2);
    auto *key12 = reinterpret_cast<unsigned long long *>(ws + L.key12);
    auto *key21 = reinterpret_cast<unsigned long long *>(ws + L.key21);
    double *acc = reinterpret_cast<double *>(ws + L.acc);
    const uint32_t most = n1 > n2 ? n1 : n2;
    hipLaunchKernelGGL(k_chamfer_clear, dim3((most + 255) / 256), dim3(256), 0, st, key12, n1, key21, n2,
                       grad2 ? acc : nullptr, reinterpret_cast<uint32_t *>(ws + L.cnt));
    const NnJob a = nn_job(s1, n1, s2, n2, key12), b = nn_job(s2, n2, s1, n1, key21);
    hipLaunchKernelGGL(k_nn, dim3(a.qblocks + b.qblocks, a.ranges > b.ranges ? a.ranges : b.ranges), dim3(kNnThreads), 0, st, a, b);
    return launch_chamfer_finish(n1, s1, n2, s2, cd, grad2, nn12, nn21, ws, st);
}

// Top-k: the lists of topk_brute (nn_brute.h), and one lane of a query's group
// averages its neighbours' rows.
template <int KM>
__global__ __launch_bounds__(kTopkBlock) void k_topk_sh(const float *s1, const float *sh1, uint32_t n1,
                                                        const float *s2, uint32_t n2, int k3, int K,
                                                        float *out_sh, int32_t *idx) {
    unsigned long long best[KM];
    topk_brute(s1, n1, s2, n2, K, blockIdx.x, best);
    const uint32_t j = topk_query(blockIdx.x);
    if (j >= n2 || threadIdx.x % (uint32_t)kTopkLanes != 0) return;
    const int kk = (int)min((uint32_t)K, n1);
    if (idx) {
#pragma unroll
        for (int k = 0; k < KM; ++k)
            if (k < K) idx[(size_t)j * K + k] = k < kk ? (int32_t)(uint32_t)(best[k] & 0xFFFFFFFFull) : -1;
    }
    for (int a = 0; a < k3; ++a) {
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < KM; ++k)
            if (k < kk) acc += (double)sh1[(size_t)k3 * (uint32_t)(best[k] & 0xFFFFFFFFull) + a];
        out_sh[(size_t)k3 * j + a] = (float)(acc / (double)kk);
    }
}

hipError_t launch_topk_sh(uint32_t n1, const float *s1, const float *sh1, uint32_t n2, const float *s2, int k3, int K,
                          float *out_sh, int32_t *idx, hipStream_t st) {
    if (n2 == 0) return hipSuccess;
    if (K < 1 || K > kTopkMax) return hipErrorInvalidValue;
    const dim3 grid((n2 + kTopkQueries - 1) / kTopkQueries);
    if (K <= 4) {
        hipLaunchKernelGGL(k_topk_sh<4>, grid, dim3(kTopkBlock), 0, st, s1, sh1, n1, s2, n2, k3, K, out_sh, idx);
    } else if (K <= 8) {
        hipLaunchKernelGGL(k_topk_sh<8>, grid, dim3(kTopkBlock), 0, st, s1, sh1, n1, s2, n2, k3, K, out_sh, idx);
    } else if (K <= 16) {
        hipLaunchKernelGGL(k_topk_sh<16>, grid, dim3(kTopkBlock), 0, st, s1, sh1, n1, s2, n2, k3, K, out_sh, idx);
    } else {
        hipLaunchKernelGGL(k_topk_sh<kTopkMax>, grid, dim3(kTopkBlock), 0, st, s1, sh1, n1, s2, n2, k3, K, out_sh,
                           idx);
    }
    return hipGetLastError();
}

// Adam with bias correction (c1 = 1 - b1^t, c2 = 1 - b2^t computed on the host)
__global__ void k_adam(uint32_t n, float *p, const float *g, float *m, float *v, float lr, float b1, float b2,
                       float c1, float c2, float eps) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

hipError_t launch_adam(uint32_t n, float *p, const float *g, float *m, float *v, int t, float lr, float b1, float b2,
                       float eps, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const float c1 = (float)(1.0 - std::pow((double)b1, (double)t));
    const float c2 = (float)(1.0 - std::pow((double)b2, (double)t));
    hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, st, n, p, g, m, v, lr, b1, b2, c1, c2, eps);
    return hipGetLastError();
}

}  // namespace dpr
