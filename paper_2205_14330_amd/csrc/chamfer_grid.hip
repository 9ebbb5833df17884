// The nearest-neighbour searches of the video warm start over a grid of cells
// (nn_grid.h): Eq. (9) in both directions, and the k nearest points of the SH
// transfer.  The results are those of the brute-force search bit for bit: the
// same float32 distances, ties to the lower index.
//
// Two frames' clouds are searched through about 45 candidates per point
// instead of the whole other cloud: Eq. (9) with its gradient of two 45k-point
// frames takes 65 us instead of 874, ten Adam steps and the transfer of the 4
// nearest points' SH 763 us instead of 9889.  Of the 65 us 18 are the search;
// the rest is nine launches whose work is mostly shorter than a launch (4 to 5
// us each).  Where the clouds do not allow that (they
// lie apart, or crowd into a few cells), more than a quarter of the queries of
// a direction is left over by the one-thread search, and that direction is
// searched by brute force instead of one wave per query: the kernel for the
// left-over queries decides it per direction from their number.
#include "nn_brute.h"
#include "nn_grid.h"

#pragma clang fp contract(off)

namespace dpr {

__global__ __launch_bounds__(kGridThreads) void k_chamfer_rest(NnQuery qa, NnQuery qb, NnJob ja, NnJob jb) {
    __shared__ NnRestLds s;
    const bool first = blockIdx.x < ja.qblocks;
    const NnQuery &q = first ? qa : qb;
    const NnJob &j = first ? ja : jb;
    const uint32_t qblk = first ? blockIdx.x : blockIdx.x - ja.qblocks;
    const uint32_t n = *q.list_n;
    if (n > q.nq / 4u) {
        nn_brute(j, qblk, blockIdx.y);
        return;
    }
    const uint32_t waves = j.qblocks * gridDim.y * (uint32_t)kRestWaves;
    for (uint32_t i = (blockIdx.y * j.qblocks + qblk) * kRestWaves + (threadIdx.x >> 6); i < n; i += waves)
        nn_rest_wave<kNnKey, false>(q, q.list[i], s);
}

uint64_t chamfer_grid_bytes(uint64_t n1, uint64_t n2) {
    auto up = [](uint64_t x) { return (x + 255) & ~255ull; };
    return chamfer_layout(n1, n2).bytes + up(grid_bytes(n1).bytes) + up(grid_bytes(n2).bytes);
}

hipError_t launch_chamfer_grid(uint32_t n1, const float *s1, uint32_t n2, const float *s2, double *cd, float *grad2,
                               int32_t *nn12, int32_t *nn21, uint8_t *ws, hipStream_t st) {
    const ChamferLayout L = chamfer_layout(n1, n2);
    uint8_t *const g1 = ws + L.bytes, *const g2 = g1 + ((grid_bytes(n1).bytes + 255) & ~255ull);
    const NnCloud a = grid_cloud(s1, n1, nn_density(1, n2), g1), b = grid_cloud(s2, n2, nn_density(1, n1), g2);
    // acc and cnt are neighbours in the layout
    hipError_t e = launch_grids(a, &b, reinterpret_cast<uint32_t *>(ws + L.acc),
                                grad2 ? (L.cnt - L.acc) / 4 + n2 : 0, st);
    if (e != hipSuccess) return e;
    NnQuery q12 = grid_query(a, b, 1, n2), q21 = grid_query(b, a, 1, n1);
    q12.key = reinterpret_cast<unsigned long long *>(ws + L.key12);
    q21.key = reinterpret_cast<unsigned long long *>(ws + L.key21);
    const uint32_t b1 = (n1 + kNearQueries - 1) / kNearQueries, b2 = (n2 + kNearQueries - 1) / kNearQueries;
    hipLaunchKernelGGL((k_nn_nearest<kNnKey, false>), dim3(b1 + b2), dim3(kGridThreads), 0, st, q12, q21, b1);
    const NnJob ja = nn_job(s1, n1, s2, n2, q12.key), jb = nn_job(s2, n2, s1, n1, q21.key);
    hipLaunchKernelGGL(k_chamfer_rest, dim3(ja.qblocks + jb.qblocks, ja.ranges > jb.ranges ? ja.ranges : jb.ranges),
                       dim3(kGridThreads), 0, st, q12, q21, ja, jb);
    return launch_chamfer_finish(n1, s1, n2, s2, cd, grad2, nn12, nn21, ws, st);
}

// out_sh[e] (e = query k3 + attribute): the mean of the attribute over the
// query's neighbours, FP64 in neighbour order.  A thread per value: a row's
// values are neighbouring lanes, so each neighbour's row is one run of loads.
__global__ void k_topk_mean(const int32_t *idx, const float *sh1, uint32_t n1, uint64_t values, uint32_t k3, int K,
                            int keff, float *out_sh) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < values;
         e += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t j = e / k3;
        const uint32_t a = (uint32_t)(e - j * k3);
        const int32_t *nb = idx + j * (uint32_t)K;
        double acc = 0.0;
#pragma unroll 4
        for (int k = 0; k < keff; ++k) acc += (double)sh1[(uint64_t)k3 * min((uint32_t)nb[k], n1 - 1u) + a];
        out_sh[e] = (float)(acc / (double)keff);
    }
}

uint64_t topk_grid_bytes(uint64_t n1, uint64_t n2, int K) {
    auto up = [](uint64_t x) { return (x + 255) & ~255ull; };
    return up(grid_bytes(n1).bytes) + up(grid_bytes(n2).bytes) + up(4 * n2 * (uint64_t)K);
}

hipError_t launch_topk_grid(uint32_t n1, const float *s1, const float *sh1, uint32_t n2, const float *s2, int k3,
                            int K, float *out_sh, int32_t *idx, uint8_t *ws, hipStream_t st) {
    if (n2 == 0) return hipSuccess;
    if (K < 1 || K > kTopkMax) return hipErrorInvalidValue;
    uint8_t *const g2 = ws + ((grid_bytes(n1).bytes + 255) & ~255ull);
    int32_t *const own = reinterpret_cast<int32_t *>(g2 + ((grid_bytes(n2).bytes + 255) & ~255ull));
    const NnCloud a = grid_cloud(s1, n1, nn_density(K, n2), ws), b = grid_cloud(s2, n2, nn_density(K, n2), g2);
    hipError_t e = launch_grids(a, &b, nullptr, 0, st);
    if (e != hipSuccess) return e;
    NnQuery q = grid_query(b, a, K, n1);
    q.idx = idx ? idx : own;
    e = launch_search<kNnIndex, false>(q, st);
    if (e != hipSuccess) return e;
    const uint64_t values = (uint64_t)n2 * (uint32_t)k3;
    const uint64_t mean_blocks = (values + 255) / 256;
    hipLaunchKernelGGL(k_topk_mean, dim3((uint32_t)(mean_blocks < 65536 ? mean_blocks : 65536)), dim3(256), 0, st, q.idx, sh1, n1,
                       values, (uint32_t)k3, K, q.keff, out_sh);
    return hipGetLastError();
}

}  // namespace dpr
