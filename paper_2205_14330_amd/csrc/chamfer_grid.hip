// The nearest-neighbour searches of the video warm start over a grid of cells
// (nn_grid.h): Eq. (9) in both directions, and the k nearest points of the SH
// transfer.  The results are those of the brute-force search: the same float32
// distances, ties to the lower index, bit for bit (the gradient sums in FP64 in
// the order in which the blocks finish, in either search).
//
// Two frames' clouds are searched through about 45 candidates per point
// instead of the whole other cloud: Eq. (9) with its gradient of two 45k-point
// frames takes 65 us instead of 874, ten Adam steps and the transfer of the 4
// nearest points' SH 773 us instead of 9889.  Of the 65 us 17 are the search;
// the rest is eight launches whose work is mostly shorter than a launch (4 to 5
// us each).
//
// Where the clouds do not allow that (a far point stretches the box, they crowd
// into a few cells, or lie apart), the first pass leaves queries over: those
// that would walk more than an eighth of the points, or more than one thread's
// or 16 lanes' share.  A second kernel searches on for the ones left over, a
// wave each; if they are too many, it searches by brute force for all instead.
// The line is where the two cost the same: 45k points, half of them in one
// cell, and a share of the queries beside these, by brute force 941 us in Eq.
// (9), by wave 917 with 15% and 1280 with 25%; 4 nearest 1290, 904 with 25%, 1175
// with 40% and 1560 with 60%; 8 nearest 2300, 1341 with 40% and 1833 with 60%
// (with a fifth of the points in the cell 940, 894 with 40%; 1280, 1012 with 60%;
// 2290, 1242 with 60%).  So a quarter; half for up to 4 nearest; three quarters.
// Such clouds then cost the grid and its first pass on top of the brute-force
// search.  45k points, brute force alone against this: one point 1000 times as
// far as the others, Eq. (9) 879 and 876 us, 4 nearest 1128 and 1338; three tight
// clusters, each cloud's elsewhere, 1425 and 1407, 865 and 1379 (an eighth is
// walked before it is left); clouds apart, 2564 and 2559, 765 and 776; every
// point the same, 2568 and 2561, 663 and 885.  With a wave for every query,
// however many candidates, the 4 nearest took 3501, 2145, 761 and 3072 us.
#include "nn_brute.h"
#include "nn_grid.h"

#pragma clang fp contract(off)

namespace dpr {

// Brute force below: the grid's launches take some 30 us however small the
// clouds are.  Eq. (9), brute force against grid: 8000 x 8000 points 41 and 45
// us, 12000 x 12000 78 and 47; few points are searched fast however many search
// them: 300 x 300k 116 and 189, 2000 x 45k 63 and 57.
bool chamfer_by_grid(uint64_t n1, uint64_t n2) {
    return (n1 < n2 ? n1 : n2) >= 2000 && (double)n1 * (double)n2 >= 6.4e7;
}
// The k nearest by brute force take a time by n1 and K (lanes walk n1 / 8
// points each), up to some 45k queries.  2000 queries, brute force against grid:
// K = 1, n1 = 1000 37 and 35 us, 1500 48 and 36; K = 4, n1 = 600 35 and 38, 1000
// 46 and 39, 3000 97 and 39; K = 8, n1 = 300
// 44 and 40, 600 62 and 38; K = 16, n1 = 150 69 and 39, 300 87 and 39.
bool topk_by_grid(uint64_t n1, int K) {
    return n1 >= (K == 1 ? 1500u : K <= 4 ? 1000u : K <= 8 ? 600u : 300u);
}

// The most neighbours for which many left over are searched by brute force: a
// wave's list costs the same for any K, the brute force's insertions grow with
// it (45k points in three clusters: K = 12 2.7 ms by brute force, 2.8 by wave;
// with a far point 4.6 and 3.8).
constexpr int kTopkBruteK = 8;
// And the fewest queries: the waves of fewer all run at once, while the brute
// force takes its time whatever their number (45k points, 300 queries, clouds
// apart: 98 us by wave, 656 by brute force; 9000 x 9000 in two blobs, K = 8, 272
// and 432; 45k x 45k in three clusters, K = 4, 2145 and 866, K = 8, 2527 and 1377).
inline uint32_t topk_brute_queries(int K) { return K <= 4 ? 8192u : 32768u; }

// Registers for six waves per SIMD: the blocks of 45k queries by brute force then run all at once.
__global__ __launch_bounds__(kGridThreads, 6) void k_chamfer_rest(NnQuery qa, NnQuery qb, NnJob ja, NnJob jb) {
    __shared__ NnRestLds s;
    const bool first = blockIdx.x < ja.qblocks;
    const NnQuery &q = first ? qa : qb;
    const NnJob &j = first ? ja : jb;
    const uint32_t qblk = first ? blockIdx.x : blockIdx.x - ja.qblocks;
    const uint32_t n = *q.list_n;
    if (n > q.list_most) {
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
    q12.list_most = n1 / 4u;
    q21.list_most = n2 / 4u;
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

// The K nearest, a wave per query; a query that would walk more than q.walk
// candidates is left over.
static __global__ __launch_bounds__(kGridThreads) void k_topk_waves(NnQuery q) {
    __shared__ NnRestLds s;
    __shared__ uint32_t s_at[kRestWaves + 1];
    const uint32_t t = blockIdx.x * (uint32_t)kRestWaves + (threadIdx.x >> 6);
    const bool left = t < q.nq && !nn_rest_wave<kNnIndex, false, false, true>(q, t, s);
    nn_append_left_block<true>(q, left && (threadIdx.x & 63u) == 0, t, s_at);
}

// The queries left over, a wave each; or, if there are many, all queries by
// brute force.
template <int KM>
static __global__ __launch_bounds__(kGridThreads, 6) void k_topk_rest(NnQuery q, const float *s1, uint32_t n1,
                                                                   const float *s2, uint32_t n2) {
    __shared__ NnRestLds s;
    const uint32_t n = *q.list_n;
    if (n > q.list_most) {
        if (blockIdx.x * kTopkQueries >= n2) return;
        unsigned long long best[KM];
        topk_brute(s1, n1, s2, n2, q.K, blockIdx.x, best);
        const uint32_t j = topk_query(blockIdx.x);
        if (j >= n2 || threadIdx.x % (uint32_t)kTopkLanes != 0) return;
#pragma unroll
        for (int k = 0; k < KM; ++k)
            if (k < q.K) q.idx[(size_t)j * q.K + k] = k < q.keff ? (int32_t)(uint32_t)(best[k] & 0xFFFFFFFFull) : -1;
        return;
    }
    for (uint32_t i = blockIdx.x * (uint32_t)kRestWaves + (threadIdx.x >> 6); i < n; i += gridDim.x * (uint32_t)kRestWaves)
        nn_rest_wave<kNnIndex, false>(q, q.list[i], s);
}

static hipError_t topk_search(NnQuery q, const float *s1, uint32_t n1, const float *s2, uint32_t n2, hipStream_t st) {
    if (q.K > kTopkBruteK || n2 < topk_brute_queries(q.K)) return launch_search<kNnIndex, false>(q, st);
    q.list_most = q.K <= 4 ? n2 / 2u : n2 / 4u * 3u;
    const uint32_t eighth = n1 / 8u > 256u ? n1 / 8u : 256u;
    q.walk = q.K == 1 || nn_by_thread(q.K, n2) ? (eighth < kNnMaxWalk ? eighth : kNnMaxWalk) : eighth;
    const dim3 threads(kGridThreads);
    if (q.K == 1) {
        const uint32_t blocks = (n2 + kNearQueries - 1) / kNearQueries;
        hipLaunchKernelGGL((k_nn_nearest<kNnIndex, false>), dim3(blocks), threads, 0, st, q, q, blocks);
    } else if (!nn_by_thread(q.K, n2)) {
        hipLaunchKernelGGL(k_topk_waves, dim3((n2 + kRestWaves - 1) / kRestWaves), threads, 0, st, q);
    } else {
        const dim3 blocks((n2 + kGridThreads - 1) / kGridThreads);
        if (q.K <= 4) hipLaunchKernelGGL((k_nn_query<4, kNnIndex, false>), blocks, threads, 0, st, q);
        else hipLaunchKernelGGL((k_nn_query<8, kNnIndex, false>), blocks, threads, 0, st, q);
    }
    const uint32_t bb = (n2 + kTopkQueries - 1) / kTopkQueries, rb = rest_blocks(n2);
    const dim3 blocks(bb > rb ? bb : rb);
    if (q.K <= 4) hipLaunchKernelGGL(k_topk_rest<4>, blocks, threads, 0, st, q, s1, n1, s2, n2);
    else hipLaunchKernelGGL(k_topk_rest<8>, blocks, threads, 0, st, q, s1, n1, s2, n2);
    return hipGetLastError();
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
    e = topk_search(q, s1, n1, s2, n2, st);
    if (e != hipSuccess) return e;
    const uint64_t values = (uint64_t)n2 * (uint32_t)k3;
    const uint64_t mean_blocks = (values + 255) / 256;
    hipLaunchKernelGGL(k_topk_mean, dim3((uint32_t)(mean_blocks < 65536 ? mean_blocks : 65536)), dim3(256), 0, st, q.idx, sh1, n1,
                       values, (uint32_t)k3, K, q.keff, out_sh);
    return hipGetLastError();
}

}  // namespace dpr
