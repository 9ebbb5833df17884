// The training loss of Eq. (8) for a batch of rendered images and its
// gradient, fused in one pass:
//   L_v = sum_{x,y,c} (R - I)^2 + lambda (sum |R(x+1,y) - R(x,y)| + sum |R(x,y+1) - R(x,y)|)
// (squared L2 plus lambda times the anisotropic total variation, forward
// differences between horizontally and vertically adjacent pixels, Sec. 3.3),
// and dL/dR = 2 (R - I) + lambda (s(R - R_left) - s(R_right - R) + s(R - R_up)
// - s(R_down - R)) with s = sign, s(0) = 0, terms dropped at the border.
//
// An image is a flat array of 3 W H floats; its horizontal neighbours are 3
// floats away and its vertical ones 3 W.  Each thread owns 4 consecutive
// floats and reads them, their horizontal neighbourhood, the target and the
// rows above and below as 16-byte loads; the gradient is written as one
// 16-byte store.  The loads and the store assume 4-byte alignment only, so one
// path serves every width and base address: a row is 3 W floats, so its
// neighbours above and below are rarely 16-byte aligned, and reading those
// float by float, under a branch each, made four 797x803 images take 49 us
// instead of 28.  All six loads are issued together, at addresses clamped to
// the image; the few groups at its ends for which that brings other floats
// than their neighbours read those one by one.  (With each load under a branch
// of its own, and the partial ones into the same registers, the loads waited
// for one another: eight 2048x1024 images 155 us instead of 142.)  A thread's pixel follows from its block's (one 64-bit
// division, uniform over the block) by 32-bit divisions.  The loss terms of a
// float are its squared difference and its differences to the right and lower
// neighbours; a block sums them in FP32, and a second kernel adds each
// image's block sums in FP64 in a fixed order, so the result does not depend
// on scheduling.  With lambda = 0 (the plain L2 loss) no neighbour is read.
// Up to kLossBatch images travel in the kernel arguments.
#include "dpr_internal.h"

namespace dpr {

constexpr int kLossThreads = 256;
constexpr int kLossFloats = 4 * kLossThreads;     // floats per block

struct LossBatch {
    LossImage img[kLossBatch];
    uint32_t block_start[kLossBatch + 1];
    int32_t n;
    float lambda;
    float *partial;      // [block_start[n]]
    double *loss;        // [n]
};

__device__ __forceinline__ float sgn(float d) { return (float)(d > 0.f) - (float)(d < 0.f); }

// Four floats at any float's address (global 16-byte accesses need 4-byte alignment).
typedef float F4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ F4 ld4(const float *p) { return *reinterpret_cast<const F4 *>(p); }

__global__ __launch_bounds__(kLossThreads) void k_loss(LossBatch bt) {
    __shared__ float s_sum[kLossThreads / 64];
    int v = 0;
    while (v + 1 < bt.n && bt.block_start[v + 1] <= blockIdx.x) ++v;
    const LossImage im = bt.img[v];
    const int W = im.width, H = im.height;
    const int64_t nf = 3ll * W * H;
    const int64_t row = 3ll * W;
    const int64_t i0 = (int64_t)(blockIdx.x - bt.block_start[v]) * kLossFloats;     // the block's first float
    const int64_t i = i0 + 4 * threadIdx.x;
    const float lambda = bt.lambda;
    float acc = 0.f;
    if (i < nf) {
        const float *R = im.render, *T = im.target;
        const bool vec = i + 4 <= nf;
        // first float's pixel and channel, from the block's; the 4 floats span at most 2 pixels
        const int64_t pb = i0 / 3;
        const int yb = (int)(pb / W), xb = (int)(pb - (int64_t)yb * W);
        const uint32_t f = (uint32_t)(i0 - 3 * pb) + 4 * threadIdx.x;
        const uint32_t xd = (uint32_t)xb + f / 3;
        const int c0 = (int)(f % 3);
        const int y0 = yb + (int)(xd / (uint32_t)W), x0 = (int)(xd % (uint32_t)W);
        F4 r = 0.f, t = 0.f, up = 0.f, dn = 0.f, lf = 0.f, rt = 0.f;
        // neighbours that the clamped loads below do not bring: the second row begins, or the image or its last row
        // ends, within the group or the next
        bool edge = !vec;
        if (vec) {
            r = ld4(R + i);
            t = ld4(T + i);
            if (lambda != 0.f) {                      // the neighbours enter only the TV term
                lf = ld4(R + max(i - 4, (int64_t)0));
                rt = ld4(R + min(i + 4, nf - 4));
                up = ld4(R + max(i - row, (int64_t)0));
                dn = ld4(R + min(i + row, nf - 4));
                edge = i + 8 > nf || (i < row && i + 4 > row) || (i + row < nf && i + row + 4 > nf);
            }
        }
        float g[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t e = i + k;
            if (e >= nf) { g[k] = 0.f; continue; }
            const int c = c0 + k;
            const bool next = c >= 3;                 // second pixel of the group
            int x = x0 + (next ? 1 : 0), y = y0;
            if (x == W) { x = 0; ++y; }
            float Rv = r[k], Tv = t[k];
            // e - 3 is float k - 3 of the group: k >= 3 in r, else float k + 1 of lf
            float Rl = k >= 3 ? r[0] : lf[(k + 1) & 3];
            // e + 3: float k + 3 of the group: k == 0 in r, else float k - 1 of rt
            float Rr = k == 0 ? r[3] : rt[(k - 1) & 3];
            float Ru = up[k], Rd = dn[k];
            if (__builtin_expect(edge, 0)) {
                Rv = R[e];
                Tv = T[e];
                if (x > 0) Rl = R[e - 3];
                if (x + 1 < W) Rr = R[e + 3];
                if (y > 0) Ru = R[e - row];
                if (y + 1 < H) Rd = R[e + row];
            }
            const float d = Rv - Tv;
            float gr = 2.f * d;
            acc = fmaf(d, d, acc);
            if (x + 1 < W) {
                const float dx = Rr - Rv;
                acc = fmaf(lambda, fabsf(dx), acc);
                gr -= lambda * sgn(dx);
            }
            if (x > 0) gr += lambda * sgn(Rv - Rl);
            if (y + 1 < H) {
                const float dy = Rd - Rv;
                acc = fmaf(lambda, fabsf(dy), acc);
                gr -= lambda * sgn(dy);
            }
            if (y > 0) gr += lambda * sgn(Rv - Ru);
            g[k] = gr;
        }
        if (vec) {
            F4 gv = {g[0], g[1], g[2], g[3]};
            *reinterpret_cast<F4 *>(im.grad + i) = gv;
        } else {
            for (int k = 0; k < 4 && i + k < nf; ++k) im.grad[i + k] = g[k];
        }
    }
    // block sum: within each wave, then across the 4 waves in a fixed order
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) bt.partial[blockIdx.x] = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
}

// One block of kLossSumThreads per image: thread l adds block sums l,
// l + kLossSumThreads, ... in FP64, then a fixed butterfly in each wave and a
// fixed order across the waves combine them.
constexpr int kLossSumThreads = 256;

__global__ __launch_bounds__(kLossSumThreads) void k_loss_sum(LossBatch bt) {
    __shared__ double s_w[kLossSumThreads / 64];
    const int v = blockIdx.x;
    const uint32_t b0 = bt.block_start[v], b1 = bt.block_start[v + 1];
    double s = 0.0;
#pragma unroll 8
    for (uint32_t b = b0 + threadIdx.x; b < b1; b += kLossSumThreads) s += (double)bt.partial[b];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) bt.loss[v] = (s_w[0] + s_w[1]) + (s_w[2] + s_w[3]);
}

uint32_t loss_blocks(int32_t width, int32_t height) {
    const uint64_t nf = 3ull * (uint64_t)width * (uint64_t)height;
    return (uint32_t)((nf + kLossFloats - 1) / kLossFloats);
}

hipError_t launch_loss(const LossImage *img, int n, float lambda, float *partial, double *loss, hipStream_t st) {
    for (int b0 = 0; b0 < n; b0 += kLossBatch) {
        LossBatch bt;
        bt.n = n - b0 < kLossBatch ? n - b0 : kLossBatch;
        bt.lambda = lambda;
        uint32_t blocks = 0;
        for (int v = 0; v < bt.n; ++v) {
            bt.img[v] = img[b0 + v];
            bt.block_start[v] = blocks;
            blocks += loss_blocks(img[b0 + v].width, img[b0 + v].height);
        }
        bt.block_start[bt.n] = blocks;
        bt.partial = partial;
        bt.loss = loss + b0;
        hipLaunchKernelGGL(k_loss, dim3(blocks), dim3(kLossThreads), 0, st, bt);
        hipLaunchKernelGGL(k_loss_sum, dim3(bt.n), dim3(kLossSumThreads), 0, st, bt);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace dpr
