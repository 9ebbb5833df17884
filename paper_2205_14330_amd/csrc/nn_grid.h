// Exact nearest neighbours over a uniform grid of cubic cells, shared by the
// neighbour search of Alg. 1 (one cloud searched for its own points) and by
// the video warm start (the points of one cloud searched in another).
//
// Building (five launches, for one cloud or two at once):
//   prep    : the box of the points, per block; scratch cleared;
//   occupy  : which cells of a coarse grid hold a point.  The occupied share
//             of the box sets the cell size, so that a cell where points are
//             holds about `density` of them, also when a few far points
//             stretch the box or the points lie on a surface;
//   count   : the points of every cell, and each point's place in its cell;
//   rows    : places for the cells of a row (consecutive x) one after the
//             other, the rows in any order (an atomic cursor per block of
//             rows), which saves the two launches of a full scan;
//   scatter : (x, y, z, index) of every point at its place, so the candidates
//             of a run of cells are consecutive 16-byte loads.
// Searching: one thread per query, in cell order, walks the 3x3 rows of three
// cells around it, nearest rows first, skips rows farther than the K-th so
// far, and keeps the K smallest keys (d2 bits << 32 | index).  It is done if
// the K-th distance is below the distance to the nearest face of the walked
// cube; if it is below that of the next cube, the thread also walks the parts
// of that shell that are closer than the K-th.  Queries that need more (far
// points), or whose cube holds more than kNnMaxWalk candidates (tight
// clusters), go to a list, and a second kernel gives each a whole wave and a
// growing cube.  (One nearest: 16 lanes per query; few queries or more than 8
// nearest: a wave each at once.)  Neither the order of the points in a cell nor
// that of the rows changes a result: the keys are distinct and totally ordered.
//
// A point that is not finite lies in the border cells of its axes and is
// searched like any other: its distances are infinite or NaN, which sort behind
// the finite ones, so a query that has too few of these walks the whole grid.
//
// The float32 distance ((dx dx + dy dy) + dz dz) rounds each operation once.
//
// Bound by the loads' latency and by the lists' upkeep, not by memory: the 8
// nearest of 255k points take 131 us by thread (51M wave instructions, 50 per
// candidate, of which most keep the list), their 33 MB of input and output 6.
#pragma once

#include <cmath>

#include "dpr_internal.h"
#include "nn_brute.h"

namespace dpr {

constexpr int kGridThreads = 256;
constexpr int kGridItems = 4 * kGridThreads;            // points per counting block
constexpr uint32_t kGridBoxBlocks = 128;                // blocks of the box reduction, per cloud
constexpr uint32_t kOccAxis = 32;                       // coarse cells per axis, at most
constexpr uint32_t kOccWords = kOccAxis * kOccAxis * kOccAxis / 32;
// Points per occupied coarse cell (some 17 in a filled box, 600 of 10M points)
// above which the cloud crowds into few cells.
constexpr uint32_t kCrowd = 640;
constexpr uint32_t kNnMaxWalk = 1024;                   // candidates a single thread walks

struct GridGeom {
    float lo[3];                // -infinity on an axis without a finite extent: one cell, which ends nowhere
    float h, inv;               // cell edge and its inverse (0: one cell)
    float hs;                   // the edge as the bounds on distances take it; 0, which bounds nothing, if its
                                // square would leave the range in which the distances' rounding is relative
    uint32_t nx, ny, nz;
};

// One cloud and its grid (pointers into scratch).
struct NnCloud {
    const float *xyz;
    uint32_t n;
    uint32_t occ_axis;          // coarse cells per axis
    uint32_t max_cells;
    uint32_t box_blocks;        // blocks of the box reduction
    float density;              // points per occupied cell to aim at
    float *part;                // [6 kGridBoxBlocks]
    uint32_t *occ;              // [kOccWords]
    GridGeom *geom;
    uint32_t *cursor;           // [2]: places given to rows; queries of this cloud left for a wave each
    uint32_t *table;            // [max_cells]: row-major cells, nx + 1 entries per row
    uint32_t *cell, *rank;      // [n] each; after the scatter, cell lists the queries left over
    float4 *pts;                // [n] sorted by cell: x, y, z, index bits
};

inline uint32_t grid_max_cells(uint64_t n) { return (uint32_t)(4 * n + 64 < 0x7FFFFF00ull ? 4 * n + 64 : 0x7FFFFF00ull); }
inline uint32_t grid_occ_axis(uint64_t n) {
    uint32_t g = 1;             // about 8 points per coarse cell of a filled box
    while (g < kOccAxis && 8ull * (g + 1) * (g + 1) * (g + 1) <= n) ++g;
    return g;
}

// K nearest, K > 1: a thread per query, or a wave.  A thread's list of up to 8
// keys stays in registers, but 64k queries are one wave per SIMD, whose loads
// nothing hides: the 8 nearest of 45k points of a ball take 115 us by thread
// and 85 us by wave, of 100k points 119 and 147, of 300k points 206 and 377.
// Longer lists are spread over the wave's lanes at any size (the 32 nearest of
// 300k points: 3762 us by thread, 820 by wave).
inline bool nn_by_thread(int K, uint64_t queries) { return K > 1 && K <= 8 && queries >= 65536; }

// Points per occupied cell to aim at: 27 cells then hold enough of them that
// the K nearest mostly lie closer than the cube's faces; a wave, which goes on
// to the next shell by itself, does best with fewer (measured at 0.15, 0.25 and
// 0.4 K on filled and surface clouds of 3k to 300k points).
inline float nn_density(int K, uint64_t queries) {
    return fmaxf(1.5f, (nn_by_thread(K, queries) ? 0.4f : 0.2f) * (float)K);
}

// Byte layout of a cloud's grid inside one buffer: 16-byte aligned regions from
// the first 16-byte aligned address on (a caller's workspace may begin anywhere).
struct GridBytes {
    uint64_t part, occ, geom, cursor, table, cell, rank, pts, bytes;
};
inline GridBytes grid_bytes(uint64_t n) {
    GridBytes b;
    uint64_t off = 0;
    auto add = [&](uint64_t bytes) {
        const uint64_t at = off;
        off += (bytes + 15) & ~15ull;
        return at;
    };
    b.pts = add(16 * n);
    b.part = add(4 * 6 * (uint64_t)kGridBoxBlocks);
    b.occ = add(4 * (uint64_t)kOccWords);
    b.geom = add(sizeof(GridGeom));
    b.cursor = add(8);
    b.table = add(4 * (uint64_t)grid_max_cells(n));
    b.cell = add(4 * n);
    b.rank = add(4 * n);
    b.bytes = off + 15;
    return b;
}

inline NnCloud grid_cloud(const float *xyz, uint64_t n, float density, uint8_t *ws) {
    const GridBytes b = grid_bytes(n);
    ws += (16 - ((uintptr_t)ws & 15)) & 15;
    NnCloud c;
    c.xyz = xyz;
    c.n = (uint32_t)n;
    c.occ_axis = grid_occ_axis(n);
    c.max_cells = grid_max_cells(n);
    c.box_blocks = (uint32_t)(n < (uint64_t)kGridItems * kGridBoxBlocks ? (n + kGridItems - 1) / kGridItems : kGridBoxBlocks);
    c.density = density;
    c.part = reinterpret_cast<float *>(ws + b.part);
    c.occ = reinterpret_cast<uint32_t *>(ws + b.occ);
    c.geom = reinterpret_cast<GridGeom *>(ws + b.geom);
    c.cursor = reinterpret_cast<uint32_t *>(ws + b.cursor);
    c.table = reinterpret_cast<uint32_t *>(ws + b.table);
    c.cell = reinterpret_cast<uint32_t *>(ws + b.cell);
    c.rank = reinterpret_cast<uint32_t *>(ws + b.rank);
    c.pts = reinterpret_cast<float4 *>(ws + b.pts);
    return c;
}

// LDS written before by any lane of the wave is readable after, and the other way round.
__device__ __forceinline__ void nn_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Cell of coordinate t (in cells from the grid's origin) on an axis of n cells;
// NaN and points outside go to the nearest border cell.
__device__ __forceinline__ uint32_t grid_axis(float t, uint32_t n) {
    if (!(t > 0.f)) return 0u;
    return t >= (float)n ? n - 1u : min((uint32_t)t, n - 1u);
}

// Minimum (a < 3) and maximum over the block of six values per thread, in s_box.
__device__ __forceinline__ void grid_block_box(float lo[3], float hi[3], float (*s_w)[kGridThreads / 64], float *s_box) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            lo[a] = fminf(lo[a], __shfl_xor(lo[a], d, 64));
            hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], d, 64));
        }
    }
    if ((threadIdx.x & 63) == 0)
        for (int a = 0; a < 3; ++a) { s_w[a][threadIdx.x >> 6] = lo[a]; s_w[3 + a][threadIdx.x >> 6] = hi[a]; }
    __syncthreads();
    if (threadIdx.x < 6) {
        float v = s_w[threadIdx.x][0];
        for (int w = 1; w < kGridThreads / 64; ++w)
            v = threadIdx.x < 3 ? fminf(v, s_w[threadIdx.x][w]) : fmaxf(v, s_w[threadIdx.x][w]);
        s_box[threadIdx.x] = v;
    }
    __syncthreads();
}

// The cloud's box from its partials (every block computes the same).
__device__ __forceinline__ void grid_box(const NnCloud &c, float (*s_w)[kGridThreads / 64], float *s_box) {
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (threadIdx.x < c.box_blocks) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = c.part[6 * threadIdx.x + a];
            hi[a] = c.part[6 * threadIdx.x + 3 + a];
        }
    }
    grid_block_box(lo, hi, s_w, s_box);
}

// Also clears zero[0 .. n_zero).
static __global__ __launch_bounds__(kGridThreads) void k_grid_prep(NnCloud a, NnCloud b, uint32_t *zero,
                                                                   uint64_t n_zero) {
    __shared__ float s_w[6][kGridThreads / 64];
    __shared__ float s_box[6];
    const bool first = blockIdx.x < a.box_blocks;
    const uint32_t bid = first ? blockIdx.x : blockIdx.x - a.box_blocks;
    const NnCloud &c = first ? a : b;
    const uint32_t i0 = bid * kGridThreads + threadIdx.x, step = c.box_blocks * kGridThreads;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
#pragma unroll 4
    for (uint32_t i = i0; i < c.n; i += step) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float v = c.xyz[3 * (size_t)i + k];
            lo[k] = fminf(lo[k], v);
            hi[k] = fmaxf(hi[k], v);
        }
    }
    for (uint32_t i = i0; i < kOccWords; i += step) c.occ[i] = 0u;
    if (i0 < 2u) c.cursor[i0] = 0u;
    for (uint64_t i = (uint64_t)blockIdx.x * kGridThreads + threadIdx.x; i < n_zero;
         i += (uint64_t)gridDim.x * kGridThreads)
        zero[i] = 0u;
    grid_block_box(lo, hi, s_w, s_box);
    if (threadIdx.x < 6) c.part[6 * bid + threadIdx.x] = s_box[threadIdx.x];
}

// Occupied coarse cells; also clears the cell table.
static __global__ __launch_bounds__(kGridThreads) void k_grid_occupy(NnCloud a, NnCloud b, uint32_t blocks_a,
                                                                     uint32_t blocks_b) {
    __shared__ float s_w[6][kGridThreads / 64];
    __shared__ float s_box[6];
    __shared__ uint32_t s_occ[kOccWords];
    const bool first = blockIdx.x < blocks_a;
    const uint32_t bid = first ? blockIdx.x : blockIdx.x - blocks_a;
    const uint32_t nb = first ? blocks_a : blocks_b;
    const NnCloud &c = first ? a : b;
    const uint32_t words = (c.occ_axis * c.occ_axis * c.occ_axis + 31u) / 32u;
    for (uint32_t i = threadIdx.x; i < words; i += kGridThreads) s_occ[i] = 0u;
    grid_box(c, s_w, s_box);
    float s[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float e = s_box[3 + k] - s_box[k];
        s[k] = e > 0.f ? (float)c.occ_axis / e : 0.f;
    }
    const uint32_t i0 = bid * kGridThreads + threadIdx.x, step = nb * kGridThreads;
#pragma unroll 4
    for (uint32_t i = i0; i < c.n; i += step) {
        uint32_t q[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) q[k] = grid_axis((c.xyz[3 * (size_t)i + k] - s_box[k]) * s[k], c.occ_axis);
        const uint32_t o = (q[2] * c.occ_axis + q[1]) * c.occ_axis + q[0];
        atomicOr(&s_occ[o >> 5], 1u << (o & 31u));
    }
    for (uint64_t i = i0; i < c.max_cells; i += step) c.table[i] = 0u;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < words; i += kGridThreads)
        if (s_occ[i]) atomicOr(&c.occ[i], s_occ[i]);
}

// Cell size and counts per axis from the box and the number of occupied
// coarse cells.  The cell edge is that of `density` points in the occupied
// volume; an axis shorter than the edge counts as one cell and drops out.
__device__ __forceinline__ GridGeom grid_geometry(const NnCloud &c, const float *box, uint32_t occupied) {
    GridGeom g;
    float e[3];
    for (int k = 0; k < 3; ++k) {
        const float d = box[3 + k] - box[k];
        g.lo[k] = d >= 0.f && d < INFINITY ? box[k] : -INFINITY;
        e[k] = d > 0.f && d < INFINITY ? d : 0.f;
    }
    const float m0 = fmaxf(e[0], fmaxf(e[1], e[2])), m2 = fminf(e[0], fminf(e[1], e[2]));
    const float m1 = fmaxf(fminf(e[0], e[1]), fminf(fmaxf(e[0], e[1]), e[2]));
    g.nx = g.ny = g.nz = 1u;
    g.h = g.inv = g.hs = 0.f;
    if (!(m0 > 0.f)) return g;
    const float G = (float)c.occ_axis;
    const float cells = fmaxf((float)c.n / c.density, 1.f);
    // relative to the longest edge, so that no product over- or underflows
    const float r1 = m1 / m0, r2 = m2 / m0;
    float x = cbrtf(r1 * r2 * fminf((float)occupied / (G * G * G), 1.f) / cells);
    if (!(x <= r2)) {
        x = sqrtf(r1 * fminf((float)occupied / (G * G), 1.f) / cells);
        if (!(x <= r1)) x = fminf((float)occupied / G, 1.f) / cells;
    }
    float h = m0 * fmaxf(x, 1e-6f);
    for (int it = 0; it < 256; ++it, h = h * 1.1f) {
        const float inv = 1.f / h;
        if (!(inv > 0.f && inv < INFINITY)) continue;
        const float fx = floorf(e[0] * inv) + 1.f, fy = floorf(e[1] * inv) + 1.f, fz = floorf(e[2] * inv) + 1.f;
        if ((fx + 1.f) * fy * fz <= 0.999f * (float)c.max_cells) {      // nx + 1 table entries per row
            g.h = h;
            g.inv = inv;
            const float hs = 0.9999f * h;
            g.hs = hs * hs >= 1e-36f && hs * hs < INFINITY ? hs : 0.f;
            g.nx = (uint32_t)fx;
            g.ny = (uint32_t)fy;
            g.nz = (uint32_t)fz;
            break;
        }
    }
    return g;
}

__device__ __forceinline__ uint32_t grid_cell(const GridGeom &g, float x, float y, float z) {
    const uint32_t cx = grid_axis((x - g.lo[0]) * g.inv, g.nx);
    const uint32_t cy = grid_axis((y - g.lo[1]) * g.inv, g.ny);
    const uint32_t cz = grid_axis((z - g.lo[2]) * g.inv, g.nz);
    return (cz * g.ny + cy) * (g.nx + 1u) + cx;
}

static __global__ __launch_bounds__(kGridThreads) void k_grid_count(NnCloud a, NnCloud b, uint32_t blocks_a) {
    __shared__ float s_w[6][kGridThreads / 64];
    __shared__ float s_box[6];
    __shared__ uint32_t s_n[kGridThreads / 64];
    constexpr int kPer = kGridItems / kGridThreads;
    __shared__ uint32_t s_cell[kGridThreads / 64][64];
    __shared__ GridGeom s_g;
    __shared__ bool s_crowd;
    const bool first = blockIdx.x < blocks_a;
    const uint32_t bid = first ? blockIdx.x : blockIdx.x - blocks_a;
    const NnCloud &c = first ? a : b;
    // the block's points, in flight while the geometry is worked out
    float p[kGridItems / kGridThreads][3];
#pragma unroll
    for (int k = 0; k < kGridItems / kGridThreads; ++k) {
        const uint32_t i = bid * (uint32_t)kGridItems + (uint32_t)k * kGridThreads + threadIdx.x;
#pragma unroll
        for (int d = 0; d < 3; ++d) p[k][d] = i < c.n ? c.xyz[3 * (size_t)i + d] : 0.f;
    }
    uint32_t occupied = 0;
    const uint32_t words = (c.occ_axis * c.occ_axis * c.occ_axis + 31u) / 32u;
    for (uint32_t i = threadIdx.x; i < words; i += kGridThreads) occupied += (uint32_t)__popc(c.occ[i]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) occupied += __shfl_xor(occupied, d, 64);
    if ((threadIdx.x & 63) == 0) s_n[threadIdx.x >> 6] = occupied;
    grid_box(c, s_w, s_box);
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int w = 0; w < kGridThreads / 64; ++w) t += s_n[w];
        s_g = grid_geometry(c, s_box, t);
        s_crowd = c.n / kCrowd > t;
        if (bid == 0) *c.geom = s_g;
    }
    __syncthreads();
    const GridGeom g = s_g;
    if (!s_crowd) {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const uint32_t i = bid * (uint32_t)kGridItems + (uint32_t)k * kGridThreads + threadIdx.x;
            if (i < c.n) {
                const uint32_t cl = grid_cell(g, p[k][0], p[k][1], p[k][2]);
                c.cell[i] = cl;
                c.rank[i] = atomicAdd(c.table + cl, 1u);
            }
        }
        return;
    }
    // groups of the wave's points in one cell take their places by one atomic each, as a cell's atomics take 10 ns each
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
#pragma unroll 1
    for (int k = 0; k < kPer; ++k) {
        const uint32_t i = bid * (uint32_t)kGridItems + (uint32_t)k * kGridThreads + threadIdx.x;
        const uint32_t cl = grid_cell(g, p[k][0], p[k][1], p[k][2]);
        s_cell[wave][lane] = cl;
        nn_wave_sync();
        uint64_t todo = __ballot(i < c.n);
        uint32_t lead = lane, at = 0, many = 1;
        for (int round = 0; round < 16 && todo != 0ull; ++round) {
            const uint32_t l = (uint32_t)__builtin_ctzll(todo);
            const uint64_t m = __ballot(((todo >> lane) & 1ull) != 0ull && s_cell[wave][l] == cl);
            const uint32_t in_cell = (uint32_t)__popcll(m);
            if (in_cell < 5u) break;                      // small groups, one by one
            if ((m >> lane) & 1ull) {
                lead = l;
                at = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                many = in_cell;
            }
            todo &= ~m;
        }
        nn_wave_sync();
        if (i < c.n && lead == lane) s_cell[wave][lane] = atomicAdd(c.table + cl, many);
        nn_wave_sync();
        if (i < c.n) {
            c.cell[i] = cl;
            c.rank[i] = s_cell[wave][lead] + at;
        }
        nn_wave_sync();
    }
}

// In place: counts -> first place of every cell; the entry after a row's last
// cell is the row's end.
static __global__ __launch_bounds__(kGridThreads) void k_grid_rows(NnCloud a, NnCloud b, uint32_t blocks_a,
                                                                   uint32_t blocks_b) {
    constexpr uint32_t kWaves = kGridThreads / 64;
    __shared__ uint32_t s_tot[kWaves], s_base;
    const bool first = blockIdx.x < blocks_a;
    const uint32_t bid = first ? blockIdx.x : blockIdx.x - blocks_a;
    const uint32_t nb = first ? blocks_a : blocks_b;
    const NnCloud &c = first ? a : b;
    const GridGeom g = *c.geom;
    const uint32_t rows = g.ny * g.nz, wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    for (uint32_t row0 = bid * kWaves; row0 < rows; row0 += nb * kWaves) {
        const uint32_t row = row0 + wave;
        uint32_t *const t = c.table + (uint64_t)row * (g.nx + 1u);
        uint32_t tot = 0;
        if (row < rows) {
#pragma unroll 4
            for (uint32_t x = lane; x < g.nx; x += 64u) tot += t[x];
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) tot += __shfl_xor(tot, d, 64);
        if (lane == 0) s_tot[wave] = tot;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t s = 0;
            for (uint32_t w = 0; w < kWaves; ++w) s += s_tot[w];
            s_base = s ? atomicAdd(c.cursor, s) : 0u;
        }
        __syncthreads();
        uint32_t run = s_base;
        for (uint32_t w = 0; w < wave; ++w) run += s_tot[w];
        if (row < rows) {
            for (uint32_t x0 = 0; x0 < g.nx; x0 += 64u) {
                const uint32_t x = x0 + lane;
                const uint32_t v = x < g.nx ? t[x] : 0u;
                uint32_t incl = v, all = v;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const uint32_t o = __shfl_up(incl, d, 64);
                    if (lane >= (uint32_t)d) incl += o;
                }
#pragma unroll
                for (int d = 32; d >= 1; d >>= 1) all += __shfl_xor(all, d, 64);
                if (x < g.nx) t[x] = run + incl - v;
                run += all;
            }
            if (lane == 0) t[g.nx] = run;
        }
        __syncthreads();
    }
}

static __global__ __launch_bounds__(kGridThreads) void k_grid_scatter(NnCloud a, NnCloud b, uint32_t blocks_a) {
    const bool first = blockIdx.x < blocks_a;
    const uint32_t bid = first ? blockIdx.x : blockIdx.x - blocks_a;
    const NnCloud &c = first ? a : b;
#pragma unroll
    for (int k = 0; k < kGridItems / kGridThreads; ++k) {
        const uint32_t i = bid * (uint32_t)kGridItems + (uint32_t)k * kGridThreads + threadIdx.x;
        if (i < c.n)
            c.pts[c.table[c.cell[i]] + c.rank[i]] = make_float4(c.xyz[3 * (size_t)i], c.xyz[3 * (size_t)i + 1],
                                                               c.xyz[3 * (size_t)i + 2], __uint_as_float(i));
    }
}

// Queries searched in a cloud's grid.
enum { kNnKey = 0, kNnIndex = 1, kNnIndexDist = 2, kNnSpread = 3 };
struct NnQuery {
    const float4 *q;            // queries in cell order: x, y, z, index bits
    uint32_t nq;
    int K, keff;                // keff = min(K, candidates)
    const GridGeom *geom;       // the searched cloud
    const uint32_t *table;
    const float4 *pts;
    uint32_t *list, *list_n;    // [nq] queries left for a wave each, their number (cleared before)
    uint32_t list_most;         // if there are more, the list is not read: the search is done otherwise
    uint32_t walk;              // candidates beyond which a query is left over
    // outputs, by the query's index
    unsigned long long *key;    // kNnKey: the nearest's (d2 bits << 32 | index), ~0 if none is at a finite distance
    int32_t *idx;               // kNnIndex, kNnIndexDist, kNnSpread: [nq][K], -1 past keff
    float *d2;                  // kNnIndexDist: [nq][K], 0 past keff
    uint32_t *keep;             // kNnSpread: 1 if the spread of the distances is at most eps
    float eps;
    // a search among the points that alive marks (FILTERED): the indices written, and the rows they are written to,
    // are pos[] of the points', ascending with them
    const uint32_t *alive, *pos;
};

// 0 if delta, the standard deviation of the keff neighbour distances, exceeds
// eps: float32, each operation rounded, in neighbour order.
template <int KMAX = kKnnMax>
__device__ __forceinline__ uint32_t nn_spread_keep(const NnQuery &a, const unsigned long long *best) {
#pragma clang fp contract(off)
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        if (k < a.keff) sum = sum + sqrtf(__uint_as_float((uint32_t)(best[k] >> 32)));
    const float mean = __fdiv_rn(sum, (float)a.keff);
    float var = 0.f;
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        if (k < a.keff) {
            const float e = sqrtf(__uint_as_float((uint32_t)(best[k] >> 32))) - mean;
            var = var + e * e;
        }
    const float delta = sqrtf(__fdiv_rn(var, (float)a.keff));
    return a.keff > 0 && delta > a.eps ? 0u : 1u;
}

// The nearest's key, ~0 (none) if it is at no finite distance, as in nn_brute.
__device__ __forceinline__ unsigned long long nn_finite(unsigned long long key) {
    return key < 0x7F800000ull << 32 ? key : ~0ull;
}

// The results of one query (one lane).
template <int KMAX, int MODE>
__device__ __forceinline__ void nn_write(const NnQuery &a, uint32_t i, const unsigned long long (&best)[KMAX]) {
    if (MODE == kNnKey) {
        a.key[i] = nn_finite(best[0]);
        return;
    }
    if (MODE == kNnSpread) a.keep[i] = nn_spread_keep<KMAX>(a, best);
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        if (k < a.K) {
            a.idx[(size_t)i * a.K + k] = k < a.keff ? (int32_t)(uint32_t)(best[k] & 0xFFFFFFFFull) : -1;
            if (MODE == kNnIndexDist)
                a.d2[(size_t)i * a.K + k] = k < a.keff ? __uint_as_float((uint32_t)(best[k] >> 32)) : 0.f;
        }
}

// Far above the float32 rounding of the cell coordinates of points in the grid
// (at most 2^-21 of them), in cells.
__device__ __forceinline__ float nn_margin(const GridGeom &g) {
    return 2e-3f + 2e-6f * (float)max(g.nx, max(g.ny, g.nz));
}

// The squared distance below which no point outside the cube of r cells around
// (cx, cy, cz) can be: the nearest face that has cells behind it, in cells from
// the query at (tx, ty, tz), less margins for the rounding of the cell
// coordinates and of the distances.  Infinite if, and only if, the cube holds
// the whole grid: a face at no finite distance (the query is not finite, or far
// beyond the grid, so that its distances are infinite or NaN) bounds nothing.
__device__ __forceinline__ float nn_bound(const GridGeom &g, float tx, float ty, float tz, int cx, int cy, int cz, int r) {
    constexpr float kMost = 3.4028235e38f;               // the largest finite value
    const bool xl = cx - r > 0, yl = cy - r > 0, zl = cz - r > 0;
    const bool xh = cx + r + 1 < (int)g.nx, yh = cy + r + 1 < (int)g.ny, zh = cz + r + 1 < (int)g.nz;
    float f = kMost;
    f = xl ? fminf(f, tx - (float)(cx - r)) : f;
    f = yl ? fminf(f, ty - (float)(cy - r)) : f;
    f = zl ? fminf(f, tz - (float)(cz - r)) : f;
    f = xh ? fminf(f, (float)(cx + r + 1) - tx) : f;
    f = yh ? fminf(f, (float)(cy + r + 1) - ty) : f;
    f = zh ? fminf(f, (float)(cz + r + 1) - tz) : f;
    f = fmaxf(f - nn_margin(g), 0.f) * g.hs;
    return xl || yl || zl || xh || yh || zh ? fminf(f * f, kMost) : INFINITY;
}

// Four candidates from i on, the last of the run repeated past its end.
__device__ __forceinline__ void nn_load4(const float4 *pts, uint32_t i, uint32_t end, float4 (&p)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) p[u] = pts[min(i + u, end - 1u)];
}

// Key of a candidate, ~0 if it is not one.
template <bool SELF>
__device__ __forceinline__ float nn_between(const float4 &q, const float4 &p) {
    return SELF ? nn_dist2(p.x, p.y, p.z, q.x, q.y, q.z) : nn_dist2(q.x, q.y, q.z, p.x, p.y, p.z);
}
template <bool SELF>
__device__ __forceinline__ unsigned long long nn_key(const float4 &q, const float4 &p, bool ok) {
    const float d = nn_between<SELF>(q, p);
    return ok ? ((unsigned long long)__float_as_uint(d) << 32) | __float_as_uint(p.w) : ~0ull;
}

// One lane's candidates [run.x, run.y).
template <int KMAX, bool SELF>
__device__ __forceinline__ void nn_walk(const NnQuery &a, const float4 &q, uint2 run, unsigned long long (&best)[KMAX],
                                        unsigned long long &worst) {
    const uint32_t self = __float_as_uint(q.w);
    for (uint32_t i = run.x; i < run.y; i += 4u) {
        float4 p[4];
        nn_load4(a.pts, i, run.y, p);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            nn_insert<KMAX>(best, a.keff, nn_key<SELF>(q, p[u], i + u < run.y && (!SELF || __float_as_uint(p[u].w) != self)),
                            worst);
    }
}

// The candidates of every lane's 9 runs (s_run), the lanes in step: each step
// takes four candidates of the lane's current run, the next four loaded before
// they are tested, and a lane that ends a run goes on to its next one, so no
// lane waits for another's longer row.  Keys below the K-th so far are put
// aside in the lane's column of s_buf; when a lane's column is full, all lanes
// insert what they hold.  (An insertion costs the whole wave some 6 KMAX
// instructions whether one lane needs it or all do.)  far(k): the squared
// distance to row k; a farther row than the K-th so far is skipped.
constexpr int kNnBuf = 8;
template <int KMAX, bool SELF, class FAR>
__device__ __forceinline__ void nn_walk_runs(const NnQuery &a, const float4 &q, bool more, const FAR &far,
                                             const uint2 (*s_run)[kGridThreads],
                                             unsigned long long (*s_buf)[kGridThreads],
                                             unsigned long long (&best)[KMAX], unsigned long long &worst) {
    const uint32_t self = __float_as_uint(q.w), tid = threadIdx.x;
    uint2 run = make_uint2(0u, 0u);
    int row = 0, held = 0;
    // the next run with candidates (none left: an empty one)
    auto next = [&]() {
        const float kth = __uint_as_float((uint32_t)(worst >> 32));
        while (run.x >= run.y && row < 9) {
            if (!(far(row) > kth)) run = s_run[row][tid];
            ++row;
        }
    };
    if (more) next();
    more = more && run.x < run.y;
    float4 p[4];
    if (more) nn_load4(a.pts, run.x, run.y, p);
    while (__ballot(more) != 0ull) {
        float4 c[4];
        const uint32_t n = more ? run.y - run.x : 0u;
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = p[u];
        if (more) {
            run.x += 4u;
            next();
            more = run.x < run.y;
            if (more) nn_load4(a.pts, run.x, run.y, p);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const unsigned long long x = nn_key<SELF>(q, c[u], (uint32_t)u < n && (!SELF || __float_as_uint(c[u].w) != self));
            if (x < worst) s_buf[held++][tid] = x;
        }
        if (__ballot(held > kNnBuf - 4) != 0ull || __ballot(more) == 0ull) {
#pragma unroll 1
            for (int k = 0; k < held; ++k) nn_insert<KMAX>(best, a.keff, s_buf[k][tid], worst);
            held = 0;
        }
    }
}

// The queries t left over, appended to the list wave by wave.
__device__ __forceinline__ void nn_append_left(const NnQuery &a, bool left, uint32_t t, uint32_t *s_at) {
    const uint32_t tid = threadIdx.x;
    const uint64_t rest = __ballot(left);
    if (rest != 0ull) {
        if ((tid & 63u) == (uint32_t)__builtin_ctzll(rest)) s_at[tid >> 6] = atomicAdd(a.list_n, (uint32_t)__popcll(rest));
        nn_wave_sync();
        if (left && a.key) a.key[__float_as_uint(a.q[t].w)] = ~0ull;     // for a search by brute force
        if (left) a.list[s_at[tid >> 6] + (uint32_t)__popcll(rest & ((1ull << (tid & 63u)) - 1ull))] = t;
    }
}

// The same block by block, where a wave has few queries (s: a word per wave and
// one): the atomics on one address take 10 ns each.  CHECK: none once the list
// is longer than it is read; the look at its length is a round trip to memory
// more, so only where few blocks leave queries over or nearly all do.
template <bool CHECK>
__device__ __forceinline__ void nn_append_left_block(const NnQuery &a, bool left, uint32_t t, uint32_t *s) {
    constexpr uint32_t kWaves = kGridThreads / 64;
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    const uint64_t rest = __ballot(left);
    if (lane == 0) s[wave] = (uint32_t)__popcll(rest);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t n = 0;
        for (uint32_t w = 0; w < kWaves; ++w) n += s[w];
        if (n) {
            const bool full = CHECK && *(const volatile uint32_t *)a.list_n > a.list_most;
            s[kWaves] = full ? 0xFFFFFFFFu : atomicAdd(a.list_n, n);
        }
    }
    __syncthreads();
    if (left) {
        if (a.key) a.key[__float_as_uint(a.q[t].w)] = ~0ull;             // for a search by brute force
        uint32_t at = s[kWaves];
        if (!CHECK || at != 0xFFFFFFFFu) {
            for (uint32_t w = 0; w < wave; ++w) at += s[w];
            a.list[at + (uint32_t)__popcll(rest & ((1ull << lane) - 1ull))] = t;
        }
    }
}

// Run k (0 .. 33) of the shell between the cubes of 1 and 2 cells around a
// query's cell, if it has points closer than the K-th: 16 outer rows, then the
// two ends of the 9 inner rows.
__device__ __forceinline__ uint2 nn_shell_run(const NnQuery &a, const GridGeom &g, int k, float tx, float ty, float tz,
                                              int cx, int cy, int cz, float m, float hs, float kth) {
    // k < 16: outer row o of the 25; else inner row (k - 16) / 2, its end (k - 16) & 1
    const int o = k < 5 ? k : k < 10 ? k + 15 : k < 13 ? 5 * (k - 9) : 5 * (k - 12) + 4;
    const int in = (k - 16) >> 1;
    const int dy = (k < 16 ? o % 5 : in % 3 + 1) - 2, dz = (k < 16 ? o / 5 : in / 3 + 1) - 2;
    const int y = cy + dy, z = cz + dz;
    if (y < 0 || y >= (int)g.ny || z < 0 || z >= (int)g.nz) return make_uint2(0u, 0u);
    const int u = k < 16 ? max(cx - 2, 0) : k & 1 ? cx + 2 : cx - 2;
    const int v = k < 16 ? min(cx + 2, (int)g.nx - 1) : u;
    if (u < 0 || v >= (int)g.nx) return make_uint2(0u, 0u);
    const float fy = dy == 0 ? 0.f : fmaxf((dy < 0 ? ty - (float)(y + 1) : (float)y - ty) - m, 0.f);
    const float fz = dz == 0 ? 0.f : fmaxf((dz < 0 ? tz - (float)(z + 1) : (float)z - tz) - m, 0.f);
    const float fx = k < 16 ? 0.f : fmaxf((k & 1 ? (float)(cx + 2) - tx : tx - (float)(cx - 1)) - m, 0.f);
    if ((fy * fy + fz * fz + fx * fx) * hs * hs > kth) return make_uint2(0u, 0u);
    const uint32_t *row = a.table + (uint64_t)((uint32_t)z * g.ny + (uint32_t)y) * (g.nx + 1u);
    return make_uint2(row[u], row[v + 1]);
}

template <int KMAX, int MODE, bool SELF>
static __global__ __launch_bounds__(kGridThreads) void k_nn_query(NnQuery a) {
    __shared__ uint2 s_run[9][kGridThreads];
    __shared__ unsigned long long s_buf[kNnBuf][kGridThreads];
    __shared__ uint32_t s_at[kGridThreads / 64 + 1];
    const uint32_t t = blockIdx.x * kGridThreads + threadIdx.x, tid = threadIdx.x;
    const bool valid = t < a.nq;
    const GridGeom g = *a.geom;
    const float4 q = a.q[valid ? t : 0u];
    const uint32_t self = __float_as_uint(q.w);
    const float tx = (q.x - g.lo[0]) * g.inv, ty = (q.y - g.lo[1]) * g.inv, tz = (q.z - g.lo[2]) * g.inv;
    const int cx = (int)grid_axis(tx, g.nx), cy = (int)grid_axis(ty, g.ny), cz = (int)grid_axis(tz, g.nz);
    // the 9 rows, the query's own first, then those that share a face with it (two bits per row: 0 the query's
    // layer, 1 below, 2 above); all their ends loaded together
    constexpr uint32_t kRowY = 0x26424u, kRowZ = 0x29640u;
    uint32_t total = 0;
    {
        const uint32_t x0 = (uint32_t)max(cx - 1, 0), x1 = (uint32_t)min(cx + 1, (int)g.nx - 1) + 1u;
        uint32_t rb[9], re[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const uint32_t sy = kRowY >> (2 * k) & 3u, sz = kRowZ >> (2 * k) & 3u;
            const int y = cy + (sy == 1u ? -1 : sy == 2u ? 1 : 0), z = cz + (sz == 1u ? -1 : sz == 2u ? 1 : 0);
            rb[k] = re[k] = 0u;
            if (y >= 0 && y < (int)g.ny && z >= 0 && z < (int)g.nz) {
                const uint32_t *row = a.table + (uint64_t)((uint32_t)z * g.ny + (uint32_t)y) * (g.nx + 1u);
                rb[k] = row[x0];
                re[k] = row[x1];
            }
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            s_run[k][tid] = make_uint2(rb[k], re[k]);
            total += re[k] - rb[k];
        }
    }
    // distances to the neighbouring rows of cells, with the margins of nn_bound
    const float m = nn_margin(g), hs = g.hs;
    const float yl = fmaxf(ty - (float)cy - m, 0.f) * hs, yh = fmaxf((float)(cy + 1) - ty - m, 0.f) * hs;
    const float zl = fmaxf(tz - (float)cz - m, 0.f) * hs, zh = fmaxf((float)(cz + 1) - tz - m, 0.f) * hs;
    const auto far = [&](int k) {
        const uint32_t sy = kRowY >> (2 * k) & 3u, sz = kRowZ >> (2 * k) & 3u;
        const float dy = sy == 1u ? yl : sy == 2u ? yh : 0.f, dz = sz == 1u ? zl : sz == 2u ? zh : 0.f;
        return dy * dy + dz * dz;
    };
    unsigned long long best[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) best[k] = ~0ull;
    unsigned long long worst = ~0ull;
    bool left = valid && total > a.walk;
    const bool walk = valid && !left;
    nn_walk_runs<KMAX, SELF>(a, q, walk && total > 0 && a.keff > 0, far, s_run, s_buf, best, worst);
    if (walk) {
        // no key so far reads as a NaN distance, which no bound exceeds
        const float kth = __uint_as_float((uint32_t)(worst >> 32));
        const float bound = nn_bound(g, tx, ty, tz, cx, cy, cz, 1);
        if (!(bound == INFINITY || kth < bound) && a.keff > 0) {
            // with K found and the K-th closer than the faces of the next cube, the parts of its shell that are
            // closer than the K-th finish the search: 9 inner rows with a cell at either end, 16 outer rows
            const float bound2 = nn_bound(g, tx, ty, tz, cx, cy, cz, 2);
            left = !(kth < bound2 || (bound2 == INFINITY && kth >= 0.f));
            if (!left) {
#pragma unroll 1
                for (int k = 0; k < 34; ++k) {
                    const uint2 run = nn_shell_run(a, g, k, tx, ty, tz, cx, cy, cz, m, hs,
                                                   __uint_as_float((uint32_t)(worst >> 32)));
                    if (run.x < run.y) nn_walk<KMAX, SELF>(a, q, run, best, worst);
                }
            }
        }
        if (!left) nn_write<KMAX, MODE>(a, self, best);
    }
    nn_append_left(a, left, t, s_at);
}
// The nearest (K = 1): 16 lanes per query.  Each lane takes a row of the cube
// (then, if the query is not done, a run of the shell around it), and the lanes
// share the candidates of those runs evenly; the nearest is the minimum of the
// lanes' keys.  A thread per query left too few waves in flight for the loads'
// latency (45k queries are 704 waves on 1024 SIMDs).
constexpr int kNearLanes = 16;
template <int MODE, bool SELF>
static __global__ __launch_bounds__(kGridThreads) void k_nn_nearest(NnQuery qa, NnQuery qb, uint32_t blocks_a) {
    __shared__ uint32_t s_beg[kGridThreads], s_pre[kGridThreads], s_end[kGridThreads];
    __shared__ uint32_t s_at[kGridThreads / 64 + 1];
    const bool first = blockIdx.x < blocks_a;
    const uint32_t bid = first ? blockIdx.x : blockIdx.x - blocks_a;
    const NnQuery &a = first ? qa : qb;
    const uint32_t tid = threadIdx.x, l = tid & (kNearLanes - 1u), g0 = tid & ~(kNearLanes - 1u);
    const uint32_t t = bid * (kGridThreads / kNearLanes) + tid / kNearLanes;
    const bool valid = t < a.nq;
    const GridGeom g = *a.geom;
    const float4 q = a.q[valid ? t : 0u];
    const uint32_t self = __float_as_uint(q.w);
    const float tx = (q.x - g.lo[0]) * g.inv, ty = (q.y - g.lo[1]) * g.inv, tz = (q.z - g.lo[2]) * g.inv;
    const int cx = (int)grid_axis(tx, g.nx), cy = (int)grid_axis(ty, g.ny), cz = (int)grid_axis(tz, g.nz);
    const float m = nn_margin(g), hs = g.hs;
    const float bound = nn_bound(g, tx, ty, tz, cx, cy, cz, 1), bound2 = nn_bound(g, tx, ty, tz, cx, cy, cz, 2);
    unsigned long long best = ~0ull;
    bool on = valid && a.keff > 0, left = false;          // the same in a query's lanes
    for (int round = 0; round < 4 && __ballot(on) != 0ull; ++round) {
        uint2 run = make_uint2(0u, 0u);
        if (on && round == 0) {
            const int y = cy + (int)(l % 3u) - 1, z = cz + (int)(l / 3u) - 1;
            if (l < 9u && y >= 0 && y < (int)g.ny && z >= 0 && z < (int)g.nz) {
                const uint32_t *row = a.table + (uint64_t)((uint32_t)z * g.ny + (uint32_t)y) * (g.nx + 1u);
                run = make_uint2(row[max(cx - 1, 0)], row[min(cx + 1, (int)g.nx - 1) + 1]);
            }
        } else if (on) {
            const int k = (round - 1) * kNearLanes + (int)l;
            if (k < 34)
                run = nn_shell_run(a, g, k, tx, ty, tz, cx, cy, cz, m, hs, __uint_as_float((uint32_t)(best >> 32)));
        }
        uint32_t incl = run.y - run.x;
#pragma unroll
        for (int d = 1; d < kNearLanes; d <<= 1) {
            const uint32_t o = __shfl_up(incl, d, 64);
            if (l >= (uint32_t)d) incl += o;
        }
        s_beg[tid] = run.x;
        s_pre[tid] = incl - (run.y - run.x);
        s_end[tid] = incl;
        nn_wave_sync();
        const uint32_t total = s_end[g0 + kNearLanes - 1u];
        if (total > a.walk) { left = on; on = false; }
        if (on) {
            for (uint32_t c = l; c < total; c += kNearLanes) {
                uint32_t lo = g0;                          // the last run that starts at or before c
#pragma unroll
                for (uint32_t d = kNearLanes / 2; d >= 1; d >>= 1)
                    if (s_pre[lo + d] <= c) lo += d;
                const float4 p = a.pts[s_beg[lo] + (c - s_pre[lo])];
                const unsigned long long x = nn_key<SELF>(q, p, !SELF || __float_as_uint(p.w) != self);
                best = x < best ? x : best;
            }
        }
#pragma unroll
        for (int d = 1; d < kNearLanes; d <<= 1) {
            const uint32_t xl = (uint32_t)__shfl_xor((int)(uint32_t)best, d, 64);
            const uint32_t xh = (uint32_t)__shfl_xor((int)(uint32_t)(best >> 32), d, 64);
            const unsigned long long x = ((unsigned long long)xh << 32) | xl;
            best = x < best ? x : best;
        }
        nn_wave_sync();                                    // the runs are read before the next are written
        // done, left over, or on to the shell (which one round does not finish)
        const float kth = __uint_as_float((uint32_t)(best >> 32));
        if (on && round == 0) {
            on = !(bound == INFINITY || kth < bound);
            left = on && !(kth < bound2 || (bound2 == INFINITY && kth >= 0.f));
            on = on && !left;
        }
    }
    if (valid && !left && l == 0) {
        unsigned long long b[1] = {best};
        nn_write<1, MODE>(a, self, b);
    }
    nn_append_left_block<false>(a, left && l == 0, t, s_at);
}

constexpr int kRestWaves = kGridThreads / 64;
constexpr int kRestRuns = 4;                    // runs per lane whose ends are loaded together
struct NnRestLds {
    uint32_t beg[kRestWaves][64], pre[kRestWaves][64], len[kRestWaves][64];
    unsigned long long key[2][kRestWaves][64], list[2][kRestWaves][64];    // the merges alternate between the halves
};

// One wave per listed query: the cube grows from 1 to 2, 3, 5, 8, ... cells
// (twofold through empty space); each step takes the rows of the new shell 64
// runs at a time, and the lanes share the candidates of those runs evenly (the
// run of a candidate is found by bisection of the runs' running total).  Lane k
// holds the k-th smallest key so far.  64 candidates of which one is below the
// K-th are merged at once: every lane counts the keys below its candidate and
// below its list entry, which are their places in the merged list.
// LIMIT: false, with nothing written, if more than a.walk candidates would have
// to be walked (it stops at the run that brings them).
template <int MODE, bool SELF, bool FILTERED = false, bool LIMIT = false>
__device__ __forceinline__ bool nn_rest_wave(const NnQuery &a, uint32_t t, NnRestLds &s) {
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    const GridGeom g = *a.geom;
    const float4 q = a.q[t];
    const uint32_t self = __float_as_uint(q.w);
    const float tx = (q.x - g.lo[0]) * g.inv, ty = (q.y - g.lo[1]) * g.inv, tz = (q.z - g.lo[2]) * g.inv;
    const int cx = (int)grid_axis(tx, g.nx), cy = (int)grid_axis(ty, g.ny), cz = (int)grid_axis(tz, g.nz);
    unsigned long long best = ~0ull, worst = ~0ull;      // worst: lane keff - 1's
    int half = 0;
    s.list[0][wave][lane] = s.list[1][wave][lane] = ~0ull;
    const float m = nn_margin(g), hs = g.hs;
    int done = -1;                                       // the cube of `done` cells has been walked
    uint32_t met = 0;                                    // candidates so far (below 2^31)
    bool any = false;                                    // a candidate was met (the same in every lane)
    for (int r = 1;;) {
        const int z0 = max(cz - r, 0), z1 = min(cz + r, (int)g.nz - 1), y0 = max(cy - r, 0), y1 = min(cy + r, (int)g.ny - 1);
        const int xa = max(cx - r, 0), xb = min(cx + r, (int)g.nx - 1);
        const uint32_t ny = (uint32_t)(y1 - y0 + 1), runs = 2u * ny * (uint32_t)(z1 - z0 + 1);
        for (uint32_t k0 = 0; k0 < runs && !(LIMIT && met > a.walk); k0 += 64u * kRestRuns) {
            // run k: row k / 2; a row inside the walked cube has a part on either side of it.  The ends of
            // kRestRuns runs per lane are loaded together: most of a large shell is empty.
            uint32_t rb[kRestRuns], re[kRestRuns];
#pragma unroll
            for (int w = 0; w < kRestRuns; ++w) {
                rb[w] = re[w] = 0u;
                const uint32_t k = k0 + 64u * (uint32_t)w + lane;
                if (k < runs) {
                    const uint32_t rw = k >> 1;
                    const int z = z0 + (int)(rw / ny), y = y0 + (int)(rw % ny);
                    const uint32_t *row = a.table + (uint64_t)((uint32_t)z * g.ny + (uint32_t)y) * (g.nx + 1u);
                    int u = xa, v = xb;
                    if (abs(z - cz) <= done && abs(y - cy) <= done) {
                        if (k & 1u) u = cx + done + 1;
                        else v = cx - done - 1;
                    } else if (k & 1u) {
                        v = u - 1;
                    }
                    // the row's part that is closer than the K-th so far (any part while there is none)
                    const float fy = y == cy ? 0.f : fmaxf((y < cy ? ty - (float)(y + 1) : (float)y - ty) - m, 0.f);
                    const float fz = z == cz ? 0.f : fmaxf((z < cz ? tz - (float)(z + 1) : (float)z - tz) - m, 0.f);
                    const float room = __uint_as_float((uint32_t)(worst >> 32)) / (hs * hs) - (fy * fy + fz * fz);
                    if (room < 0.f) {
                        v = u - 1;
                    } else if (room < 1e9f && fabsf(tx) < INFINITY) {
                        const float x = sqrtf(room) + m;
                        u = max(u, (int)fmaxf(fminf(tx - x, 1e9f), 0.f));
                        v = min(v, (int)fmaxf(fminf(tx + x, 1e9f), -1.f));
                    }
                    if (u <= v) { rb[w] = row[u]; re[w] = row[v + 1]; }
                }
            }
#pragma unroll 1
            for (int w = 0; w < kRestRuns; ++w) {
                uint32_t b = rb[0], e = re[0];
#pragma unroll
                for (int o = 1; o < kRestRuns; ++o)
                    if (w == o) { b = rb[o]; e = re[o]; }
                if (__ballot(e > b) == 0ull) continue;
                any = true;
                uint32_t incl = e - b;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const uint32_t o = __shfl_up(incl, d, 64);
                    if (lane >= (uint32_t)d) incl += o;
                }
                s.beg[wave][lane] = b;
                s.pre[wave][lane] = incl - (e - b);
                s.len[wave][lane] = incl;
                nn_wave_sync();
                uint32_t all = s.len[wave][63];
                if (LIMIT) {                                 // the same in every lane
                    met = min(met + all, a.walk + 1u);
                    all = met > a.walk ? 0u : all;
                }
                for (uint32_t c0 = 0; c0 < all; c0 += 64u) {
                    const uint32_t c = c0 + lane;
                    unsigned long long x = ~0ull;
                    if (c < all) {
                        uint32_t lo = 0;                     // the last run that starts at or before c
#pragma unroll
                        for (uint32_t d = 32; d >= 1; d >>= 1)
                            if (s.pre[wave][lo + d] <= c) lo += d;
                        const float4 p = a.pts[s.beg[wave][lo] + (c - s.pre[wave][lo])];
                        const uint32_t j = __float_as_uint(p.w);
                        const float d = nn_between<SELF>(q, p);
                        if ((!SELF || j != self) && (!FILTERED || a.alive[j])) x = ((unsigned long long)__float_as_uint(d) << 32) | j;
                    }
                    if (__ballot(x < worst) == 0ull) continue;
                    unsigned long long *const key = s.key[half][wave], *const list = s.list[half][wave];
                    half ^= 1;
                    unsigned long long *const next = s.list[half][wave];
                    key[lane] = x;
                    nn_wave_sync();
                    uint32_t rx = 0, rb = lane;              // places of the candidate and of the list entry
#pragma unroll 8
                    for (int k = 0; k < 64; ++k) {
                        const unsigned long long y = key[k];
                        rx += y < x ? 1u : 0u;
                        rb += y < best ? 1u : 0u;
                    }
                    for (int k = 0; k < a.keff; ++k) rx += list[k] < x ? 1u : 0u;
                    // the list only grows, so every place below its new length is written
                    if (x != ~0ull && rx < (uint32_t)a.keff) next[rx] = x;
                    if (best != ~0ull && rb < (uint32_t)a.keff) next[rb] = best;
                    nn_wave_sync();
                    best = next[lane];
                    worst = next[a.keff > 0 ? a.keff - 1 : 0];
                }
                nn_wave_sync();                              // the runs are read before the next are written
            }
        }
        const float kth = __uint_as_float((uint32_t)(worst >> 32));
        const float bound = nn_bound(g, tx, ty, tz, cx, cy, cz, r);
        if (LIMIT && met > a.walk) return false;
        if (bound == INFINITY || kth < bound) break;     // the same in every lane
        done = r;
        r += any ? (r + 1) / 2 : r;
    }
    if (MODE == kNnKey) {
        if (lane == 0) a.key[self] = nn_finite(best);
        return true;
    }
    if (MODE == kNnSpread) {
        s.key[0][wave][lane] = best;
        nn_wave_sync();
        if (lane == 0) a.keep[self] = nn_spread_keep(a, s.key[0][wave]);
        nn_wave_sync();
    }
    if ((int)lane < a.K) {
        const bool ok = (int)lane < a.keff && best != ~0ull;
        const uint32_t j = (uint32_t)(best & 0xFFFFFFFFull), i = FILTERED ? a.pos[self] : self;
        a.idx[(size_t)i * a.K + lane] = !ok ? -1 : (int32_t)(FILTERED ? a.pos[j] : j);
        if (MODE == kNnIndexDist) a.d2[(size_t)i * a.K + lane] = ok ? __uint_as_float((uint32_t)(best >> 32)) : 0.f;
    }
    return true;
}

// ALL: every query, not only the listed ones.
template <int MODE, bool SELF, bool ALL, bool FILTERED = false>
static __global__ __launch_bounds__(kGridThreads) void k_nn_rest(NnQuery qa) {
    __shared__ NnRestLds s;
    const uint32_t n = ALL ? qa.nq : *qa.list_n;
    for (uint32_t i = blockIdx.x * kRestWaves + (threadIdx.x >> 6); i < n; i += gridDim.x * kRestWaves)
        nn_rest_wave<MODE, SELF, FILTERED>(qa, ALL ? i : qa.list[i], s);
}

// The neighbours of every point that is left, from its neighbours among all
// points (idx): where none of those was removed they are the same, numbered by
// pos.  The other points that are left are listed for a search.
static __global__ __launch_bounds__(kGridThreads) void k_nn_renumber(NnQuery a, const int32_t *idx) {
    __shared__ uint32_t s_at[kGridThreads / 64 + 1];
    const uint32_t t = blockIdx.x * kGridThreads + threadIdx.x;
    bool left = false;
    if (t < a.nq) {
        const uint32_t i = __float_as_uint(a.q[t].w);
        if (a.alive[i]) {
            const int32_t *from = idx + (size_t)i * a.K;
            int32_t *const to = a.idx + (size_t)a.pos[i] * a.K;
            uint32_t all = 1u;
#pragma unroll 8
            for (int k = 0; k < a.K; ++k) {
                const uint32_t j = (uint32_t)from[k];
                const bool ok = j != 0xFFFFFFFFu;
                all &= ok ? a.alive[j] : 0u;
                if (ok) to[k] = (int32_t)a.pos[j];
            }
            left = all == 0u;
        }
    }
    nn_append_left(a, left, t, s_at);
}

// The queries of cloud q searched in cloud c (q's list of queries left over takes its cell numbers' place).
static inline NnQuery grid_query(const NnCloud &q, const NnCloud &c, int K, uint64_t candidates) {
    NnQuery a;
    a.q = q.pts;
    a.nq = q.n;
    a.K = K;
    a.keff = (int)((uint64_t)K < candidates ? (uint64_t)K : candidates);
    a.geom = c.geom;
    a.table = c.table;
    a.pts = c.pts;
    a.list = q.cell;
    a.list_n = q.cursor + 1;
    a.list_most = 0xFFFFFFFFu;
    a.walk = kNnMaxWalk;
    a.key = nullptr;
    a.idx = nullptr;
    a.d2 = nullptr;
    a.keep = nullptr;
    a.eps = 0.f;
    a.alive = a.pos = nullptr;
    return a;
}

// Blocks of the search of the queries left over: a wave each, at most 4096 at once.
static inline uint32_t rest_blocks(uint32_t nq) {
    const uint32_t b = (nq + kRestWaves - 1) / kRestWaves;
    return b < 1024u ? b : 1024u;
}

template <int KMAX, int MODE, bool SELF>
static inline void launch_query(const NnQuery &q, hipStream_t st) {
    const uint32_t blocks = (q.nq + kGridThreads - 1) / kGridThreads;
    hipLaunchKernelGGL((k_nn_query<KMAX, MODE, SELF>), dim3(blocks), dim3(kGridThreads), 0, st, q);
    hipLaunchKernelGGL((k_nn_rest<MODE, SELF, false>), dim3(rest_blocks(q.nq)), dim3(kGridThreads), 0, st, q);
}

constexpr uint32_t kNearQueries = kGridThreads / kNearLanes;      // queries per block of k_nn_nearest

// One search for the K nearest.
template <int MODE, bool SELF>
static inline hipError_t launch_search(const NnQuery &q, hipStream_t st) {
    if (q.K == 1) {
        const uint32_t blocks = (q.nq + kNearQueries - 1) / kNearQueries;
        hipLaunchKernelGGL((k_nn_nearest<MODE, SELF>), dim3(blocks), dim3(kGridThreads), 0, st, q, q, blocks);
        hipLaunchKernelGGL((k_nn_rest<MODE, SELF, false>), dim3(rest_blocks(q.nq)), dim3(kGridThreads), 0, st, q);
    } else if (!nn_by_thread(q.K, q.nq)) {
        hipLaunchKernelGGL((k_nn_rest<MODE, SELF, true>), dim3((q.nq + kRestWaves - 1) / kRestWaves), dim3(kGridThreads),
                           0, st, q);
    } else if (q.K <= 4) {
        launch_query<4, MODE, SELF>(q, st);
    } else {
        launch_query<8, MODE, SELF>(q, st);
    }
    return hipGetLastError();
}

// Builds the grids of one cloud (b == nullptr) or two; clears zero[0 .. n_zero).
static inline hipError_t launch_grids(const NnCloud &a, const NnCloud *b, uint32_t *zero, uint64_t n_zero,
                                      hipStream_t st) {
    const NnCloud &b_ = b ? *b : a;
    auto items = [](const NnCloud &c) { return (c.n + kGridItems - 1) / kGridItems; };
    auto some = [](uint64_t blocks, uint64_t most) { return (uint32_t)(blocks < 1 ? 1 : blocks > most ? most : blocks); };
    hipLaunchKernelGGL(k_grid_prep, dim3(a.box_blocks + (b ? b->box_blocks : 0u)), dim3(kGridThreads), 0, st, a, b_, zero, n_zero);
    const uint32_t oa = some(items(a), 256), ob = b ? some(items(b_), 256) : 0u;
    hipLaunchKernelGGL(k_grid_occupy, dim3(oa + ob), dim3(kGridThreads), 0, st, a, b_, oa, ob);
    const uint32_t ca = items(a), cb = b ? items(b_) : 0u;
    hipLaunchKernelGGL(k_grid_count, dim3(ca + cb), dim3(kGridThreads), 0, st, a, b_, ca);
    const uint32_t ra = some(a.max_cells / 64, 512), rb = b ? some(b_.max_cells / 64, 512) : 0u;
    hipLaunchKernelGGL(k_grid_rows, dim3(ra + rb), dim3(kGridThreads), 0, st, a, b_, ra, rb);
    hipLaunchKernelGGL(k_grid_scatter, dim3(ca + cb), dim3(kGridThreads), 0, st, a, b_, ca);
    return hipGetLastError();
}

}  // namespace dpr
