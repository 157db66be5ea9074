// The voxel radiance cache of Sec. 4.2 for gfx950: average pooling of the
// observed pixels onto a grid over the scene (the L' that the query of Eq. 9
// reads), and the conversion of a grid into the scene's sparse form.
//
// The pixel-to-voxel map is fixed by the cameras, so a plan sorts the pixels
// by voxel once (host counting sort, pixels of a voxel in index order) and
// keeps a dense start array over all voxels.  The pooling kernel then runs
// one thread per voxel over the whole grid (a wavefront per voxel of many
// pixels): it sums the pixels' observations in double, in pixel order, and
// writes the mean, or zero for an empty voxel, so every voxel is written once
// and the result does not depend on scheduling.  The grid is ~4 (R^3 + n)
// bytes of plan and 12 R^3 bytes of output: 268 MB in all at R = 256 for a
// million pixels, which HBM holds with room to spare.
//
// The bake reads the grid at random surface points, so the scene keeps it
// sparse: pixels only ever land on surfaces, and of the 16.8 M voxels of a
// 256^3 grid over a room a few per cent are occupied.  One 16-byte word per
// brick of 4 x 4 x 4 voxels (occupancy bits and the number of occupied
// voxels in earlier bricks) and the occupied values in brick order take
// ~9 MB instead of 268 MB, and hits close together on a surface read the
// same words and value lines.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "fipt_internal.hpp"

struct fipt_voxel_plan_s {
    int32_t device = 0;
    int64_t n = 0;           // pixels
    int32_t res = 0;
    int64_t n_vox = 0;       // res^3
    int32_t* start = nullptr;  // [n_vox + 1] ranges into order
    int32_t* order = nullptr;  // [n] pixels grouped by voxel, index order within one
    int32_t* large = nullptr;  // [n_large] the voxels of more than kManyPixels pixels
    int32_t n_large = 0;
    int64_t bytes = 0;
};

namespace fipt {
namespace {

constexpr int kBlock = 256;

// LDS written by a wavefront's lanes before, read by its lanes after.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Add the first min(N, left) of `order`'s pixels to the sums, in order.  All N
// pixels' loads are in flight at once (past the end they repeat the last
// pixel, whose lines are already on their way).
template <int N>
__device__ __forceinline__ void add_pixels(const int32_t* __restrict__ order, const float* __restrict__ obs,
                                           int64_t os, uint32_t left, double& r, double& g, double& b) {
    int64_t p[N];
    float q[N][3];
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) p[u] = order[min(u, left - 1)];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        q[u][0] = obs[p[u]];
        q[u][1] = obs[os + p[u]];
        q[u][2] = obs[2 * os + p[u]];
    }
#pragma unroll
    for (uint32_t u = 0; u < N; ++u) {
        if (u < left) {
            r += q[u][0];
            g += q[u][1];
            b += q[u][2];
        }
    }
}

// Streaming the start array and the planes is 16 bytes per voxel; what takes
// longer is the voxels near a camera, up to thousands of pixels that have to
// be added in order while every batch waits for two dependent loads.  So a
// voxel of up to kManyPixels pixels is one batch of its thread, and each
// larger one, which the plan lists, has a wavefront of its own among the
// launch's first workgroups: 256 pixels' loads at once, through LDS, then one
// lane per channel adds them in order.  614,400 pixels on 256^3 voxels (the
// largest 2,015 pixels, 17 % of the occupied ones more than 4): 243 us with
// every voxel on one thread, 137 with the wavefront sharing the large voxels
// of its 64; with the list 84 from 9 pixels on, 99 from 17, 113 from 33, 118
// from 49 (longer batches cost registers, and with them wavefronts).
constexpr int kManyPixels = 8;
constexpr int kShare = 256;          // pixels of a large voxel staged together
constexpr int kWaves = kBlock / 64;

__device__ __forceinline__ void pool_large(const int32_t* __restrict__ start, const int32_t* __restrict__ order,
                                           const float* __restrict__ obs, int64_t os, float* __restrict__ out,
                                           int64_t cs, int64_t v, int lane, float (*q)[kShare]) {
    const int32_t s = start[v], k = start[v + 1] - s;
    double sum = 0.0;        // of channel `lane`, in lanes 0 to 2
    for (int32_t left = k; left > 0; left -= kShare) {
        const int32_t* __restrict__ run = order + s + (k - left);
        int64_t p[kShare / 64];
        float x[kShare / 64][3];
#pragma unroll
        for (int u = 0; u < kShare / 64; ++u) p[u] = run[min(64 * u + lane, left - 1)];
#pragma unroll
        for (int u = 0; u < kShare / 64; ++u)
            for (int c = 0; c < 3; ++c) x[u][c] = obs[c * os + p[u]];
#pragma unroll
        for (int u = 0; u < kShare / 64; ++u)
            for (int c = 0; c < 3; ++c) q[c][64 * u + lane] = x[u][c];
        wave_sync();
        if (lane < 3) {
            const int32_t cnt = min(left, kShare);
            for (int32_t j = 0; j < cnt; j += 16) {
                float y[16];
#pragma unroll
                for (int t = 0; t < 16; ++t) y[t] = q[lane][j + t];
#pragma unroll
                for (int t = 0; t < 16; ++t)
                    if (j + t < cnt) sum += y[t];
            }
        }
        wave_sync();
    }
    if (lane < 3) out[lane * cs + v] = (float)(sum / (double)k);
}

__global__ __launch_bounds__(kBlock) void k_voxel_pool(const int32_t* __restrict__ start,
                                                       const int32_t* __restrict__ order,
                                                       int64_t n_vox, const int32_t* __restrict__ large,
                                                       int32_t n_large, int32_t large_blocks,
                                                       const float* __restrict__ obs, int64_t os,
                                                       float* __restrict__ out, int64_t cs) {
    __shared__ float s_q[kWaves][3][kShare];
    if ((int32_t)blockIdx.x < large_blocks) {
        const int wave = threadIdx.x >> 6;
        for (int64_t i = (int64_t)blockIdx.x * kWaves + wave; i < n_large; i += (int64_t)large_blocks * kWaves)
            pool_large(start, order, obs, os, out, cs, large[i], threadIdx.x & 63, s_q[wave]);
        return;
    }
    const int64_t step = (int64_t)(gridDim.x - large_blocks) * kBlock;
    for (int64_t v = (int64_t)(blockIdx.x - large_blocks) * kBlock + threadIdx.x; v < n_vox; v += step) {
        const int32_t s = start[v], k = start[v + 1] - s;
        if (k > kManyPixels) continue;
        float mr = 0.0f, mg = 0.0f, mb = 0.0f;
        if (k > 0) {
            double r = 0.0, g = 0.0, b = 0.0;
            if (k <= 4) {
                add_pixels<4>(order + s, obs, os, (uint32_t)k, r, g, b);
            } else {
                add_pixels<kManyPixels>(order + s, obs, os, (uint32_t)k, r, g, b);
            }
            mr = (float)(r / (double)k);
            mg = (float)(g / (double)k);
            mb = (float)(b / (double)k);
        }
        out[v] = mr;
        out[cs + v] = mg;
        out[2 * cs + v] = mb;
    }
}

// Voxel of lane `lane` of brick `w` (B bricks per axis): lane bits
// (k % 4, j % 4, i % 4) from high to low.
__device__ __forceinline__ void brick_voxel(int64_t w, int lane, int32_t nb, int32_t& i,
                                            int32_t& j, int32_t& k) {
    const int32_t bx = (int32_t)(w % nb), by = (int32_t)((w / nb) % nb), bz = (int32_t)(w / ((int64_t)nb * nb));
    i = 4 * bx + (lane & 3);
    j = 4 * by + ((lane >> 2) & 3);
    k = 4 * bz + (lane >> 4);
}

// Occupancy of an R^3 grid given as planes [3][cs], one wavefront per brick
// of 4 x 4 x 4 voxels (one word): a voxel is occupied when any channel is
// non-zero; .z holds the brick's occupied count until the scan turns it
// into a rank.
__global__ __launch_bounds__(kBlock) void k_voxel_words(uint4* __restrict__ words,
                                                        const float* __restrict__ cache,
                                                        int64_t cs, int32_t res) {
    const int lane = threadIdx.x & 63;
    const int32_t nb = (res + 3) / 4;
    const int64_t n_words = (int64_t)nb * nb * nb;
    const int64_t wave0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int64_t step = ((int64_t)gridDim.x * kBlock) >> 6;
    for (int64_t w = wave0; w < n_words; w += step) {
        int32_t i, j, k;
        brick_voxel(w, lane, nb, i, j, k);
        bool occ = false;
        if (i < res && j < res && k < res) {
            const int64_t v = ((int64_t)k * res + j) * res + i;
            occ = (cache[v] != 0.0f) | (cache[cs + v] != 0.0f) | (cache[2 * cs + v] != 0.0f);
        }
        const uint64_t m = __builtin_amdgcn_ballot_w64(occ);
        if (lane == 0)
            words[w] = make_uint4((uint32_t)m, (uint32_t)(m >> 32), (uint32_t)__popcll(m), 0u);
    }
}

// The same for R a multiple of 4 and planes of 16-byte alignment (256^3: 38 us
// against 91): one wavefront takes four bricks side by side, lane 16 b + r the row r of four
// voxels of brick b with one load per plane (64 contiguous bytes per row of
// the four, where the general form reads 16), and the rows' bits meet by
// four steps of 16-lane rotations.
template <int N>
__device__ __forceinline__ uint32_t or_rotated(uint32_t v) {
    return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + N, 0xF, 0xF, true);   // row_ror:N
}
__global__ __launch_bounds__(kBlock) void k_voxel_words4(uint4* __restrict__ words,
                                                         const float* __restrict__ cache,
                                                         int64_t cs, int32_t res) {
    const int lane = threadIdx.x & 63, row = lane & 15;
    const int32_t nb = res / 4;
    const int64_t n_words = (int64_t)nb * nb * nb;
    const int64_t wave0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int64_t step = ((int64_t)gridDim.x * kBlock) >> 6;
    for (int64_t w0 = 4 * wave0; w0 < n_words; w0 += 4 * step) {
        const int64_t w = w0 + (lane >> 4);
        uint32_t bits = 0;
        if (w < n_words) {
            int32_t i, j, k;
            brick_voxel(w, 4 * row, nb, i, j, k);
            const int64_t v = ((int64_t)k * res + j) * res + i;
            const float4 a = *reinterpret_cast<const float4*>(cache + v);
            const float4 b = *reinterpret_cast<const float4*>(cache + cs + v);
            const float4 c = *reinterpret_cast<const float4*>(cache + 2 * cs + v);
            bits = (uint32_t)((a.x != 0.0f) | (b.x != 0.0f) | (c.x != 0.0f)) |
                   (uint32_t)((a.y != 0.0f) | (b.y != 0.0f) | (c.y != 0.0f)) << 1 |
                   (uint32_t)((a.z != 0.0f) | (b.z != 0.0f) | (c.z != 0.0f)) << 2 |
                   (uint32_t)((a.w != 0.0f) | (b.w != 0.0f) | (c.w != 0.0f)) << 3;
        }
        bits <<= 4 * (row & 7);
        uint32_t lo = row < 8 ? bits : 0u, hi = row < 8 ? 0u : bits;
        lo = or_rotated<8>(or_rotated<4>(or_rotated<2>(or_rotated<1>(lo))));
        hi = or_rotated<8>(or_rotated<4>(or_rotated<2>(or_rotated<1>(hi))));
        if (row == 0 && w < n_words) words[w] = make_uint4(lo, hi, (uint32_t)(__popc(lo) + __popc(hi)), 0u);
    }
}

// Exclusive scan of the words' counts (.z) into ranks, in three passes over
// tiles of 1024 words: each tile scanned by one workgroup (its total kept),
// the tile totals scanned by one workgroup (the grand total to *total), the
// tile offsets added.
constexpr int kScanTile = (int)kVoxelScanTile;

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* lds, uint32_t& sum) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    uint32_t incl = x;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t up = __shfl_up(incl, d, 64);
        if (lane >= d) incl += up;
    }
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    if (t == 0) {
        uint32_t run = 0;
        for (int w = 0; w < kScanTile / 64; ++w) {
            const uint32_t v = lds[w];
            lds[w] = run;
            run += v;
        }
        lds[kScanTile / 64] = run;
    }
    __syncthreads();
    sum = lds[kScanTile / 64];
    const uint32_t r = lds[wave] + incl - x;
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(kScanTile) void k_voxel_scan_tiles(uint4* __restrict__ words,
                                                                int64_t n_words,
                                                                uint32_t* __restrict__ tile_sum) {
    __shared__ uint32_t lds[kScanTile / 64 + 1];
    const int64_t i = (int64_t)blockIdx.x * kScanTile + threadIdx.x;
    const uint32_t x = i < n_words ? words[i].z : 0u;
    uint32_t sum;
    const uint32_t r = block_exclusive_scan(x, lds, sum);
    if (i < n_words) words[i].z = r;
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = sum;
}

__global__ __launch_bounds__(kScanTile) void k_voxel_scan_totals(uint32_t* __restrict__ tile_sum,
                                                                 int64_t n_tiles,
                                                                 int64_t* __restrict__ total) {
    __shared__ uint32_t lds[kScanTile / 64 + 1];
    uint32_t carry = 0;
    for (int64_t base = 0; base < n_tiles; base += kScanTile) {
        const int64_t i = base + threadIdx.x;
        const uint32_t x = i < n_tiles ? tile_sum[i] : 0u;
        uint32_t sum;
        const uint32_t r = block_exclusive_scan(x, lds, sum);
        if (i < n_tiles) tile_sum[i] = carry + r;
        carry += sum;
    }
    if (threadIdx.x == 0) *total = carry;
}

__global__ __launch_bounds__(kScanTile) void k_voxel_scan_add(uint4* __restrict__ words,
                                                              int64_t n_words,
                                                              const uint32_t* __restrict__ tile_sum) {
    const int64_t i = (int64_t)blockIdx.x * kScanTile + threadIdx.x;
    if (i < n_words) words[i].z += tile_sum[blockIdx.x];
}

// Occupied voxels' values in brick order, one wavefront per brick.
__global__ __launch_bounds__(kBlock) void k_voxel_compact(float4* __restrict__ dst,
                                                          const uint4* __restrict__ words,
                                                          const float* __restrict__ cache,
                                                          int64_t cs, int32_t res) {
    const int lane = threadIdx.x & 63;
    const int32_t nb = (res + 3) / 4;
    const int64_t n_words = (int64_t)nb * nb * nb;
    const int64_t wave0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int64_t step = ((int64_t)gridDim.x * kBlock) >> 6;
    for (int64_t w = wave0; w < n_words; w += step) {
        const uint4 wd = words[w];
        const uint64_t m = ((uint64_t)wd.y << 32) | wd.x;
        if ((m >> lane) & 1ull) {
            int32_t i, j, k;
            brick_voxel(w, lane, nb, i, j, k);
            const int64_t v = ((int64_t)k * res + j) * res + i;
            const uint32_t idx = wd.z + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
            dst[idx] = make_float4(cache[v], cache[cs + v], cache[2 * cs + v], 0.0f);
        }
    }
}

int grid_for(int64_t n) {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    return (int)std::max<int64_t>(1, std::min<int64_t>((n + kBlock - 1) / kBlock, (int64_t)cus * 32));
}

int check_voxel(const char* what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FIPT_EHIP, "%s launch failed: %s", what, hipGetErrorString(e));
    return FIPT_OK;
}

}  // namespace

int launch_voxel_words(uint4* words, const float* cache, int64_t stride, int32_t res,
                       uint32_t* tile_sum, int64_t* total, void* stream) {
    const int64_t nb = (res + 3) / 4;
    const int64_t n_words = nb * nb * nb;
    const int64_t n_tiles = (n_words + kScanTile - 1) / kScanTile;
    hipStream_t st = (hipStream_t)stream;
    if (res % 4 == 0 && stride % 4 == 0 && reinterpret_cast<uintptr_t>(cache) % 16 == 0)
        hipLaunchKernelGGL(k_voxel_words4, dim3(grid_for(n_words * 16)), dim3(kBlock), 0, st, words, cache,
                           stride, res);
    else
        hipLaunchKernelGGL(k_voxel_words, dim3(grid_for(n_words * 64)), dim3(kBlock), 0, st, words,
                           cache, stride, res);
    int rc = check_voxel("voxel_words");
    if (rc) return rc;
    hipLaunchKernelGGL(k_voxel_scan_tiles, dim3((unsigned)n_tiles), dim3(kScanTile), 0, st, words,
                       n_words, tile_sum);
    rc = check_voxel("voxel_scan_tiles");
    if (rc) return rc;
    hipLaunchKernelGGL(k_voxel_scan_totals, dim3(1), dim3(kScanTile), 0, st, tile_sum, n_tiles, total);
    rc = check_voxel("voxel_scan_totals");
    if (rc) return rc;
    hipLaunchKernelGGL(k_voxel_scan_add, dim3((unsigned)n_tiles), dim3(kScanTile), 0, st, words,
                       n_words, tile_sum);
    return check_voxel("voxel_scan_add");
}

int launch_voxel_compact(float4* dst, const uint4* words, const float* cache, int64_t stride,
                         int32_t res, void* stream) {
    const int64_t nb = (res + 3) / 4;
    hipLaunchKernelGGL(k_voxel_compact, dim3(grid_for(nb * nb * nb * 64)), dim3(kBlock), 0,
                       (hipStream_t)stream, dst, words, cache, stride, res);
    return check_voxel("voxel_compact");
}

}  // namespace fipt

using namespace fipt;

extern "C" {

int fipt_voxel_plan_create(const float* pos_host, int64_t n, int32_t res, const float* bmin_host,
                           const float* bmax_host, int32_t device, fipt_voxel_plan* out) {
    clear_error();
    if (!out) return fail(FIPT_EINVAL, "out is NULL");
    *out = nullptr;
    if (!pos_host || !bmin_host || !bmax_host) return fail(FIPT_EINVAL, "NULL argument");
    if (n < 1 || n >= (int64_t(1) << 31)) return fail(FIPT_EINVAL, "n must be in [1, 2^31)");
    if (res < 1 || res > kMaxVoxelRes)
        return fail(FIPT_EINVAL, "res must be in [1, %d], got %d", kMaxVoxelRes, res);
    for (int a = 0; a < 3; ++a)
        if (!std::isfinite(bmin_host[a]) || !std::isfinite(bmax_host[a]) ||
            !(bmax_host[a] > bmin_host[a]))
            return fail(FIPT_EINVAL, "the box must be finite with bmin < bmax on every axis");
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev)
        return fail(FIPT_EINVAL, "device %d not available", device);
    const int64_t n_vox = (int64_t)res * res * res;
    // voxel of every pixel (double arithmetic on the float inputs), then a
    // stable counting sort
    std::vector<int32_t> vox(n);
    for (int64_t p = 0; p < n; ++p) {
        int64_t ijk[3];
        for (int a = 0; a < 3; ++a) {
            const double lo = bmin_host[a], hi = bmax_host[a];
            const double u = ((double)pos_host[a * n + p] - lo) * res / (hi - lo);
            double f = std::floor(u);
            if (!(f >= 0.0)) f = 0.0;   // also NaN
            if (f > res - 1) f = res - 1;
            ijk[a] = (int64_t)f;
        }
        vox[p] = (int32_t)((ijk[2] * res + ijk[1]) * res + ijk[0]);
    }
    std::vector<int32_t> start(n_vox + 1, 0);
    for (int64_t p = 0; p < n; ++p) ++start[vox[p] + 1];
    std::vector<int32_t> large;
    for (int64_t v = 0; v < n_vox; ++v) {
        if (start[v + 1] > kManyPixels) large.push_back((int32_t)v);
        start[v + 1] += start[v];
    }
    std::vector<int32_t> order(n);
    {
        std::vector<int32_t> fill(start.begin(), start.end() - 1);
        for (int64_t p = 0; p < n; ++p) order[fill[vox[p]]++] = (int32_t)p;
    }

    int prev = -1;
    (void)hipGetDevice(&prev);
    if (hipSetDevice(device) != hipSuccess) return fail(FIPT_EHIP, "hipSetDevice(%d) failed", device);
    fipt_voxel_plan pl = new fipt_voxel_plan_s();
    pl->device = device;
    pl->n = n;
    pl->res = res;
    pl->n_vox = n_vox;
    pl->n_large = (int32_t)large.size();
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&pl->start), sizeof(int32_t) * start.size());
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&pl->order), sizeof(int32_t) * order.size());
    if (e == hipSuccess)
        e = hipMemcpy(pl->start, start.data(), sizeof(int32_t) * start.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(pl->order, order.data(), sizeof(int32_t) * order.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess && !large.empty()) {
        e = hipMalloc(reinterpret_cast<void**>(&pl->large), sizeof(int32_t) * large.size());
        if (e == hipSuccess)
            e = hipMemcpy(pl->large, large.data(), sizeof(int32_t) * large.size(), hipMemcpyHostToDevice);
    }
    if (e != hipSuccess) {
        if (pl->large) (void)hipFree(pl->large);
        if (pl->start) (void)hipFree(pl->start);
        if (pl->order) (void)hipFree(pl->order);
        delete pl;
        if (prev >= 0) (void)hipSetDevice(prev);
        return fail(e == hipErrorOutOfMemory ? FIPT_ENOMEM : FIPT_EHIP, "voxel plan upload: %s",
                    hipGetErrorString(e));
    }
    pl->bytes = (int64_t)(sizeof(int32_t) * (start.size() + order.size() + large.size()));
    if (prev >= 0) (void)hipSetDevice(prev);
    *out = pl;
    return FIPT_OK;
}

int fipt_voxel_plan_destroy(fipt_voxel_plan pl) {
    clear_error();
    if (!pl) return FIPT_OK;
    int prev = -1;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(pl->device);
    (void)hipDeviceSynchronize();
    (void)hipFree(pl->start);
    (void)hipFree(pl->order);
    if (pl->large) (void)hipFree(pl->large);
    delete pl;
    if (prev >= 0) (void)hipSetDevice(prev);
    return FIPT_OK;
}

int fipt_voxel_pool(fipt_voxel_plan pl, const float* observed, int64_t obs_stride, float* cache,
                    int64_t cache_stride, void* stream) {
    clear_error();
    if (!pl || !observed || !cache) return fail(FIPT_EINVAL, "NULL argument");
    if (obs_stride < pl->n) return fail(FIPT_EINVAL, "obs_stride < the plan's pixel count");
    if (cache_stride < pl->n_vox) return fail(FIPT_EINVAL, "cache_stride < res^3");
    // (a wavefront for each large voxel, up to the 32 workgroups per CU that
    // bound every launch here: of 2^32 threads and more HIP runs only some,
    // without an error)
    const int32_t large_blocks = pl->n_large ? grid_for((int64_t)pl->n_large * 64) : 0;
    hipLaunchKernelGGL(k_voxel_pool, dim3((unsigned)(large_blocks + grid_for(pl->n_vox))), dim3(kBlock), 0,
                       (hipStream_t)stream, pl->start, pl->order, pl->n_vox, pl->large, pl->n_large, large_blocks,
                       observed, obs_stride, cache, cache_stride);
    return check_voxel("voxel_pool");
}

}  // extern "C"
