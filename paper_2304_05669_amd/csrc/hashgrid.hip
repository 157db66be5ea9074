// The paper's material network for gfx950 (Eq. 14; architecture from its
// network paragraph): (a, sigma, m) = Sigmoid(MLP(hash encoding of x)), with
// a multiresolution hash encoding of 32 levels x 2^19 entries x 2 features
// (base resolution 16, scale 2 per level: level l has 16 * 2^l cells per
// axis over the scene box; levels whose vertices fit the table are indexed
// densely, the others by the spatial hash with the primes 1, 2654435761,
// 805459861) and an MLP of two hidden layers of 64 (ReLU, no biases).
//
// Parameters, one float array: tables [32][2^19][2], then W1 [64][64],
// W2 [64][64], W3 [5][64] (row = output).
//
// Forward: the encoding (256 table gathers per point, 8 vertices x 32 levels of
// 8 bytes) as a kernel of its own, one level of all points before the next, so
// that a level's 4 MB table stays in each XCD's L2; then the two hidden layers
// on the matrix cores over a wavefront's 64 points (see below), the weights in
// LDS, and the five outputs on the vector ALUs.  Without room for the encoding
// one kernel does both, a lane going through all levels of its point.
//
// Backward: a workgroup recomputes the forward pass of 64 points from their
// encoding, back-propagates through the MLP, stores the per-level feature
// gradients (W1^T d1, two per level) and accumulates the weight gradients of
// its run of points, all on the matrix cores; a last kernel adds the runs'
// weight gradients in order.  The table gradient is a gather: a plan built
// once for the point set lists, per level, every (point, corner) with a
// nonzero trilinear weight sorted by table slot (then point, then corner),
// and one group of lanes per slot sums weight x feature gradient over its
// list in that order, in double, adding the total into the slot's entry.
// Everything is summed in a fixed order, without float atomics, so the
// gradient is reproducible bit for bit.
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <cmath>

#include "fipt_internal.hpp"

namespace fipt {
namespace {

constexpr int kLevels = FIPT_HG_LEVELS;
constexpr int kFeat = 2;
constexpr uint32_t kT = 1u << FIPT_HG_LOG2_TABLE;
constexpr int kIn = kLevels * kFeat;   // 64
constexpr int kHid = 64;
constexpr int kOut = 5;
constexpr int64_t kTable = (int64_t)kLevels * kT * kFeat;
constexpr int kW1 = kHid * kIn, kW2 = kHid * kHid, kW3 = kOut * kHid;
constexpr int kWeights = kW1 + kW2 + kW3;   // 8512
constexpr int kBlock = 256;
// the workspace: 325 floats per point beside the feature gradients and 12,288
// per 2048 points, of which the encoding (64 per point) and the runs' weight
// gradients are used
constexpr int kChunk = 2048;
constexpr int kWsRows = 3 * 64 + 2 * 64 + kOut;
constexpr int kFeatGradRows = kLevels * kFeat;     // per-level feature gradients, [32][n] float2

struct HgArgs {
    const float* params;
    const float* pos;
    int64_t ps;
    int64_t n;
    float lo[3];
    float inv[3];
};

// Cell of coordinate p in [0, 1] at a level of N cells: lower vertex (low 32
// bits of the integer coordinate) and fraction, exact in single precision.
__device__ __forceinline__ void cell(float p, float nl, uint32_t& c, float& f) {
    const float u = p * nl;
    const float cf = fminf(floorf(u), nl - 1.0f);
    f = u - cf;
    c = (uint32_t)(uint64_t)cf;
}

// Table slots and trilinear weights of the 8 vertices of the point's cell at
// level l (corner bit 0/1/2 = +1 along x/y/z).  The level is a run-time
// value so that no register array is indexed by it.
__device__ __forceinline__ void corners(int l, const float p[3], uint32_t idx[8], float w[8]) {
    const float nl = 16.0f * (float)(1u << l);   // exact power of two
    uint32_t cx, cy, cz;
    float fx, fy, fz;
    cell(p[0], nl, cx, fx);
    cell(p[1], nl, cy, fy);
    cell(p[2], nl, cz, fz);
    const bool dense = l < 3;   // (16 * 2^l + 1)^3 <= 2^19
    const uint32_t r = (16u << (l & 3)) + 1u;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t dx = k & 1, dy = (k >> 1) & 1, dz = (k >> 2) & 1;
        w[k] = (dx ? fx : 1.0f - fx) * (dy ? fy : 1.0f - fy) * (dz ? fz : 1.0f - fz);
        const uint32_t x = cx + dx, y = cy + dy, z = cz + dz;
        idx[k] = dense ? x + y * r + z * r * r
                       : (x ^ (y * 2654435761u) ^ (z * 805459861u)) & (kT - 1u);
    }
}

// Unit-cube position of point i (single precision, as specified).
__device__ __forceinline__ void unit_pos(const HgArgs& a, int64_t i, float p[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
        p[k] = fminf(fmaxf((a.pos[k * a.ps + i] - a.lo[k]) * a.inv[k], 0.0f), 1.0f);
}

// ---- the layers on the matrix cores ------------------------------------------
// One wavefront holds 64 points as two tiles of 32 (points 0-31 and 32-63 of
// the wavefront).  A 64 x 64 layer over them is four 32 x 32 output tiles of
// v_mfma_f32_32x32x2f32, two input features per instruction: lane l supplies
// A[l % 32][l / 32] and B[l / 32][l % 32], and accumulator register r of lane
// l holds D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32] (dfeat below).  The
// encoding arrives one level (two features) at a time with a lane per point;
// v_permlane32_swap turns the two feature registers into the B operands of
// both point tiles.  A layer's output feeds the next layer as B without any
// data movement: its reduction takes the features in the order the output
// registers hold them (register r of the two half-waves, features f and
// f + 4), and the weights are read from LDS in that same order.  The weights
// live in LDS with rows of 65 floats, so that a row-wise read (W) and a
// column-wise read (W^T) both reach distinct banks across the 32 lanes.
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kWs = 65;                                      // LDS row stride of W1 and W2
constexpr int kLdsW = 2 * kHid * kWs + kW3;                  // floats of weights in LDS

__device__ __forceinline__ int dfeat(int i, int r, int h) { return 32 * i + 8 * (r >> 2) + 4 * h + (r & 3); }

__device__ __forceinline__ v16f mfma2(float a, float b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// (lanes 0-31 of x, lanes 0-31 of y) and (lanes 32-63 of x, lanes 32-63 of y)
__device__ __forceinline__ void swap_halves(float x, float y, float& lo_pair, float& hi_pair) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    lo_pair = __uint_as_float(r[0]);
    hi_pair = __uint_as_float(r[1]);
}

// The weights of all three layers into LDS (rows of kWs floats for W1, W2).
__device__ __forceinline__ void load_weights(const float* __restrict__ params, float* w) {
    const float* src = params + kTable;
    for (int q = threadIdx.x; q < kW1 + kW2; q += kBlock) {
        const int m = q / kW1, rc = q % kW1;
        w[m * kHid * kWs + (rc / kIn) * kWs + rc % kIn] = src[q];
    }
    for (int q = threadIdx.x; q < kW3; q += kBlock) w[2 * kHid * kWs + q] = src[kW1 + kW2 + q];
    __syncthreads();
}

// One workgroup takes 64 points at a time through the whole backward pass,
// each of its four wavefronts owning one 32 x 32 tile (u, j) of every product:
// outputs (or rows of a weight gradient) 32 u .., points (or columns) 32 j ...
// Activations and layer gradients never leave the chip: they pass from one
// product to the next through two LDS tiles of 64 x 64 (rows of kWs floats),
// written [feature][point] from the accumulators and read by rows (B of the
// next layer) or by columns (both operands of a weight gradient, whose
// reduction runs over the points).  A tile's own pre-activations stay in
// registers as the ReLU masks.  The weight gradients accumulate in 36 registers
// over a run of consecutive tiles and leave at its end.  Runs are cut from the
// number of points alone (see BackwardRuns): at most 2,048 points, so that a
// single-precision chain has a bound, and as many for all workgroups.  The
// products that decide the masks (z1, z2) are formed as in the forward pass.
// Bound by the single-precision matrix rate: 200 products of 64 cycles per
// wavefront and 64 points, 0.6 ms on the room's 1,843,200 points.  It takes
// 1.02 ms there (two wavefronts per SIMD, 69 KB of LDS per workgroup, and the
// barriers between the products), with its reduction 1.04; as a per-point
// kernel that wrote every activation and layer gradient (1.3 KB per point) and
// a split-K kernel that read them back it took 1.20 + 0.55 + 0.11 ms.
constexpr int kTilePts = 64;

// acc += the N products of a(k), b(k), k ascending, eight at a time: the next
// eight operands are read from LDS while these are multiplied (left to itself
// the compiler reads all of them first and runs out of registers).
template <int N, class A, class B>
__device__ __forceinline__ void product(v16f& acc, A a, B b) {
    constexpr int G = 8;
    float av[2][G], bv[2][G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
        av[0][q] = a(q);
        bv[0][q] = b(q);
    }
#pragma unroll
    for (int g = 0; g < N / G; ++g) {
        __builtin_amdgcn_sched_barrier(0);
        if (g + 1 < N / G) {
#pragma unroll
            for (int q = 0; q < G; ++q) {
                av[(g + 1) & 1][q] = a((g + 1) * G + q);
                bv[(g + 1) & 1][q] = b((g + 1) * G + q);
            }
        }
#pragma unroll
        for (int q = 0; q < G; ++q) acc = mfma2(av[g & 1][q], bv[g & 1][q], acc);
    }
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ v16f zero16() {
    v16f v;
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = 0.0f;
    return v;
}

__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_hg_backward(
    HgArgs a, const float* __restrict__ gy, int64_t gs, const float* __restrict__ ws, int64_t wn,
    float2* __restrict__ fgrad, float* __restrict__ part, int run_tiles, int n_runs) {
    __shared__ float w[kLdsW];
    __shared__ float Q[kHid * kWs];            // h1, then d1
    __shared__ float R[kHid * kWs];            // h2, then d2, then the encoding
    __shared__ float D3[kOut][kTilePts];
    load_weights(a.params, w);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, h = lane >> 5, lo = lane & 31;
    const int u = wave >> 1, j = wave & 1;
    const int l16 = lane & 15, k16 = lane >> 4;
    const float* W1 = w;                   // W1[o][c] at o * kWs + c
    const float* W2 = w + kHid * kWs;      // W2[o][c] at o * kWs + c
    const float* W3 = w + 2 * kHid * kWs;  // W3[o][c] at o * 64 + c
    // this wavefront's operands, step k of a reduction over features (pairs f,
    // f + 4 in accumulator order) or over points (pairs p, p + 1)
    const float* W1row = W1 + (32 * u + lo) * kWs + h;
    const float* W2row = W2 + (32 * u + lo) * kWs + 4 * h;
    const float* W1col = W1 + 4 * h * kWs + 32 * u + lo;
    const float* W2col = W2 + 4 * h * kWs + 32 * u + lo;
    const float* Qcol = Q + 4 * h * kWs + 32 * j + lo;
    const float* Rcol = R + 4 * h * kWs + 32 * j + lo;
    float* Qout = Q + (32 * u + 4 * h) * kWs + 32 * j + lo;   // accumulator register r at row dfeat(0, r, 0)
    float* Rout = R + (32 * u + 4 * h) * kWs + 32 * j + lo;
    const int64_t run_pts = (int64_t)run_tiles * kTilePts;
    float e[kLevels];   // the next tile's encoding: feature 2 l + h of this lane's point
    auto fetch = [&](int64_t base) {
        const int64_t pt = base + 32 * j + lo;
        const float* src = ws + (int64_t)h * wn + (pt < a.n ? pt : 0);
#pragma unroll
        for (int l = 0; l < kLevels; ++l) e[l] = src[(int64_t)(2 * l) * wn];
        if (pt >= a.n) {
#pragma unroll
            for (int l = 0; l < kLevels; ++l) e[l] = 0.0f;
        }
    };
    fetch(blockIdx.x * run_pts);
    for (int run = (int)blockIdx.x; run < n_runs; run += (int)gridDim.x) {
        const int64_t end = min(a.n, (run + 1) * run_pts);
        v16f dw1 = zero16(), dw2 = zero16();
        v4f dw3;
#pragma unroll
        for (int r = 0; r < 4; ++r) dw3[r] = 0.0f;
        for (int64_t base = run * run_pts; base < end; base += kTilePts) {
            asm volatile("" ::: "memory");   // (the weights are read from LDS where they are used)
            const int64_t pt = base + 32 * j + lo;   // this lane's point in a tile
            // z1 = W1 e
            v16f z = zero16();
            product<kLevels>(z, [&](int l) { return W1row[2 * l]; }, [&](int l) { return e[l]; });
            __syncthreads();   // (the previous tile's reads of Q and R)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                z[r] = fmaxf(z[r], 0.0f);
                Qout[dfeat(0, r, 0) * kWs] = z[r];
            }
            __syncthreads();
            // z2 = W2 h1
            v16f y = zero16();
            product<32>(y, [&](int k) { return W2row[dfeat(k >> 4, k & 15, 0)]; },
                        [&](int k) { return Qcol[dfeat(k >> 4, k & 15, 0) * kWs]; });
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                y[r] = fmaxf(y[r], 0.0f);
                Rout[dfeat(0, r, 0) * kWs] = y[r];
            }
            __syncthreads();
            // outputs o = wave (and 4 on the first wavefront): each lane sums its
            // half of the features of two points, the halves meet with a swap
            for (int o = wave; o < kOut; o += kBlock / 64) {
                float s0 = 0.0f, s1 = 0.0f;
                const float* w3 = W3 + o * kHid + 4 * h;
                const float* hr = R + 4 * h * kWs + lo;
#pragma unroll
                for (int k = 0; k < 32; ++k) {
                    const int c = dfeat(k >> 4, k & 15, 0);
                    s0 = fmaf(w3[c], hr[c * kWs], s0);
                    s1 = fmaf(w3[c], hr[c * kWs + 32], s1);
                    if ((k & 7) == 7) __builtin_amdgcn_sched_barrier(0);
                }
                float pa, pb;
                swap_halves(s0, s1, pa, pb);
                const float yv = 1.0f / (1.0f + expf(-(pa + pb)));
                const int64_t i = base + lane;
                D3[o][lane] = i < a.n ? gy[o * gs + i] * yv * (1.0f - yv) : 0.0f;
            }
            __syncthreads();
            // dW3 += d3 h2^T (16 columns per wavefront); d2 = (W3^T d3) masked
#pragma unroll
            for (int k0 = 0; k0 < kTilePts; k0 += 4) {
                const float av = l16 < kOut ? D3[l16 < kOut ? l16 : 0][k0 + k16] : 0.0f;
                dw3 = __builtin_amdgcn_mfma_f32_16x16x4f32(av, R[(16 * wave + l16) * kWs + k0 + k16], dw3, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            {
                float d3[kOut];
#pragma unroll
                for (int o = 0; o < kOut; ++o) d3[o] = D3[o][32 * j + lo];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float s = 0.0f;
#pragma unroll
                    for (int o = 0; o < kOut; ++o) s = fmaf(W3[o * kHid + dfeat(u, r, h)], d3[o], s);
                    y[r] = y[r] > 0.0f ? s : 0.0f;
                    if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
                }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 16; ++r) Rout[dfeat(0, r, 0) * kWs] = y[r];
            __syncthreads();
            // (the encoding again, a row per wavefront and step, for dW1)
            float er[kHid / 4];
            {
                const int64_t i = base + lane;
                const float* src = ws + (int64_t)wave * wn + (i < a.n ? i : 0);
#pragma unroll
                for (int q = 0; q < kHid / 4; ++q) er[q] = src[(int64_t)(4 * q) * wn];
                if (i >= a.n) {
#pragma unroll
                    for (int q = 0; q < kHid / 4; ++q) er[q] = 0.0f;
                }
            }
            // dW2 += d2 h1^T; d1 = (W2^T d2) masked
            product<32>(dw2, [&](int k) { return R[(32 * u + lo) * kWs + h + 2 * k]; },
                        [&](int k) { return Q[(32 * j + lo) * kWs + h + 2 * k]; });
            v16f g = zero16();
            product<32>(g, [&](int k) { return W2col[dfeat(k >> 4, k & 15, 0) * kWs]; },
                        [&](int k) { return Rcol[dfeat(k >> 4, k & 15, 0) * kWs]; });
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 16; ++r) Qout[dfeat(0, r, 0) * kWs] = z[r] > 0.0f ? g[r] : 0.0f;
#pragma unroll
            for (int q = 0; q < kHid / 4; ++q) R[(4 * q + wave) * kWs + lane] = er[q];
            __syncthreads();
            // (the run's next tile, or the first of the workgroup's next run)
            const int64_t next = base + kTilePts < end ? base + kTilePts : (run + (int)gridDim.x) * run_pts;
            if (next < a.n) fetch(next);
            // dW1 += d1 e^T; feature gradients W1^T d1: features 2l and 2l + 1 sit
            // in registers r, r + 1 (r even) of one lane, one float2 per level
            product<32>(dw1, [&](int k) { return Q[(32 * u + lo) * kWs + h + 2 * k]; },
                        [&](int k) { return R[(32 * j + lo) * kWs + h + 2 * k]; });
            g = zero16();
            product<32>(g, [&](int k) { return W1col[dfeat(k >> 4, k & 15, 0) * kWs]; },
                        [&](int k) { return Qcol[dfeat(k >> 4, k & 15, 0) * kWs]; });
            if (pt < a.n) {
#pragma unroll
                for (int r = 0; r < 16; r += 2)
                    fgrad[(int64_t)(dfeat(u, r, h) >> 1) * wn + pt] = make_float2(g[r], g[r + 1]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        float* out = part + (int64_t)run * kWeights;
        int at = dfeat(u, 0, h) * kHid + 32 * j + lo;
        asm volatile("" : "+v"(at));   // (no address of the partial kept across the tiles)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            out[at + dfeat(0, r, 0) * kIn] = dw1[r];
            out[at + kW1 + dfeat(0, r, 0) * kHid] = dw2[r];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * k16 + r < kOut) out[kW1 + kW2 + (4 * k16 + r) * kHid + 16 * wave + l16] = dw3[r];
    }
}

// The forward pass in the same layout: the two hidden layers on the matrix
// cores, the five outputs summed per half-wave on the vector ALUs.
// For callers without room for the encoding and for the sizes where it is the
// faster form (see one_kernel_forward); k_hg_encode and k_hg_mlp, which keep the
// encoding, take 1.2 against 1.67 ms on 1,843,200 points.
__global__ __launch_bounds__(kBlock) void k_hg_forward(HgArgs a, float* __restrict__ out, int64_t os) {
    __shared__ float w[kLdsW];
    load_weights(a.params, w);
    const float* W1 = w;
    const float* W2 = w + kHid * kWs;
    const float* W3 = w + 2 * kHid * kWs;
    const int lane = threadIdx.x & 63, h = lane >> 5, lo = lane & 31;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool live = i < a.n;
    v16f z[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) z[u][j][r] = 0.0f;
    {
        float p[3] = {0.0f, 0.0f, 0.0f};
        if (live) unit_pos(a, i, p);
        const float2* t2 = reinterpret_cast<const float2*>(a.params);
#pragma unroll 1
        for (int l = 0; l < kLevels; ++l) {
            uint32_t idx[8];
            float wt[8];
            corners(l, p, idx, wt);
            const float2* t = t2 + (int64_t)l * kT;
            float e0 = 0.0f, e1 = 0.0f;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (wt[k] != 0.0f) {
                    const float2 v = t[idx[k]];
                    e0 = fmaf(wt[k], v.x, e0);
                    e1 = fmaf(wt[k], v.y, e1);
                }
            }
            float b0, b1;
            swap_halves(e0, e1, b0, b1);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float av = W1[(32 * u + lo) * kWs + 2 * l + h];
                z[u][0] = mfma2(av, b0, z[u][0]);
                z[u][1] = mfma2(av, b1, z[u][1]);
            }
        }
    }
    v16f y[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) y[u][j][r] = 0.0f;
#pragma unroll
    for (int ui = 0; ui < 2; ++ui)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int c = dfeat(ui, r, h);
            const float h0 = fmaxf(z[ui][0][r], 0.0f), h1 = fmaxf(z[ui][1][r], 0.0f);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float av = W2[(32 * u + lo) * kWs + c];
                y[u][0] = mfma2(av, h0, y[u][0]);
                y[u][1] = mfma2(av, h1, y[u][1]);
            }
        }
#pragma unroll
    for (int o = 0; o < kOut; ++o) {
        float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float wv = W3[o * kHid + dfeat(u, r, h)];
                s0 = fmaf(wv, fmaxf(y[u][0][r], 0.0f), s0);
                s1 = fmaf(wv, fmaxf(y[u][1][r], 0.0f), s1);
            }
        float pa, pb;
        swap_halves(s0, s1, pa, pb);
        if (live) out[o * os + i] = 1.0f / (1.0f + expf(-(pa + pb)));
    }
}

// ---- the encoding as a kernel of its own ------------------------------------
// One level of one point per thread, into rows 2l and 2l + 1 of ws[.][wn], all
// points of a level before the next (the grid's y).  What
// bounds the gathers is where a level's 4 MB table is found: with every
// wavefront going through all 32 levels (k_hg_forward) the tables in use at
// once are the whole 134 MB, and each 8-byte entry brings a line from beyond
// the L2, 6 KB per point.  One level at a time fits each XCD's 4 MB L2 (91 %
// of the requests hit), and what is left is the L2's rate of requests, about
// 85 per point: 0.91 ms on the room's 1,843,200 points in camera order (0.94
// with a level's points on one XCD only: the levels are not equal; 1.00 with
// non-temporal positions and stores), against 1.72 ms for all of
// k_hg_forward's gathers and products, with the encoding kept.
// PAIR: vertices x and x + 1 of an even x differ in the lowest bit of the
// slot only (the hash multiplies x by 1), so one 16-byte load brings both;
// for an odd x the second is loaded apart (6 requests per cell instead of 8).
// Needs the parameters 16-byte aligned.
template <bool PAIR>
__global__ __launch_bounds__(kBlock) void k_hg_encode(HgArgs a, float* __restrict__ ws,
                                                      int64_t wn) {
    const int l = (int)blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= a.n) return;
    float p[3];
    unit_pos(a, i, p);
    uint32_t idx[8];
    float wt[8];
    corners(l, p, idx, wt);
    const float2* t = reinterpret_cast<const float2*>(a.params) + (int64_t)l * kT;
    float2 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = make_float2(0.0f, 0.0f);
    if (PAIR) {
#pragma unroll
        for (int q = 0; q < 8; q += 2) {
            const bool both = (idx[q] ^ 1u) == idx[q + 1];
            if (wt[q] != 0.0f || (both && wt[q + 1] != 0.0f)) {
                const float4 f = *reinterpret_cast<const float4*>(t + (idx[q] & ~1u));
                const float2 even = make_float2(f.x, f.y), odd = make_float2(f.z, f.w);
                v[q] = (idx[q] & 1u) ? odd : even;
                v[q + 1] = (idx[q] & 1u) ? even : odd;
            }
        }
#pragma unroll
        for (int q = 0; q < 8; q += 2)
            if ((idx[q] ^ 1u) != idx[q + 1] && wt[q + 1] != 0.0f) v[q + 1] = t[idx[q + 1]];
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (wt[q] != 0.0f) v[q] = t[idx[q]];
    }
    float e0 = 0.0f, e1 = 0.0f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        if (wt[q] != 0.0f) {
            e0 = fmaf(wt[q], v[q].x, e0);
            e1 = fmaf(wt[q], v[q].y, e1);
        }
    }
    ws[(int64_t)(2 * l) * wn + i] = e0;
    ws[(int64_t)(2 * l + 1) * wn + i] = e1;
}

// The layers of k_hg_forward on an encoding read from ws (same products in
// the same order, so the same bits): a persistent grid, each wavefront taking
// 64 points at a time, the weights read into LDS once per workgroup.  Bound by
// the single-precision matrix rate: 256 products of 64 cycles per wavefront
// and tile are 0.19 ms on the room's 1,843,200 points; it takes 0.32.
constexpr int kMlpAhead = 4;   // levels whose features are in flight
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_hg_mlp(const float* __restrict__ params,
                                                   const float* __restrict__ ws, int64_t wn, int64_t n,
                                                   float* __restrict__ out, int64_t os) {
    __shared__ float w[kLdsW];
    load_weights(params, w);
    const float* W1 = w;
    const float* W2 = w + kHid * kWs;
    const float* W3 = w + 2 * kHid * kWs;
    const int lane = threadIdx.x & 63, h = lane >> 5, lo = lane & 31;
    const int64_t step = (int64_t)gridDim.x * kBlock;
    for (int64_t base = (int64_t)blockIdx.x * kBlock + (threadIdx.x & ~63); base < n; base += step) {
        const int64_t i = base + lane;
        const bool live = i < n;
        const float* src = ws + (live ? i : 0);
        asm volatile("" ::: "memory");   // (the weights are read from LDS where they are used)
        v16f z[2][2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) z[u][j][r] = 0.0f;
        // the next levels' features are in flight while these are multiplied
        float e[2 * kMlpAhead], en[2 * kMlpAhead];
#pragma unroll
        for (int q = 0; q < 2 * kMlpAhead; ++q) en[q] = src[(int64_t)q * wn];
#pragma unroll 1
        for (int l0 = 0; l0 < kLevels; l0 += kMlpAhead) {
#pragma unroll
            for (int q = 0; q < 2 * kMlpAhead; ++q) e[q] = en[q];
            const float* nx = src + (int64_t)(2 * min(l0 + kMlpAhead, kLevels - kMlpAhead)) * wn;
#pragma unroll
            for (int q = 0; q < 2 * kMlpAhead; ++q) en[q] = nx[(int64_t)q * wn];
#pragma unroll
            for (int q = 0; q < kMlpAhead; ++q) {
                const float e0 = live ? e[2 * q] : 0.0f, e1 = live ? e[2 * q + 1] : 0.0f;
                float b0, b1;
                swap_halves(e0, e1, b0, b1);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const float av = W1[(32 * u + lo) * kWs + 2 * (l0 + q) + h];
                    z[u][0] = mfma2(av, b0, z[u][0]);
                    z[u][1] = mfma2(av, b1, z[u][1]);
                }
            }
        }
        v16f y[2][2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) y[u][j][r] = 0.0f;
#pragma unroll
        for (int ui = 0; ui < 2; ++ui)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int c = dfeat(ui, r, h);
                const float h0 = fmaxf(z[ui][0][r], 0.0f), h1 = fmaxf(z[ui][1][r], 0.0f);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const float av = W2[(32 * u + lo) * kWs + c];
                    y[u][0] = mfma2(av, h0, y[u][0]);
                    y[u][1] = mfma2(av, h1, y[u][1]);
                }
            }
#pragma unroll
        for (int o = 0; o < kOut; ++o) {
            float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float wv = W3[o * kHid + dfeat(u, r, h)];
                    s0 = fmaf(wv, fmaxf(y[u][0][r], 0.0f), s0);
                    s1 = fmaf(wv, fmaxf(y[u][1][r], 0.0f), s1);
                }
            float pa, pb;
            swap_halves(s0, s1, pa, pb);
            if (live) out[o * os + i] = 1.0f / (1.0f + expf(-(pa + pb)));
        }
    }
}

// ---- table-gradient plan ---------------------------------------------------
// Sort keys of level l: the slot of each (point, corner) with a nonzero
// weight, kT (after every slot) for the others; values p << 3 | corner, in
// point order, so the stable radix sort leaves each slot's list in (point,
// corner) order.  `nnz` counts the nonzero weights.
__global__ __launch_bounds__(kBlock) void k_hgp_keys(HgArgs a, int l, uint32_t* __restrict__ keys,
                                                     uint32_t* __restrict__ vals,
                                                     unsigned long long* __restrict__ nnz) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    int c = 0;
    if (i < a.n) {
        float p[3];
        unit_pos(a, i, p);
        uint32_t idx[8];
        float w[8];
        corners(l, p, idx, w);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            keys[8 * i + k] = w[k] != 0.0f ? idx[k] : kT;
            vals[8 * i + k] = (uint32_t)(i << 3) | (uint32_t)k;
            c += w[k] != 0.0f;
        }
    }
    for (int m = 32; m >= 1; m >>= 1) c += __shfl_xor(c, m, 64);
    if ((threadIdx.x & 63) == 0 && c) atomicAdd(nnz, (unsigned long long)c);
}

// Entries (p << 3 | corner, weight bits) of the sorted nonzero list.
__global__ __launch_bounds__(kBlock) void k_hgp_entries(HgArgs a, int l, const uint32_t* __restrict__ vals,
                                                        int64_t nnz, int2* __restrict__ ent) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= nnz) return;
    const uint32_t e = vals[i];
    float p[3];
    unit_pos(a, e >> 3, p);
    uint32_t idx[8];
    float w[8];
    corners(l, p, idx, w);
    float wk = 0.0f;
#pragma unroll
    for (int k = 0; k < 8; ++k) wk = (int)(e & 7) == k ? w[k] : wk;
    ent[i] = make_int2((int)e, __float_as_int(wk));
}

// Slot ranges: off[s] = the first sorted entry whose slot is >= s (a binary
// search per slot), so off[kT] = nnz.
__global__ __launch_bounds__(kBlock) void k_hgp_offsets(const uint32_t* __restrict__ keys, int64_t nnz,
                                                        uint32_t* __restrict__ off) {
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s > (int64_t)kT) return;
    int64_t lo = 0, hi = nnz;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)keys[mid] < s) lo = mid + 1;
        else hi = mid;
    }
    off[s] = (uint32_t)lo;
}

// The slots that have entries, light ones (at most kHeavy) and heavy ones, as
// two lists; stats: light slots, their entries, heavy slots.  A workgroup's
// slots stay together and in order; the order of the workgroups is free (each
// slot's sum depends on its own entries only).
constexpr uint32_t kHeavy = 256;
__global__ __launch_bounds__(kBlock) void k_hgp_lists(const uint32_t* __restrict__ off, int64_t n_slots,
                                                      uint32_t* __restrict__ light, uint32_t* __restrict__ heavy,
                                                      unsigned long long* __restrict__ stats) {
    __shared__ uint32_t n_w[kBlock / 64][2], base[2];
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t c = s < n_slots ? off[s + 1] - off[s] : 0;
    const bool is_light = c > 0 && c <= kHeavy, is_heavy = c > kHeavy;
    const uint64_t ml = __builtin_amdgcn_ballot_w64(is_light), mh = __builtin_amdgcn_ballot_w64(is_heavy);
    uint32_t entries = is_light ? c : 0;
    for (int m = 32; m >= 1; m >>= 1) entries += __shfl_xor(entries, m, 64);
    if (lane == 0) {
        n_w[wave][0] = (uint32_t)__popcll(ml);
        n_w[wave][1] = (uint32_t)__popcll(mh);
        if (entries) atomicAdd(stats + 1, (unsigned long long)entries);
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        uint32_t t = 0;
        for (int q = 0; q < kBlock / 64; ++q) t += n_w[q][threadIdx.x];
        base[threadIdx.x] = t ? (uint32_t)atomicAdd(stats + 2 * threadIdx.x, (unsigned long long)t) : 0u;
    }
    __syncthreads();
    uint32_t at[2] = {base[0], base[1]};
    for (int q = 0; q < wave; ++q) {
        at[0] += n_w[q][0];
        at[1] += n_w[q][1];
    }
    const uint64_t below = (1ull << lane) - 1ull;
    if (is_light) light[at[0] + __popcll(ml & below)] = (uint32_t)s;
    if (is_heavy) heavy[at[1] + __popcll(mh & below)] = (uint32_t)s;
}

// Table gradient of one level, slots of at most kHeavy entries: L lanes per
// slot (a power of two up to 64); lane j sums entries j, j + L, ... of the
// slot's list in double (four entries' loads, then their four gradient
// loads, in flight together), a fixed butterfly adds the L partial sums, and
// the first lane adds the total into the slot's two features.

__device__ __forceinline__ void gather_sum(const int2* __restrict__ ent, const float2* __restrict__ fg,
                                           uint32_t first, uint32_t e1, uint32_t stride, double& s0,
                                           double& s1) {
    for (uint32_t e = first; e < e1; e += 4 * stride) {
        int2 en[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) en[u] = ent[min(e + u * stride, e1 - 1)];
        float2 d[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) d[u] = fg[(uint32_t)en[u].x >> 3];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (e + u * stride < e1) {
                const double w = (double)__int_as_float(en[u].y);
                s0 += w * (double)d[u].x;
                s1 += w * (double)d[u].y;
            }
        }
    }
}

// The table gradient of every level in one launch, so that a level's last
// workgroups run beside the next level's first (and a small batch pays one
// launch, not one per level): per level its heavy slots (one workgroup each),
// then its light ones, the finest level first, whose longest heavy slots
// would otherwise be the launch's tail.
struct TableLevel {
    const int2* ent;
    const uint32_t* off;
    const uint32_t* light;
    const uint32_t* heavy;
    uint32_t first;      // the level's first workgroup
    uint32_t n_heavy;    // its workgroups of heavy slots
    uint32_t n_light;    // its light slots
    int32_t lanes;       // lanes per light slot
};
struct TableGrad {
    TableLevel lv[kLevels];   // in launch order: level kLevels - 1 first
    const float2* fg;         // feature gradients [kLevels][n]
    int64_t n;
    float* grad;              // tables [kLevels][kT][2]
};

__global__ __launch_bounds__(kBlock) void k_hg_table_grad(TableGrad g) {
    __shared__ double part[kBlock / 64][2];
    int q = 0;
#pragma unroll
    for (int s = kLevels / 2; s > 0; s >>= 1)
        if (blockIdx.x >= g.lv[q + s].first) q += s;
    const TableLevel lv = g.lv[q];
    const int l = kLevels - 1 - q;
    const int2* __restrict__ ent = lv.ent;
    const float2* __restrict__ fg = g.fg + (int64_t)l * g.n;
    float* __restrict__ t = g.grad + (int64_t)l * kT * kFeat;
    const uint32_t blk = blockIdx.x - lv.first;
    double s0 = 0.0, s1 = 0.0;
    if (blk >= lv.n_heavy) {
        // Consecutive workgroups run on different XCDs; each XCD gets a run of
        // neighbouring slots instead (the last few workgroups as they come),
        // so that on the levels whose neighbouring slots share points their
        // gradients are fetched into one L2 and not into several.  What bounds
        // the kernel is those fetches: 101 of its 141 million requests miss L2
        // at 1.84 M points, 7 TB/s of 128-byte lines, most of them from the
        // levels finer than the points' spacing, whose slots hold unrelated
        // points.  1.80 -> 1.74 ms there.
        const uint32_t blocks = (lv.n_light * (uint32_t)lv.lanes + kBlock - 1) / kBlock, run = blocks / kXcdCount;
        uint32_t rel = blk - lv.n_heavy;
        if (rel < run * kXcdCount) rel = rel % kXcdCount * run + rel / kXcdCount;
        const uint32_t id = rel * kBlock + threadIdx.x;
        const uint32_t at = id / (uint32_t)lv.lanes, j = id % (uint32_t)lv.lanes;
        uint32_t slot = 0;
        if (at < lv.n_light) {
            slot = lv.light[at];
            gather_sum(ent, fg, lv.off[slot] + j, lv.off[slot + 1], lv.lanes, s0, s1);
        }
        for (int m = 1; m < lv.lanes; m <<= 1) {
            s0 += __shfl_xor(s0, m, 64);
            s1 += __shfl_xor(s1, m, 64);
        }
        if (j == 0 && at < lv.n_light) {
            t[2 * slot] += (float)s0;
            t[2 * slot + 1] += (float)s1;
        }
        return;
    }
    // a heavy slot: thread j sums entries j, j + kBlock, ...; each wavefront's
    // butterfly, then the four wavefront totals in order
    const uint32_t slot = lv.heavy[blk];
    gather_sum(ent, fg, lv.off[slot] + threadIdx.x, lv.off[slot + 1], kBlock, s0, s1);
    for (int m = 1; m < 64; m <<= 1) {
        s0 += __shfl_xor(s0, m, 64);
        s1 += __shfl_xor(s1, m, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        part[threadIdx.x >> 6][0] = s0;
        part[threadIdx.x >> 6][1] = s1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double x = 0.0, y = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) {
            x += part[w][0];
            y += part[w][1];
        }
        t[2 * slot] += (float)x;
        t[2 * slot + 1] += (float)y;
    }
}

// gparams[weights] += the runs' partials: eight threads per weight sum an
// eighth of the runs each, in order and in double, and the eighths are added in
// order.
constexpr int kRedParts = 8, kRedCols = kBlock / kRedParts;
__global__ __launch_bounds__(kBlock) void k_hg_wreduce(const float* __restrict__ part, int n_parts,
                                                       float* __restrict__ gparams) {
    __shared__ double sum[kRedParts][kRedCols];
    const int c = threadIdx.x % kRedCols, q = threadIdx.x / kRedCols;
    const int j = blockIdx.x * kRedCols + c;
    static_assert(kWeights % kRedCols == 0, "whole workgroups of weights");
    const int b0 = (int)((int64_t)n_parts * q / kRedParts), b1 = (int)((int64_t)n_parts * (q + 1) / kRedParts);
    double s = 0.0;
#pragma unroll 8
    for (int b = b0; b < b1; ++b) s += (double)part[(int64_t)b * kWeights + j];
    sum[q][c] = s;
    __syncthreads();
    if (q == 0) {
        double t = 0.0;
        for (int k = 0; k < kRedParts; ++k) t += sum[k][c];
        gparams[kTable + j] += (float)t;
    }
}

int grid_points(int64_t n) { return (int)((n + kBlock - 1) / kBlock); }

int check_hg(const char* what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FIPT_EHIP, "%s launch failed: %s", what, hipGetErrorString(e));
    return FIPT_OK;
}

// (params may be NULL for the plan, which reads only positions)
int make_args(const float* params, const float* pos, int64_t ps, int64_t n, const float* lo,
              const float* hi, HgArgs& a, bool need_params = true) {
    if ((need_params && !params) || !pos || !lo || !hi) return fail(FIPT_EINVAL, "NULL argument");
    if (n < 1 || n >= (int64_t(1) << 31)) return fail(FIPT_EINVAL, "n must be in [1, 2^31)");
    if (ps < n) return fail(FIPT_EINVAL, "pos_stride < n");
    for (int k = 0; k < 3; ++k) {
        if (!std::isfinite(lo[k]) || !std::isfinite(hi[k]) || !(hi[k] > lo[k]))
            return fail(FIPT_EINVAL, "the box must be finite with bmin < bmax on every axis");
        a.lo[k] = lo[k];
        a.inv[k] = 1.0f / (hi[k] - lo[k]);
        if (!std::isfinite(a.inv[k])) return fail(FIPT_EINVAL, "the box is too thin");
    }
    a.params = params;
    a.pos = pos;
    a.ps = ps;
    a.n = n;
    return FIPT_OK;
}

int launch_encode(const HgArgs& a, float* ws, int64_t wn, hipStream_t st) {
    const dim3 grid(grid_points(a.n), kLevels);
    if (reinterpret_cast<uintptr_t>(a.params) % 16 == 0)
        hipLaunchKernelGGL(k_hg_encode<true>, grid, dim3(kBlock), 0, st, a, ws, wn);
    else
        hipLaunchKernelGGL(k_hg_encode<false>, grid, dim3(kBlock), 0, st, a, ws, wn);
    return check_hg("hashgrid_encode");
}

int device_cus() {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    return cus;
}

// Workgroups of k_hg_mlp: one per 256 points, up to the three that a CU holds.
int mlp_blocks(int64_t n) { return (int)std::min<int64_t>(grid_points(n), (int64_t)device_cus() * 3); }

// Whether inference runs k_hg_forward although there is room for the encoding:
// from three quarters of a workgroup per CU to the three that a CU holds it is
// one round, whose latency grows with the workgroups per CU only, while the
// encoding by levels takes its time per point from the first (us, one kernel
// against two: 40,000 points 98 and 86, 50,000 98 and 98, 65,536 99 and 113,
// 120,000 128 and 161, 196,608 178 and 196, 200,000 228 and 211).
bool one_kernel_forward(int64_t n) {
    const int64_t groups = grid_points(n), cus = device_cus();
    return 4 * groups > 3 * cus && groups <= 3 * cus;
}

// The runs of tiles whose weight gradients k_hg_backward sums in single
// precision: at most kRunTiles tiles (2,048 points) each, and for a larger point
// set as few as keep kRunSlots workgroups (two for each of the 256 CUs; one per
// CU: 1.23 against 1.01 ms on 1,843,200 points) at the same number of runs.
// They depend on the number of points only, not on the device, and so do the
// sums.  A run's partial takes 8512 floats, less than the 261 rows of the
// workspace that its first 64 points leave unused.
constexpr int kRunTiles = 32, kRunSlots = 512;
struct BackwardRuns {
    int tiles;   // of one run
    int runs;
    explicit BackwardRuns(int64_t n) {
        const int64_t t = (n + kTilePts - 1) / kTilePts;
        const int64_t each = (t + (int64_t)kRunSlots * kRunTiles - 1) / ((int64_t)kRunSlots * kRunTiles);
        tiles = (int)((t + kRunSlots * each - 1) / (kRunSlots * each));
        runs = (int)((t + tiles - 1) / tiles);
    }
};

// Lanes per slot of a level's table gather: the power of two nearest above
// a quarter of the mean list length of the level's (light, nonempty) slots,
// at most 64.
int lanes_per_slot(int64_t nnz, int64_t n_slots) {
    const int64_t mean = nnz / std::max<int64_t>(n_slots, 1);
    int L = 1;
    while (L < 64 && 4 * L < mean) L *= 2;
    return L;
}

// Slots of level l: the dense levels index (16 2^l + 1)^3 vertices.
int64_t level_slots(int l) {
    if (l < 3) {
        const int64_t r = (16 << l) + 1;
        return r * r * r;
    }
    return kT;
}

}  // namespace
}  // namespace fipt

struct fipt_hashgrid_plan_s {
    int32_t device = 0;
    int64_t n = 0;
    float lo[3], hi[3];
    float* pos = nullptr;                 // [3][n] device copy of the positions
    int2* ent[FIPT_HG_LEVELS] = {};       // per level: (p << 3 | corner, weight bits), by slot
    uint32_t* off[FIPT_HG_LEVELS] = {};   // per level: [2^19 + 1] slot ranges into ent
    uint32_t* light[FIPT_HG_LEVELS] = {}; // per level: the slots of 1 to kHeavy entries
    uint32_t* heavy[FIPT_HG_LEVELS] = {}; // per level: the slots of more than kHeavy entries
    int64_t n_light[FIPT_HG_LEVELS] = {};
    int64_t n_heavy[FIPT_HG_LEVELS] = {};
    int64_t nnz[FIPT_HG_LEVELS] = {};
    int lanes[FIPT_HG_LEVELS] = {};
};

using namespace fipt;

namespace {
void hg_plan_free(fipt_hashgrid_plan p) {
    if (!p) return;
    (void)hipFree(p->pos);
    for (int l = 0; l < FIPT_HG_LEVELS; ++l) {
        (void)hipFree(p->ent[l]);
        (void)hipFree(p->off[l]);
        (void)hipFree(p->light[l]);
        (void)hipFree(p->heavy[l]);
    }
    delete p;
}
}  // namespace

extern "C" {

int64_t fipt_hashgrid_workspace_floats(int64_t n) {
    if (n < 1) return 0;
    const int64_t chunks = (n + kChunk - 1) / kChunk;
    return (int64_t)(kWsRows + kFeatGradRows) * n + 3 * chunks * 4096;
}

int fipt_hashgrid_plan_create(const float* pos, int64_t pos_stride, int64_t n, const float* bmin_host,
                              const float* bmax_host, void* stream, fipt_hashgrid_plan* out) {
    clear_error();
    if (!out) return fail(FIPT_EINVAL, "out is NULL");
    *out = nullptr;
    HgArgs a;
    int rc = make_args(nullptr, pos, pos_stride, n, bmin_host, bmax_host, a, false);
    if (rc) return rc;
    if (n >= (int64_t(1) << 28)) return fail(FIPT_EINVAL, "n must be below 2^28");
    hipStream_t st = (hipStream_t)stream;
    fipt_hashgrid_plan p = new fipt_hashgrid_plan_s();
    (void)hipGetDevice(&p->device);
    p->n = n;
    for (int k = 0; k < 3; ++k) {
        p->lo[k] = bmin_host[k];
        p->hi[k] = bmax_host[k];
    }
    const int64_t m = 8 * n;
    uint32_t *k_in = nullptr, *k_out = nullptr, *v_in = nullptr, *v_out = nullptr;
    unsigned long long* d_nnz = nullptr;
    void* tmp = nullptr;
    size_t tmp_bytes = 0;
    auto cleanup = [&]() {
        (void)hipFree(k_in);
        (void)hipFree(k_out);
        (void)hipFree(v_in);
        (void)hipFree(v_out);
        (void)hipFree(d_nnz);
        (void)hipFree(tmp);
    };
    auto bail = [&](int code, const char* what) {
        (void)hipStreamSynchronize(st);
        cleanup();
        hg_plan_free(p);
        return fail(code, "hashgrid plan: %s", what);
    };
    if (hipMalloc(reinterpret_cast<void**>(&p->pos), sizeof(float) * 3 * n) != hipSuccess ||
        hipMalloc(reinterpret_cast<void**>(&k_in), sizeof(uint32_t) * m) != hipSuccess ||
        hipMalloc(reinterpret_cast<void**>(&k_out), sizeof(uint32_t) * m) != hipSuccess ||
        hipMalloc(reinterpret_cast<void**>(&v_in), sizeof(uint32_t) * m) != hipSuccess ||
        hipMalloc(reinterpret_cast<void**>(&v_out), sizeof(uint32_t) * m) != hipSuccess ||
        hipMalloc(reinterpret_cast<void**>(&d_nnz), sizeof(unsigned long long) * 4 * kLevels) != hipSuccess)
        return bail(FIPT_ENOMEM, "hipMalloc failed");
    for (int k = 0; k < 3; ++k)
        if (hipMemcpyAsync(p->pos + k * n, pos + k * pos_stride, sizeof(float) * n, hipMemcpyDeviceToDevice,
                           st) != hipSuccess)
            return bail(FIPT_EHIP, "copying the positions failed");
    a.pos = p->pos;
    a.ps = n;
    unsigned long long* d_stats = d_nnz + kLevels;   // k_hgp_lists' three counts per level
    if (hipMemsetAsync(d_nnz, 0, sizeof(unsigned long long) * 4 * kLevels, st) != hipSuccess)
        return bail(FIPT_EHIP, "hipMemsetAsync failed");
    if (hipcub::DeviceRadixSort::SortPairs(nullptr, tmp_bytes, k_in, k_out, v_in, v_out, (int)m, 0, 20, st) !=
            hipSuccess ||
        hipMalloc(&tmp, tmp_bytes) != hipSuccess)
        return bail(FIPT_ENOMEM, "radix sort scratch");
    for (int l = 0; l < kLevels; ++l) {
        hipLaunchKernelGGL(k_hgp_keys, dim3(grid_points(n)), dim3(kBlock), 0, st, a, l, k_in, v_in,
                           d_nnz + l);
        if (hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, k_in, k_out, v_in, v_out, (int)m, 0, 20, st) !=
            hipSuccess)
            return bail(FIPT_EHIP, "radix sort failed");
        // the nonzero count sizes the level's entry list
        unsigned long long h_nnz = 0;
        if (hipMemcpyAsync(&h_nnz, d_nnz + l, sizeof(h_nnz), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return bail(FIPT_EHIP, "counting the entries failed");
        p->nnz[l] = (int64_t)h_nnz;
        if (hipMalloc(reinterpret_cast<void**>(&p->ent[l]), sizeof(int2) * std::max<int64_t>(p->nnz[l], 1)) !=
                hipSuccess ||
            hipMalloc(reinterpret_cast<void**>(&p->off[l]), sizeof(uint32_t) * (kT + 1)) != hipSuccess)
            return bail(FIPT_ENOMEM, "hipMalloc entries failed");
        if (p->nnz[l] > 0)
            hipLaunchKernelGGL(k_hgp_entries, dim3(grid_points(p->nnz[l])), dim3(kBlock), 0, st, a, l, v_out,
                               p->nnz[l], p->ent[l]);
        hipLaunchKernelGGL(k_hgp_offsets, dim3(grid_points(kT + 1)), dim3(kBlock), 0, st, k_out, p->nnz[l],
                           p->off[l]);
        // slots of more than kHeavy entries get a workgroup each; the others
        // share lanes by the mean length of their lists
        const int64_t slots = level_slots(l);
        const int64_t most_heavy = std::min<int64_t>(slots, p->nnz[l] / kHeavy);
        if (hipMalloc(reinterpret_cast<void**>(&p->light[l]),
                      sizeof(uint32_t) * std::max<int64_t>(1, std::min<int64_t>(slots, p->nnz[l]))) != hipSuccess ||
            hipMalloc(reinterpret_cast<void**>(&p->heavy[l]), sizeof(uint32_t) * std::max<int64_t>(1, most_heavy)) !=
                hipSuccess)
            return bail(FIPT_ENOMEM, "hipMalloc slot lists failed");
        hipLaunchKernelGGL(k_hgp_lists, dim3(grid_points(slots)), dim3(kBlock), 0, st, p->off[l], slots, p->light[l],
                           p->heavy[l], d_stats + 3 * l);
        unsigned long long h_stats[3] = {0, 0, 0};
        if (hipMemcpyAsync(h_stats, d_stats + 3 * l, sizeof(h_stats), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return bail(FIPT_EHIP, "listing the slots failed");
        p->n_light[l] = (int64_t)h_stats[0];
        p->n_heavy[l] = (int64_t)h_stats[2];
        p->lanes[l] = lanes_per_slot((int64_t)h_stats[1], p->n_light[l]);
    }
    if (check_hg("hashgrid plan") != FIPT_OK || hipStreamSynchronize(st) != hipSuccess)
        return bail(FIPT_EHIP, "building the entry lists failed");
    cleanup();
    *out = p;
    return FIPT_OK;
}

int fipt_hashgrid_plan_destroy(fipt_hashgrid_plan p) {
    clear_error();
    if (!p) return FIPT_OK;
    int prev = -1;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(p->device);
    (void)hipDeviceSynchronize();
    hg_plan_free(p);
    if (prev >= 0) (void)hipSetDevice(prev);
    return FIPT_OK;
}

int fipt_hashgrid_forward(const float* params, const float* pos, int64_t pos_stride, int64_t n,
                          const float* bmin_host, const float* bmax_host, float* material,
                          int64_t mat_stride, void* stream) {
    clear_error();
    HgArgs a;
    int rc = make_args(params, pos, pos_stride, n, bmin_host, bmax_host, a);
    if (rc) return rc;
    if (!material) return fail(FIPT_EINVAL, "material is NULL");
    if (mat_stride < n) return fail(FIPT_EINVAL, "mat_stride < n");
    hipLaunchKernelGGL(k_hg_forward, dim3(grid_points(n)), dim3(kBlock), 0, (hipStream_t)stream, a, material,
                       mat_stride);
    return check_hg("hashgrid_forward");
}

int fipt_hashgrid_forward_scratch(const float* params, const float* pos, int64_t pos_stride, int64_t n,
                                  const float* bmin_host, const float* bmax_host, float* material,
                                  int64_t mat_stride, float* scratch, int64_t scratch_floats,
                                  void* stream) {
    clear_error();
    HgArgs a;
    int rc = make_args(params, pos, pos_stride, n, bmin_host, bmax_host, a);
    if (rc) return rc;
    if (!material || !scratch) return fail(FIPT_EINVAL, "NULL argument");
    if (mat_stride < n) return fail(FIPT_EINVAL, "mat_stride < n");
    if (scratch_floats < kIn)
        return fail(FIPT_EINVAL, "scratch holds %lld floats, at least %d needed", (long long)scratch_floats, kIn);
    const int64_t run = std::min(n, scratch_floats / kIn);
    for (int64_t first = 0; first < n; first += run) {
        a.pos = pos + first;
        a.n = std::min(run, n - first);
        if (one_kernel_forward(a.n)) {
            hipLaunchKernelGGL(k_hg_forward, dim3(grid_points(a.n)), dim3(kBlock), 0, (hipStream_t)stream, a,
                               material + first, mat_stride);
            if ((rc = check_hg("hashgrid_forward_scratch"))) return rc;
            continue;
        }
        rc = launch_encode(a, scratch, a.n, (hipStream_t)stream);
        if (rc) return rc;
        hipLaunchKernelGGL(k_hg_mlp, dim3(mlp_blocks(a.n)), dim3(kBlock), 0, (hipStream_t)stream, params, scratch,
                           a.n, a.n, material + first, mat_stride);
        rc = check_hg("hashgrid_forward_scratch");
        if (rc) return rc;
    }
    return FIPT_OK;
}

int fipt_hashgrid_forward_save(const float* params, const float* pos, int64_t pos_stride, int64_t n,
                               const float* bmin_host, const float* bmax_host, float* material,
                               int64_t mat_stride, float* workspace, int64_t workspace_floats,
                               void* stream) {
    clear_error();
    HgArgs a;
    int rc = make_args(params, pos, pos_stride, n, bmin_host, bmax_host, a);
    if (rc) return rc;
    if (!material || !workspace) return fail(FIPT_EINVAL, "NULL argument");
    if (mat_stride < n) return fail(FIPT_EINVAL, "mat_stride < n");
    if (workspace_floats < fipt_hashgrid_workspace_floats(n))
        return fail(FIPT_EINVAL, "workspace holds %lld floats, %lld needed", (long long)workspace_floats,
                    (long long)fipt_hashgrid_workspace_floats(n));
    rc = launch_encode(a, workspace, n, (hipStream_t)stream);
    if (rc) return rc;
    hipLaunchKernelGGL(k_hg_mlp, dim3(mlp_blocks(n)), dim3(kBlock), 0, (hipStream_t)stream, params, workspace, n,
                       n, material, mat_stride);
    return check_hg("hashgrid_forward_save");
}

static int hashgrid_backward(fipt_hashgrid_plan plan, const float* params, const float* grad_material,
                             int64_t gm_stride, float* grad_params, float* workspace,
                             int64_t workspace_floats, bool saved, void* stream) {
    if (!plan) return fail(FIPT_EINVAL, "plan is NULL");
    const int64_t n = plan->n;
    HgArgs a;
    int rc = make_args(params, plan->pos, n, n, plan->lo, plan->hi, a);
    if (rc) return rc;
    if (!grad_material || !grad_params || !workspace) return fail(FIPT_EINVAL, "NULL argument");
    if (gm_stride < n) return fail(FIPT_EINVAL, "gm_stride < n");
    if (workspace_floats < fipt_hashgrid_workspace_floats(n))
        return fail(FIPT_EINVAL, "workspace holds %lld floats, %lld needed", (long long)workspace_floats,
                    (long long)fipt_hashgrid_workspace_floats(n));
    hipStream_t st = (hipStream_t)stream;
    // workspace: the encoding (64 n floats), the feature gradients (64 n), the
    // runs' weight-gradient partials
    float2* fgrad = reinterpret_cast<float2*>(workspace + (int64_t)kIn * n);
    float* part = workspace + (int64_t)(kIn + kFeatGradRows) * n;
    const BackwardRuns br(n);
    if (!saved && (rc = launch_encode(a, workspace, n, st))) return rc;
    hipLaunchKernelGGL(k_hg_backward, dim3(std::min(br.runs, kRunSlots)), dim3(kBlock), 0, st, a, grad_material,
                       gm_stride, workspace, n, fgrad, part, br.tiles, br.runs);
    rc = check_hg("hashgrid_backward");
    if (rc) return rc;
    TableGrad tg;
    tg.fg = fgrad;
    tg.n = n;
    tg.grad = grad_params;
    int64_t first = 0;
    for (int q = 0; q < kLevels; ++q) {
        const int l = kLevels - 1 - q;
        TableLevel& v = tg.lv[q];
        v.ent = plan->ent[l];
        v.off = plan->off[l];
        v.light = plan->light[l];
        v.heavy = plan->heavy[l];
        v.first = (uint32_t)first;
        v.n_heavy = (uint32_t)plan->n_heavy[l];
        v.n_light = (uint32_t)plan->n_light[l];
        v.lanes = plan->lanes[l];
        first += v.n_heavy + ((int64_t)v.n_light * v.lanes + kBlock - 1) / kBlock;
    }
    if (first > 0) hipLaunchKernelGGL(k_hg_table_grad, dim3((unsigned)first), dim3(kBlock), 0, st, tg);
    rc = check_hg("hashgrid_table_grad");
    if (rc) return rc;
    hipLaunchKernelGGL(k_hg_wreduce, dim3(kWeights / kRedCols), dim3(kBlock), 0, st, part, br.runs, grad_params);
    return check_hg("hashgrid_wreduce");
}

int fipt_hashgrid_backward(fipt_hashgrid_plan plan, const float* params, const float* grad_material,
                           int64_t gm_stride, float* grad_params, float* workspace,
                           int64_t workspace_floats, void* stream) {
    clear_error();
    return hashgrid_backward(plan, params, grad_material, gm_stride, grad_params, workspace,
                             workspace_floats, false, stream);
}

int fipt_hashgrid_backward_saved(fipt_hashgrid_plan plan, const float* params,
                                 const float* grad_material, int64_t gm_stride, float* grad_params,
                                 float* workspace, int64_t workspace_floats, void* stream) {
    clear_error();
    return hashgrid_backward(plan, params, grad_material, gm_stride, grad_params, workspace,
                             workspace_floats, true, stream);
}

}  // extern "C"
