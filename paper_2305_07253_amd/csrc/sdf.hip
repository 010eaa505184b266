// The stored forms of a grid and its step bounds: the kernels' bricked copy in
// each format, the dequantized samples, and the Lipschitz and slope bounds of
// their interpolant.
//
//   k_block_scales   (I8) one scale per block of 8^3 cells
//   k_store          everything else, in one pass over the samples
//   k_finish_bounds  the step bounds from the maxima of k_store's blocks
#include "hyb_device.hpp"
#include "kernels.hpp"

namespace hyb {
namespace {

constexpr int kWave = 64;
constexpr int kThreads = 256;
constexpr float kMaxFinite = 3.402823466e38f;

__device__ bool finite(float v) { return fabsf(v) <= kMaxFinite; }  // false for NaN

// I8 block scales: one wavefront per block of 8^3 cells (its nodes [8b, 8b + 8]
// on each axis, a face shared with the next block): 2^e with e the smallest
// integer >= -126 such that max |f| <= 127 * 2^e (exact comparisons).
__global__ __launch_bounds__(kThreads) void k_block_scales(const float* __restrict__ in, int32_t n, int32_t nb,
                                                           float* __restrict__ scales) {
    const int64_t b = (int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
    if (b >= (int64_t)nb * nb * nb) return;
    constexpr int S = kScaleBlock + 1;
    const int bi = (int)(b % nb), bj = (int)((b / nb) % nb), bk = (int)(b / ((int64_t)nb * nb));
    float m = 0.0f;
    for (int q = threadIdx.x % kWave; q < S * S * S; q += kWave) {
        const int i = bi * kScaleBlock + q % S, j = bj * kScaleBlock + q / S % S, k = bk * kScaleBlock + q / (S * S);
        if (i < n && j < n && k < n) m = fmaxf(m, fabsf(in[i + (int64_t)n * (j + (int64_t)n * k)]));
    }
    for (int o = kWave / 2; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, kWave));
    if (threadIdx.x % kWave != 0) return;
    int e = -126;
    if (m > 0.0f) {
        e = max(ilogbf(m) - 7, -126);  // 127 * 2^e < m here: 127 < 2^7
        while (ldexpf(127.0f, e) < m) ++e;
    }
    scales[b] = ldexpf(1.0f, e);
}

// The I8 blocks holding node i along one axis: lo to hi (equal unless the
// node lies on a face between two blocks).
__device__ inline void node_blocks(int i, int nb, int& lo, int& hi) {
    lo = min(max((i - 1) / kScaleBlock, 0), nb - 1);
    hi = min(i / kScaleBlock, nb - 1);
}

// A node's value as the kernels see it.
template <int FMT>
__device__ float dequantized(float f, int i, int j, int k, int nb, const float* __restrict__ scales) {
    if constexpr (FMT == kF32) {
        return f;
    } else if constexpr (FMT == kF16 || FMT == kF16B2) {
        return (float)(_Float16)f;
    } else {
        // the largest and smallest scale of the 1 to 8 blocks holding the
        // node: code rint(f / s_max), clamped to what the smallest-scale
        // block can hold, times s_max (all exact: powers of two)
        int il, ih, jl, jh, kl, kh;
        node_blocks(i, nb, il, ih);
        node_blocks(j, nb, jl, jh);
        node_blocks(k, nb, kl, kh);
        float smax = 0.0f, smin = __builtin_inff();
        for (int bk = kl; bk <= kh; ++bk)
            for (int bj = jl; bj <= jh; ++bj)
                for (int bi = il; bi <= ih; ++bi) {
                    const float sc = scales[bi + nb * (bj + nb * bk)];
                    smax = fmaxf(smax, sc);
                    smin = fminf(smin, sc);
                }
        const float lim = floorf(127.0f * (smin / smax));
        return fminf(fmaxf(rintf(f / smax), -lim), lim) * smax;
    }
}

// One block's share of the grid: kTileX x kTileY x kTileZ cells, whose nodes it
// keeps in LDS.
constexpr int kTileX = 32, kTileY = 8, kTileZ = 4;
constexpr int kNodesX = kTileX + 1, kNodesY = kTileY + 1;
constexpr int kNodes = kNodesX * kNodesY * (kTileZ + 1);
constexpr int kMaxBlocks = 2048;

__host__ __device__ inline int64_t store_tiles(int n) {
    const int64_t x = (n - 1 + kTileX - 1) / kTileX, y = (n - 1 + kTileY - 1) / kTileY,
                  z = (n - 1 + kTileZ - 1) / kTileZ;
    return x * y * z;
}

// Slot `at` of the two-cell brick at cell (x, y, z) of the tile (even).
__device__ float brick_sample(const float* __restrict__ node, int x, int y, int z, int at) {
    return at < 27 ? node[x + at % 3 + kNodesX * (y + at / 3 % 3 + kNodesY * (z + at / 9))] : 0.0f;
}

// Every output of one pass over the samples: the kernels' copy in the storage
// format and its bricks, the dequantized samples (`values`, unless null), and
// per block the maxima block_max[5 b ..] = (squared gradient bound, edge
// differences along x, y and z, 1 if some sample is not finite else 0).  The
// bounds are of the dequantized samples; a sample is not finite when it was not
// or is not any more (F16).
//
// Bound by the bytes it writes on large grids (FP32 four per sample byte: 256^3
// in 115 us with the bounds, 400 MB moved), by the latency of its phases on small
// ones; tiles of 4 layers rather than 8 give those twice the blocks (F16 at 96^3
// 13.5 against 15 us).  It replaced passes of their own for the copy of the
// samples, the bounds (twice for the compact formats), the dequantization and the
// bricks, whose every slot divided its way to its node.  An update without a wait,
// before and after: FP32 128^3 47 -> 21 us, 256^3 259 -> 115; F16 86 -> 19 and 346
// -> 80; I8 271 -> 36 and 1,242 -> 182.  `values` may be the input: then a node may be read again once it is
// dequantized, which gives the same value.
template <int FMT>
__global__ __launch_bounds__(kThreads) void k_store(const float* in, int32_t n, int32_t nb, float* values,
                                                    void* __restrict__ out, const float* __restrict__ scales,
                                                    float* __restrict__ block_max) {
    constexpr int V = kBoundValues;
    using B = Brick<FMT>;
    __shared__ float node[kNodes];
    __shared__ float red[V][kThreads / kWave];
    const int t = threadIdx.x, cells = n - 1, per = B::per_axis(n);
    const int tx = (cells + kTileX - 1) / kTileX, ty = (cells + kTileY - 1) / kTileY;
    float best[V] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    for (int64_t tile = blockIdx.x; tile < store_tiles(n); tile += gridDim.x) {
        const int x0 = (int)(tile % tx) * kTileX, y0 = (int)(tile / tx % ty) * kTileY,
                  z0 = (int)(tile / ((int64_t)tx * ty)) * kTileZ;
        __syncthreads();  // the last tile's nodes have been read
        for (int q = t; q < kNodes; q += kThreads) {
            const int x = q % kNodesX, y = q / kNodesX % kNodesY, z = q / (kNodesX * kNodesY);
            const int i = x0 + x, j = y0 + y, k = z0 + z;
            float v = 0.0f;
            if (i < n && j < n && k < n) {
                const int64_t id = i + (int64_t)n * (j + (int64_t)n * k);
                const float f = in[id];
                v = dequantized<FMT>(f, i, j, k, nb, scales);
                if (!finite(f) || !finite(v)) best[4] = 1.0f;
                // a face shared with the next tile is that tile's to write
                const bool mine =
                    (x < kTileX || i == cells) && (y < kTileY || j == cells) && (z < kTileZ || k == cells);
                if (values && mine) values[id] = v;
            }
            node[q] = v;
        }
        __syncthreads();
        const int cx = t % kTileX, cy = t / kTileX;
        for (int cz = 0; cz < kTileZ; ++cz) {
            const int i = x0 + cx, j = y0 + cy, k = z0 + cz;
            if (i >= cells || j >= cells || k >= cells) break;
            const float* p = node + cx + kNodesX * (cy + kNodesY * cz);
            constexpr int sy = kNodesX, sz = kNodesX * kNodesY;
            const float f[8] = {p[0], p[1], p[sy], p[sy + 1], p[sz], p[sz + 1], p[sz + sy], p[sz + sy + 1]};
            float s[3];
            cell_slopes(f, 1.0f, s);
            best[0] = fmaxf(best[0], cell_gradient2(f));
            for (int a = 0; a < 3; ++a) best[1 + a] = fmaxf(best[1 + a], s[a]);
            if constexpr (B::kCells == 1) {
                const int64_t cell = i + (int64_t)cells * (j + (int64_t)cells * k);
                if constexpr (FMT == kF16) {
                    struct alignas(16) Halves {
                        _Float16 h[8];
                    } c;
                    for (int q = 0; q < 8; ++q) c.h[q] = (_Float16)f[q];
                    static_cast<Halves*>(out)[cell] = c;
                } else {
                    // each node's value is an integer multiple of the scale of
                    // every block holding it, here the block of the cell
                    const float sc =
                        scales[i / kScaleBlock + nb * (j / kScaleBlock + nb * (k / kScaleBlock))];
                    const float inv = 1.0f / sc;
                    uint32_t word[3] = {0u, 0u, __builtin_bit_cast(uint32_t, sc)};
                    for (int q = 0; q < 8; ++q)
                        word[q / 4] |= (uint32_t)(uint8_t)(int8_t)(f[q] * inv) << (8 * (q % 4));
                    uint32_t* to = static_cast<uint32_t*>(out) + 3 * cell;
                    to[0] = word[0];
                    to[1] = word[1];
                    to[2] = word[2];
                }
            }
        }
        if constexpr (B::kCells == 2) {
            // eight lanes per brick, four slots each: a brick's bytes in one run
            const int part = t % 8;
            for (int b = t / 8; b < (kTileX / 2) * (kTileY / 2) * (kTileZ / 2); b += kThreads / 8) {
                const int bx = b % (kTileX / 2), by = b / (kTileX / 2) % (kTileY / 2),
                          bz = b / ((kTileX / 2) * (kTileY / 2));
                const int gx = x0 / 2 + bx, gy = y0 / 2 + by, gz = z0 / 2 + bz;
                if (gx >= per || gy >= per || gz >= per) continue;
                float s[4];
                for (int q = 0; q < 4; ++q) s[q] = brick_sample(node, 2 * bx, 2 * by, 2 * bz, 4 * part + q);
                const int64_t at = (((int64_t)gz * per + gy) * per + gx) * 8 + part;
                if constexpr (FMT == kF32) {
                    static_cast<float4*>(out)[at] = make_float4(s[0], s[1], s[2], s[3]);
                } else {
                    struct alignas(8) Halves {
                        _Float16 h[4];
                    } c;
                    for (int q = 0; q < 4; ++q) c.h[q] = (_Float16)s[q];
                    static_cast<Halves*>(out)[at] = c;
                }
            }
        }
    }
    for (int c = 0; c < V; ++c) {
        for (int o = kWave / 2; o > 0; o >>= 1) best[c] = fmaxf(best[c], __shfl_xor(best[c], o, kWave));
        if (t % kWave == 0) red[c][t / kWave] = best[c];
    }
    __syncthreads();
    if (t < V) {
        float m = red[t][0];
        for (int w = 1; w < kThreads / kWave; ++w) m = fmaxf(m, red[t][w]);
        block_max[V * blockIdx.x + t] = m;
    }
}

// The step bounds (kDeviceBounds floats) from the maxima of k_store's blocks.
// Root and 1 / h come last: both keep the order of the values they are taken
// of, so this is the largest of the cells' own bounds.
__global__ __launch_bounds__(kThreads) void k_finish_bounds(const float* __restrict__ block_max, int32_t n_blocks,
                                                            float inv_h, float two_e, float* __restrict__ out) {
    constexpr int V = kBoundValues;
    __shared__ float red[V][kThreads / kWave];
    float m[V] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    for (int b = threadIdx.x; b < n_blocks; b += kThreads)
        for (int c = 0; c < V; ++c) m[c] = fmaxf(m[c], block_max[V * b + c]);
    for (int c = 0; c < V; ++c) {
        for (int o = kWave / 2; o > 0; o >>= 1) m[c] = fmaxf(m[c], __shfl_xor(m[c], o, kWave));
        if (threadIdx.x % kWave == 0) red[c][threadIdx.x / kWave] = m[c];
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int c = 0; c < V; ++c)
        for (int w = 0; w < kThreads / kWave; ++w) m[c] = fmaxf(m[c], red[c][w]);
    m[0] = sqrtf(m[0]) * inv_h;
    for (int c = 1; c < 4; ++c) m[c] *= inv_h;
    bool bad = m[4] != 0.0f;
    for (int c = 0; c < 4; ++c) bad = bad || !finite(m[c]);
    const float L = finish_lipschitz(m[0]);
    out[kBBad] = bad ? 1.0f : 0.0f;
    out[kBLipschitz] = L;
    out[kBInvL] = inv_step(L);
    out[kBSlopeX] = finish_slope(m[1]);
    out[kBSlopeY] = finish_slope(m[2]);
    out[kBSlopeZ] = finish_slope(m[3]);
    out[kBTwoE] = two_e;
}

}  // namespace

int32_t store_blocks(int32_t n) {
    const int64_t tiles = store_tiles(n);
    return (int32_t)(tiles < kMaxBlocks ? tiles : kMaxBlocks);
}

hipError_t launch_store(int fmt, const float* in, int32_t n, float h, float* values, void* out, float* scales,
                        float* block_max, float two_e, float* bounds, hipStream_t stream) {
    const int32_t nb = i8_blocks(n);
    const dim3 blocks((unsigned)store_blocks(n)), threads(kThreads);
    if (fmt == kF32) {
        hipLaunchKernelGGL(k_store<kF32>, blocks, threads, 0, stream, in, n, nb, values == in ? nullptr : values, out,
                           scales, block_max);
    } else if (fmt == kF16) {
        hipLaunchKernelGGL(k_store<kF16>, blocks, threads, 0, stream, in, n, nb, values, out, scales, block_max);
    } else if (fmt == kF16B2) {
        hipLaunchKernelGGL(k_store<kF16B2>, blocks, threads, 0, stream, in, n, nb, values, out, scales, block_max);
    } else if (fmt == kI8) {
        const int64_t nbb = (int64_t)nb * nb * nb;
        constexpr int per = kThreads / kWave;
        hipLaunchKernelGGL(k_block_scales, dim3((unsigned)((nbb + per - 1) / per)), threads, 0, stream, in, n, nb,
                           scales);
        hipLaunchKernelGGL(k_store<kI8>, blocks, threads, 0, stream, in, n, nb, values, out, scales, block_max);
    } else {
        return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(k_finish_bounds, dim3(1), threads, 0, stream, block_max, (int32_t)blocks.x, 1.0f / h, two_e,
                       bounds);
    return hipGetLastError();
}

}  // namespace hyb
