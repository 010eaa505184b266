// Device build of the traversal entry pyramid (BvhHost::entry has the
// definition): for every window the lowest common ancestor of the leaves whose
// boxes overlap it.
//
// Taking the common ancestor is associative and commutative, so the leaves join
// the finest windows in any order with a compare-and-swap loop in the entry
// array itself; no scratch memory.  A coarser window is the union of 2 x 2 x 2
// windows of the level below.  Bound by latency: each join is a chain of
// dependent reads up the tree and an atomic, so the joins are spread over as
// many lanes as there are windows.  About 0.17 ms for 1,052 triangles (clear 5,
// leaves 42, large leaves 46, levels 38, tail 26 us); on the host the pyramid
// took 23 of the 26 ms of loading that mesh (2.1M half-cells, eight common
// ancestors per window, whatever the mesh).
#include "entry.hpp"
#include "kernels.hpp"

namespace hyb {
namespace {

constexpr int kWave = 64;
constexpr int kThreads = 256;
constexpr int kTailRes = 4;  // levels up to this resolution share one block
constexpr int kLargeLeaf = 512;    // windows of a leaf that one wavefront joins
constexpr int kLargeBlocks = 1024;

__global__ __launch_bounds__(kThreads) void k_entry_clear(int32_t* __restrict__ entry, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads)
        entry[i] = kEmptyRef;
}

// The finest windows [w0, w0 + side) that a leaf's box overlaps; their count.
__device__ int leaf_windows(const float* __restrict__ q, int c, const EntryGrid& g, int w0[3], int side[3]) {
    const int W = 2 * g.res - 1;
    for (int a = 0; a < 3; ++a) {
        int v0, v1;
        entry_range(q[8 * a + c], q[8 * a + 4 + c], g.lo[a], g.size, g.res, v0, v1);
        // window w holds the half-cells w and w + 1
        w0[a] = v0 > 0 ? v0 - 1 : 0;
        side[a] = (v1 < W ? v1 : W - 1) - w0[a] + 1;
    }
    return side[0] * side[1] * side[2];
}

// Leaf `ref` joins the k-th of its windows: every pass either ends or sees
// another leaf's ancestor, which only moves toward the root.
__device__ void join_window(const float* __restrict__ nodes4, const float* __restrict__ tris, int W, int32_t* entry,
                            const int w0[3], const int side[3], int k, int32_t ref) {
    const int yz = k / side[0];
    const int x = w0[0] + k - yz * side[0], z = w0[2] + yz / side[1], y = w0[1] + yz % side[1];
    int32_t* slot = entry + x + (int64_t)W * (y + (int64_t)W * z);
    int32_t seen = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (;;) {
        const int32_t join = entry_lca(nodes4, tris, seen, ref);
        if (join == seen) return;
        const int32_t old = atomicCAS(slot, seen, join);
        if (old == seen) return;
        seen = old;
    }
}

// One wavefront per four-wide node: its leaf children join their windows (most
// leaves 8 to 64).  A leaf of more than kLargeLeaf windows, a wall's, would
// keep its wavefront for a millisecond (32k windows, each a chain of dependent
// reads and an atomic): it goes to a list for the whole grid.  The list lies in
// the words of the levels above, which are written later; its count is the
// first word, one less than the leaves because the words start at -1.
__global__ __launch_bounds__(kThreads) void k_entry_leaves(const float* __restrict__ nodes4,
                                                           const float* __restrict__ tris, int64_t n_nodes,
                                                           EntryGrid g, int32_t* entry, int32_t* list, int room) {
    const int64_t node = (int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
    if (node >= n_nodes) return;
    const int lane = threadIdx.x & (kWave - 1);
    const float* q = nodes4 + 32 * node;
    for (int c = 0; c < 4; ++c) {
        const int32_t ref = entry_word(q + 24 + c);
        if (ref >= 0 || ref == kEmptyRef) continue;
        int w0[3], side[3];
        const int count = leaf_windows(q, c, g, w0, side);
        if (count > kLargeLeaf) {
            int at = room;
            if (lane == 0) at = atomicAdd(list, 1) + 1;
            at = __shfl(at, 0, kWave);
            if (at < room) {
                if (lane == 0) list[1 + at] = (int32_t)(4 * node + c);  // n_nodes < 2^29: at most one per triangle
                continue;
            }
        }
        for (int k = lane; k < count; k += kWave) join_window(nodes4, tris, 2 * g.res - 1, entry, w0, side, k, ref);
    }
}

// The listed leaves, each over an equal share of the grid's blocks.
__global__ __launch_bounds__(kThreads) void k_entry_large(const float* __restrict__ nodes4,
                                                          const float* __restrict__ tris, EntryGrid g, int32_t* entry,
                                                          const int32_t* __restrict__ list, int room) {
    const int leaves = min(list[0] + 1, room);
    if (leaves == 0) return;
    const int parts = max(1, (int)gridDim.x / leaves);
    for (int w = blockIdx.x; w < leaves * parts; w += gridDim.x) {
        const int32_t which = list[1 + w / parts];
        const float* q = nodes4 + 32 * (int64_t)(which >> 2);
        const int32_t ref = entry_word(q + 24 + (which & 3));
        int w0[3], side[3];
        const int count = leaf_windows(q, which & 3, g, w0, side);
        for (int k = (w % parts) * kThreads + threadIdx.x; k < count; k += parts * kThreads)
            join_window(nodes4, tris, 2 * g.res - 1, entry, w0, side, k, ref);
    }
}

__device__ void entry_window(const float* __restrict__ nodes4, const float* __restrict__ tris, const int32_t* below,
                             int32_t* out, int W, int i) {
    const int x = i % W, y = (i / W) % W, z = i / (W * W);
    const int64_t B = 2 * W + 1;  // windows per axis of the level below
    int32_t acc = kEmptyRef;
    for (int c = 0; c < 8; ++c) {
        const int bx = 2 * (x + (c & 1)), by = 2 * (y + ((c >> 1) & 1)), bz = 2 * (z + (c >> 2));
        acc = entry_lca(nodes4, tris, acc, below[bx + B * (by + B * bz)]);
    }
    out[i] = acc;
}

// One level from the level below it.
__global__ __launch_bounds__(kThreads) void k_entry_level(const float* __restrict__ nodes4,
                                                          const float* __restrict__ tris, const int32_t* below,
                                                          int32_t* out, int W) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i < W * W * W) entry_window(nodes4, tris, below, out, W, i);
}

// The coarsest levels in one block: too small to fill the chip, and each waits
// for the one below.
__global__ __launch_bounds__(kThreads) void k_entry_tail(const float* __restrict__ nodes4,
                                                         const float* __restrict__ tris, const int32_t* below,
                                                         int32_t* out, int res) {
    for (; res >= 1; res >>= 1) {
        const int W = 2 * res - 1;
        for (int i = threadIdx.x; i < W * W * W; i += kThreads) entry_window(nodes4, tris, below, out, W, i);
        __syncthreads();
        below = out;
        out += W * W * W;
    }
}

}  // namespace

hipError_t launch_entries(const float4* nodes4, const float4* tris, int64_t n_nodes, const EntryGrid& g,
                          int32_t* entry, hipStream_t stream) {
    if (g.res < 1 || n_nodes < 1) return hipErrorInvalidValue;
    const float* nd = reinterpret_cast<const float*>(nodes4);
    const float* tr = reinterpret_cast<const float*>(tris);
    hipLaunchKernelGGL(k_entry_clear, dim3(2048), dim3(kThreads), 0, stream, entry, entry_total(g.res));
    const int per = kThreads / kWave;
    const int64_t finest = (int64_t)(2 * g.res - 1) * (2 * g.res - 1) * (2 * g.res - 1);
    int32_t* list = entry + finest;  // of the words above the finest level, one for the count
    const int room = (int)(entry_total(g.res) - finest) - 1;
    if (room < 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_entry_leaves, dim3((unsigned)((n_nodes + per - 1) / per)), dim3(kThreads), 0, stream, nd, tr,
                       n_nodes, g, entry, list, room);
    hipLaunchKernelGGL(k_entry_large, dim3(kLargeBlocks), dim3(kThreads), 0, stream, nd, tr, g, entry, list, room);
    int32_t* below = entry;
    int res = g.res;
    for (;;) {
        const int64_t W = 2 * res - 1;
        int32_t* out = below + W * W * W;
        res >>= 1;
        if (res < 1) break;
        if (res <= kTailRes) {
            hipLaunchKernelGGL(k_entry_tail, dim3(1), dim3(kThreads), 0, stream, nd, tr, below, out, res);
            break;
        }
        const int w = 2 * res - 1;
        hipLaunchKernelGGL(k_entry_level, dim3((unsigned)((w * w * w + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                           stream, nd, tr, below, out, w);
        below = out;
    }
    return hipGetLastError();
}

}  // namespace hyb
