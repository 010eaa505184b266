// Backward of the distance-field hit distance (hyb_df_backward): for every
// ray with a crossing, the 8 implicit derivatives d t / d sample of the
// corners of its hit cell, times grad_t, added into the grid gradient.
//
// The float atomic adds are nearly the whole cost of a plain scatter (8 per
// hit, 17 to 22 G adds/s, and 4 ns for every add at the same node; recomputing the
// hits is a few percent of it).  So workgroups sum by node in LDS before they add: up to
// 2^18 rays in the caller's order, more of them after a radix sort by the block of 8^3
// cells that they hit, since hits cluster on surfaces.
#include <rocprim/device/device_radix_sort.hpp>

#include "hyb_device.hpp"
#include "kernels.hpp"

namespace hyb {
namespace {

constexpr int kBwdBlock = 256;

// The (block, ray) pairs are sorted by rocPRIM's onesweep radix sort: its default
// is a block sort plus merge passes up to 1M pairs, which took 154 us of a 241 us
// backward on 1M rays (ten merge passes) where onesweep takes two passes over the 13
// bits of a block at 128^3.
using BwdSortConfig =
    rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config, rocprim::default_config, 65536>;

// Contributions of ray i (grad_t times d t / d sample of its cell's 8
// corners, corner order of `corners`) and the linear index of the cell's
// corner 0; false when the ray adds nothing.
HYB_HD bool ray_gradient(const TraceArgs& a, const Grid& g, int64_t i, const float* __restrict__ t_hit,
                         const float* __restrict__ grad_t, int64_t& cell, float v[8]) {
    const float gt = grad_t[i];
    if (gt == 0.0f) return false;
    const float tmin = a.tmin ? a.tmin[i] : 0.0f;
    const float tmax = a.tmax_ray ? fminf(a.tmax_ray[i], a.tmax) : a.tmax;
    if (!(tmin <= tmax)) return false;
    int64_t node[8];
    float dt[8];
    if (!df_hit_gradient(g, a.ox[i], a.oy[i], a.oz[i], a.dx[i], a.dy[i], a.dz[i], tmin, tmax, t_hit[i], node, dt))
        return false;
    for (int c = 0; c < 8; ++c) v[c] = gt * dt[c];
    cell = node[0];
    return true;
}

constexpr int kCells = 8;               // cells of a block per axis
constexpr int kSide = kCells + 1;       // its nodes
constexpr int kNodes = kSide * kSide * kSide;
constexpr int kOpen = 8;                // blocks that a workgroup sums at a time
constexpr int kSparse = 32;             // distinct blocks above which it sums none
constexpr int kRuns = 48;               // runs of a wavefront up to which they are summed first
constexpr int kSumBlock = 512;
constexpr int kSlotBits = 13;
constexpr int kSlots = 1 << kSlotBits;  // of a workgroup's hash table
constexpr int kGroupBits = 4;           // nodes in a row that the table keeps together
constexpr int kGroup = 1 << kGroupBits;
static_assert(kSlots >= 2 * 8 * kSumBlock, "at least half of the table stays empty");
constexpr uint32_t kEmpty = 0xffffffffu;

// Rays up to which no sort pays, whatever their order: its passes take 40 us and more
// whatever the count, the unsorted rays' additional global adds take time per ray.
// Unsorted against sorted by block: 128k rays of an image on 128^3 13 us and 80, random
// ones 43 and 90; 256k 22 and 90, 80 and 102 (on 32^3 62 and 66); 400k random rays 123
// and 119, 1M 279 and 222.
constexpr int64_t kUnsorted = 1 << 18;

__host__ __device__ inline int blocks_per_axis(int n) { return (n - 1 + kCells - 1) / kCells; }

// Cell coordinates of a linear node index (below 2^30).
__device__ void cell_of(int64_t cell, int n, int& i, int& j, int& k) {
    const uint32_t c = (uint32_t)cell, row = c / (uint32_t)n;
    i = (int)(c - row * n);
    k = (int)(row / (uint32_t)n);
    j = (int)(row - (uint32_t)k * n);
}

// Sort keys: the hit cell's block, or `none` for a ray that adds nothing; the
// values are the ray indices.
__global__ __launch_bounds__(kBwdBlock) void k_bwd_keys(TraceArgs a, const float* __restrict__ t_hit,
                                                        const float* __restrict__ grad_t, uint32_t* __restrict__ keys,
                                                        uint32_t* __restrict__ rays, uint32_t none) {
    const int64_t i = (int64_t)blockIdx.x * kBwdBlock + threadIdx.x;
    if (i >= a.n) return;
    const Grid g = grid_of(a);
    int64_t cell = 0;
    float v[8];
    uint32_t key = none;
    if (ray_gradient(a, g, i, t_hit, grad_t, cell, v)) {
        int ci, cj, ck;
        cell_of(cell, a.n_grid, ci, cj, ck);
        const uint32_t nb = blocks_per_axis(a.n_grid);
        key = ci / kCells + nb * (cj / kCells + nb * (ck / kCells));
    }
    keys[i] = key;
    rays[i] = (uint32_t)i;
}

__device__ void add_corners(float* __restrict__ grad_grid, int64_t cell, int64_t n, const float v[8]) {
    for (int c = 0; c < 8; ++c)
        unsafeAtomicAdd(grad_grid + cell + (c & 1) + n * (((c >> 1) & 1) + n * (c >> 2)), v[c]);
}

// Neighbours of an image hit one cell: where the wavefront's rays form kRuns runs of one
// cell or fewer, each run's contributions are summed into its last lane.  Whether this
// lane adds `v`.  (All lanes active.)  Without it the lanes of a run add at the same
// addresses in LDS, one after the other: 2M rays of an image on 128^3 230 us instead of
// 157, 1M 157 instead of 121 (at 32 runs or fewer 121, 512^3 248 instead of 220).
__device__ bool sum_runs(bool found, int64_t cell, float v[8]) {
    const int lane = threadIdx.x & 63;
    const uint32_t id = found ? (uint32_t)cell : kEmpty, left = __shfl_up(id, 1);
    const uint64_t starts = __ballot(lane == 0 || left != id);
    if (__popcll(starts) > kRuns) return found;
    const int start = 63 - __builtin_clzll(starts & (~uint64_t(0) >> (63 - lane)));
    for (int c = 0; c < 8; ++c) v[c] = found ? v[c] : 0.0f;
    for (int o = 1; o < 64; o <<= 1)
        for (int c = 0; c < 8; ++c) {
            const float w = __shfl_up(v[c], o);
            if (lane - o >= start) v[c] += w;
        }
    return found && (lane == 63 || (starts >> (lane + 1) & 1));
}

// Above kUnsorted rays.  Over the sorted keys, 256 rays per workgroup: each thread
// recomputes its ray's contributions, the workgroup sums up to kOpen blocks at a time
// in LDS, a block per table of 9^3 nodes (23 KB: six workgroups per CU; 4 tables and 16
// the same within 1%, 16 fewer workgroups), and adds what got something.  A workgroup
// whose rays hit more than kSparse blocks, 8 rays or fewer in each, has little to sum:
// each ray adds for itself (the line at 64 is the same on grids up to 256^3, where few
// workgroups are near it).  1M rays on 128^3: keys 14 us, sort 66 us, this 76 us, 164 us
// with the gaps; sorted by cell, and the runs of equal keys summed in each wavefront
// (8 global adds for each cell of a wavefront), 193 us.
__global__ __launch_bounds__(kBwdBlock) void k_bwd_blocks(TraceArgs a, const float* __restrict__ t_hit,
                                                          const float* __restrict__ grad_t,
                                                          const uint32_t* __restrict__ keys,
                                                          const uint32_t* __restrict__ rays,
                                                          float* __restrict__ grad_grid, uint32_t none) {
    __shared__ float acc[kOpen * kNodes];
    __shared__ uint32_t s_block[kBwdBlock];  // the distinct blocks, in order
    __shared__ int s_heads[kBwdBlock / 64];
    const int t = threadIdx.x, n = a.n_grid, nb = blocks_per_axis(n), wave = t / 64;
    const int64_t j = (int64_t)blockIdx.x * kBwdBlock + t;
    const uint32_t key = j < a.n ? keys[j] : none;
    const uint32_t left = t > 0 && j - 1 < a.n ? keys[j - 1] : none;
    const bool head = key != none && (t == 0 || key != left);
    const uint64_t heads = __ballot(head);
    if (t % 64 == 0) s_heads[wave] = __popcll(heads);
    for (int q = t; q < kOpen * kNodes; q += kBwdBlock) acc[q] = 0.0f;
    float v[8];
    int ci = 0, cj = 0, ck = 0;
    int64_t cell = 0;
    // the same computation as for the key: it succeeds again
    const bool found = key != none && ray_gradient(a, grid_of(a), rays[j], t_hit, grad_t, cell, v);
    if (found) cell_of(cell, n, ci, cj, ck);
    const bool adds = sum_runs(found, cell, v);
    __syncthreads();
    int before = 0, total = 0;
    for (int w = 0; w < kBwdBlock / 64; ++w) {
        if (w < wave) before += s_heads[w];
        total += s_heads[w];
    }
    // this ray's block among the workgroup's (the keys are sorted)
    const int mine = before + __popcll(heads & (~uint64_t(0) >> (63 - t % 64))) - 1;
    if (total > kSparse) {
        if (adds) add_corners(grad_grid, cell, n, v);
        return;
    }
    if (head) s_block[mine] = key;
    for (int base = 0; base < total; base += kOpen) {
        __syncthreads();  // s_block written; the tables cleared
        if (adds && mine >= base && mine < base + kOpen) {
            const int i = ci - (int)(key % nb) * kCells, jj = cj - (int)(key / nb % nb) * kCells,
                      k = ck - (int)(key / nb / nb) * kCells;
            if ((unsigned)i < kCells && (unsigned)jj < kCells && (unsigned)k < kCells) {
                float* p = acc + (mine - base) * kNodes + i + kSide * (jj + kSide * k);
                for (int c = 0; c < 8; ++c) atomicAdd(p + (c & 1) + kSide * (((c >> 1) & 1) + kSide * (c >> 2)), v[c]);
            } else {  // a recomputation that rounded to another block than the key's
                add_corners(grad_grid, cell, n, v);
            }
        }
        __syncthreads();
        const int open = min(kOpen, total - base);
        for (int q = t; q < open * kNodes; q += kBwdBlock) {
            const float sum = acc[q];
            if (sum == 0.0f) continue;  // a node that no ray touched, or beyond the grid
            acc[q] = 0.0f;
            const uint32_t block = s_block[base + q / kNodes];
            const int r = q % kNodes;
            const int i = (int)(block % nb) * kCells + r % kSide,
                      jj = (int)(block / nb % nb) * kCells + r / kSide % kSide,
                      k = (int)(block / nb / nb) * kCells + r / (kSide * kSide);
            unsafeAtomicAdd(grad_grid + i + (int64_t)n * (jj + (int64_t)n * k), sum);
        }
    }
}

// Up to kUnsorted rays: one launch over the rays in the caller's order, each
// workgroup's 512 rays summed by node in a hash table in LDS before the nodes are added.
// At most 8 * 512 of its 8,192 slots are taken, and the probes' odd stride meets every
// slot, so that every probe ends.  Neighbouring rays of an image share nodes, and what
// narrow views or small grids need is that few workgroups add at one node: 64k rays into
// about 20 cells take 15 us so and 280 us when each wavefront sums its own.
//
// Bound by the global adds.  Sixteen nodes in a row along x keep their order in the table
// (a probe that goes on leaves the group), so that a wavefront adds to few lines at once
// where the rays hit a surface here and there: 256k random rays on 32^3 62 us instead of
// 186 with every node hashed by itself, on 128^3 80 instead of 128; those of an image 23
// instead of 33 and 22 instead of 39 (groups of 8 and 32 the same within 10%).  64 KB:
// two workgroups per CU.
__global__ __launch_bounds__(kSumBlock) void k_bwd_sum(TraceArgs a, const float* __restrict__ t_hit,
                                                       const float* __restrict__ grad_t,
                                                       float* __restrict__ grad_grid) {
    __shared__ uint32_t s_node[kSlots];
    __shared__ float s_sum[kSlots];
    const int64_t i = (int64_t)blockIdx.x * kSumBlock + threadIdx.x;
    for (int q = threadIdx.x; q < kSlots; q += kSumBlock) {
        s_node[q] = kEmpty;
        s_sum[q] = 0.0f;
    }
    int64_t cell = 0;
    float v[8];
    const bool found = i < a.n && ray_gradient(a, grid_of(a), i, t_hit, grad_t, cell, v);
    __syncthreads();
    if (found) {
        const uint32_t n = (uint32_t)a.n_grid;
        uint32_t node[8], slot[8], old[8];
        for (int c = 0; c < 8; ++c) {
            node[c] = (uint32_t)cell + (c & 1) + n * (((c >> 1) & 1) + n * (c >> 2));
            slot[c] = (((node[c] >> kGroupBits) * 2654435769u) >> (32 - kSlotBits + kGroupBits) << kGroupBits) +
                      (node[c] & (kGroup - 1));
            old[c] = atomicCAS(&s_node[slot[c]], kEmpty, node[c]);
        }
        for (int c = 0; c < 8; ++c) {
            while (old[c] != kEmpty && old[c] != node[c]) {
                slot[c] = (slot[c] + kGroup + 1) % kSlots;
                old[c] = atomicCAS(&s_node[slot[c]], kEmpty, node[c]);
            }
            atomicAdd(&s_sum[slot[c]], v[c]);
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < kSlots; q += kSumBlock)
        if (s_node[q] != kEmpty) unsafeAtomicAdd(grad_grid + s_node[q], s_sum[q]);
}

uint32_t key_none(int32_t n_grid) {
    const uint32_t nb = blocks_per_axis(n_grid);
    return nb * nb * nb;
}

int key_bits(int32_t n_grid) {
    const uint32_t none = key_none(n_grid);
    return 32 - __builtin_clz(none);
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

size_t sort_temp_bytes(int64_t n, int32_t n_grid) {
    size_t bytes = 0;
    rocprim::double_buffer<uint32_t> keys(nullptr, nullptr), rays(nullptr, nullptr);
    const hipError_t e = rocprim::radix_sort_pairs<BwdSortConfig>(nullptr, bytes, keys, rays, static_cast<int>(n), 0,
                                                                  key_bits(n_grid), hipStream_t(nullptr));
    return e == hipSuccess ? bytes : 0;
}

}  // namespace

bool df_backward_sorts(int64_t n) { return n > kUnsorted; }

size_t df_backward_workspace(int64_t n, int32_t n_grid) {
    if (n <= 0) return 0;
    const size_t t = sort_temp_bytes(n, n_grid);
    if (t == 0) return 0;
    return 4 * align256(sizeof(uint32_t) * (size_t)n) + align256(t);
}

hipError_t launch_df_backward(const TraceArgs& a, const float* t_hit, const float* grad_t, float* grad_grid,
                              void* workspace, size_t workspace_bytes, hipStream_t stream) {
    if (a.n <= 0) return hipSuccess;
    if (!df_backward_sorts(a.n)) {
        hipLaunchKernelGGL(k_bwd_sum, dim3((unsigned)((a.n + kSumBlock - 1) / kSumBlock)), dim3(kSumBlock), 0, stream,
                           a, t_hit, grad_t, grad_grid);
        return hipGetLastError();
    }
    // four arrays of n words (keys and ray indices, each twice for the sort's
    // passes), then the sort's scratch: the caller sized it with
    // df_backward_workspace(a.n, a.n_grid)
    const size_t arr = align256(sizeof(uint32_t) * (size_t)a.n);
    if (!workspace || workspace_bytes <= 4 * arr) return hipErrorInvalidValue;
    char* p = static_cast<char*>(workspace);
    rocprim::double_buffer<uint32_t> keys(reinterpret_cast<uint32_t*>(p), reinterpret_cast<uint32_t*>(p + arr));
    rocprim::double_buffer<uint32_t> rays(reinterpret_cast<uint32_t*>(p + 2 * arr),
                                          reinterpret_cast<uint32_t*>(p + 3 * arr));
    size_t temp_bytes = workspace_bytes - 4 * arr;
    const uint32_t none = key_none(a.n_grid);
    const unsigned blocks = (unsigned)((a.n + kBwdBlock - 1) / kBwdBlock);
    hipLaunchKernelGGL(k_bwd_keys, dim3(blocks), dim3(kBwdBlock), 0, stream, a, t_hit, grad_t, keys.current(),
                       rays.current(), none);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = rocprim::radix_sort_pairs<BwdSortConfig>(p + 4 * arr, temp_bytes, keys, rays, static_cast<int>(a.n), 0,
                                                 key_bits(a.n_grid), stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bwd_blocks, dim3(blocks), dim3(kBwdBlock), 0, stream, a, t_hit, grad_t, keys.current(),
                       rays.current(), grad_grid, none);
    return hipGetLastError();
}

}  // namespace hyb
