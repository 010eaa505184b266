// Distance-field construction from the triangle BVH: every grid node's exact
// signed distance in FP64 (point/triangle distance and crossing tests of
// sdf_device.hpp), rounded once to FP32.
//
//   k_mesh_boundary   (with the tree) is the mesh a closed surface?
//   k_sdf_nearest     unsigned distances, one wavefront per 4^3 nodes, or
//   k_sdf_nearest_apart  four lanes per node
//   k_sdf_components  nodes joined across surface-free balls, per 8^3 nodes
//   k_sdf_cast        the winding number of one node per component
//   k_sdf_sign        every other node takes its component's sign
//   k_sdf_few         all of it for meshes of a few triangles
#include "kernels.hpp"
#include "sdf_device.hpp"

namespace hyb {
namespace {

constexpr int kWave = 64;
constexpr int kThreads = 256;

// ---------------------------------------------------------------------------
// closed surface
// ---------------------------------------------------------------------------

__device__ uint64_t mix64(uint64_t x) {  // Steele et al., "Fast splittable pseudorandom number generators", 2014
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    return x ^ (x >> 31);
}

__device__ uint64_t vertex_hash(float4 v) {
    const uint32_t x = __builtin_bit_cast(uint32_t, v.x + 0.0f), y = __builtin_bit_cast(uint32_t, v.y + 0.0f),
                   z = __builtin_bit_cast(uint32_t, v.z + 0.0f);  // + 0: one zero
    return mix64(mix64(((uint64_t)x << 32 | y) + 0x9e3779b97f4a7c15ull) + z);
}

__device__ uint64_t edge_hash(uint64_t a, uint64_t b) { return mix64(a + mix64(b + 1)) - mix64(b + mix64(a + 1)); }

// Adds a hash of every directed edge (by its end positions), a -> b and b -> a
// opposite: the sum is 0 when every edge is run through as often one way as the
// other (up to one chance in 2^64), so the triangles form closed surfaces and
// the winding number is constant on any path that meets none of them.
__global__ __launch_bounds__(kThreads) void k_mesh_boundary(const float4* __restrict__ tris, int64_t n,
                                                            unsigned long long* __restrict__ sum) {
    uint64_t acc = 0;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
        const uint64_t a = vertex_hash(tris[3 * i]), b = vertex_hash(tris[3 * i + 1]), c = vertex_hash(tris[3 * i + 2]);
        acc += edge_hash(a, b) + edge_hash(b, c) + edge_hash(c, a);
    }
    for (int o = kWave / 2; o > 0; o >>= 1) acc += __shfl_xor((unsigned long long)acc, o, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0 && acc) atomicAdd(sum, (unsigned long long)acc);
}

// ---------------------------------------------------------------------------
// unsigned distances
// ---------------------------------------------------------------------------

__device__ D3 node_position(const SdfBuildArgs& a, int i, int j, int k) {
    return d3((double)a.lo_x + (double)i * (double)a.h, (double)a.lo_y + (double)j * (double)a.h,
              (double)a.lo_z + (double)k * (double)a.h);
}

// A coordinate rounded to FP32 downward and upward (by an ulp more than needed).
struct Around {
    float lo, hi;
};

__device__ Around around(double p) {
    const float f = (float)p, e = fabsf(f) * 1.2e-7f;
    return {f - e, f + e};
}

// Squared distance of a point to a box from below, but for a rounding error (relative,
// at most 4e-7, and 3e-45 of products below the normal range) that every use allows for.
__device__ float box_below(Around x, Around y, Around z, float lx, float hx, float ly, float hy, float lz, float hz) {
    const float dx = fmaxf(fmaxf(lx - x.hi, x.lo - hx), 0.0f), dy = fmaxf(fmaxf(ly - y.hi, y.lo - hy), 0.0f),
                dz = fmaxf(fmaxf(lz - z.hi, z.lo - hz), 0.0f);
    return fmaf(dx, dx, fmaf(dy, dy, dz * dz));
}

// The same for a triangle's box.
__device__ float triangle_below(Around x, Around y, Around z, float4 a, float4 b, float4 c) {
    return box_below(x, y, z, fminf(fminf(a.x, b.x), c.x), fmaxf(fmaxf(a.x, b.x), c.x), fminf(fminf(a.y, b.y), c.y),
                     fmaxf(fmaxf(a.y, b.y), c.y), fminf(fminf(a.z, b.z), c.z), fmaxf(fmaxf(a.z, b.z), c.z));
}

// A squared distance in FP32, from above by the error that box_below may have (the
// constant: of its products below the normal range).
__device__ float bound_of(double d2) { return fmaf((float)d2, 1.0f + 2e-6f, 1e-43f); }

// Largest value of the wavefront, in every lane (all lanes active).
__device__ float wave_max(float v) {
#define HYB_MAX_STEP(ctrl, rows)                                                                                      \
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, v),                   \
                                                                       __builtin_bit_cast(int, v), ctrl, rows, 0xf, \
                                                                       false)))
    HYB_MAX_STEP(0x111, 0xf);  // row_shr 1, 2, 4, 8: the last lane of each row of 16 has its maximum
    HYB_MAX_STEP(0x112, 0xf);
    HYB_MAX_STEP(0x114, 0xf);
    HYB_MAX_STEP(0x118, 0xf);
    HYB_MAX_STEP(0x142, 0xa);  // row_bcast 15, 31
    HYB_MAX_STEP(0x143, 0xc);
#undef HYB_MAX_STEP
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), kWave - 1));
}

__device__ void order_keys(uint32_t& ka, int& ra, uint32_t& kb, int& rb) {
    const bool sw = kb < ka;
    const uint32_t k = sw ? kb : ka;
    const int r = sw ? rb : ra;
    kb = sw ? ka : kb;
    rb = sw ? ra : rb;
    ka = k;
    ra = r;
}

// Nearest triangle of 4 x 4 x 4 nodes by one traversal of the four-wide tree
// per wavefront.  The node and triangle a wavefront reads are the same for all
// lanes, so they come through scalar loads, the loop does not diverge and the
// stack is a register across the lanes.  A child is entered when its box may be
// nearer than the nearest triangle so far for any lane, nearest first as seen
// from one lane near the middle; a popped child is dropped when even from the
// farthest lane it is no nearer.  Boxes of children and triangles are tested in
// FP32 from below; only triangles that pass are measured, in FP64.
//
// Bound by VALU issue, more than half of it the FP64 tests: at 128^3 on the
// 188,572-triangle scene a wavefront visits 58 nodes and measures 62 triangles.
// 1.25 ms there.  One thread per node with its own FP64 traversal and its stack in
// scratch took 6.26 ms, the sign included.
__global__ __launch_bounds__(kWave) void k_sdf_nearest(SdfBuildArgs a, const float4* __restrict__ nodes4,
                                                       const float4* __restrict__ tris, float* __restrict__ out) {
    constexpr int kMiddle = 1 + 4 + 16;  // lane of node (1, 1, 1): at most 2 sqrt(3) h from any lane
    constexpr uint32_t kSkip = 0xffffffffu;
    static_assert(kStackDepth4 <= 2 * kWave, "the stack is two registers across the lanes");
    const int lane = threadIdx.x, n = a.n_grid, nt = (n + 3) / 4;
    const uint32_t tile = xcd_block(blockIdx.x, gridDim.x, kXcdRun);
    const int i = (int)(tile % nt) * 4 + (lane & 3), j = (int)(tile / nt % nt) * 4 + (lane >> 2 & 3),
              k = (int)(tile / nt / nt) * 4 + (lane >> 4);
    const D3 p = node_position(a, min(i, n - 1), min(j, n - 1), min(k, n - 1));
    const Around x = around(p.x), y = around(p.y), z = around(p.z);
    const float reach = 3.4642f * a.h;

    double best = __builtin_inf();
    float bound = __builtin_inff();  // best from above
    float limit = __builtin_inff();  // squared distance from the middle beyond which no lane needs a box
    int refs0 = 0, refs1 = 0, keys0 = 0, keys1 = 0;
    int sp = 0, ref = 0;
    for (;;) {
        if (ref >= 0) {
            const float4* nd = nodes4 + 8 * (int64_t)ref;
            const float4 lx = nd[0], hx = nd[1], ly = nd[2], hy = nd[3], lz = nd[4], hz = nd[5], rf = nd[6];
            const float b0 = box_below(x, y, z, lx.x, hx.x, ly.x, hy.x, lz.x, hz.x);
            const float b1 = box_below(x, y, z, lx.y, hx.y, ly.y, hy.y, lz.y, hz.y);
            const float b2 = box_below(x, y, z, lx.z, hx.z, ly.z, hy.z, lz.z, hz.z);
            const float b3 = box_below(x, y, z, lx.w, hx.w, ly.w, hy.w, lz.w, hz.w);
            int r0 = bits_i(rf.x), r1 = bits_i(rf.y), r2 = bits_i(rf.z), r3 = bits_i(rf.w);
            const auto key = [&](float b, int r) {
                const uint32_t mid = (uint32_t)__builtin_amdgcn_readlane(bits_i(b), kMiddle);
                return __ballot(b <= bound) != 0 && r != kEmptyRef ? mid : kSkip;
            };
            uint32_t k0 = key(b0, r0), k1 = key(b1, r1), k2 = key(b2, r2), k3 = key(b3, r3);
            order_keys(k0, r0, k1, r1);
            order_keys(k2, r2, k3, r3);
            order_keys(k0, r0, k2, r2);
            order_keys(k1, r1, k3, r3);
            order_keys(k1, r1, k2, r2);
            const uint32_t ks[3] = {k3, k2, k1};
            const int rs[3] = {r3, r2, r1};
            for (int c = 0; c < 3; ++c) {
                if (ks[c] == kSkip) continue;
                if (sp < kWave) {
                    refs0 = lane == sp ? rs[c] : refs0;
                    keys0 = lane == sp ? (int)ks[c] : keys0;
                } else {
                    refs1 = lane == sp - kWave ? rs[c] : refs1;
                    keys1 = lane == sp - kWave ? (int)ks[c] : keys1;
                }
                ++sp;
            }
            if (k0 != kSkip) {
                ref = r0;
                continue;
            }
        } else {
            const int first = (~ref) >> 3, count = (~ref) & 7;
            bool nearer = false;
            for (int q = 0; q < count; ++q) {
                const float4* tp = tris + 3 * (int64_t)(first + q);
                const float4 v0 = tp[0], v1 = tp[1], v2 = tp[2];
                const float b = triangle_below(x, y, z, v0, v1, v2);
                if (b <= bound) {
                    const double t = tri_dist2(p, dvert(v0), dvert(v1), dvert(v2));
                    if (t < best) {
                        best = t;
                        bound = bound_of(t);
                        nearer = true;
                    }
                }
            }
            if (__ballot(nearer) != 0) {
                const float far = sqrtf(wave_max(bound)) + reach;
                limit = fmaf(far * far, 1.0f + 4e-6f, 1e-43f);
            }
        }
        bool found = false;
        while (sp > 0) {
            --sp;
            const float mid = __builtin_bit_cast(float, sp < kWave ? __builtin_amdgcn_readlane(keys0, sp)
                                                                   : __builtin_amdgcn_readlane(keys1, sp - kWave));
            if (mid <= limit) {
                ref = sp < kWave ? __builtin_amdgcn_readlane(refs0, sp) : __builtin_amdgcn_readlane(refs1, sp - kWave);
                found = true;
                break;
            }
        }
        if (!found) break;
    }
    if (blockIdx.x == 0 && lane == 0) *a.count = 0;
    if (i < n && j < n && k < n) out[i + (int64_t)n * (j + (int64_t)n * k)] = (float)sqrt(best);
}

constexpr int kQuads = kWave / 4;  // nodes or rays of a wavefront that gives four lanes to each

__device__ float quad_min(float v) {
    v = fminf(v, __shfl_xor(v, 1, kWave));
    return fminf(v, __shfl_xor(v, 2, kWave));
}

// The same for nodes that lie far apart beside the triangles (nodes_apart): a traversal
// for each node, four lanes to a node, one for each child of a tree node and each
// triangle of a leaf, nearest child first, with the stack in LDS.  The same triangles'
// distances, so the same result.  Bound by the chain of visits of its longest node,
// some 300 to 500 of them at half a microsecond: 188,572 triangles at 12^3 take 0.3 ms,
// field and all, where one thread per node took 0.9 and packets, which visit 4,263 nodes and
// measure 7,168 triangles in one wavefront, 6.7.
__global__ __launch_bounds__(kWave) void k_sdf_nearest_apart(SdfBuildArgs a) {
    __shared__ int s_refs[kQuads * kStackDepth4];
    __shared__ float s_keys[kQuads * kStackDepth4];
    const int lane = threadIdx.x, c = lane & 3, base = lane & ~3;
    int* refs = s_refs + (lane >> 2);  // entries kQuads apart
    float* keys = s_keys + (lane >> 2);
    const int64_t n = a.n_grid, id = (int64_t)blockIdx.x * kQuads + (lane >> 2);
    if (blockIdx.x == 0 && lane == 0) *a.count = 0;
    if (id >= n * n * n) return;
    const D3 p = node_position(a, (int)(id % n), (int)(id / n % n), (int)(id / (n * n)));
    const Around x = around(p.x), y = around(p.y), z = around(p.z);
    double best = __builtin_inf();  // of this lane's triangles
    float bound = __builtin_inff();  // of all four lanes', from above
    int sp = 0, ref = 0;
    for (;;) {
        bool found = false;
        if (ref >= 0) {
            const float* q = reinterpret_cast<const float*>(a.nodes4 + 8 * (int64_t)ref) + c;
            const float b = box_below(x, y, z, q[0], q[4], q[8], q[12], q[16], q[20]);
            const int child = bits_i(q[24]);
            const bool hit = b <= bound && child != kEmptyRef;
            const int hits = (int)(__ballot(hit) >> base) & 15;
            // place among the children to visit, nearest first (equal ones in slot order)
            int place = 0;
            for (int o = 1; o < 4; ++o) {
                const float other = __shfl_xor(b, o, kWave);
                if ((hits >> (c ^ o) & 1) && (other < b || (other == b && (c ^ o) < c))) ++place;
            }
            const int behind = __popc(hits) - 1;
            if (hit && place > 0) {
                refs[(sp + behind - place) * kQuads] = child;
                keys[(sp + behind - place) * kQuads] = b;
            }
            if (behind >= 0) {
                const int first = (int)(__ballot(hit && place == 0) >> base) & 15;
                ref = __shfl(child, base + __ffs(first) - 1, kWave);
                sp += behind;
                found = true;
            }
        } else {
            const int first = (~ref) >> 3, count = (~ref) & 7;
            for (int t = c; t < count; t += 4) {
                const float4* tp = a.tris + 3 * (int64_t)(first + t);
                const float4 v0 = tp[0], v1 = tp[1], v2 = tp[2];
                const float b = triangle_below(x, y, z, v0, v1, v2);
                if (b <= bound) best = fmin(best, tri_dist2(p, dvert(v0), dvert(v1), dvert(v2)));
            }
            bound = quad_min(bound_of(best));
        }
        // the four lanes read what each other wrote
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        while (!found && sp > 0) {
            --sp;
            ref = refs[sp * kQuads];
            found = keys[sp * kQuads] <= bound;
        }
        if (!found) break;
    }
    best = fmin(best, __shfl_xor(best, 1, kWave));
    best = fmin(best, __shfl_xor(best, 2, kWave));
    if (c == 0) a.out[id] = (float)sqrt(best);
}

// ---------------------------------------------------------------------------
// signs
// ---------------------------------------------------------------------------

constexpr int kTile = 8;
constexpr int kTileNodes = kTile * kTile * kTile;

__device__ int64_t tile_node(int n, uint32_t tile, int in_tile, int& i, int& j, int& k) {
    const int nt = (n + kTile - 1) / kTile;
    i = (int)(tile % nt) * kTile + in_tile % kTile;
    j = (int)(tile / nt % nt) * kTile + in_tile / kTile % kTile;
    k = (int)(tile / nt / nt) * kTile + in_tile / (kTile * kTile);
    return i + (int64_t)n * (j + (int64_t)n * k);
}

// No triangle lies within a node's distance of it, so when the balls of two
// neighbouring nodes overlap the segment between them meets no surface, and on
// a closed surface both have one sign.  Joins the nodes of a tile that way (26
// neighbours, so a node 0.07 h off a surface already joins one away from it)
// and lists each component's first node; each node keeps its component's first
// node in the tile.  The winding number, a traversal of the whole ray, is then
// found for a few percent of the nodes.  On an open surface every node is
// listed.
__global__ __launch_bounds__(kTileNodes) void k_sdf_components(SdfBuildArgs a) {
    __shared__ float dist[kTileNodes];
    __shared__ int label[kTileNodes];
    __shared__ int before[kTileNodes / kWave + 1];
    const int t = threadIdx.x, n = a.n_grid;
    int i, j, k;
    const int64_t id = tile_node(n, blockIdx.x, t, i, j, k);
    const bool inside = i < n && j < n && k < n;
    const bool closed = *a.boundary == 0;
    const float d = inside ? a.out[id] : -__builtin_inff();
    dist[t] = d;
    label[t] = t;
    __syncthreads();
    // a tile whose nodes all join their neighbours along the axes is one component
    const bool one = closed && __syncthreads_and(!inside || d > 0.501f * a.h);
    uint32_t joined = 0;
    const int x = t % kTile, y = t / kTile % kTile, z = t / (kTile * kTile);
    int bit = 0;
    for (int dz = -1; dz <= 1 && !one; ++dz)
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx) {
                if (dx == 0 && dy == 0 && dz == 0) continue;
                const int steps = dx * dx + dy * dy + dz * dz;
                const float apart = (steps == 1 ? 1.0f : (steps == 2 ? 1.4142136f : 1.7320508f)) * a.h * 1.0001f;
                const bool in = (unsigned)(x + dx) < kTile && (unsigned)(y + dy) < kTile && (unsigned)(z + dz) < kTile;
                if (closed && in && d + dist[t + dx + kTile * (dy + kTile * dz)] > apart) joined |= 1u << bit;
                ++bit;
            }
    int mine = one ? 0 : t;
    while (!one) {
        int m = mine;
        bit = 0;
        for (int dz = -1; dz <= 1; ++dz)
            for (int dy = -1; dy <= 1; ++dy)
                for (int dx = -1; dx <= 1; ++dx) {
                    if (dx == 0 && dy == 0 && dz == 0) continue;
                    if (joined >> bit & 1) m = min(m, label[t + dx + kTile * (dy + kTile * dz)]);
                    ++bit;
                }
        m = min(m, label[m]);
        __syncthreads();
        const bool changed = m != mine;
        mine = label[t] = m;
        if (!__syncthreads_or(changed)) break;
    }
    // the listed nodes of a tile stay together: they cast neighbouring rays
    const bool first = inside && mine == t;
    const uint64_t firsts = __ballot(first);
    const int wave = t / kWave;
    if (t % kWave == 0) before[wave + 1] = __popcll(firsts);
    __syncthreads();
    if (t == 0) {
        int sum = 0;
        for (int w = 1; w <= kTileNodes / kWave; ++w) {
            const int c = before[w];
            before[w] = sum;
            sum += c;
        }
        before[0] = (int)atomicAdd(a.count, (uint32_t)sum);
    }
    __syncthreads();
    if (first) {
        const uint64_t lower = firsts & ((uint64_t(1) << (t % kWave)) - 1);
        a.list[(uint32_t)before[0] + before[wave + 1] + __popcll(lower)] = (uint32_t)id;
    }
    if (inside) a.label[id] = (uint16_t)mine;
}

// The direction of the winding number's rays: one that no mesh edge is likely
// to contain.  All components are positive, which the box test uses.
__device__ D3 cast_direction() {
    const double len = sqrt(0.61 * 0.61 + 0.5177 * 0.5177 + 0.6003 * 0.6003);
    return d3(0.61 / len, 0.5177 / len, 0.6003 / len);
}

constexpr int kCastBlocks = 8192;

// Winding number of every listed node: signed crossings of its ray with the
// triangles, boxes tested in FP32 widened over its rounding, triangles in FP64.
// Four lanes per ray, one for each child of a node and each triangle of a leaf:
// the rays are few (some tens of thousands at 128^3), so the kernel is bound by
// the chain of node visits of the longest ray, and a visit is a quarter as long
// this way, on four times the wavefronts (0.42 -> 0.15 ms at 128^3 against one
// lane per ray).
__global__ __launch_bounds__(kWave) void k_sdf_cast(SdfBuildArgs a) {
    __shared__ int s_stack[kQuads * kStackAll4];
    const int lane = threadIdx.x, c = lane & 3;
    int* stack = s_stack + (lane >> 2);  // entries kQuads apart
    const int64_t n = a.n_grid;
    const D3 D = cast_direction();
    const float ix = (float)(1.0 / D.x), iy = (float)(1.0 / D.y), iz = (float)(1.0 / D.z);
    const uint32_t total = *a.count;
    for (uint32_t at = blockIdx.x * kQuads + (lane >> 2); at < total; at += gridDim.x * kQuads) {
        const uint32_t id = a.list[at];
        const D3 p = node_position(a, (int)(id % n), (int)(id / n % n), (int)(id / (n * n)));
        const Around x = around(p.x), y = around(p.y), z = around(p.z);
        int wind = 0;
        int sp = 0, ref = 0;
        for (;;) {
            if (ref >= 0) {
                const float* q = reinterpret_cast<const float*>(a.nodes4 + 8 * (int64_t)ref) + c;
                const float lx = q[0], hx = q[4], ly = q[8], hy = q[12], lz = q[16], hz = q[20];
                const int child = bits_i(q[24]);
                const float in = fmaxf(fmaxf((lx - x.hi) * ix, (ly - y.hi) * iy), fmaxf((lz - z.hi) * iz, 0.0f));
                const float out = fminf(fminf((hx - x.lo) * ix, (hy - y.lo) * iy), (hz - z.lo) * iz);
                const bool hit = in <= out * (1.0f + 2e-6f) && child != kEmptyRef;
                const int hits = (int)(__ballot(hit) >> (lane & ~3)) & 15;
                if (hit) stack[(sp + __popc(hits & ((1 << c) - 1))) * kQuads] = child;
                sp += __popc(hits);
            } else {
                const int first = (~ref) >> 3, count = (~ref) & 7;
                for (int t = c; t < count; t += 4) {
                    const float4* tp = a.tris + 3 * (int64_t)(first + t);
                    wind += crossing(p, D, dvert(tp[0]), dvert(tp[1]), dvert(tp[2]));
                }
            }
            if (sp == 0) break;
            // the four lanes read what one of them wrote
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            ref = stack[--sp * kQuads];
        }
        wind += __shfl_xor(wind, 1, kWave);
        wind += __shfl_xor(wind, 2, kWave);
        if (c == 0 && wind + (a.exterior_solid ? 1 : 0) >= 1) a.out[id] = -a.out[id];
    }
}

// Nodes that were not listed take the sign of their component's listed node.
__global__ __launch_bounds__(kThreads) void k_sdf_sign(SdfBuildArgs a) {
    const int64_t n = a.n_grid, id = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (id >= n * n * n) return;
    const int i = (int)(id % n), j = (int)(id / n % n), k = (int)(id / (n * n));
    const int mine = i % kTile + kTile * (j % kTile + kTile * (k % kTile)), root = a.label[id];
    if (root == mine) return;
    const int64_t at = (i / kTile * kTile + root % kTile) +
                       n * ((j / kTile * kTile + root / kTile % kTile) +
                            n * (k / kTile * kTile + root / (kTile * kTile)));
    if (__builtin_bit_cast(uint32_t, a.out[at]) >> 31) a.out[id] = -a.out[id];
}

// Few triangles: every node goes through all of them and counts its own ray's crossings,
// in one pass.  The passes for larger meshes cost launches and n^3 labels whatever the
// mesh: 2 triangles at 128^3 229 us with them, 127 in this one (155 by one thread per node
// and a tree), 30 at 128^3 326 and 304, at 256^3 2,036 and 1,820, 40 there 1,981 and 2,165.
__global__ __launch_bounds__(kThreads) void k_sdf_few(SdfBuildArgs a) {
    const int64_t n = a.n_grid, id = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (id >= n * n * n) return;
    const D3 p = node_position(a, (int)(id % n), (int)(id / n % n), (int)(id / (n * n))), D = cast_direction();
    const Around x = around(p.x), y = around(p.y), z = around(p.z);
    double best = __builtin_inf();
    int wind = a.exterior_solid ? 1 : 0;
    for (int t = 0; t < (int)a.n_tris; ++t) {
        const float4 v0 = a.tris[3 * t], v1 = a.tris[3 * t + 1], v2 = a.tris[3 * t + 2];
        if (triangle_below(x, y, z, v0, v1, v2) <= bound_of(best))
            best = fmin(best, tri_dist2(p, dvert(v0), dvert(v1), dvert(v2)));
        wind += crossing(p, D, dvert(v0), dvert(v1), dvert(v2));
    }
    const float dist = (float)sqrt(best);
    a.out[id] = wind >= 1 ? -dist : dist;
}

}  // namespace

size_t sdf_build_scratch(int32_t n) { return 16 + (sizeof(uint32_t) + sizeof(uint16_t)) * (size_t)n * n * n; }

hipError_t launch_mesh_boundary(const float4* tris, int64_t n_tris, unsigned long long* sum, hipStream_t stream) {
    if (n_tris <= 0) return hipSuccess;
    const int64_t blocks = (n_tris + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(k_mesh_boundary, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(kThreads), 0, stream,
                       tris, n_tris, sum);
    return hipGetLastError();
}

constexpr int64_t kFewTriangles = 32;  // k_sdf_few

// Whether the nodes of a grid lie too far apart beside the triangles for a wavefront to
// search for 64 of them at once.  `spacing` is a voxel in triangles of a surface that
// spans the mesh once.  A packet visits what any of its nodes needs, one after the
// other; four lanes to a node visit what that node needs, on four times the wavefronts,
// and share none of it.  Packets against lanes of their own, the whole field in us:
// 188,572 triangles at 16^3 (spacing 39) 4,380 and 340, 32^3 (16) 1,550 and 505, 48^3
// (10) 1,230 and 720, 64^3 (7) 1,090 and 1,170, 128^3 (3.5) 1,600 and 5,700; on a grid
// four times the mesh 64^3 (27) 2,800 and 630, 128^3 (13) 1,850 and 3,500; 25,740 on
// that grid at 64^3 (9.9) 1,080 and 550.  Up to 40^3 packets leave SIMDs without a
// wavefront: 1,324 triangles at 32^3 (1.3) 215 and 191, 44^3 (0.9) 224 and 221, 64^3
// (0.6) 240 and 450.
static bool nodes_apart(const SdfBuildArgs& a) {
    const float spacing = a.h * sqrtf((float)a.n_tris) / a.extent;
    return a.n_grid <= 512 && spacing > (a.n_grid <= 40 ? 1.0f : 0.15f * (float)a.n_grid);
}

hipError_t launch_sdf_build(const SdfBuildArgs& args, void* scratch, size_t scratch_bytes, hipStream_t stream) {
    const size_t n = (size_t)args.n_grid, total = n * n * n;
    if (n < 2 || n > 1024 || !scratch || scratch_bytes < sdf_build_scratch(args.n_grid)) return hipErrorInvalidValue;
    SdfBuildArgs a = args;
    a.count = static_cast<uint32_t*>(scratch);
    a.list = a.count + 4;
    a.label = reinterpret_cast<uint16_t*>(a.list + total);
    const unsigned nt = (unsigned)(n + 3) / 4, tiles = (unsigned)(n + kTile - 1) / kTile;
    if (a.n_tris <= kFewTriangles) {
        hipLaunchKernelGGL(k_sdf_few, dim3((unsigned)((total + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream,
                           a);
        return hipGetLastError();
    }
    if (nodes_apart(a))
        hipLaunchKernelGGL(k_sdf_nearest_apart, dim3((unsigned)((total + kQuads - 1) / kQuads)), dim3(kWave), 0, stream,
                           a);
    else
        hipLaunchKernelGGL(k_sdf_nearest, dim3(nt * nt * nt), dim3(kWave), 0, stream, a, a.nodes4, a.tris, a.out);
    hipLaunchKernelGGL(k_sdf_components, dim3(tiles * tiles * tiles), dim3(kTileNodes), 0, stream, a);
    hipLaunchKernelGGL(k_sdf_cast, dim3(kCastBlocks), dim3(kWave), 0, stream, a);
    hipLaunchKernelGGL(k_sdf_sign, dim3((unsigned)((total + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

}  // namespace hyb
