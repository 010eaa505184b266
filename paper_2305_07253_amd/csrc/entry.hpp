// Traversal entry points (internal header): what the device build of the
// pyramid (entry.hip) and its host build (bvh_build.cpp) share.  Plain C++, so
// both compilers take it.
#pragma once

#include <cstdint>
#include <cstring>

#include "bvh_build.hpp"

#if defined(__HIPCC__)
#define HYB_ENTRY_HD __host__ __device__ inline
#else
#define HYB_ENTRY_HD inline
#endif

namespace hyb {

HYB_ENTRY_HD int32_t entry_word(const float* p) {
    int32_t v;
    __builtin_memcpy(&v, p, 4);
    return v;
}

// Parent node and depth of a nodes4 index or leaf reference: stored in the
// node's unused last column, and beside the leaf's first triangle.
HYB_ENTRY_HD int32_t entry_up(const float* nodes4, const float* tris, int32_t r) {
    return r >= 0 ? entry_word(nodes4 + 32 * static_cast<int64_t>(r) + kNode4Parent)
                  : entry_word(tris + 12 * static_cast<int64_t>((~r) >> 3) + kTriLeafParent);
}

HYB_ENTRY_HD int32_t entry_depth(const float* nodes4, const float* tris, int32_t r) {
    return r >= 0 ? entry_word(nodes4 + 32 * static_cast<int64_t>(r) + kNode4Depth)
                  : entry_word(nodes4 + 32 * static_cast<int64_t>(entry_up(nodes4, tris, r)) + kNode4Depth) + 1;
}

// Lowest common ancestor of two references (kEmptyRef: none yet).
HYB_ENTRY_HD int32_t entry_lca(const float* nodes4, const float* tris, int32_t a, int32_t b) {
    if (a == b || b == kEmptyRef) return a;
    if (a == kEmptyRef) return b;
    if (a == 0 || b == 0) return 0;  // the root
    int32_t da = entry_depth(nodes4, tris, a), db = entry_depth(nodes4, tris, b);
    for (; da > db; --da) a = entry_up(nodes4, tris, a);
    for (; db > da; --db) b = entry_up(nodes4, tris, b);
    while (a != b) {
        a = entry_up(nodes4, tris, a);
        b = entry_up(nodes4, tris, b);
    }
    return a;
}

// The finest half-cells [v0, v1] that a leaf's box [lo, hi] overlaps along
// one axis, the box grown by a margin (FP32 rounding of segment end points is
// far below it).  The cube has 2 res half-cells per axis.
HYB_ENTRY_HD void entry_range(float lo, float hi, float cube_lo, float size, int res, int& v0, int& v1) {
#if defined(__clang__)
#pragma clang fp contract(off)
#endif
    const double half = 0.5 * static_cast<double>(size), top = 2 * res - 1.0;
    const double a = lo < 0.0f ? -static_cast<double>(lo) : lo, b = hi < 0.0f ? -static_cast<double>(hi) : hi;
    const double slack = 1e-3 * size + 1e-6 * (1.0 + (a > b ? a : b));
    const double u0 = (lo - slack - cube_lo) / half, u1 = (hi + slack - cube_lo) / half;
    v0 = static_cast<int>(u0 < 0.0 ? 0.0 : (u0 > top ? top : u0));  // truncation is floor: never negative
    v1 = static_cast<int>(u1 < 0.0 ? 0.0 : (u1 > top ? top : u1));
}

// Entries of all levels of a pyramid of res^3 finest voxels.
inline int64_t entry_total(int res) {
    int64_t total = 0;
    for (int e = res; e >= 1; e >>= 1) total += static_cast<int64_t>(2 * e - 1) * (2 * e - 1) * (2 * e - 1);
    return total;
}

}  // namespace hyb
