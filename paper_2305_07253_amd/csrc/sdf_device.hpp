// Exact signed distance at one grid node (internal header), host+device so a
// CPU build can check it: the distance of a point to a triangle, the signed
// crossing of a ray with one, and, as the definition of a node's value, a query
// of one point that uses them.  The build kernels (sdf_build.hip) evaluate the
// same two functions over many nodes at once.
//   distance  nearest-triangle query over the BVH in FP64: children in order of
//             their box distance, a subtree skipped once its box is no closer
//             than the best triangle; point/triangle distance = plane distance
//             when the projection falls inside, else the nearest edge segment;
//   sign      winding number from signed ray crossings along a fixed generic
//             direction (leaving through the front of a face +1, entering -1),
//             plus 1 when the exterior is solid; solid iff the total is >= 1.
#pragma once

#include "bvh_build.hpp"
#include "hyb_device.hpp"

namespace hyb {

struct D3 {
    double x, y, z;
};

HYB_HD D3 d3(double x, double y, double z) { return D3{x, y, z}; }
HYB_HD D3 dsub(D3 a, D3 b) { return d3(a.x - b.x, a.y - b.y, a.z - b.z); }
HYB_HD double ddot(D3 a, D3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
HYB_HD D3 dcross(D3 a, D3 b) {
    return d3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
HYB_HD D3 dvert(float4 v) { return d3(v.x, v.y, v.z); }

// Reciprocal to about 2^-46, for positive normal x: the hardware's estimate (2^-23)
// after one Newton step, tens of units in the last place.  Callers correct for it or
// use it where its error enters squared.  (Exact division in the CPU build.)
HYB_HD double rcp64(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
    const double r = __builtin_amdgcn_rcp(x);
    return fma(fma(-x, r, 1.0), r, r);
#else
    return 1.0 / x;
#endif
}

// squared length of w - s e at the s in [0, 1] that makes it least: the distance
// from a point w off the start of an edge e.  An error of s enters only squared (s is
// at the minimum), so the reciprocal need not be rounded correctly.
HYB_HD double edge_dist2(D3 w, D3 e) {
    const double ee = ddot(e, e);
    double s = ee > 0.0 ? ddot(w, e) * rcp64(ee) : 0.0;
    s = fmin(fmax(s, 0.0), 1.0);
    const D3 r = d3(fma(-s, e.x, w.x), fma(-s, e.y, w.y), fma(-s, e.z, w.z));
    return ddot(r, r);
}

// squared distance from p to triangle abc: to its plane when the projection of
// p lies inside, else to the nearest edge.  Inside is the inner side of the three
// planes that hold an edge and the normal: each test is good to a rounding of p
// against its own edge, however thin the triangle.  (Barycentric coordinates from
// the Gram matrix of two edges take nine FP64 products less, 1,525 against 1,610 us
// for the grid of sdf_build.hip, but their determinant is a difference of nearly
// equal products, mere rounding once the height is 1e-8 of the length: points beyond
// an end then pass for inside, and get the distance to the plane.)
HYB_HD double tri_dist2(D3 p, D3 a, D3 b, D3 c) {
    const D3 e = dsub(b, a), f = dsub(c, a), g = dsub(c, b), w = dsub(p, a), x = dsub(p, b);
    const D3 n = dcross(e, f);
    const double nn = ddot(n, n);
    if (nn > 0.0 && ddot(dcross(e, w), n) >= 0.0 && ddot(dcross(g, x), n) >= 0.0 &&
        ddot(dcross(f, dsub(p, c)), n) <= 0.0) {
        const double h = ddot(w, n), hh = h * h, r = rcp64(nn), q = hh * r;
        return fma(fma(-q, nn, hh), r, q);
    }
    return fmin(edge_dist2(w, e), fmin(edge_dist2(w, f), edge_dist2(x, g)));
}

HYB_HD double box_dist2(D3 p, float lx, float hx, float ly, float hy, float lz, float hz) {
    const double dx = fmax(fmax((double)lx - p.x, 0.0), p.x - (double)hx);
    const double dy = fmax(fmax((double)ly - p.y, 0.0), p.y - (double)hy);
    const double dz = fmax(fmax((double)lz - p.z, 0.0), p.z - (double)hz);
    return dx * dx + dy * dy + dz * dz;
}

// ray (o + t D, t > 0) against a box, FP64
HYB_HD bool ray_box64(D3 o, D3 inv, float lx, float hx, float ly, float hy, float lz, float hz) {
    const double t0x = ((double)lx - o.x) * inv.x, t1x = ((double)hx - o.x) * inv.x;
    const double t0y = ((double)ly - o.y) * inv.y, t1y = ((double)hy - o.y) * inv.y;
    const double t0z = ((double)lz - o.z) * inv.z, t1z = ((double)hz - o.z) * inv.z;
    const double tn = fmax(fmax(fmin(t0x, t1x), fmin(t0y, t1y)), fmax(fmin(t0z, t1z), 0.0));
    const double tf = fmin(fmin(fmax(t0x, t1x), fmax(t0y, t1y)), fmax(t0z, t1z));
    return tn <= tf * (1.0 + 1e-12);
}

// signed crossing of the ray o + t D (t > 0) with triangle abc: +1 when the ray
// leaves through the front side (D . n > 0), -1 when it enters, 0 when it misses
// (edge functions of the triangle seen along D, all of one sign)
HYB_HD int crossing(D3 o, D3 D, D3 a, D3 b, D3 c) {
    const D3 pa = dsub(a, o), pb = dsub(b, o), pc = dsub(c, o);
    const double wa = ddot(D, dcross(pb, pc));
    const double wb = ddot(D, dcross(pc, pa));
    const double wc = ddot(D, dcross(pa, pb));
    if (!((wa >= 0.0 && wb >= 0.0 && wc >= 0.0) || (wa <= 0.0 && wb <= 0.0 && wc <= 0.0))) return 0;
    const double s = wa + wb + wc;
    if (s == 0.0) return 0;
    const D3 n = dcross(dsub(b, a), dsub(c, a));
    const double t = ddot(n, pa) / ddot(n, D);
    if (!(t > 0.0)) return 0;
    return ddot(D, n) > 0.0 ? 1 : -1;
}

// BVH2 queries push at most one entry per level, and the BVH2 is at most 64 deep.
constexpr int kStack2 = 64;

HYB_HD double sdf_node_value(const float4* __restrict__ nodes, const float4* __restrict__ tris, D3 p,
                             int exterior_solid) {
    int stack[kStack2];

    // nearest triangle: children in order of box distance; a popped subtree is
    // skipped when its box is no closer than the best triangle found since
    double best = __builtin_inf();
    double dstack[kStack2];
    int sp = 0;
    int ref = 0;
    for (;;) {
        if (ref >= 0) {
            const float4* nd = nodes + 4 * (int64_t)ref;
            const float4 A = nd[0], B = nd[1], C = nd[2], E = nd[3];
            const double d0 = box_dist2(p, A.x, A.y, A.z, A.w, C.x, C.y);
            const double d1 = box_dist2(p, B.x, B.y, B.z, B.w, C.z, C.w);
            const int r0 = bits_i(E.x), r1 = bits_i(E.y);
            const bool h0 = d0 < best && r0 != kEmptyRef, h1 = d1 < best && r1 != kEmptyRef;
            if (h0 && h1) {
                const bool first0 = d0 <= d1;
                dstack[sp] = first0 ? d1 : d0;
                stack[sp++] = first0 ? r1 : r0;
                ref = first0 ? r0 : r1;
                continue;
            }
            if (h0) { ref = r0; continue; }
            if (h1) { ref = r1; continue; }
        } else {
            const int info = ~ref;
            const int first = info >> 3, count = info & 7;
            for (int q = 0; q < count; ++q) {
                const float4* tp = tris + 3 * (int64_t)(first + q);
                best = fmin(best, tri_dist2(p, dvert(tp[0]), dvert(tp[1]), dvert(tp[2])));
            }
        }
        bool found = false;
        while (sp > 0) {
            --sp;
            if (dstack[sp] < best) {
                ref = stack[sp];
                found = true;
                break;
            }
        }
        if (!found) break;
    }

    // winding number along a fixed direction that no mesh edge is likely to contain
    const double Dn = sqrt(0.61 * 0.61 + 0.5177 * 0.5177 + 0.6003 * 0.6003);
    const D3 D = d3(0.61 / Dn, 0.5177 / Dn, 0.6003 / Dn);
    const D3 inv = d3(1.0 / D.x, 1.0 / D.y, 1.0 / D.z);
    int wind = exterior_solid ? 1 : 0;
    sp = 0;
    ref = 0;
    for (;;) {
        if (ref >= 0) {
            const float4* nd = nodes + 4 * (int64_t)ref;
            const float4 A = nd[0], B = nd[1], C = nd[2], E = nd[3];
            const int r0 = bits_i(E.x), r1 = bits_i(E.y);
            const bool h0 = r0 != kEmptyRef && ray_box64(p, inv, A.x, A.y, A.z, A.w, C.x, C.y);
            const bool h1 = r1 != kEmptyRef && ray_box64(p, inv, B.x, B.y, B.z, B.w, C.z, C.w);
            if (h0 && h1) {
                stack[sp++] = r1;
                ref = r0;
                continue;
            }
            if (h0) { ref = r0; continue; }
            if (h1) { ref = r1; continue; }
        } else {
            const int info = ~ref;
            const int first = info >> 3, count = info & 7;
            for (int q = 0; q < count; ++q) {
                const float4* tp = tris + 3 * (int64_t)(first + q);
                wind += crossing(p, D, dvert(tp[0]), dvert(tp[1]), dvert(tp[2]));
            }
        }
        if (sp == 0) break;
        ref = stack[--sp];
    }
    const double dist = sqrt(best);
    return wind >= 1 ? -dist : dist;
}

}  // namespace hyb
